"""GPU selection against a stable sort at the row lengths where its kernels change (csrc/select.hip), on the key
distributions that steer the search: distinct entropies, one bin with more than 64 keys at every level of the range
division, ties everywhere, one outlier that stretches the range, infinities, NaN and signed zeros.  Exact."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _rows(N, g):
    u = torch.rand(N, generator=g) * 8.0
    near = 3.0 + torch.randint(0, 900, (N,), generator=g) * 2.0 ** -21       # a few hundred neighbouring keys
    ties = torch.randint(0, 3, (N,), generator=g).float()
    outlier = u.clone() * 1e-3 + 5.0
    outlier[N // 2] = -float("inf")
    mixed = u.clone()
    mixed[torch.rand(N, generator=g) < 0.2] = float("nan")
    mixed[torch.rand(N, generator=g) < 0.1] = -0.0
    mixed[torch.rand(N, generator=g) < 0.1] = 0.0
    mixed[torch.rand(N, generator=g) < 0.05] = float("inf")
    mixed[torch.rand(N, generator=g) < 0.05] = -float("inf")
    return torch.stack([u, near, ties, outlier, mixed, torch.full((N,), 2.5), torch.full((N,), float("nan"))])


def _reference(h, k):
    v = h.astype(np.float64) + 0.0                                           # -0 == +0
    order = np.lexsort((np.arange(len(v)), np.where(np.isnan(v), np.inf, -v), np.isnan(v)))
    kept = np.sort(order[:k])
    mask = np.zeros(len(v), np.uint8)
    mask[kept] = 1
    return kept, mask


@pytest.mark.parametrize("N", [1, 2, 63, 65, 169, 256, 257, 1000, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193])
def test_every_row_length(N):
    from paper_2602_01345_amd import Nova
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU and the built libnova.so (no fallback)")
    print(f"select N={N}", flush=True)
    nova = Nova(0)
    h = _rows(N, torch.Generator().manual_seed(N))
    B = h.shape[0]
    d = h.cuda()
    for k in sorted({1, N // 3, N // 2, N - 1, N} - {0}):
        idx = torch.full((B, k), -7, dtype=torch.int32, device="cuda")
        mask = torch.full((B, N), 9, dtype=torch.uint8, device="cuda")
        nova.select(d, k, idx, mask)
        per = torch.tensor([(k * (b + 1)) // B for b in range(B)], dtype=torch.int32)
        idx2, mask2 = torch.full_like(idx, -7), torch.full_like(mask, 9)
        nova.select(d, k, idx2, mask2, k_per_row=per.cuda())
        for b in range(B):
            kept, m = _reference(h[b].numpy(), k)
            assert np.array_equal(idx[b].cpu().numpy(), kept) and np.array_equal(mask[b].cpu().numpy(), m), (N, k, b)
            n = int(per[b])
            kept, m = _reference(h[b].numpy(), n)
            got = idx2[b].cpu().numpy()
            assert np.array_equal(got[:n], kept) and (got[n:] == -1).all(), (N, k, b, "per row")
            assert np.array_equal(mask2[b].cpu().numpy(), m), (N, k, b, "per row")
