"""GPU: entropies, means and selections of several blocks in one call (nova_entropy_blocks, nova_select_blocks) are the bits of
one call per block: counts around the 32 tensors of a launch, regular and odd rows, tensors of different alignment (other
kernels), fewer rows than waves, rows for the long selection, keep counts 0 and N among them."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nova():
    import harness
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU and the built libnova.so (no fallback)")
    return harness.nova()


def _logits(n, B, N, V, dtype, odd):
    g = torch.Generator(device="cuda").manual_seed(n * 1000 + V)
    out = []
    for i in range(n):
        flat = torch.empty(B * N * V + 8, dtype=dtype, device="cuda")
        t = flat[odd if i % 3 == 1 else 0:][:B * N * V].view(B, N, V)        # every third one element off, if asked for
        t.copy_(torch.randn((B, N, V), generator=g, device="cuda") * (1 + i))
        out.append(t)
    return out


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("n,B,N,V,odd", [(1, 2, 9, 512, 0), (2, 1, 1, 4096, 0), (5, 3, 700, 512, 0), (33, 2, 25, 1024, 0),
                                         (4, 2, 50, 1000, 0), (7, 2, 36, 512, 1), (65, 1, 4, 333, 0)])
def test_entropies_and_means(nova, dtype, n, B, N, V, odd):
    print(f"entropy blocks n={n} B={B} N={N} V={V} {dtype} odd={odd}", flush=True)
    logits = _logits(n, B, N, V, dtype, odd)
    new = lambda shape: [torch.full(shape, -1.0, device="cuda") for _ in range(n)]
    H, m, H2, m2, H3 = new((B, N)), new((B,)), new((B, N)), new((B,)), new((B, N))
    nova.entropy_blocks(logits, H, m)
    nova.entropy_blocks(logits, H3)
    for i in range(n):
        nova.entropy(logits[i], H2[i], m2[i])
    for i in range(n):
        assert torch.equal(H[i], H2[i]) and torch.equal(m[i], m2[i]) and torch.equal(H3[i], H2[i]), i


@pytest.mark.parametrize("n,B,N", [(1, 2, 9), (3, 2, 256), (33, 3, 257), (4, 1, 1025), (2, 2, 4096), (3, 1, 8193)])
def test_selections(nova, n, B, N):
    print(f"select blocks n={n} B={B} N={N}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(N + n)
    H = [torch.randint(0, 50, (B, N), generator=g, device="cuda").float() for _ in range(n)]     # many ties
    ks = [(0, N, N // 2, 1)[i % 4] for i in range(n)]
    new = lambda: ([torch.full((B, max(k, 1)), -7, dtype=torch.int32, device="cuda") for k in ks],
                   [torch.full((B, N), 9, dtype=torch.uint8, device="cuda") for _ in ks])
    (idx, mask), (idx2, mask2) = new(), new()
    nova.select_blocks(H, ks, idx, mask)
    for i in range(n):
        nova.select(H[i], ks[i], idx2[i], mask2[i])
        assert torch.equal(idx[i], idx2[i]) and torch.equal(mask[i], mask2[i]), (i, ks[i])


def test_bad_arguments_launch_nothing(nova):
    import ctypes as C
    p = (C.c_void_p * 2)(None, None)
    k = (C.c_int32 * 2)(1, 5)
    bad = -1                                           # NOVA_ERR_INVALID_ARG
    assert nova.lib.nova_entropy_blocks(nova.ctx, None, 2, p, 0, 4, 1, 16, 16, p, None) == bad
    assert nova.lib.nova_select_blocks(nova.ctx, None, 2, p, 1, 4, k, p, p) == bad
    assert nova.lib.nova_entropy_blocks(nova.ctx, None, 0, None, 0, 4, 1, 16, 16, None, None) == 0
    assert nova.lib.nova_select_blocks(nova.ctx, None, 0, None, 1, 4, None, None, None) == 0
