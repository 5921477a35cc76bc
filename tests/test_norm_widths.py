"""LayerNorm at every count of 16-byte vectors that a lane holds (csrc/norm.hip: 1 ... 8 have a kernel each, longer rows take
three passes), the last of them partly filled, modulated and not.  Seen through the block, whose other parts are switched
off: the query projection is the only consumer of LN(x) here, read back as the appended key rows (w_qkv's key part is the
identity, so k_cache = LN(x) (1 + scale) + shift, one rounding to the storage type).  Tolerance: bf16 rounding of u and of
the key (2^-7 of the value; the sums are fp32), fp32 1e-5."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,per_vector", [("bf16", 8), ("f32", 4)])
@pytest.mark.parametrize("vectors", [1, 2, 3, 4, 5, 6, 7, 8, 9])
@pytest.mark.parametrize("modulated", [False, True])
def test_every_vector_count(dtype, per_vector, vectors, modulated):
    from paper_2602_01345_amd import NOVA_BF16, NOVA_F32, BlockShape, Nova
    from paper_2602_01345_amd.binding import BlockVariant
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU and the built libnova.so (no fallback)")
    C = 64 * per_vector * vectors - 64                 # the last vector only in some lanes
    print(f"layernorm {dtype} C={C} modulated={modulated}", flush=True)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    heads, B, k, cap, dh = C // 64, 2, 3, 64, 64
    nova = Nova(0)
    shape = BlockShape(NOVA_F32 if dtype == "f32" else NOVA_BF16, B, k, C, heads, 0, cap, k, 1)
    g = torch.Generator().manual_seed(C)
    rnd = lambda *s: torch.randn(s, generator=g).to(tdt).cuda()
    zeros = lambda *s: torch.zeros(s, dtype=tdt, device="cuda")
    w_qkv = zeros(3 * C, C)
    w_qkv[C:2 * C] = torch.eye(C, dtype=tdt, device="cuda")
    W = {"w_qkv": w_qkv, "w_o": zeros(C, C), "w_fc1": zeros(C, C), "w_fc2": zeros(C, C)}
    x, ada = rnd(B, k, C) * 3.0 + 1.0, rnd(B, 6, C)
    idx = torch.arange(k, dtype=torch.int32, device="cuda").repeat(B, 1)
    kc, vc, y = zeros(B, heads, cap, dh), zeros(B, heads, dh, cap), zeros(B, k, C)
    ws = torch.empty(nova.workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    nova.pruned_block_variant(shape, W, BlockVariant(ada=ada) if modulated else None, x, idx, kc, vc, y, ws)
    torch.cuda.synchronize()
    xd, ad = x.double().cpu(), ada.double().cpu()
    u = (xd - xd.mean(-1, keepdim=True)) / torch.sqrt(xd.var(-1, unbiased=False, keepdim=True) + 1e-6)
    bound = u.abs()
    if modulated:
        bound = (u * (1 + ad[:, 1:2])).abs() + ad[:, 0:1].abs()
        u = u * (1 + ad[:, 1:2]) + ad[:, 0:1]
    got = kc[:, :, :k].transpose(1, 2).reshape(B, k, C).double().cpu()
    tol = 1e-5 * (bound + 1.0) + (2.0 ** -7 * u.abs() if dtype == "bf16" else 0.0)
    assert bool(((got - u).abs() <= tol).all()), float((got - u).abs().max())
