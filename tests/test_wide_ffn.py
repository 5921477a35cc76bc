"""GPU parity of the FFN down projection where K is too long for the tiles' 32-bit offsets (csrc/gemm_plan.h, kNearK): few
features and a very wide FFN, in one launch and in K slices, gated or not.  The hidden units are zero but for 640, the first
and the last among them and the others anywhere, so the oracle computes those only (the others add exact zeros).
Tolerance: bf16 tensors max|d| / max|ref| <= 2e-2, as everywhere (the sums have the 640 terms of any other block)."""
import pytest
import torch

import workloads as WL

pytestmark = pytest.mark.gpu
C, LIVE = 64, 640


def _check(monkeypatch, M, F, variant=None, **knobs):
    import harness as hx
    from paper_2602_01345_amd import Nova
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU and the built libnova.so (no fallback)")
    for name, v in knobs.items():
        monkeypatch.setenv("NOVA_GEMM_" + name, str(v))
    monkeypatch.setattr(hx, "_NOVA", Nova(0))          # the knobs are read when a context is created
    print(f"wide FFN M={M} F={F} {variant} {knobs}", flush=True)
    wl = WL.Workload("wide-ffn", "bf16", B=1, C=C, heads=1, L=1, V=64, keep_hi=.5, keep_lo=.5, ffn_mult=LIVE // C,
                     scales=(WL.Scale(grid=18, prev_grid=16, kv_len=20),), seed=23)
    hb = hx.make_host_block(wl, 0, k=M, variant=variant)
    hb.weights["w_fc2"] *= 64                           # the down projection outweighs the residual
    runner, st, x = hx.to_gpu(hb, poison=True)
    g = torch.Generator().manual_seed(M)
    inner = torch.randint(1, F - 1, (4 * LIVE,), generator=g).unique()
    inner = inner[torch.randperm(len(inner), generator=g)[:LIVE - 2]]
    live = torch.cat([torch.tensor([0, F - 1]), inner]).sort().values.cuda()
    assert len(live) == LIVE == len(live.unique())
    for n, shape, dim in (("w_fc1", (F, C), 0), ("b_fc1", (F,), 0), ("w_fc2", (C, F), 1)):
        st.weights[n] = torch.zeros(shape, dtype=torch.bfloat16, device="cuda").index_copy_(dim, live, st.weights[n])
    runner.ffn_mult = F // C
    runner.blocks.clear()
    runner.add_block(st)
    runner.run_block(st, x)
    torch.cuda.synchronize()
    ref = hx.oracle_block(hb, st.entropy.cpu().numpy())
    assert hx.nerr(st.y_kept, ref["y"]) <= hx.BF16_TOL
    assert hx.nerr(st.out, ref["out"]) <= hx.BF16_TOL


@pytest.mark.parametrize("ksplit", [0, 4], ids=["whole", "sliced"])
@pytest.mark.parametrize("variant", [None, frozenset({"ada"})], ids=["base", "gated"])
@pytest.mark.parametrize("F", [1 << 21, (1 << 21) + 256, (1 << 23) + 2048])
def test_ring_tiles(monkeypatch, F, variant, ksplit):
    _check(monkeypatch, 300, F, variant, CFG=2, KSPLIT=ksplit)


@pytest.mark.parametrize("M,F", [(5, 1 << 23), (300, 1 << 23), (5, (1 << 23) + 2048), (300, (1 << 23) + 2048),
                                 (300, (1 << 24) + 2048), (5, 1 << 26)])
def test_few_rows_tiles(monkeypatch, M, F):
    """Smaller tiles of the few-rows kernels as K grows: 64 rows or features end at 2^23, 32 at 2^24, 8 at 2^26."""
    _check(monkeypatch, M, F)
