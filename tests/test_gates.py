"""Gated residuals in every kernel that adds one: the few-rows kernels, every tile configuration of the projections, and the
second pass of a K-sliced down projection; 2 x 130 rows, so that tiles are ragged and hold rows of both images.  Exact: a
zero gate leaves the residual, whatever the projection is; gates of one (and no modulation) are the block without them."""
import pytest
import torch

import workloads as WL

pytestmark = pytest.mark.gpu

PATHS = [(None, None), ("1", None), ("2", None), ("5", None), ("6", None), ("1", "2"), ("2", "4")]


@pytest.mark.parametrize("cfg,ksplit", PATHS)
def test_gates_of_zero_and_one(cfg, ksplit, monkeypatch):
    import harness as hx
    from paper_2602_01345_amd import BlockVariant, Nova
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU and the built libnova.so (no fallback)")
    for name, v in (("NOVA_GEMM_CFG", cfg), ("NOVA_GEMM_KSPLIT", ksplit)):
        if v is not None:
            monkeypatch.setenv(name, v)
    monkeypatch.setattr(hx, "_NOVA", Nova(0))          # the knobs are read when a context is created
    print(f"gates cfg={cfg} ksplit={ksplit}", flush=True)
    C = 1024
    wl = WL.Workload("gates", "bf16", B=2, C=C, heads=8, L=1, V=64, keep_hi=.5, keep_lo=.5,
                     scales=(WL.Scale(grid=17, prev_grid=13, kv_len=40),), seed=31)
    hb = hx.make_host_block(wl, 0, k=130)
    hb.x = hb.x * 2.0 ** -17                           # projections some 10^7 times the residual
    for n in ("b_o", "b_fc2"):
        hb.weights[n] = torch.full_like(hb.weights[n], 96.0)

    def run(variant):
        runner, st, x = hx.to_gpu(hb)
        st.variant = variant
        runner.run_block(st, x)
        torch.cuda.synchronize()
        kept = torch.gather(x, 1, st.kept_idx[:, :130].long().unsqueeze(-1).expand(-1, -1, C))
        return st.y_kept.clone(), kept

    ada = (torch.randn(2, 6, C, generator=torch.Generator().manual_seed(3)) * 0.2).to(torch.bfloat16).cuda()
    ada[:, 2], ada[:, 5] = 0.0, 0.0
    y, kept = run(BlockVariant(ada=ada))
    assert torch.equal(y, kept), f"{int((y != kept).sum())} of {y.numel()} elements are not the residual"
    ones = torch.zeros_like(ada)
    ones[:, 2], ones[:, 5] = 1.0, 1.0
    assert torch.equal(run(BlockVariant(ada=ones))[0], run(None)[0])
