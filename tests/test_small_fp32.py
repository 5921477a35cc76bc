"""GPU parity of the fp32 block's kernels (csrc/block_f32.hip) against the oracle at the edges of their loops: widths that
end inside a K step or a tile, head sizes below and beside the sixteen and four channels taken at a time, fewer keys than
threads, and the most cached keys the entry point accepts (with heads of four channels the scores and what the waves
exchange are then a little more than 64 KiB of LDS).  Tolerance: the fp32 tolerance of the harness."""
import pytest
import torch

import workloads as WL

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hx():
    import harness
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU and the built libnova.so (no fallback)")
    return harness


@pytest.mark.parametrize("B,grid,P,C,heads,k", [(2, 5, 3, 36, 3, 7), (1, 7, 300, 68, 4, 33), (3, 4, 0, 20, 5, 1),
                                                (1, 6, 70, 132, 2, 17), (2, 6, 60, 256, 1, 16), (1, 3, 16375, 8, 2, 5)])
def test_fp32_block_edges(hx, B, grid, P, C, heads, k):
    print(f"fp32 edges B={B} P={P} C={C} heads={heads} k={k}", flush=True)
    wl = WL.Workload("edges", "f32", B=B, C=C, heads=heads, L=1, V=64, keep_hi=.5, keep_lo=.5,
                     scales=(WL.Scale(grid=grid, prev_grid=max(grid - 2, 1), kv_len=P),), seed=23)
    hx.check_block(hx.make_host_block(wl, 0, k=k), hx.F32_TOL)
