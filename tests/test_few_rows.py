"""GPU parity of the few-rows projection kernels (csrc/gemm_rows_bf16.hip) against the oracle at the edges of their tiles:
row counts around 8, 16, 32 and multiples of 64, a K with fewer runs of 64 than a workgroup has waves (C = 64, 320), every
tile the plan can pick in every projection it picks it for (tests/test_gemm_plan.py holds SIZES to that), the long K of the
down projection.
Tolerance: bf16 tensors max|d| / max|ref| <= 2e-2, as everywhere (the products and their sums are fp32)."""
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


def _block(B, grid, P, C, heads):
    return WL.Workload("few", "bf16", B=B, C=C, heads=heads, L=1, V=64, keep_hi=.5, keep_lo=.5,
                       scales=(WL.Scale(grid=grid, prev_grid=max(grid - 2, 1), kv_len=P),), seed=17)


AROUND_THE_TILES = [(64, 1), (320, 5), (1024, 8)], [1, 8, 9, 16, 17, 32, 33, 64, 65, 129, 257]
WIDTHS = [(2048, 16, 5), (2048, 16, 12), (2048, 16, 30), (2048, 16, 50), (2048, 16, 100), (1920, 30, 72), (512, 8, 511),
          (1024, 8, 512)]
# tiles that the widths above do not reach, or not in every projection: 8 x 32 (of more rows than a projection normalises itself),
# 16 x 32, 32 x 64, 64 x 64 with one unit in flight
OTHER_TILES = [(1152, 18, 1), (1152, 18, 8), (1536, 24, 7), (1536, 24, 165), (704, 11, 87), (384, 6, 330), (2112, 33, 5),
               (2112, 33, 9), (2112, 33, 451), (2304, 36, 213), (384, 6, 36), (384, 6, 50)]
BEYOND_512 = [(1024, 8, 257), (1024, 8, 511), (512, 8, 600)]
SIZES = ([(C, M) for C, _ in AROUND_THE_TILES[0] for M in AROUND_THE_TILES[1]] + [(C, M) for C, _, M in WIDTHS + OTHER_TILES] +
         [(C, 2 * k) for C, _, k in BEYOND_512])


@pytest.mark.parametrize("C,heads", AROUND_THE_TILES[0])
@pytest.mark.parametrize("M", AROUND_THE_TILES[1])
def test_row_counts_around_the_tiles(hx, C, heads, M):
    print(f"few rows C={C} M={M}", flush=True)
    wl = _block(1, 17, 40, C, heads)
    hx.check_block(hx.make_host_block(wl, 0, k=M), hx.BF16_TOL)


@pytest.mark.parametrize("C,heads,M", WIDTHS + OTHER_TILES)
def test_widths_and_long_k(hx, C, heads, M):
    print(f"few rows C={C} M={M}", flush=True)
    wl = _block(1, 23, 20, C, heads)
    hx.check_block(hx.make_host_block(wl, 0, k=M), hx.BF16_TOL)


@pytest.mark.parametrize("C,heads,k", BEYOND_512)
def test_one_workgroup_per_cu_beyond_512_rows(hx, C, heads, k):
    print(f"few rows C={C} M={2 * k}", flush=True)
    wl = _block(2, 25, 20, C, heads)
    hx.check_block(hx.make_host_block(wl, 0, k=k), hx.BF16_TOL)
