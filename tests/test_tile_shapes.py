"""GPU parity of the projection tiles that stand in where others leave CUs idle (csrc/gemm_bf16.hip) against the oracle, by force
where their K loops and edges change: one, two, three and more K steps than stages, an odd number, rows and features that end inside
a tile and on its edge, gated residuals, more tiles than compute units (a workgroup then walks several, each starting in the
first LDS buffer), and at sizes where the plan chooses them, for all rows and for the first or last of two launches.  Tolerance: bf16 tensors max|d| / max|ref| <= 2e-2, as everywhere (the products and
their sums are fp32)."""
import pytest
import torch

import workloads as WL

pytestmark = pytest.mark.gpu
TILES = {"192x256": "9", "128x64": "8"}


@pytest.fixture(params=list(TILES.values()), ids=list(TILES))
def hx(request, monkeypatch):
    import harness
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU and the built libnova.so (no fallback)")
    from paper_2602_01345_amd import Nova
    monkeypatch.setenv("NOVA_GEMM_CFG", request.param)
    monkeypatch.setattr(harness, "_NOVA", Nova(0))     # the knob is read when a context is created
    return harness


def _block(B, grid, P, C, heads):
    return WL.Workload("shapes", "bf16", B=B, C=C, heads=heads, L=1, V=64, keep_hi=.5, keep_lo=.5,
                       scales=(WL.Scale(grid=grid, prev_grid=max(grid - 2, 1), kv_len=P),), seed=23)


@pytest.mark.parametrize("C,heads,k", [(64, 1, 1), (64, 1, 191), (128, 2, 192), (192, 3, 193), (320, 5, 64), (448, 7, 129), (640, 5, 289)])
@pytest.mark.parametrize("variant", [None, frozenset({"ada"})], ids=["base", "gated"])
def test_k_steps_and_edges(hx, C, heads, k, variant):
    print(f"tile shapes C={C} k={k} {variant}", flush=True)
    wl = _block(2, 17, 40, C, heads)
    hx.check_block(hx.make_host_block(wl, 0, k=k, variant=variant), hx.BF16_TOL)


def test_several_tiles_per_workgroup_with_an_odd_number_of_k_steps(hx):
    print("tile shapes C=832 M=6480", flush=True)      # 13 K steps
    wl = _block(16, 21, 30, 832, 13)
    hx.check_block(hx.make_host_block(wl, 0, k=405), hx.BF16_TOL, rows=[0, 7, 15])


def test_128_x_128_with_a_long_k(monkeypatch):
    """From K = 2048 on that tile has one more stage."""
    import harness as hx
    from paper_2602_01345_amd import Nova
    monkeypatch.setenv("NOVA_GEMM_CFG", "5")
    monkeypatch.setattr(hx, "_NOVA", Nova(0))
    print("tile shapes C=2048 128 x 128", flush=True)
    hx.check_block(hx.make_host_block(_block(1, 13, 40, 2048, 16), 0, k=129), hx.BF16_TOL)


# C, heads, images, kept tokens, image compared, and (projection: 0 QKV, 1 output, 2 up, 3 down; launch of it; tile) of its rows
CHOSEN = [(704, 11, 6, 249, 5, [(1, 0, 128, 64), (3, 0, 128, 64)]), (768, 12, 2, 257, 1, [(0, 0, 128, 64), (2, 0, 128, 64)]),
          (1344, 21, 14, 425, 13, [(0, 0, 192, 256), (3, 0, 192, 256)]), (2304, 36, 8, 512, 3, [(1, 0, 192, 256), (3, 0, 192, 256)]),
          (1984, 31, 7, 404, 6, [(0, 1, 192, 256), (2, 0, 192, 256)]), (2368, 37, 4, 418, 3, [(0, 0, 192, 256), (2, 1, 192, 256)]),
          (960, 15, 9, 667, 8, [(0, 1, 128, 64), (2, 0, 192, 256)]), (960, 15, 11, 518, 0, [(0, 0, 128, 64)])]


@pytest.mark.parametrize("C,heads,B,k,image,tiles", CHOSEN)
def test_sizes_where_the_plan_chooses_them(C, heads, B, k, image, tiles):
    import harness as hx
    print(f"tile shapes chosen C={C} M={B * k}", flush=True)
    hx.check_block(hx.make_host_block(_block(B, 27, 30, C, heads), 0, k=k), hx.BF16_TOL, rows=[image])
