"""GPU parity of the 256 x 256 projection tile (csrc/gemm_bf16.hip, configuration 1) against the oracle where its K loop
and its edges change: one, two, three and an odd number of K steps, rows and features that end inside a tile, gated
residuals, more tiles than compute units (a workgroup then walks several, each starting in the first LDS buffer), and
per-image keep counts.  Tolerance: bf16 tensors max|d| / max|ref| <= 2e-2, as everywhere."""
import pytest
import torch

import workloads as WL

pytestmark = pytest.mark.gpu


@pytest.fixture
def hx(monkeypatch):
    import harness
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU and the built libnova.so (no fallback)")
    from paper_2602_01345_amd import Nova
    monkeypatch.setenv("NOVA_GEMM_CFG", "1")
    monkeypatch.setattr(harness, "_NOVA", Nova(0))     # the knob is read when a context is created
    return harness


def _block(B, grid, P, C, heads):
    return WL.Workload("large", "bf16", B=B, C=C, heads=heads, L=1, V=64, keep_hi=.5, keep_lo=.5,
                       scales=(WL.Scale(grid=grid, prev_grid=max(grid - 2, 1), kv_len=P),), seed=19)


@pytest.mark.parametrize("C,heads,k", [(64, 1, 255), (128, 2, 256), (192, 3, 257), (320, 5, 130), (640, 5, 289)])
@pytest.mark.parametrize("variant", [None, frozenset({"ada"})], ids=["base", "gated"])
def test_k_steps_and_edges(hx, C, heads, k, variant):
    print(f"large tiles C={C} k={k} {variant}", flush=True)
    wl = _block(2, 17, 40, C, heads)
    hx.check_block(hx.make_host_block(wl, 0, k=k, variant=variant), hx.BF16_TOL)


def test_several_tiles_per_workgroup_with_an_odd_number_of_k_steps(hx):
    # C = 832: 13 K steps; 6480 rows: 26 tile rows, 260 QKV and 338 FFN tiles
    print("large tiles C=832 M=6480", flush=True)
    wl = _block(16, 21, 30, 832, 13)
    hx.check_block(hx.make_host_block(wl, 0, k=405), hx.BF16_TOL, rows=[0, 7, 15])
