"""GPU parity of the few-queries attention kernel (csrc/attention_few_bf16.hip) against the oracle where it can go wrong: fewer
key tiles than waves, keys that end on, one before and one behind a tile, queries that end on and next to a block of 32, one,
four and eight waves, both head sizes, scores spread over tens of nats (the softmax reference moves in every wave), images
with counts of their own (one with none), waves none of whose keys has a finite score.
Tolerance: bf16 tensors max|d| / max|ref| <= 2e-2, as everywhere."""
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


def _wl(B, P, C, heads, grid=17):
    return WL.Workload("fewq", "bf16", B=B, C=C, heads=heads, L=1, V=64, keep_hi=.5, keep_lo=.5,
                       scales=(WL.Scale(grid=grid, prev_grid=grid - 4, kv_len=P),), seed=23)


@pytest.mark.parametrize("C,heads", [(128, 2), (256, 2)])                     # dh = 64 and dh = 128
@pytest.mark.parametrize("P,k", [(0, 1), (31, 1), (32, 32), (30, 33), (63, 64), (127, 2), (256, 65), (700, 97), (1500, 31)])
def test_tile_and_block_edges(hx, C, heads, P, k):
    print(f"few queries C={C} P={P} k={k}", flush=True)
    hx.check_block(hx.make_host_block(_wl(2, P, C, heads), 0, k=k), hx.BF16_TOL)


@pytest.mark.parametrize("C,heads", [(128, 2), (256, 2)])
def test_wide_scores_move_the_reference(hx, C, heads):
    print(f"few queries, wide rising scores C={C}", flush=True)
    hb = hx.make_host_block(_wl(2, 900, C, heads), 0, k=70)
    w = hb.weights["w_qkv"].to(torch.float32)
    w[:C] *= 24.0
    hb.weights["w_qkv"] = w.to(hb.weights["w_qkv"].dtype)
    ramp = torch.linspace(0.25, 4.0, hb.k_prior.shape[1]).reshape(1, -1, 1)
    hb.k_prior = (hb.k_prior.to(torch.float32) * ramp).to(hb.k_prior.dtype)
    hx.check_block(hb, hx.BF16_TOL)


@pytest.mark.parametrize("C,heads", [(128, 2), (256, 2)])
def test_images_with_their_own_counts(hx, C, heads):
    print(f"few queries, per-image counts C={C}", flush=True)
    hb = hx.make_host_block(_wl(3, 300, C, heads), 0)
    hx.check_block_rows(hb, [100, 0, 33], [300, 17, 64], hx.BF16_TOL)


@pytest.mark.parametrize("C,heads", [(128, 2), (256, 2)])
def test_one_tile_of_keys_with_counts(hx, C, heads):
    """At most one tile of keys (64 at dh = 64, 32 at dh = 128): a single wave per workgroup, which writes its output itself."""
    print(f"few queries, one tile, per-image counts C={C}", flush=True)
    hb = hx.make_host_block(_wl(4, 12, C, heads, grid=9), 0, k=20)
    hx.check_block_rows(hb, [20, 0, 1, 7], [12, 5, 0, 3], hx.BF16_TOL)


@pytest.mark.parametrize("C,heads", [(128, 2), (256, 2)])
def test_one_forced_run_is_the_many_query_kernel_uncut(hx, C, heads, monkeypatch):
    """NOVA_ATTN_SPLIT=1 reaches csrc/attention_bf16.hip without key runs, whatever the size: the bits of its default
    workgroup shape forced (too few key tiles here for the launcher to cut any)."""
    from paper_2602_01345_amd import Nova
    print(f"forced uncut attention C={C}", flush=True)
    hb = hx.make_host_block(_wl(2, 700, C, heads), 0, k=70)
    outs = []
    for knob in ("NOVA_ATTN_SPLIT", "NOVA_ATTN_CFG"):
        with monkeypatch.context() as m:
            m.setenv(knob, "1")
            m.setattr(hx, "_NOVA", Nova(0))            # the knobs are read when a context is created
            runner, st, x = hx.to_gpu(hb)
            runner.run_block(st, x)
            torch.cuda.synchronize()
            outs.append(st.y_kept.clone())
    assert torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("C,heads", [(128, 2), (256, 2)])
@pytest.mark.parametrize("P", [200, 700])                                    # four and eight waves
def test_keys_whose_scores_overflow_weigh_nothing(hx, C, heads, P):
    """Behind the first 64 prior keys every prior key scores -inf (about -3e39 before fp32 ends): whole tiles, and all tiles
    of some waves, without a finite score."""
    print(f"few queries, scores of -inf C={C} P={P}", flush=True)
    hb = hx.make_host_block(_wl(2, P, C, heads), 0, k=32)
    dh = C // heads
    hb.weights["w_qkv"][:C:dh] = 0.0                                         # the first query channel of every head is 64
    hb.weights["b_qkv"][:C:dh] = 64.0
    hb.k_prior[:, 64:, ::dh] = -3.0e38
    hx.check_block(hb, hx.BF16_TOL)
