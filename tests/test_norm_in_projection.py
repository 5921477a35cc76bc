"""GPU parity of the projections that normalise their rows themselves (csrc/gemm_rows_bf16.hip, block_f32.hip) against the oracle:
row counts around their tiles of 8 and 16 rows and around the last one they take (16 in wide projections, which pick tiles of 32
rows beyond, else 24 or 32), widths at the ends of the range and with a last vector that only some lanes hold, every tile in
every projection that picks it (tests/test_gemm_plan.py holds the sizes to that), per-image keep counts (dead slots, an image
without rows, cache lengths written by the launch), the unmodulated variants.  Tolerance: bf16 tensors max|d| / max|ref| <=
2e-2, as everywhere; fp32 2e-5.  The norm's bits are those of the separate kernel: an image alone, whose projections normalise,
against the same image among others, whose do not, and fp32 blocks against blocks with a modulation of zeros and ones."""
import dataclasses

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
    return WL.Workload("norm", "bf16", B=B, C=C, heads=heads, L=1, V=64, keep_hi=.5, keep_lo=.5,
                       scales=(WL.Scale(grid=grid, prev_grid=max(grid - 2, 1), kv_len=P),), seed=29)


# below, at and inside the range of K (256 ... 2560), 512-element vectors whole and in part
WIDTHS = [(192, 3), (256, 4), (576, 9), (1024, 8), (1600, 25), (2496, 39), (2560, 20), (2624, 41)]
ROWS = [1, 9, 16, 17, 32, 33]


@pytest.mark.parametrize("C,heads", WIDTHS)
@pytest.mark.parametrize("M", ROWS)
def test_widths_and_row_counts(hx, C, heads, M):
    print(f"norm in projection C={C} M={M}", flush=True)
    hx.check_block(hx.make_host_block(_block(1, 6, 20, C, heads), 0, k=M), hx.BF16_TOL)


# every tile in front of the cross-attention and of the tanh form
CROSS = [(512, 8, 3), (576, 9, 13), (1088, 17, 26), (1536, 12, 3), (1792, 28, 9), (2112, 33, 17), (704, 11, 17)]


@pytest.mark.parametrize("C,heads,M", CROSS)
def test_cross_attention_and_tanh(hx, C, heads, M):
    print(f"norm in projection, cross C={C} M={M}", flush=True)
    hx.check_block(hx.make_host_block(_block(1, 6, 20, C, heads), 0, k=M, variant={"gelu_tanh", "cross"}), hx.BF16_TOL)


# images of k rows, and as many of them as make a separate launch of the norm
AMONG_OTHERS = [(256, 4, 1, 33), (512, 8, 26, 2), (1088, 17, 26, 2), (1600, 25, 9, 4), (1792, 28, 9, 4), (2112, 33, 17, 2),
                (2304, 36, 8, 5), (2560, 20, 16, 3)]


@pytest.mark.parametrize("C,heads,k,B", AMONG_OTHERS)
@pytest.mark.parametrize("variant", [None, {"gelu_tanh", "cross"}], ids=["base", "cross"])
def test_bits_of_the_separate_norm(hx, monkeypatch, C, heads, k, B, variant):
    print(f"norm in projection, bits C={C} k={k} {variant}", flush=True)
    from paper_2602_01345_amd import Nova
    monkeypatch.setenv("NOVA_ATTN_SPLIT", "1")           # keys of an item are not cut, whatever the number of items
    monkeypatch.setattr(hx, "_NOVA", Nova(0))
    hb = hx.make_host_block(_block(B, 6, 20, C, heads), 0, k=k, variant=variant)
    first = {f.name: getattr(hb, f.name)[:1] for f in dataclasses.fields(hb) if f.name in ("logits", "x", "k_prior", "v_prior", "cache_prev")}
    if variant:
        cross = {n: t[:1] if n in ("k_text", "v_text") else t for n, t in hb.variant["cross"].items()}
        first["variant"] = {**hb.variant, "cross": cross}
    alone = dataclasses.replace(hb, wl=dataclasses.replace(hb.wl, B=1), **first)
    for got, ref in zip(_outputs(hx, alone), _outputs(hx, hb)):
        assert torch.equal(got[0], ref[0])


@pytest.mark.parametrize("k_rows,kv_rows", [([5, 0, 1, 7], [20, 3, 0, 11]), ([0, 0, 8, 0], [0, 20, 1, 2]), ([0, 0, 0, 1], [4, 4, 4, 4])])
@pytest.mark.parametrize("C,heads", [(320, 5), (1024, 8)])
def test_per_image_counts(hx, C, heads, k_rows, kv_rows):
    print(f"norm in projection, counts {k_rows} C={C}", flush=True)
    hx.check_block_rows(hx.make_host_block(_block(4, 6, 20, C, heads), 0), k_rows, kv_rows, hx.BF16_TOL, kpitch=8)


@pytest.mark.parametrize("variant", [{"gelu_tanh", "cross", "qk_norm"}, {"ada", "cross"}], ids=lambda v: "+".join(sorted(v)))
@pytest.mark.parametrize("M", [3, 16])
def test_variants(hx, variant, M):
    """Modulated norms keep their own launch, the one in front of the cross-attention has no modulation."""
    print(f"norm in projection {sorted(variant)} M={M}", flush=True)
    hx.check_block(hx.make_host_block(_block(1, 6, 20, 512, 8), 0, k=M, variant=variant), hx.BF16_TOL)


# fp32: rows of up to 256, a sixteenth per thread (multiples of four, not of sixteen), around the 16-row tiles
@pytest.mark.parametrize("C,heads", [(4, 1), (60, 3), (252, 9), (256, 8), (260, 10)])
@pytest.mark.parametrize("M", [1, 16, 17, 36])
def test_fp32_widths_and_row_counts(hx, C, heads, M):
    print(f"norm in projection fp32 C={C} M={M}", flush=True)
    wl = WL.Workload("norm", "f32", B=1, C=C, heads=heads, L=1, V=64, keep_hi=.5, keep_lo=.5,
                     scales=(WL.Scale(grid=6, prev_grid=4, kv_len=20),), seed=31)
    hx.check_block(hx.make_host_block(wl, 0, k=M), hx.F32_TOL)


@pytest.mark.parametrize("variant", [{"gelu_tanh", "cross", "qk_norm"}, {"ada", "cross"}], ids=lambda v: "+".join(sorted(v)))
def test_fp32_variants(hx, variant):
    print(f"norm in projection fp32 {sorted(variant)}", flush=True)
    wl = WL.Workload("norm", "f32", B=2, C=48, heads=3, L=1, V=64, keep_hi=.5, keep_lo=.5,
                     scales=(WL.Scale(grid=6, prev_grid=4, kv_len=20),), seed=31)
    hx.check_block(hx.make_host_block(wl, 0, k=19, variant=variant), hx.F32_TOL)


@pytest.mark.parametrize("dtype,C,heads,M,own", [("bf16", 1024, 8, 8, 0), ("bf16", 1024, 8, 36, 1), ("f32", 64, 4, 8, 0),
                                                 ("f32", 260, 10, 8, 1)])
@pytest.mark.parametrize("variant", [None, {"ada", "cross"}], ids=["base", "ada"])
def test_stages_count_the_launches_made(hx, dtype, C, heads, M, own, variant):
    print(f"norm in projection, stages {dtype} C={C} M={M} {variant}", flush=True)
    from paper_2602_01345_amd.binding import STAGES
    wl = dataclasses.replace(_block(1, 6, 20, C, heads), dtype=dtype)
    hb, n = hx.make_host_block(wl, 0, k=M, variant=variant), hx.nova()
    runner, st, x = hx.to_gpu(hb)
    n.profile_stages(range(len(STAGES)))
    try:
        runner.run_block(st, x)
    finally:
        n.profile_stages([])
    torch.cuda.synchronize()
    got = {name: n.profile_collect(i)[1] for i, name in enumerate(STAGES)}
    assert got == {**dict.fromkeys(got, 1), **dict.fromkeys(("gather_ln", "ln2"), 1 if variant else own)}


def _outputs(hx, hb):
    runner, st, x = hx.to_gpu(hb)
    runner.run_block(st, x)
    torch.cuda.synchronize()
    return st.y_kept, st.k_cache, st.v_cache, st.out


def _neutral_ada(hb):
    """The block with a modulation that changes no bit: shifts and scales of zero, gates of one."""
    ada = torch.zeros((hb.wl.B, 6, hb.wl.C), dtype=WL.torch_dtype(hb.wl.dtype))
    ada[:, 2] = ada[:, 5] = 1.0
    return dataclasses.replace(hb, variant={**(hb.variant or {}), "ada": ada})


@pytest.mark.parametrize("C,heads", [(4, 1), (60, 3), (64, 4), (192, 12), (252, 9), (256, 8)])
@pytest.mark.parametrize("variant", [None, {"gelu_tanh"}], ids=["erf", "tanh"])
def test_fp32_bits_of_the_separate_norm(hx, C, heads, variant):
    """Rows of a mean of three deviations: what another order of a row's sums would lose most of."""
    print(f"norm in projection fp32 bits C={C}", flush=True)
    wl = WL.Workload("norm", "f32", B=1, C=C, heads=heads, L=1, V=64, keep_hi=.5, keep_lo=.5,
                     scales=(WL.Scale(grid=6, prev_grid=4, kv_len=20),), seed=37)
    hb = hx.make_host_block(wl, 0, k=36, variant=variant)
    hb.x += 3.0
    for got, ref in zip(_outputs(hx, hb), _outputs(hx, _neutral_ada(hb))):
        assert torch.equal(got, ref)
