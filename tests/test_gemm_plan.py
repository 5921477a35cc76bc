"""The launch plans of csrc/gemm_plan.h on the CPU, compiled for the host alone (gemm_plan_probe.cpp)."""
import os
import re
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2602_01345_amd", "csrc")
QKV, ATTN_OUT, GELU, RESIDUAL, PLAIN = 0, 1, 2, 3, 6   # EpiMode of csrc/epilogue.h
NORM = 16                                              # added: behind a LayerNorm without modulation


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plan") / "probe")
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    subprocess.run([hipcc, "--offload-arch=gfx950", "--offload-host-only", "-std=c++20", "-x", "hip", "-I" + CSRC,
                    os.path.join(HERE, "gemm_plan_probe.cpp"), "-o", exe], check=True, capture_output=True)

    def answers(requests):
        r = subprocess.run([exe], input="".join(requests), text=True, check=True, capture_output=True)
        return [line.split() for line in r.stdout.split("\n")]

    def ask(mode, M, Nout, K, part_floats=10 ** 9, cfg=-1, parts=-1, ksplit=-1, fields=4):
        """[(rows, configuration, tiles or workgroups, K slices)] of the launches, with fields=5 the end of each launch's 32-bit
        offsets behind them (0: 64-bit addresses), with fields=7 a tile's rows and columns"""
        line = answers([f"{mode} {M} {Nout} {K} {part_floats} {cfg} {parts} {ksplit}\n"])[0]
        return [tuple(int(v) for v in p.split(":")[:fields]) for p in line]

    def few_rows_tiles(sizes, norm=None):
        """{(mode, rg, ng, kw, s)} of the few-rows launches of blocks of (C, M).  norm=None: their norms are launches of their
        own (modulated blocks), norm=False / True: of the other blocks, in the projections that do not / do normalise their rows"""
        blocks = ((QKV, 3, 1), (ATTN_OUT, 1, 1), (GELU, 4, 1), (RESIDUAL, 1, 4)) + (((PLAIN, 1, 1),) if norm else ())
        asked = [(mode, f"{mode + (NORM if norm is not None and mode in (QKV, GELU, PLAIN) else 0)} {M} {N * C} {K * C} "
                        f"{_part_floats(M, C)} -1 -1 -1\n") for C, M in sizes for mode, N, K in blocks]
        return {(mode, *(int(v) for v in p.split(":")[5:9])) for (mode, _), line in zip(asked, answers(q for _, q in asked))
                for p in line if p.split(":")[1] == "7" and p.endswith("norm") == bool(norm)}
    ask.few_rows_tiles = few_rows_tiles
    ask.exe = exe
    return ask


@pytest.mark.parametrize("K", [(1 << 21) + 64, 1 << 22, 1 << 23])
@pytest.mark.parametrize("M,Nout", [(600, 16384), (2049, 8192), (4097, 16384), (9000, 8192)])
def test_the_tile_with_32_bit_offsets_stops_where_they_end(plan, M, Nout, K):
    """255 rows of 2 K bytes and the offset along K of the 256 x 256 tile have to stay below 2^31 bytes: neither one launch,
    nor the parts of two, nor a forced choice may take it beyond K = 2^21."""
    for cfg in (-1, 1, 9):
        parts = plan(RESIDUAL, M, Nout, K, cfg=cfg)
        assert all(c not in (1, 9) for _, c, _, _ in parts), parts
        assert sum(p[0] for p in parts) == M


@pytest.mark.parametrize("M,Nout,K", [(m, 64, k) for m in (1, 64, 200, 300, 600, 5000) for k in
                                      (1 << 21, (1 << 21) + 256, (1 << 22) + 4096, 1 << 23, (1 << 23) + 2048)] +
                         [(600, 2048, 2049 * 2048), (1100, 2048, 2049 * 2048), (2100, 2048, 1025 * 2048)])
def test_no_launch_leaves_its_32_bit_offsets(plan, M, Nout, K):
    """The FFN down projection of few features and a very wide FFN, cut into K slices or not: every launch's offsets stay
    below 2^31 - 1 bytes, the length its buffer loads are bounded by, or it takes 64-bit addresses."""
    cut = 0
    for cfg in (-1, 0, 1, 2, 3, 4, 5, 6, 8, 9):
        for ksplit in (-1, 0, 2, 4):
            parts = plan(RESIDUAL, M, Nout, K, _part_floats(M, Nout), cfg=cfg, ksplit=ksplit, fields=5)
            assert sum(p[0] for p in parts) == M
            assert all(p[4] < (1 << 31) - 1 for p in parts), (cfg, ksplit, parts)
            assert K <= 1 << 21 or all(p[1] == 7 or p[4] == 0 for p in parts), (cfg, ksplit, parts)
            cut += any(p[3] > 1 for p in parts)
    assert cut or 2 * M * Nout > _part_floats(M, Nout)


def test_a_projection_that_normalises_reads_its_rows_and_no_more(plan):
    """Rows shorter than the 512 elements that a wave reads at a time among them: the last row of the activations ends where
    the caller's memory may end."""
    r = subprocess.run([plan.exe, "norm"], text=True, check=True, capture_output=True)
    rows = [[int(v) for v in line.split()] for line in r.stdout.splitlines()]
    assert [row[0] for row in rows] == list(range(64, 2561, 64))
    assert all((first, end, missing) == (0, K, 0) for K, first, end, missing in rows), rows


def test_entropies_of_many_images_with_their_means(plan):
    """Sizes where one launch takes up to 24 % longer than two (0), and neighbours of them where it takes less (1)."""
    sizes = {(2, 9, 256, 4096): 1, (2, 9, 257, 4096): 0, (2, 9, 4096, 4096): 0, (2, 8, 800, 4096): 1, (2, 9, 3000, 2048): 0,
             (2, 16, 3000, 2048): 0, (2, 16, 3000, 2560): 1, (2, 9, 3000, 1536): 1, (2, 5, 256, 8192): 1, (2, 5, 800, 8192): 0,
             (2, 4, 4096, 4096): 1, (2, 4, 2048, 32768): 1, (4, 9, 2048, 2048): 1, (4, 6, 256, 6144): 1,
             (4, 6, 300, 6144): 0, (2, 16, 1, 2560): 1, (2, 16, 1, 4096): 0, (4, 16, 1, 4096): 0, (2, 17, 1, 512): 0}
    r = subprocess.run([plan.exe, "entropy"], input="".join("%d %d %d %d\n" % s for s in sizes), text=True, check=True,
                       capture_output=True)
    assert [int(v) for v in r.stdout.split()] == list(sizes.values())


@pytest.mark.parametrize("K,few", [(1 << 23, True), ((1 << 23) + 2048, True), (1 << 26, True), ((1 << 26) + 64, False)])
def test_few_rows_keep_their_kernels_while_a_tile_fits(plan, K, few):
    """Eight rows of 2 K bytes are within 32-bit offsets up to K = 2^26: no reason to leave the few-rows kernels before."""
    for M in (1, 8, 64, 200):
        assert [p[1] == 7 for p in plan(RESIDUAL, M, 64, K, _part_floats(M, 64))] == [few], (M, K)


def test_eight_rows_of_features_that_divide_unevenly(plan):
    """288 or 864 workgroups of 8 x 8 give some CUs one more than others: wider tiles, one workgroup per CU at most."""
    for M in (1, 8):
        assert plan.few_rows_tiles([(2304, M)]) == {(QKV, 1, 4, 4, 4), (ATTN_OUT, 1, 2, 4, 4), (GELU, 1, 2, 4, 4),
                                                    (RESIDUAL, 1, 2, 4, 4)}
        assert plan.few_rows_tiles([(2048, M)]) == {(mode, 1, 1, 8 if mode == RESIDUAL else 4, 4) for mode in range(4)}


def test_the_taller_of_two_tiles_that_load_as_much(plan):
    """64 x 32 fetches the weights half as often as 32 x 64 (C = 2304, 64 rows, QKV: 1.6 us less)."""
    assert (QKV, 8, 4, 4, 2) in plan.few_rows_tiles([(2304, 64)]) and (ATTN_OUT, 8, 4, 4, 2) in plan.few_rows_tiles([(1920, 200)])


def test_the_tile_with_32_bit_offsets_up_to_there(plan):
    assert plan(RESIDUAL, 2049, 8192, 1 << 21, cfg=1)[0][1] == 1


@pytest.mark.parametrize("mode,M,C,cfg,slices", [(QKV, 1500, 1920, 1, 1), (GELU, 1500, 1920, 1, 1), (QKV, 1500, 2048, 1, 1),
                                                 (GELU, 1500, 2048, 1, 1), (QKV, 3072, 1024, 1, 1), (QKV, 4096, 768, 1, 1),
                                                 (GELU, 4096, 768, 1, 1), (RESIDUAL, 1800, 1024, 5, 2),
                                                 (RESIDUAL, 2048, 1024, 5, 2)])
def test_tiles_are_priced_with_weights_from_memory(plan, mode, M, C, cfg, slices):
    """One round of wide tiles against two of narrow ones, which read the weights more often: blocks of these sizes are 3 to
    7 % slower with what launches on weights in L2 would choose."""
    N, K = {QKV: (3 * C, C), GELU: (4 * C, C), RESIDUAL: (C, 4 * C)}[mode]
    (_, got, _, ks), = plan(mode, M, N, K, _part_floats(M, C))
    assert (got, ks) == (cfg, slices)


def _part_floats(M, C):
    return min(4 * M * C, 128 * 256 * 256)             # K-slice scratch of the block's workspace


ANY_BLOCK = [(C, M) for C in range(64, 2560, 64) for M in [*range(1, 66), *range(66, 1100, 11)]]


def test_sizes_of_the_gpu_tests_reach_every_few_rows_tile(plan):
    """Every tile of csrc/gemm_plan.h, in every projection that picks it over the widths of up to 2496 with up to 1100 rows,
    in launches that do not normalise their rows."""
    import test_few_rows as F
    tested = plan.few_rows_tiles(F.SIZES, norm=False)
    with open(os.path.join(CSRC, "gemm_plan.h")) as f:
        tiles = {tuple(int(v) for v in t.split(",")[:4]) for t in re.findall(r" T\((\d+(?:, \d+){4})\)", f.read())}
    assert len(tiles) == 13 and {t[1:] for t in tested} == tiles
    picked = plan.few_rows_tiles(ANY_BLOCK)
    assert picked <= tested, picked - tested


def test_sizes_of_the_gpu_tests_reach_every_tile_that_normalises(plan):
    """The same for projections that normalise their rows, QKV, up (both forms of the GELU) and cross-attention query."""
    import test_norm_in_projection as T
    picked = plan.few_rows_tiles(ANY_BLOCK + [(2560, M) for M in range(1, 40)], norm=True)
    assert len(picked) == 12
    base = plan.few_rows_tiles([(C, M) for C, _ in T.WIDTHS for M in T.ROWS], norm=True)
    assert {t for t in picked if t[0] != PLAIN} <= base, picked - base
    cross = plan.few_rows_tiles([(C, M) for C, _, M in T.CROSS], norm=True)
    assert {t for t in picked if t[0] != QKV} <= cross, picked - cross
    alone = [(C, k) for C, _, k, _ in T.AMONG_OTHERS]
    # but for 8 x 32 in the up projection, whose blocks' down projections split K over eight waves if alone
    assert picked - {(GELU, 1, 4, 4, 4)} <= plan.few_rows_tiles(alone, norm=True)
    # ... against launches that do not normalise, whose waves split K in the same way
    assert not plan.few_rows_tiles([(C, B * k) for C, _, k, B in T.AMONG_OTHERS], norm=True)
    assert all(t[3] == 4 for t in plan.few_rows_tiles(alone, norm=False) |
               plan.few_rows_tiles([(C, B * k) for C, _, k, B in T.AMONG_OTHERS], norm=False))


def test_sizes_of_the_gpu_tests_reach_the_tiles_for_half_filled_rounds(plan):
    """192 x 256 and 128 x 64 as the plan chooses them, in one launch and in two."""
    import test_tile_shapes as T
    nk = {QKV: (3, 1), ATTN_OUT: (1, 1), GELU: (4, 1), RESIDUAL: (1, 4)}
    for C, _, B, k, image, tiles in T.CHOSEN:
        for mode, part, bm, bn in tiles:
            N, K = nk[mode]
            parts = plan(mode, B * k, N * C, K * C, _part_floats(B * k, C), fields=7)
            assert parts[part][5:] == (bm, bn) and parts[part][1] == (8 if bn == 64 else 1) and parts[part][3] == 1, parts
            first = sum(p[0] for p in parts[:part])
            assert first < (image + 1) * k and image * k < first + parts[part][0]       # rows of the image that is compared
    assert {(bm, part > 0) for *_, tiles in T.CHOSEN for _, part, bm, _ in tiles} == {(192, False), (192, True), (128, False), (128, True)}


@pytest.mark.parametrize("mode,M,C,bm,bn", [(ATTN_OUT, 4096, 2304, 192, 256), (RESIDUAL, 4096, 2304, 192, 256),
                                            (ATTN_OUT, 4915, 2048, 192, 256), (QKV, 4096, 2304, 256, 256),
                                            (ATTN_OUT, 820, 2304, 128, 64), (ATTN_OUT, 1640, 1024, 128, 64),
                                            (RESIDUAL, 1640, 1024, 128, 128), (ATTN_OUT, 2458, 1024, 128, 128)])
def test_tiles_that_fill_more_of_the_compute_units(plan, mode, M, C, bm, bn):
    """One round of them in place of tiles that leave half of the compute units idle; not in a second round, and a long K that
    is cut stays with the tiles that can be."""
    N, K = {QKV: (3, 1), ATTN_OUT: (1, 1), RESIDUAL: (1, 4)}[mode]
    (part,) = plan(mode, M, N * C, K * C, _part_floats(M, C), fields=7)
    assert part[5:] == (bm, bn)
    assert (part[3] > 1) == (mode == RESIDUAL and bm == 128)


def test_a_forced_height_of_the_alternating_tile(plan):
    for cfg, bm in ((1, 256), (9, 192)):
        (part,) = plan(RESIDUAL, 4096, 2304, 9216, _part_floats(4096, 2304), cfg=cfg, fields=7)
        assert part[1] == cfg and part[5:] == (bm, 256)
        (part,) = plan(RESIDUAL, 600, 1024, 4096, _part_floats(600, 1024), cfg=cfg, ksplit=2, fields=7)
        assert part[3] == (2 if cfg == 1 else 1) and part[5] == bm
    assert plan(RESIDUAL, 600, 1024, 4096, _part_floats(600, 1024), cfg=8, ksplit=2)[0][3] == 1


def test_sizes_of_the_gpu_tests_reach_what_they_test(plan):
    import test_gpu_parity as G
    M, C = 2 * G.TWO_LAUNCHES_K, 768
    assert len(plan(GELU, M, 4 * C, C)) == 2 and len(plan(GELU, M, 4 * C, C, parts=0)) == 1
    (_, cfg, tiles, _), = plan(GELU, 2 * G.MANY_TILES_K, 4 * C, C)
    assert cfg != 7 and tiles > 256
    for M, slices in ((1100, 4), (1400, 4), (3100, 1)):                    # the down projection of C = 1024
        (_, cfg, _, got), = plan(RESIDUAL, M, 1024, 4096, _part_floats(M, 1024))
        assert cfg != 7 and got == slices, (M, cfg, got)
        for forced in (2, 4):
            (_, _, _, got), = plan(RESIDUAL, M, 1024, 4096, _part_floats(M, 1024), ksplit=forced)
            assert got == (forced if forced * M * 1024 <= _part_floats(M, 1024) else 1), (M, forced, got)
    for cfg in (1, 2, 5, 6):                           # forced tiles take few rows away from the few-rows kernels
        assert plan(ATTN_OUT, 260, 1024, 1024, cfg=cfg)[0][1] == cfg
        assert plan(RESIDUAL, 260, 1024, 4096, _part_floats(260, 1024), cfg=cfg, ksplit=2)[0][3] == 2
    assert plan(QKV, 300, 384, 128)[0][1] == 7         # and unforced they go there
