// bf16 matrix-core GEMM of the pruned block's four projections (Sec. 3.3, "Residual Cache
// Reuse", first equation: Layer_j on the kept rows):  out = epilogue(A W^T),
// A [M, K] activations, W [Nout, K] weights, both K-contiguous, fp32 accumulation.
//
// gfx950 design:
//  * v_mfma_f32_32x32x16_bf16; a workgroup owns a BM x BN tile, WM x WN waves own
//    (BM/WM) x (BN/WN) sub-tiles, the K loop advances 64 elements (128 bytes per row).
//  * Global -> LDS copies bypass the registers (buffer_load_dwordx4 ... lds): a wave instruction
//    drops 8 rows x 128 bytes straight into LDS.  Because the LDS side of that instruction is
//    lane-linear, the bank-conflict-avoiding XOR swizzle is applied on the global side: the
//    lane that fills 16-byte slot p of row r fetches chunk p ^ ((r >> 1) & 7) of that row, and
//    the MFMA operand reads look the chunk up at the same swizzled slot.
//  * The 256 x 256 tile: two LDS buffers filled and freed in halves, the two waves of a SIMD alternating between the
//    matrix cores and LDS (see the K loop).  Against one ring of K steps for all waves, same box, weights from HBM:
//    4096 x 6912 x 2304 (QKV) 150 -> 124 us, 4096 x 9216 x 2304 (GELU) 225 -> 180, 8192 x 8192 x 8192 968 -> 833
//    (1.14 -> 1.32 PFLOP/s; a large library product on the same card 1.40).
//    192 x 256 alternates in the same way, where it fills the CUs better (gemm_plan.h).
//  * The smaller tiles: an NST-stage LDS ring (3 to 6 stages, per tile configuration): the loads of tiles
//    t+1 .. t+NST-1 are in flight while tile t feeds the MFMAs; one bare barrier per K step with explicit
//    vmcnt / lgkmcnt waits.
//  * What surrounds the K loop is vector instructions at two waves per SIMD, some 4 ns each: the accumulators start from
//    the bias, no epilogue goes through LDS, and no division is left in front of the first load.
//    (That is K / 16 roundings at the bias's magnitude, 2^-28 K |bias| at most: nothing next to the rounding to bf16.)
//  * The projection p is summed apart from the residual r and meets it once, as p + r or fma(gate, p, r), as in the few-rows
//    kernels and the second pass of a K-sliced launch: a zero gate leaves r, and a large r costs p no bits.
//  * Workgroup ids are remapped so that each XCD (ids are dealt round-robin to the 8 XCDs) works
//    on a contiguous run of tiles, ordered in bands of 8 tile rows, so that the tiles in flight on
//    one XCD form a compact rectangle and share A rows and W columns in that XCD's L2.
#include "common.h"
#include "epilogue.h"
#include "gemm_plan.h"
#include "nova_internal.h"

namespace {

typedef const __attribute__((address_space(1))) void* gptr_t;

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// s_waitcnt with only vmcnt = n constrained (gfx9 encoding: vmcnt in bits 3:0 and 15:14)
#define WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(0x0F70 | ((n) & 15) | (((n) >> 4) << 14))

// LDS byte offset of 16-byte chunk `c` of tile row `r`; a row holds 64 elements (128 bytes).
// The XOR term changes with every group of rows that shares a bank window, so that 16 consecutive
// rows reading the same chunk index hit 16 different 16-byte bank groups.
__device__ __forceinline__ int swz(int r, int c) { return r * 128 + ((c ^ ((r >> 1) & 7)) << 4); }

// Whether a workgroup walks several tiles (one workgroup per CU): the modes without a residual (the next tile's would
// have to wait for the registers that this tile's is held in).
constexpr bool persistent_tiles(bool stagger, int mode) {
  return !stagger && (mode == EPI_QKV || mode == EPI_GELU || mode == EPI_GELU_TANH || mode == EPI_PLAIN);
}

// Workgroup id -> tile, with the divisions made on the host: a scalar division is some 30 dependent instructions, and
// everything in front of a workgroup's first load is latency that nothing hides.
struct TileMap {
  int nblk, xcd_base, xcd_rem;             // tiles, tiles per XCD, XCDs with one more
  int band_tiles, full_bands, last_rows;   // tiles per band of 8 tile rows, such bands, rows of the last, lower band
  uint32_t band_inv, last_inv;             // div_inv of band_tiles / last_rows
  int tiles_n, KT;                         // tile columns, K steps per workgroup
};

// GATED (residual modes): the projection is multiplied by ep.gate before the residual is added
// FAR: 64-bit addresses instead of 32-bit offsets into the tile (K > kNearK, and the staggered kernels)
template <int BM, int BN, int WM, int WN, int BK, int NST, bool STAGGER, int MODE, bool GATED, bool FAR = STAGGER>
__global__ __launch_bounds__(WM* WN * 64) void gemm_bf16_kernel(const bf16_t* __restrict__ A,
                                                                const bf16_t* __restrict__ W, int M, int Nout,
                                                                int K, int m_base, TileMap map,
                                                                EpiParams<bf16_t> ep) {
  constexpr int NW = WM * WN;
  constexpr int TM = BM / WM / 32, TN = BN / WN / 32;      // MFMA tiles per wave
  constexpr int ROW_BYTES = BK * 2;
  constexpr int CH = ROW_BYTES / 16;                       // 16-byte chunks per tile row
  constexpr int RPI = 64 / CH;                             // tile rows filled by one wave load instruction
  constexpr int LA = BM / RPI / NW, LB = BN / RPI / NW;    // load instructions per wave per stage
  constexpr int LPW = LA + LB;
  static_assert(BK == 64, "the swizzle is that of 128-byte rows");
  constexpr int KS = BK / 16;                              // MFMA K steps per stage
  constexpr int A_BYTES = BM * ROW_BYTES, B_BYTES = BN * ROW_BYTES, STAGE = A_BYTES + B_BYTES;
  // PP: the two waves of a SIMD alternate between the matrix cores and LDS (see the K loop); PP3: in three phases
  constexpr bool PP3 = BM == 192 && BN == 256 && NST == 2 && WM == 2 && WN == 4;
  constexpr bool PP = PP3 || (BM == 256 && BN == 256 && NST == 2 && WM == 2 && WN == 4);
  constexpr int LDS_BYTES = PP ? 131072 : NST * STAGE;
  static_assert(BM % (RPI * NW) == 0 && BN % (RPI * NW) == 0, "tile rows must split over the waves");
  static_assert((NST - 2) * LPW < 64, "vmcnt is a 6-bit counter");
  __shared__ __attribute__((aligned(1024))) char lds[LDS_BYTES];

  // all arguments in one round trip, not one per branch below that needs some
  asm volatile("" ::"s"(A), "s"(W), "s"(M), "s"(Nout), "s"(K), "s"(m_base), "s"(map.xcd_base), "s"(map.xcd_rem),
               "s"(map.band_tiles), "s"(map.full_bands), "s"(map.last_rows), "s"(map.band_inv), "s"(map.last_inv),
               "s"(map.KT), "s"(ep.bias), "s"(ep.k_rows), "s"(ep.ldo));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: LDS fill addresses stay scalar
  const int wm = wave / WN, wn = wave % WN;

  // ---- workgroup id -> tile, XCD-contiguous, M fastest -------------------------------
  // blockIdx.y: K slice (EPI_PARTIAL only)
  // PERSIST (see persistent_tiles): the grid is one workgroup per CU and a
  // workgroup takes the tiles L, L + gridDim.x, ...; the first K stages of its next tile are requested
  // before the epilogue of the current one, so their latency passes behind the epilogue.
  constexpr bool PERSIST = persistent_tiles(STAGGER, MODE);
  // first tile row / column of MFMA tile i / jn of this wave
  auto row_of = [&](int i) { return PP3 ? i * 64 + wm * 32 : PP ? (i >> 1) * 128 + wm * 64 + (i & 1) * 32 : wm * (BM / WM) + i * 32; };
  auto col_of = [&](int jn) { return PP ? jn * 128 + wn * 32 : wn * (BN / WN) + jn * 32; };
  const int kslice = PERSIST ? 0 : blockIdx.y;
  int L = blockIdx.x;
  // ---- global -> LDS: instruction i of this wave fills tile rows (i * NW + wave) * RPI + lane / CH
  const int lr = lane / CH, lp = lane % CH;
  const bf16_t* ga[FAR ? LA : 1];
  const bf16_t* gb[FAR ? LB : 1];
  const bf16_t *tile_a = nullptr, *tile_w = nullptr;               // the tile's first row / column and the lanes' offsets
  uint32_t oa[LA], ob[LB];
  int tn = 0, m0 = 0, n0 = 0;
  auto set_tile = [&](int Lt) {
    // Lt -> tile, XCD-contiguous (gridDim.x is a multiple of 8 when a workgroup takes several tiles, so all of
    // them have its XCD's residue)
    const int xcd = Lt & 7, j = Lt >> 3;
    const int id = xcd * map.xcd_base + min(xcd, map.xcd_rem) + j;
    // bands of 8 tile rows, column by column inside a band: the workgroups an XCD runs at the same
    // time then cover a compact 8 x (slots / 8) rectangle and share A and W tiles in its L2
    int in_band = 0, tr = 0;
    const int band = div_by(id, map.band_tiles, map.band_inv, in_band);
    tn = div_by(in_band, map.last_rows, map.last_inv, tr);
    const bool full = band < map.full_bands;
    tn = full ? in_band >> 3 : tn;
    const int tm = band * 8 + (full ? in_band & 7 : tr);
    m0 = m_base + tm * BM;                                 // this launch covers rows [m_base, M)
    n0 = tn * BN;
    tile_a = A + (int64_t)m0 * K;
    tile_w = W + (int64_t)n0 * K;
    // byte offset of the chunk of row r that lands in slot lp; rows past the edge re-read the last row
#pragma unroll
    for (int i = 0; i < LA; ++i) {
      const int r = (i * NW + wave) * RPI + lr, c = swz(r, lp) - r * ROW_BYTES;
      if constexpr (FAR) ga[i] = tile_a + (int64_t)min(r, M - 1 - m0) * K + c / 2;
      else oa[i] = (uint32_t)min(r, M - 1 - m0) * (uint32_t)(2 * K) + c;
    }
#pragma unroll
    for (int i = 0; i < LB; ++i) {
      const int r = (i * NW + wave) * RPI + lr, c = swz(r, lp) - r * ROW_BYTES;
      if constexpr (FAR) gb[i] = tile_w + (int64_t)min(r, Nout - 1 - n0) * K + c / 2;
      else ob[i] = (uint32_t)min(r, Nout - 1 - n0) * (uint32_t)(2 * K) + c;
    }
  };
  set_tile(L);
  if (ep.k_rows) {
    // Per-image keep counts: the rows are B segments of ep.k slots and image b fills only the first k_rows[b] of
    // its segment.  A tile none of whose rows is a live slot has nothing to compute (launches with per-image counts
    // give every tile its own workgroup, so leaving here skips exactly this tile).  The whole workgroup leaves
    // together, before the first barrier.
    const int m_hi = min(m0 + BM, M);
    bool live = false;
    for (int b = m0 / ep.k; b * ep.k < m_hi; ++b)
      live = live || max(m0 - b * ep.k, 0) < image_count(ep.k_rows, b, ep.k);
    if (!live) return;
  }
  // Load instructions lo..hi-1 (A first, then W) of the tile at K offset k0 into `stage`.  With an offset per lane and a
  // scalar one for K no vector instruction stands between the matrix instructions (64-bit addresses: two per load, and
  // a wave's MFMAs wait behind them): K = 1024, one round, 128 x 128 tiles 11.7 -> 11.3 us, 192 x 128 14.9 -> 14.0,
  // 256 x 128 17.5 -> 17.1; K = 8192 126.6 -> 123.8, 96.0 -> 93.0, 106.6 -> 104.5.
  auto issue = [&](int stage, int k0, int lo, int hi) {
    char* sa = lds + stage * STAGE;
    char* sb = sa + A_BYTES;
#pragma unroll
    for (int i = 0; i < LA; ++i)
      if (i >= lo && i < hi) {
        char* d = sa + (i * NW + wave) * RPI * ROW_BYTES;
        if constexpr (FAR) __builtin_amdgcn_global_load_lds((gptr_t)(ga[i] + k0), (lptr_t)d, 16, 0, 0);
        else fill_lds(tile_a, d, oa[i], k0 * 2);
      }
#pragma unroll
    for (int i = 0; i < LB; ++i)
      if (LA + i >= lo && LA + i < hi) {
        char* d = sb + (i * NW + wave) * RPI * ROW_BYTES;
        if constexpr (FAR) __builtin_amdgcn_global_load_lds((gptr_t)(gb[i] + k0), (lptr_t)d, 16, 0, 0);
        else fill_lds(tile_w, d, ob[i], k0 * 2);
      }
  };

  f32x16 acc[TM][TN];

  const int KT = map.KT;                                   // K steps of this workgroup's slice
  const int k_begin = kslice * KT * BK;
  // With few rows every tile column is streamed by one workgroup (or a few that share it), and all
  // of them would walk K in step: the same 128-byte slice of every weight row at the same time,
  // rows a power-of-two stride apart, i.e. a handful of memory channels.  Each tile column
  // therefore starts its (cyclic) walk over K at its own offset.
  const int kt_first = STAGGER ? (int)(((int64_t)tn * KT) / map.tiles_n) : 0;
  auto k_of = [&](int t) { const int q = t + kt_first; return k_begin + (q >= KT ? q - KT : q) * BK; };
  // PP: half h of the tile's rows (part h) or columns (part 2 + h) at K step t into LDS buffer buf
  auto pp_fill = [&](int part, int buf, int t) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int j = (part & 1) * 2 + i;
      char* d = lds + (part >> 1) * 65536 + buf * 32768 + (j * NW + wave) * RPI * ROW_BYTES;
      fill_lds(part >> 1 ? tile_w : tile_a, d, part >> 1 ? ob[j] : oa[j], (k_begin + t * BK) * 2);
    }
  };
  // PP3: 64 rows (part 0 ... 2) or all columns (part 3) of the tile at K step t into LDS buffer buf
  auto pp3_fill = [&](int part, int buf, int t) {
#pragma unroll
    for (int j = 0; j < (part == 3 ? 4 : 1); ++j) {
      const int i = part == 3 ? j : part;
      char* d = lds + (part == 3 ? 65536 : 0) + buf * 32768 + (i * NW + wave) * RPI * ROW_BYTES;
      fill_lds(part == 3 ? tile_w : tile_a, d, part == 3 ? ob[i] : oa[i], (k_begin + t * BK) * 2);
    }
  };
  // prologue: NST-1 K stages in flight (PP: one and three quarters, PP3: two but for 64 rows)
  auto prologue_first = [&]() {
    if constexpr (PP3) {
      pp3_fill(3, 0, 0); pp3_fill(0, 0, 0); pp3_fill(1, 0, 0); pp3_fill(2, 0, 0);
    } else if constexpr (PP) {
      pp_fill(0, 0, 0); pp_fill(2, 0, 0); pp_fill(3, 0, 0); pp_fill(1, 0, 0);
    } else {
      issue(0, k_of(0), 0, LPW);
    }
  };
  auto prologue_rest = [&]() {
    if constexpr (PP3) {
      if (KT > 1) { pp3_fill(3, 1, 1); pp3_fill(0, 1, 1); pp3_fill(1, 1, 1); }
    } else if constexpr (PP) {
      if (KT > 1) { pp_fill(0, 1, 1); pp_fill(2, 1, 1); pp_fill(3, 1, 1); }
    } else {
#pragma unroll
      for (int t = 1; t < NST - 1; ++t)
        if (t < KT) issue(t, k_of(t), 0, LPW);
    }
  };

  // ---- bias (what the accumulators start from) and residual row, requested ahead of the tile's second K stage, so that
  // what waits for them does not wait for more than the first stage.  The residual waits in registers for the epilogue;
  // PP has none to spare and requests it there, all but the kept index that its address takes.
  const int half = lane >> 5, r32 = lane & 31;
  constexpr bool HAS_RES = MODE == EPI_ATTN_OUT || MODE == EPI_RESIDUAL;
  constexpr bool HAS_BIAS = MODE != EPI_PARTIAL && MODE != EPI_ENTROPY;
  bf16x4 bvec[HAS_BIAS ? TN : 1][4];         // this lane's bias entries, packed
  auto load_bias = [&]() {
    if constexpr (HAS_BIAS) {
#pragma unroll
      for (int jn = 0; jn < TN; ++jn)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) bvec[jn][g4] = bf16x4{(bf16_t)0.f, (bf16_t)0.f, (bf16_t)0.f, (bf16_t)0.f};
      if (ep.bias) {
#pragma unroll
        for (int jn = 0; jn < TN; ++jn) {
          // 32 columns are all inside or all outside (Nout is a multiple of 64): outside, some that are inside stand in
          const bf16_t* bp = ep.bias + min(n0 + col_of(jn), Nout - 32) + 4 * half;
#pragma unroll
          for (int g4 = 0; g4 < 4; ++g4) bvec[jn][g4] = *reinterpret_cast<const bf16x4*>(bp + 8 * g4);
        }
      }
    }
  };
  // residual row of this lane in MFMA tile row i (rows past the edge: the last one)
  int kept[MODE == EPI_ATTN_OUT ? TM : 1];
  if constexpr (MODE == EPI_ATTN_OUT) {
#pragma unroll
    for (int i = 0; i < TM; ++i) kept[i] = ep.idx[min(m0 + row_of(i) + r32, M - 1)];
  }
  auto res_row = [&](int i) -> const bf16_t* {
    const int row = min(m0 + row_of(i) + r32, M - 1);
    int64_t roff = (int64_t)row * ep.ldo;
    if constexpr (MODE == EPI_ATTN_OUT)
      roff = ((int64_t)ep.image(row) * ep.Ntok + min(max(kept[i], 0), ep.Ntok - 1)) * ep.C;
    return ep.res + roff + n0 + 8 * half;
  };
  // eight features of this lane's row in MFMA tile rows lo .. hi - 1: 16 gp + 8 half .. of a 32-column block
  auto load_res = [&](u32x4* dst, int lo, int hi) {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if (i < lo || i >= hi) continue;
      const bf16_t* rp = res_row(i);
#pragma unroll
      for (int jn = 0; jn < TN; ++jn) {
        const int c = n0 + col_of(jn) < Nout ? col_of(jn) : 0;        // columns past the edge: not used
#pragma unroll
        for (int gp = 0; gp < 2; ++gp) dst[(i * TN + jn) * 2 + gp] = *reinterpret_cast<const u32x4*>(rp + c + 16 * gp);
      }
    }
  };
  u32x4 rs[HAS_RES ? TM * TN * 2 : 1];
  load_bias();
  prologue_first();
  if constexpr (HAS_RES && !PP) load_res(rs, 0, TM);
  prologue_rest();

  const int arow0 = row_of(0) + r32;   // tile row of this lane's A operand in MFMA tile 0
  const int brow0 = col_of(0) + r32;
  // swizzled byte offsets of this lane's operand chunk for the 16-wide K steps of a stage
  int aoff[KS], boff[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    aoff[ks] = swz(arow0, ks * 2 + half);
    boff[ks] = swz(brow0, ks * 2 + half) + (PP ? 65536 : 0);
  }
  // Operand fragments are double buffered in registers and the schedule is pinned with
  // sched_barrier: the LDS reads of K step ks+1 are issued right after the first MFMA of K step
  // ks, so the remaining MFMAs of that step cover their latency.  The reads of the next stage's
  // first K step are issued right after the barrier, under the MFMAs of this stage's last K step.
  bf16x8 a[2][TM], b[2][TN];
  auto read_frags = [&](int buf, int stage, int ks) {
    const char* sa = lds + stage * STAGE;
    const char* sb = sa + A_BYTES;
#pragma unroll
    for (int i = 0; i < TM; ++i) a[buf][i] = *reinterpret_cast<const bf16x8*>(sa + aoff[ks] + i * 32 * ROW_BYTES);
#pragma unroll
    for (int jn = 0; jn < TN; ++jn) b[buf][jn] = *reinterpret_cast<const bf16x8*>(sb + boff[ks] + jn * 32 * ROW_BYTES);
  };
  // MFMAs lo..hi-1 (flattened over the wave's TM x TN tiles) of one K step
  auto mfmas = [&](int buf, int lo, int hi) {
#pragma unroll
    for (int t = 0; t < TM * TN; ++t)
      if (t >= lo && t < hi) acc[t / TN][t % TN] = mfma32(b[buf][t % TN], a[buf][t / TN], acc[t / TN][t % TN]);
  };
  constexpr int LEAD = 1;                   // MFMAs issued before the next K step's LDS reads
  static_assert(KS % 2 == 0, "fragment buffers alternate per K step");

  bool first_tile = true;
  for (;;) {   // tiles of this workgroup (one, unless PERSIST)
  auto bias_of = [&](int jn, int r) {
    if constexpr (MODE == EPI_ENTROPY) {
      const int col = n0 + col_of(jn) + 8 * (r >> 2) + 4 * half + (r & 3);
      return col >= Nout ? -INFINITY : (ep.bias ? (float)ep.bias[col] : 0.0f);   // -inf masks the edge
    } else if constexpr (HAS_BIAS) {
      return (float)bvec[jn][r >> 2][r & 3];
    } else {
      return 0.0f;
    }
  };
#pragma unroll
  for (int jn = 0; jn < TN; ++jn)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float b = bias_of(jn, r);
#pragma unroll
      for (int i = 0; i < TM; ++i) acc[i][jn][r] = b;
    }
  if constexpr (PP) {
    // ---- 256 x 256 tile, K steps of 64, two LDS buffers, each filled and freed in halves of its rows and columns.
    // A wave computes a 64 x 32 quadrant per phase (rows half x columns half), four phases per K step:
    //   phase 1: read rows half 0, columns half 0 | quadrant 00     fill rows half 1 of step t + 1
    //   phase 2: read columns half 1              | quadrant 01     fill rows half 0 of step t + 2
    //   phase 3: read rows half 1                 | quadrant 11     fill columns half 0 of step t + 2
    //   phase 4: nothing to read                  | quadrant 10     fill columns half 1 of step t + 2
    // The waves of the upper row group run one barrier behind those of the lower one, so that of the two waves of a
    // SIMD one issues its MFMAs while the other reads its next fragments.  A part is refilled a phase or more after
    // the last reads of it were waited for in front of a barrier; it is read five phases later at the earliest,
    // with five parts (80 KB of the CU's) still in flight.
    bf16x8 fa[2][4], fb[2][4];
    auto rd_a = [&](int h) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
          fa[i][ks] = *reinterpret_cast<const bf16x8*>(lds + aoff[ks] + h * 16384 + i * 4096);
    };
    auto rd_b = [&](int h) {
#pragma unroll
      for (int ks = 0; ks < 4; ++ks)
        fb[h][ks] = *reinterpret_cast<const bf16x8*>(lds + boff[ks] + h * 16384);
    };
    auto bar = [&]() {
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    };
    // between two barriers: the products of MFMA tiles (i0, j0) and (i1, j1), rows' fragments a0 and a1
    auto products = [&](int i0, int j0, int a0, int i1, int j1, int a1) {
      __builtin_amdgcn_s_waitcnt(0xC07F);     // lgkmcnt(0): the fragments are here, their LDS may be refilled
      bar();
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        acc[i0][j0] = mfma32(fb[j0][ks], fa[a0][ks], acc[i0][j0]);
        acc[i1][j1] = mfma32(fb[j1][ks], fa[a1][ks], acc[i1][j1]);
      }
      __builtin_amdgcn_s_setprio(0);
      bar();
    };
    auto toggle = [&]() {                     // to the other LDS buffer
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) { aoff[ks] ^= 32768; boff[ks] ^= 32768; }
    };
    if constexpr (PP3) {
      // 192 x 256 tile: three phases per K step, 64 rows (32 of them the wave's) x all columns each: eight products a phase as
      // above, and all columns are read in the first.
      //   phase 1: read columns, rows 0 .. 63   fill rows 128 .. 191 of step t + 1
      //   phase 2: read rows 64 .. 127          fill columns and rows 0 .. 63 of step t + 2
      //   phase 3: read rows 128 .. 191         fill rows 64 .. 127 of step t + 2
      // What a phase reads, both wave groups have read in front of the barrier that the next phase's fills come behind; the
      // wait in a phase is for what the next one reads, requested four phases before.
      auto rd = [&](int i) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) fa[0][ks] = *reinterpret_cast<const bf16x8*>(lds + aoff[ks] + i * 8192);
      };
      if (!first_tile) { WAIT_VMCNT(0); } else if (KT > 1) { WAIT_VMCNT(8); } else { WAIT_VMCNT(2); }
      first_tile = false;
      bar();
      if (wm == 1) bar();
      for (int t = 0; t < KT; ++t) {
        const int left = KT - 1 - t, buf = t & 1;   // K steps after this one
        rd(0);
        rd_b(0);
        rd_b(1);
        if (left >= 1) { pp3_fill(2, buf ^ 1, t + 1); WAIT_VMCNT(8); } else { WAIT_VMCNT(1); }
        products(0, 0, 0, 0, 1, 0);
        rd(1);
        if (left >= 2) { pp3_fill(3, buf, t + 2); pp3_fill(0, buf, t + 2); WAIT_VMCNT(12); }
        else if (left == 1) { WAIT_VMCNT(7); }
        else { WAIT_VMCNT(0); }
        products(1, 0, 0, 1, 1, 0);
        rd(2);
        if (left >= 2) { pp3_fill(1, buf, t + 2); WAIT_VMCNT(8); }
        else if (left == 1) { WAIT_VMCNT(2); }
        toggle();
        products(2, 0, 0, 2, 1, 0);
      }
      if (wm == 0) bar();
      if (PERSIST && (KT & 1)) toggle();            // the next tile starts in buffer 0 again
    } else {
    auto quad = [&](int h, int jn) { products(2 * h, jn, 0, 2 * h + 1, jn, 1); };
    if (!first_tile) { WAIT_VMCNT(0); } else if (KT > 1) { WAIT_VMCNT(10); } else { WAIT_VMCNT(4); }
    first_tile = false;
    bar();
    if (wm == 1) bar();
    for (int t = 0; t < KT; ++t) {
      const int left = KT - 1 - t, buf = t & 1;   // K steps after this one
      rd_a(0);
      rd_b(0);
      if (left >= 1) { pp_fill(1, buf ^ 1, t + 1); WAIT_VMCNT(10); } else { WAIT_VMCNT(2); }
      quad(0, 0);
      rd_b(1);
      if (left >= 2) { pp_fill(0, buf, t + 2); WAIT_VMCNT(10); }
      else if (left == 1) { WAIT_VMCNT(8); }
      else { WAIT_VMCNT(0); }
      quad(0, 1);
      rd_a(1);
      if (left >= 2) pp_fill(2, buf, t + 2);
      quad(1, 1);
      if (left >= 2) { pp_fill(3, buf, t + 2); WAIT_VMCNT(10); }
      else if (left == 1) { WAIT_VMCNT(4); }
      toggle();
      quad(1, 0);
    }
    if (wm == 0) bar();
    if (PERSIST && (KT & 1)) toggle();              // the next tile starts in buffer 0 again
    }
  } else {
  // wait for the first K stage.  After a prefetch the epilogue's own loads and stores are in flight as well and
  // the counter does not tell them apart: wait for everything.
  if (first_tile && KT >= NST - 1) { WAIT_VMCNT((NST - 2) * LPW); } else { WAIT_VMCNT(0); }
  first_tile = false;
  __syncthreads();
  int stage = 0, fill = NST - 1;            // stage being computed / stage being refilled
  read_frags(0, 0, 0);
  // A loop body of 0.8 KB that every wave fetches in step: where it lies in the 64-byte lines of the instruction cache moves
  // a launch by up to 4 % and changes with every edit around it (192 x 128 tiles, 3280 x 2048 rows x features, K = 8192:
  // 174.9 us where the compiler happened to put it well, 184.2 where not, 174.7 with its first line aligned; 256 x 128
  // 133.9 / 135.0 / 131.3).  The 256 x 256 tile's loop does not mind.
  asm volatile(".p2align 6");
  for (int kt = 0; kt < KT; ++kt) {
    // the stage refilled now was read during the previous iteration and freed by its barrier
    const bool more = kt + NST - 1 < KT;
    constexpr int LPS = (LPW + KS - 2) / (KS - 1);   // fill instructions issued per K step (all but the last step)
#pragma unroll
    for (int ks = 0; ks < KS - 1; ++ks) {
      mfmas(ks & 1, 0, LEAD);
      __builtin_amdgcn_sched_barrier(0);
      if (more) issue(fill, k_of(kt + NST - 1), ks * LPS, ks + 2 == KS ? LPW : (ks + 1) * LPS);
      read_frags((ks + 1) & 1, stage, ks + 1);
      __builtin_amdgcn_sched_barrier(0);
      mfmas(ks & 1, LEAD, TM * TN);
      __builtin_amdgcn_sched_barrier(0);
    }
    // tile kt+1 must have landed (younger tiles may stay in flight) and this wave's reads of
    // the current stage must be complete before anyone may refill it
    if (more) { WAIT_VMCNT((NST - 2) * LPW); } else { WAIT_VMCNT(0); }
    __builtin_amdgcn_s_waitcnt(0xC07F);     // lgkmcnt(0)
    // a bare barrier: __syncthreads() would add a wait for ALL outstanding loads, i.e. also for the
    // tiles requested for later iterations, and a ring deeper than two stages would gain nothing
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    const int next = stage + 1 == NST ? 0 : stage + 1;
    mfmas((KS - 1) & 1, 0, LEAD);
    __builtin_amdgcn_sched_barrier(0);
    if (kt + 1 < KT) read_frags(0, next, 0);
    __builtin_amdgcn_sched_barrier(0);
    mfmas((KS - 1) & 1, LEAD, TM * TN);
    __builtin_amdgcn_sched_barrier(0);
    stage = next;
    fill = fill + 1 == NST ? 0 : fill + 1;
  }
  }
  if constexpr (MODE == EPI_ENTROPY) {
    // The accumulators (+ bias) are logits that never leave the chip: each lane reduces the columns
    // it holds of a token row to (max, S, T), the two half-waves and then the waves that share the
    // row merge their partials, and one (m, S, T) per row and column tile goes to memory.
    constexpr float kLog2e = 1.4426950408889634f;
    f32x4* lp = reinterpret_cast<f32x4*>(lds);           // [WN][BM]; the stage ring is free after the last barrier
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      float m = -INFINITY;
#pragma unroll
      for (int jn = 0; jn < TN; ++jn)
#pragma unroll
        for (int r = 0; r < 16; ++r) m = fmaxf(m, acc[i][jn][r]);
      float S = 0.0f, T = 0.0f;
      if (m != -INFINITY) {
#pragma unroll
        for (int jn = 0; jn < TN; ++jn)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const float d = fmaxf(acc[i][jn][r] - m, -200.0f);     // e^-200 == 0: masked columns add nothing
            const float e = __builtin_amdgcn_exp2f(d * kLog2e);
            S += e;
            T = fmaf(-d, e, T);
          }
      }
      entropy_merge(m, S, T, __shfl_xor(m, 32, 64), __shfl_xor(S, 32, 64), __shfl_xor(T, 32, 64));
      if (half == 0) lp[wn * BM + row_of(i) + r32] = f32x4{m, S, T, 0.0f};
    }
    __syncthreads();
    for (int row = tid; row < BM; row += NW * 64) {
      const f32x4 a = lp[row];
      float pm = a[0], pS = a[1], pT = a[2];
#pragma unroll
      for (int w = 1; w < WN; ++w) {
        const f32x4 b2 = lp[w * BM + row];
        entropy_merge(pm, pS, pT, b2[0], b2[1], b2[2]);
      }
      if (m0 + row < M) ep.ent_part[(int64_t)tn * M + m0 + row] = f32x4{pm, pS, pT, 0.0f};
    }
    return;
  }
  // The MFMAs ran with the weight rows as the A operand, so a lane owns token l % 32 of each MFMA
  // tile and, per register group r / 4, four consecutive output features.
  if constexpr (MODE == EPI_PARTIAL) {
    float* pp = ep.part + ((int64_t)kslice * (M - m_base) - m_base) * Nout;     // [slice][row - m_base][Nout]
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int row = m0 + row_of(i) + r32;
#pragma unroll
      for (int jn = 0; jn < TN; ++jn)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          const int col = n0 + col_of(jn) + 8 * g4 + 4 * half;
          if (row < M && col < Nout) {
            f32x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = acc[i][jn][g4 * 4 + e];
            *reinterpret_cast<f32x4*>(pp + (int64_t)row * Nout + col) = v;
          }
        }
    }
    return;
  }
  {
    const int em0 = m0, en0 = n0;            // origin of the tile whose accumulators are written out below
    // ---- epilogue, without LDS staging.  A lane owns token l % 32
    // and, per register group g4, four consecutive features (8 g4 + 4 half ..); swapping the upper lanes'
    // group g4 with the lower lanes' group g4 + 1 (v_permlane32_swap) leaves every lane with eight
    // consecutive features of its token: one 16-byte store, and the two halves of the wave cover 32
    // contiguous bytes of each row.  The value columns of the QKV projection (key index minor) need no swap: the
    // lanes of a half wave hold consecutive tokens.
    bool more_tiles = false;
    if constexpr (PERSIST) {
      // Every wave has passed the last barrier of the K loop, nobody reads the ring any more: request the
      // bias and the first stages of this workgroup's next tile now; they land behind the conversion work.
      if (L + (int)gridDim.x < map.nblk) {
        more_tiles = true;
        L += gridDim.x;
        set_tile(L);
        load_bias();
        prologue_first();
        prologue_rest();
      }
    }
    // p -> p + r or fma(gate, p, r) for MFMA tile row i.  The gates, and PP's residual with them, come one tile row
    // ahead (registers for more there are none); PP's residual alone comes whole.
    u32x4 gate[GATED ? TM * TN * 2 : 1];
    auto load_gate = [&](int i) {
      const bf16_t* gr = ep.gate + (int64_t)ep.image(min(em0 + row_of(i) + r32, M - 1)) * ep.gate_pitch + en0 + 8 * half;
#pragma unroll
      for (int jn = 0; jn < TN; ++jn) {
        const int c = en0 + col_of(jn) < Nout ? col_of(jn) : 0;       // columns past the edge: not used
#pragma unroll
        for (int gp = 0; gp < 2; ++gp) gate[(i * TN + jn) * 2 + gp] = *reinterpret_cast<const u32x4*>(gr + c + 16 * gp);
      }
    };
    // eight consecutive features of a row -> the lane's groups 2 gp and 2 gp + 1
    auto spread = [&](const u32x4& v, float (&f)[8]) {
#pragma unroll
      for (int w2 = 0; w2 < 2; ++w2) {
        const auto sw = __builtin_amdgcn_permlane32_swap(v[w2], v[2 + w2], false, false);
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          f[g * 4 + 2 * w2] = __uint_as_float(sw[g] << 16);
          f[g * 4 + 2 * w2 + 1] = __uint_as_float(sw[g] & 0xFFFF0000u);
        }
      }
    };
    auto add_residual = [&](int i) {
      if constexpr (GATED) {
        if (i + 1 < TM) {
          if constexpr (PP) load_res(rs, i + 1, i + 2);
          load_gate(i + 1);
        }
      }
#pragma unroll
      for (int jn = 0; jn < TN; ++jn)
#pragma unroll
        for (int gp = 0; gp < 2; ++gp) {
          float r[8], g[8];
          spread(rs[(i * TN + jn) * 2 + gp], r);
          if constexpr (GATED) spread(gate[(i * TN + jn) * 2 + gp], g);
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float v = acc[i][jn][gp * 8 + e];
            acc[i][jn][gp * 8 + e] = GATED ? fmaf(g[e], v, r[e]) : v + r[e];
          }
        }
    };
    if constexpr (HAS_RES) {
      if constexpr (PP) load_res(rs, 0, GATED ? 1 : TM);
      if constexpr (GATED) load_gate(0);
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int row = em0 + row_of(i) + r32;
      if constexpr (HAS_RES) add_residual(i);
      if (row < M) {
        bf16_t* op = ep.out + (int64_t)row * ep.ldo + (MODE == EPI_QKV ? 0 : en0) + 8 * half;
        int image = 0, pos = 0;
        bool live = true;
        if constexpr (MODE == EPI_QKV) {
          int slot;
          image = ep.image(row, slot);
          live = slot < image_count(ep.k_rows, image, ep.k);         // slots past an image's keep count append nothing
          pos = image_prior(ep.kv_rows, image, ep.P) + slot;
        }
#pragma unroll
        for (int jn = 0; jn < TN; ++jn) {
          if (en0 + col_of(jn) >= Nout) continue;                     // wave-uniform
          bf16_t* dst = op + col_of(jn);
          float qs = MODE == EPI_PLAIN ? ep.q_scale : 1.0f;
          if constexpr (MODE == EPI_QKV) {
            // C and dh are multiples of 64: 32 columns lie in one part and one head
            const int cb = en0 + col_of(jn), part = (cb >= ep.C) + (cb >= 2 * ep.C), cf = cb - part * ep.C;
            const int head = cf >> ep.dh_log2, d = cf & (ep.dh - 1);
            const int64_t bh = (int64_t)image * ep.heads + head;
            if (part == 2) {
              if (live) {
                bf16_t* vp = ep.vc + (bh * ep.dh + d + 4 * half) * ep.cap + pos;
#pragma unroll
                for (int r = 0; r < 16; ++r) vp[(int64_t)(8 * (r >> 2) + (r & 3)) * ep.cap] = (bf16_t)acc[i][jn][r];
              }
              continue;
            }
            if (part == 0) qs = ep.q_scale;
            dst = part == 0 ? op + cf : ep.kc + (bh * ep.cap + pos) * ep.dh + d + 8 * half;
            if (part == 1 && !live) continue;
          }
#pragma unroll
          for (int gp = 0; gp < 2; ++gp) {                            // register groups (2 gp, 2 gp + 1)
            u32x2 lo, hi;                                             // packed bf16 pairs of the two groups
#pragma unroll
            for (int g = 0; g < 2; ++g) {
              bf16x4 o;
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                float v = acc[i][jn][(2 * gp + g) * 4 + e];
                if (MODE == EPI_GELU) v = gelu_erf(v);
                if (MODE == EPI_GELU_TANH) v = gelu_tanh(v);
                if (MODE == EPI_PLAIN || MODE == EPI_QKV) v *= qs;
                o[e] = (bf16_t)v;
              }
              (g == 0 ? lo : hi) = __builtin_bit_cast(u32x2, o);
            }
            u32x4 out16;
#pragma unroll
            for (int w2 = 0; w2 < 2; ++w2) {
              const auto sw = __builtin_amdgcn_permlane32_swap(lo[w2], hi[w2], false, false);
              out16[w2] = sw[0];        // lower lanes: own group 2 gp;       upper lanes: lower partner's group 2 gp + 1
              out16[2 + w2] = sw[1];    // lower lanes: upper partner's 2 gp; upper lanes: own group 2 gp + 1
            }
            *reinterpret_cast<u32x4*>(dst + 16 * gp) = out16;
          }
        }
      }
    }
    if (more_tiles) continue;
    return;
  }
  }
}

template <int BM, int BN, int WM, int WN, int BK, int NST, bool STAGGER, int MODE, bool FAR = STAGGER>
hipError_t launch_cfg(hipStream_t st, const bf16_t* A, const bf16_t* W, int m_base, int M, int Nout, int K,
                      const EpiParams<bf16_t>& ep, int slots, int kslices = 1) {
  const int tiles_m = (M - m_base + BM - 1) / BM, tiles_n = (Nout + BN - 1) / BN;   // rows [m_base, M)
  TileMap map;
  map.nblk = tiles_m * tiles_n;
  map.xcd_base = map.nblk / 8; map.xcd_rem = map.nblk % 8;
  map.band_tiles = 8 * tiles_n; map.band_inv = div_inv(map.band_tiles);
  map.full_bands = tiles_m / 8; map.last_rows = std::max(tiles_m % 8, 1); map.last_inv = div_inv(map.last_rows);
  map.tiles_n = tiles_n; map.KT = K / BK / kslices;
  // the kernel's PERSIST modes walk several tiles per workgroup: one workgroup per CU then (a multiple of 8, so
  // that a workgroup's tiles share its XCD)
  constexpr bool PERSIST = persistent_tiles(STAGGER, MODE);
  int grid = map.nblk;
  // (not with per-image keep counts: a workgroup that finds its tile without a live row leaves at once)
  if (PERSIST && slots > 0 && slots % 8 == 0 && grid > slots && !ep.k_rows) grid = slots;
  if constexpr (MODE == EPI_ATTN_OUT || MODE == EPI_RESIDUAL) {
    if (ep.gate) {
      gemm_bf16_kernel<BM, BN, WM, WN, BK, NST, STAGGER, MODE, true, FAR><<<grid, WM * WN * 64, 0, st>>>(A, W, M, Nout, K, m_base, map, ep);
      return hipGetLastError();
    }
  }
  gemm_bf16_kernel<BM, BN, WM, WN, BK, NST, STAGGER, MODE, false, FAR><<<dim3(grid, kslices), WM * WN * 64, 0, st>>>(
      A, W, M, Nout, K, m_base, map, ep);
  return hipGetLastError();
}

// Second pass of a K-sliced launch (EPI_RESIDUAL): out = residual + gate (sum of the slices + bias) for rows [m_base, M).
// One thread per 8 output features.
__global__ __launch_bounds__(256) void gemm_reduce_kernel(const float* __restrict__ part, int kslices, int m_base,
                                                          int M, int Nout, uint32_t cpr_inv, EpiParams<bf16_t> ep) {
  const int cpr = Nout / 8;
  int c8;
  const int row = m_base + div_by(blockIdx.x * 256 + threadIdx.x, cpr, cpr_inv, c8), col = c8 * 8;
  if (row >= M) return;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < kslices; ++s) {
    const float* p = part + ((int64_t)s * (M - m_base) + row - m_base) * Nout + col;
    const f32x4 a = *reinterpret_cast<const f32x4*>(p), b = *reinterpret_cast<const f32x4*>(p + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) { acc[e] += a[e]; acc[4 + e] += b[e]; }
  }
  bf16x8 bias;
#pragma unroll
  for (int e = 0; e < 8; ++e) bias[e] = (bf16_t)0.f;
  if (ep.bias) bias = *reinterpret_cast<const bf16x8*>(ep.bias + col);
  const bf16x8 r = *reinterpret_cast<const bf16x8*>(ep.res + (int64_t)row * ep.ldo + col);
  bf16x8 o;
  if (ep.gate) {
    const bf16x8 gt = *reinterpret_cast<const bf16x8*>(ep.gate + (int64_t)ep.image(row) * ep.gate_pitch + col);
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (bf16_t)fmaf((float)gt[e], acc[e] + (float)bias[e], (float)r[e]);
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (bf16_t)(acc[e] + (float)bias[e] + (float)r[e]);
  }
  *reinterpret_cast<bf16x8*>(ep.out + (int64_t)row * ep.ldo + col) = o;
}

template <int MODE>
hipError_t launch_part(const nova_ctx* ctx, hipStream_t st, int cfg, const bf16_t* A, const bf16_t* W, int m_base, int M, int Nout,
                       int K, const EpiParams<bf16_t>& ep) {
  const int cus = ctx ? ctx->num_cus : 256, slots = ctx && ctx->gemm_persist == 0 ? 0 : cus;
  if (cfg == kRowsCfg) {
    const RowsPlan plan = gemm_rows_plan(cus, MODE, M - m_base, Nout, K);
    return launch_gemm_rows_bf16(st, plan, MODE, A, W, m_base, M, Nout, K, ep);
  }
  const bool low = low_launch(ctx, cfg, MODE, M - m_base, Nout, K, ep.part ? ep.part_floats : 0);
  if constexpr (MODE == EPI_RESIDUAL) {
    // see k_slices; the scratch buffer holds 4 x rows x C floats, hence Nout == C
    if (cut_in_k(cfg, low) && ep.part && Nout == ep.C && Nout % 8 == 0) {
      const int bm = cfg == 5 ? 128 : cfg == 6 ? 192 : 256, bn = cfg == 1 ? 256 : 128;
      const int tiles = ((M - m_base + bm - 1) / bm) * ((Nout + bn - 1) / bn);
      const int ks = k_slices(cus, MODE, tiles, M - m_base, Nout, K, ep.part_floats, ctx ? ctx->gemm_ksplit : -1);
      if (ks > 1) {
        hipError_t e;
        if (far_tile(K)) e = launch_cfg<256, 128, 4, 2, 64, 3, false, EPI_PARTIAL, true>(st, A, W, m_base, M, Nout, K, ep, 0, ks);
        else if (cfg == 1) e = launch_cfg<256, 256, 2, 4, 64, 2, false, EPI_PARTIAL>(st, A, W, m_base, M, Nout, K, ep, 0, ks);
        else if (cfg == 2) e = launch_cfg<256, 128, 4, 2, 64, 3, false, EPI_PARTIAL>(st, A, W, m_base, M, Nout, K, ep, 0, ks);
        else if (cfg == 6) e = launch_cfg<192, 128, 2, 4, 64, 3, false, EPI_PARTIAL>(st, A, W, m_base, M, Nout, K, ep, 0, ks);
        else e = launch_cfg<128, 128, 2, 4, 64, 3, false, EPI_PARTIAL>(st, A, W, m_base, M, Nout, K, ep, 0, ks);
        if (e != hipSuccess) return e;
        const int64_t nvec = (int64_t)(M - m_base) * (Nout / 8);
        gemm_reduce_kernel<<<(unsigned)((nvec + 255) / 256), 256, 0, st>>>(ep.part, ks, m_base, M, Nout, div_inv(Nout / 8), ep);
        return hipGetLastError();
      }
    }
  }
  if constexpr (MODE == EPI_ENTROPY) {
    if (cfg == 3) return launch_cfg<64, 32, 2, 1, 64, 6, true, MODE>(st, A, W, m_base, M, Nout, K, ep, slots);
    if (cfg == 4) return launch_cfg<128, 32, 4, 1, 64, 4, true, MODE>(st, A, W, m_base, M, Nout, K, ep, slots);
  }
  if (far_tile(K)) {
    // the FFN down projection of a very wide FFN and a prediction head of very wide tokens; K of the other projections is
    // the width itself, and C x C weights of more than 8 TB are in no memory
    if constexpr (MODE == EPI_RESIDUAL || MODE == EPI_ENTROPY)
      return launch_cfg<256, 128, 4, 2, 64, 3, false, MODE, true>(st, A, W, m_base, M, Nout, K, ep, slots);
    else
      return hipErrorInvalidValue;
  }
  if constexpr (MODE != EPI_ENTROPY) {
    if (low) return launch_cfg<192, 256, 2, 4, 64, 2, false, MODE>(st, A, W, m_base, M, Nout, K, ep, slots);
    if (cfg == 8) return launch_cfg<128, 64, 4, 2, 64, 6, false, MODE>(st, A, W, m_base, M, Nout, K, ep, slots);
  }
  switch (cfg) {
    case 1: return launch_cfg<256, 256, 2, 4, 64, 2, false, MODE>(st, A, W, m_base, M, Nout, K, ep, slots);
    case 5:
      if constexpr (MODE != EPI_ENTROPY)
        if (K >= kDeepK) return launch_cfg<128, 128, 2, 4, 64, 4, false, MODE>(st, A, W, m_base, M, Nout, K, ep, slots);
      return launch_cfg<128, 128, 2, 4, 64, 3, false, MODE>(st, A, W, m_base, M, Nout, K, ep, slots);
    case 6: return launch_cfg<192, 128, 2, 4, 64, 3, false, MODE>(st, A, W, m_base, M, Nout, K, ep, slots);
    default: return launch_cfg<256, 128, 4, 2, 64, 3, false, MODE>(st, A, W, m_base, M, Nout, K, ep, slots);
  }
}

template <int MODE>
hipError_t launch_mode(const nova_ctx* ctx, hipStream_t st, const bf16_t* A, const bf16_t* W, int M, int Nout,
                       int K, const EpiParams<bf16_t>& ep, bool norm) {
  if (norm)
    return launch_gemm_rows_bf16(st, gemm_norm_plan(ctx ? ctx->num_cus : 256, MODE, M, Nout, K), MODE, A, W, 0, M, Nout, K, ep, true);
  const Plan p = plan_rows(ctx, MODE, M, Nout, K, ep.part ? ep.part_floats : 0);
  for (int i = 0; i < p.n; ++i) {
    const hipError_t e = launch_part<MODE>(ctx, st, p.cfg[i], A, W, p.m_base[i], p.m_end[i], Nout, K, ep);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace

// Output columns per tile of the configuration launch_gemm_bf16 uses for this shape.
int gemm_bf16_tile_cols(const nova_ctx* ctx, int M, int Nout, int K) {
  switch (pick_cfg(ctx, EPI_ENTROPY, M, Nout, K, 0)) {
    case 1: return 256;
    case 3: case 4: return 32;
    default: return 128;
  }
}

hipError_t launch_gemm_bf16(const nova_ctx* ctx, hipStream_t st, int mode, const void* A, const void* W, int M,
                            int Nout, int K, const EpiParams<bf16_t>& params, bool norm) {
  EpiParams<bf16_t> ep = params;
  ep.k_inv = ep.k > 0 ? div_inv(ep.k) : 0;
  ep.dh_log2 = ep.dh == 128 ? 7 : 6;
  const bf16_t* a = static_cast<const bf16_t*>(A);
  const bf16_t* w = static_cast<const bf16_t*>(W);
  switch (mode) {
    case EPI_QKV: return launch_mode<EPI_QKV>(ctx, st, a, w, M, Nout, K, ep, norm);
    case EPI_ATTN_OUT: return launch_mode<EPI_ATTN_OUT>(ctx, st, a, w, M, Nout, K, ep, norm);
    case EPI_GELU: return launch_mode<EPI_GELU>(ctx, st, a, w, M, Nout, K, ep, norm);
    case EPI_GELU_TANH: return launch_mode<EPI_GELU_TANH>(ctx, st, a, w, M, Nout, K, ep, norm);
    case EPI_PLAIN: return launch_mode<EPI_PLAIN>(ctx, st, a, w, M, Nout, K, ep, norm);
    case EPI_ENTROPY: return launch_mode<EPI_ENTROPY>(ctx, st, a, w, M, Nout, K, ep, norm);
    default: return launch_mode<EPI_RESIDUAL>(ctx, st, a, w, M, Nout, K, ep, norm);
  }
}
