// out = epilogue(A W^T) for few rows (the projections of the early, small scales and of row remainders): the weights
// are read once and everything else is latency.
//
// The floor of such a projection is its weight stream, 2 Nout K bytes (0.4 ... 6.5 us at the rate of a large copy), plus
// the launch (1.6 us inside a graph).  A kernel that walks K step by step through an LDS ring shared by the workgroup,
// with a barrier per step and 20 KB in flight, takes 8 ... 17 us whatever the size.  Here:
//  * The KW waves of a workgroup share one output tile (8 RG rows x 8 NG features) and split K among themselves: wave w
//    takes the runs ("units") of 64 elements w, w + KW, ...  The narrow tile gives every projection enough workgroups
//    to stream its weights from all over the chip, and no wave waits for another one until the end, when the partial
//    sums meet once in LDS and are added in a fixed order.
//  * A wave keeps S units in flight in an LDS ring of its own (global -> LDS loads of eight rows x 128 bytes, so that
//    the eight lanes of a row ask for one line; operands loaded straight into the MFMA's register layout, 16 rows per
//    16 lanes, cost one line look-up per lane: measured 1.3x slower with one row, 2x with 64).  No barrier: the wave
//    waits for its own loads only.
//  * What surrounds the K walk is one lone wave per SIMD, some 5 cycles an instruction: no division (two of 64 bits to
//    divide K over slices were 0.4 us of every launch), the arguments in one round trip, loads whose addresses are one
//    lane offset and a scalar, no accumulation registers to move out of.
//  * The epilogue works on eight consecutive features of one row per thread, rows fastest, so that value-cache
//    columns (key index minor) are written in runs of rows; its bias and residual are requested before the K walk.
//  * In tiles of 8 or 16 rows, K of 256 ... 2560 and at most 32 rows (gemm_norm_plan), a projection behind a LayerNorm without
//    modulation takes it along (NORM): the norm's own launch is 2.8 us of which half is starting and ending, and its rows are
//    a latency that the weights' covers (a block of one / eight rows of 1024 in a graph 22.4 / 23.4 -> 19.6 / 19.9 us).
// Measured in a graph, weights from HBM (us; with the divisions and 64-row tiles whatever the width / now / a stream of the
// same bytes): K = 1024, Nout = 1024 / 3072 / 4096, one row 3.1 / 4.2 / 4.5 -> 2.7 / 3.6 / 3.9 (- / 2.9 / 3.3), 64 rows
// 4.3 / 5.9 / 6.1 -> 3.0 / 4.9 / 5.1; K = 4096, Nout = 1024, one row 4.8 -> 4.4, 64 rows 9.3 -> 6.7.
#include <type_traits>

#include "common.h"
#include "epilogue.h"
#include "gemm_plan.h"
#include "nova_internal.h"

namespace {

#define WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(0x0F70 | ((n) & 15) | (((n) >> 4) << 14))

// s_waitcnt vmcnt(younger * LPU) for a wave-uniform younger in 0 .. MAXJ
template <int MAXJ, int LPU>
__device__ __forceinline__ void wait_younger(int younger) {
  if constexpr (MAXJ == 0) {
    WAIT_VMCNT(0);
  } else {
    if (younger == MAXJ) { WAIT_VMCNT(MAXJ * LPU); } else { wait_younger<MAXJ - 1, LPU>(younger); }
  }
}

typedef float f32x4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x4v mfma16(bf16x8 a, bf16x8 b, f32x4v c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// LDS of a kernel: of a fixed size, or with the rows of A in front, as long as K has it
template <bool DYNAMIC, int BYTES>
__device__ __forceinline__ char* rows_lds() {
  if constexpr (DYNAMIC) {
    extern __shared__ __attribute__((aligned(1024))) char dyn[];
    return dyn;
  } else {
    __shared__ __attribute__((aligned(1024))) char fixed[BYTES];
    return fixed;
  }
}

// RG, NG: groups of eight rows / features of a tile (an MFMA tile is 16 x 16: with an odd count its other half is
// whatever lies in LDS behind and is never used); KW: waves; S: units in flight per wave.
// NORM: A's rows are gathered and normalised here (see normalise), then lie in LDS whole, and the waves' rings hold
// weights only.
template <int RG, int NG, int KW, int S, int MODE, bool NORM>
__global__ __launch_bounds__(KW* 64) __attribute__((amdgpu_waves_per_eu(!NORM && KW * S * (NG + RG) <= 79 ? 2 : 1))) void gemm_rows_kernel(
    const bf16_t* __restrict__ A, const bf16_t* __restrict__ W, int M, int Nout, int K, int m_base, EpiParams<bf16_t> ep) {
  constexpr int MT = (RG + 1) / 2, NF = (NG + 1) / 2;
  constexpr int ROWS = MT * 16, LROWS = RG * 8, COLS = NG * 8, NT = KW * 64;
  constexpr int COL8 = COLS / 8;                         // eight-feature groups per row: one thread each in the epilogue
  constexpr int LPU = NORM ? NG : NG + RG;               // 1 KB load instructions per unit
  constexpr int SLOT = LPU * 1024;                       // rows 8 .. 15 of an odd group count are whatever follows: never used
  constexpr int NO = (ROWS * COL8 + NT - 1) / NT;        // of which a thread takes this many
  static_assert(S * LPU < 64, "vmcnt is a 6-bit counter");
  static_assert(S * SLOT >= ROWS * NF * 16 * 4, "a wave's partial sums take the place of its ring");
  char* const a_lds = rows_lds<NORM, KW * S * SLOT + 1024>();
  char* const lds = a_lds + (NORM ? RG * 16 * K : 0);

  // all arguments in one round trip, not one per branch below that needs some
  asm volatile("" ::"s"(A), "s"(W), "s"(M), "s"(Nout), "s"(K), "s"(m_base), "s"(ep.bias), "s"(ep.out),
               "s"(ep.ldo), "s"(ep.k), "s"(ep.k_inv), "s"(ep.k_rows), "s"(ep.res), "s"(ep.idx), "s"(ep.Ntok), "s"(ep.gate));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n0 = blockIdx.x * COLS, m0 = m_base + blockIdx.y * LROWS;
  auto advance_kv = [&]() {
    // per-image cache lengths after this block: prior rows + kept rows (the up-projection: everything that reads the old
    // lengths has run, so the output may be the input array)
    if (!NORM || !ep.kv_next || blockIdx.x != 0 || blockIdx.y != 0) return;
    for (int b = tid; b * ep.k < M; b += NT) ep.kv_next[b] = image_prior(ep.kv_rows, b, ep.P) + image_count(ep.k_rows, b, ep.k);
  };
  if (ep.k_rows) {
    // per-image keep counts: a tile without a live row has nothing to compute (the whole workgroup leaves together)
    const int m_hi = min(m0 + LROWS, M);
    bool live = false;
    for (int b = ep.image(m0); b * ep.k < m_hi; ++b)
      live = live || max(m0 - b * ep.k, 0) < image_count(ep.k_rows, b, ep.k);
    if (!live) {
      advance_kv();
      return;
    }
  }

  // ---- fills: instruction j of a unit drops 8 rows x 128 bytes into LDS; slot p of row r holds chunk p ^ ((r >> 1) & 7)
  const int n_units = (K / 64 - wave + KW - 1) / KW;     // runs of 64 elements of this wave: wave, wave + KW, ...
  const int lr = lane >> 3, lp = lane & 7;
  const bf16_t* Ab = A + (int64_t)m0 * K;
  const bf16_t* Wb = W + (int64_t)n0 * K;
  // byte offsets from the tile's first row (32 bits: gemm_rows_plan keeps K that short); rows past the last one re-read it
  uint32_t ow[2], oa[RG];
#pragma unroll
  for (int j = 0; j < 2; ++j) ow[j] = (uint32_t)lr * (uint32_t)(2 * K) + ((lp ^ (lr >> 1) ^ (j * 4)) << 4);
#pragma unroll
  for (int j = 0; j < RG; ++j) {
    const int r = j * 8 + lr;
    oa[j] = (uint32_t)min(r, M - 1 - m0) * (uint32_t)(2 * K) + ((lp ^ ((r >> 1) & 7)) << 4);
  }
  char* mine_lds = lds + wave * (S * SLOT);
  auto issue_at = [&](int slot, int i) {
    char* d = mine_lds + slot * SLOT;
    const uint32_t k0 = (uint32_t)(wave + i * KW) * 128;
#pragma unroll
    for (int j = 0; j < NG; ++j) fill_lds(Wb, d + j * 1024, ow[j & 1], k0 + (uint32_t)(j * 16 * K));
    if constexpr (!NORM) {
#pragma unroll
      for (int j = 0; j < RG; ++j) fill_lds(Ab, d + (NG + j) * 1024, oa[j], k0);
    }
  };
  // ---- NORM: wave w takes rows w, w + KW, ... of the tile, a row per wave as in norm.hip and with its sums in the same
  // order, so that the bits are those of its output.  The rows are requested in front of the weights, whose latency then
  // covers the sums.  NU: 512 elements a time per row, the last ones perhaps fewer.
  auto normalise = [&](auto nu_tag) {
    constexpr int NU = decltype(nu_tag)::value, NR = LROWS / KW;
    constexpr bool GATHER = MODE == EPI_QKV;
    const bool last = ((NU - 1) * 64 + lane) * 8 < K;    // whether this lane has elements in the last vector of a row
    int m[NR], image[NR], slot[NR], token[NR], count[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      m[i] = min(m0 + wave + i * KW, M - 1);             // rows past the last one: the last one, never stored
      image[i] = ep.image(m[i], slot[i]);
      count[i] = ep.k;
    }
    if (ep.k_rows) {
#pragma unroll
      for (int i = 0; i < NR; ++i) count[i] = image_count(ep.k_rows, image[i], ep.k);
    }
    if constexpr (GATHER) {
#pragma unroll
      for (int i = 0; i < NR; ++i) token[i] = ep.idx[m[i]];
    }
    bf16x8 x[NR][NU];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int64_t row = GATHER ? (int64_t)image[i] * ep.Ntok + min(max(token[i], 0), ep.Ntok - 1) : m[i];
#pragma unroll
      for (int u = 0; u < NU; ++u)
        x[i][u] = *reinterpret_cast<const bf16x8*>(A + row * K + (u + 1 < NU ? u * 64 + lane : norm_vector(u, lane, K)) * 8);
    }
    // the weights behind the rows, gathered ones too (in front of them: 0.6 us slower), and without branches, so that the
    // wait for the rows is not one for everything: with few units the last one comes twice
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < S; ++i) issue_at(i, min(i, n_units - 1));
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    float mean[NR], rstd[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      float sum = 0.f;
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int e = 0; e < 8; ++e) sum += u + 1 < NU || last ? (float)x[i][u][e] : 0.f;
      mean[i] = wave_sum(sum) / (float)K;
    }
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      float sq = 0.f;
#pragma unroll
      for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float d = u + 1 < NU || last ? (float)x[i][u][e] - mean[i] : 0.f;
          sq = fmaf(d, d, sq);
        }
      rstd[i] = 1.0f / sqrtf(wave_sum(sq) / (float)K + kNormEps);
    }
#pragma unroll
    for (int i = 0; i < NR; ++i) {
      const int r = wave + i * KW;
#pragma unroll
      for (int u = 0; u < NU; ++u) {
        const int c = u * 64 + lane;                     // chunk of eight elements: unit c / 8, slot as the fills have it
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (bf16_t)(((float)x[i][u][e] - mean[i]) * rstd[i]);
        if (slot[i] >= count[i]) {                       // a slot past its image's keep count: zeros
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = (bf16_t)0.f;
        }
        if (u + 1 < NU || last)
          *reinterpret_cast<bf16x8*>(a_lds + (c >> 3) * (RG * 1024) + r * 128 + (((c & 7) ^ ((r >> 1) & 7)) << 4)) = o;
      }
    }
    __builtin_amdgcn_s_waitcnt(0xC07F);                  // lgkmcnt(0), and a bare barrier: the weights stay in flight
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  static_assert(!NORM || LROWS % KW == 0, "rows split over the waves");
  auto issue = [&](int i) { issue_at(i % S, i); };
  // This thread's outputs: row m0 + o % ROWS, features n0 + 8 (o / ROWS) .. for o = tid, tid + NT, ...  Their bias,
  // residual and gate are requested behind the first units; only the gathered residual's index, which its address
  // waits for, goes ahead of them.  (vmcnt counts in order: the waits below are then for a few loads more than needed.)
  constexpr bool HAS_RES = MODE == EPI_ATTN_OUT || MODE == EPI_RESIDUAL;
  auto has_output = [&](int o) { return o < ROWS * COL8 && o % ROWS < LROWS && m0 + o % ROWS < M; };
  bf16x8 bias[NO], res[HAS_RES ? NO : 1], gate[HAS_RES ? NO : 1];
  int src[NO];
#pragma unroll
  for (int q = 0; q < NO; ++q) {
    const int o = tid + q * NT;
    src[q] = MODE == EPI_ATTN_OUT && has_output(o) ? ep.idx[m0 + o % ROWS] : 0;
  }
  asm volatile("" ::: "memory");
#pragma unroll
  for (int i = 0; i < S; ++i)
    if (!NORM && i < n_units) issue(i);
  if constexpr (NORM) {
    switch ((K + 511) / 512) {
      case 1: normalise(std::integral_constant<int, 1>{}); break;
      case 2: normalise(std::integral_constant<int, 2>{}); break;
      case 3: normalise(std::integral_constant<int, 3>{}); break;
      case 4: normalise(std::integral_constant<int, 4>{}); break;
      default: normalise(std::integral_constant<int, kNormMaxK / 512>{}); break;
    }
    advance_kv();
  }
  asm volatile("" ::: "memory");
#pragma unroll
  for (int q = 0; q < NO; ++q) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      bias[q][e] = (bf16_t)0.f;
      if (HAS_RES) { res[q][e] = (bf16_t)0.f; gate[q][e] = (bf16_t)1.f; }
    }
    const int o = tid + q * NT, row = m0 + o % ROWS, col = n0 + o / ROWS * 8;
    if (!has_output(o)) continue;
    if (ep.bias) bias[q] = *reinterpret_cast<const bf16x8*>(ep.bias + col);
    if constexpr (HAS_RES) {
      int64_t roff = (int64_t)row * ep.ldo;
      if (MODE == EPI_ATTN_OUT) roff = ((int64_t)ep.image(row) * ep.Ntok + min(max(src[q], 0), ep.Ntok - 1)) * ep.C;
      res[q] = *reinterpret_cast<const bf16x8*>(ep.res + roff + col);
      if (ep.gate) gate[q] = *reinterpret_cast<const bf16x8*>(ep.gate + (int64_t)ep.image(row) * ep.gate_pitch + col);
    }
  }
  asm volatile("" ::: "memory");

  const int r16 = lane & 15, kg = lane >> 4;
  int off[2];                                            // byte offset of this lane's chunk of K step s in a 16-row tile
#pragma unroll
  for (int s = 0; s < 2; ++s) off[s] = r16 * 128 + (((s * 4 + kg) ^ ((r16 >> 1) & 7)) << 4);
  f32x4v acc[MT][NF];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int f = 0; f < NF; ++f) acc[i][f] = f32x4v{0.f, 0.f, 0.f, 0.f};

  for (int i = 0; i < n_units; ++i) {
    // unit i has landed once at most the younger ones are in flight
    const int younger = min(n_units - 1 - i, S - 1);
    wait_younger<S - 1, LPU>(younger);
    asm volatile("" ::: "memory");
    const char* d = mine_lds + (i % S) * SLOT;
    bf16x8 wf[2][NF], af[2][MT];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
#pragma unroll
      for (int f = 0; f < NF; ++f) wf[s][f] = *reinterpret_cast<const bf16x8*>(d + f * 2048 + off[s]);
#pragma unroll
      for (int t = 0; t < MT; ++t)
        af[s][t] = *reinterpret_cast<const bf16x8*>((NORM ? a_lds + (wave + i * KW) * (RG * 1024) : d + NG * 1024) + t * 2048 + off[s]);
    }
    if (i + S < n_units) {
      __builtin_amdgcn_s_waitcnt(0xC07F);                // lgkmcnt(0): the slot has been read
      asm volatile("" ::: "memory");
      issue(i + S);
    }
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int f = 0; f < NF; ++f) acc[t][f] = mfma16(wf[s][f], af[s][t], acc[t][f]);
  }

  // a lane holds features 4 kg .. 4 kg + 3 of row l % 16 of every tile
#pragma unroll
  for (int t = 0; t < MT; ++t)
#pragma unroll
    for (int f = 0; f < NF; ++f) *reinterpret_cast<f32x4v*>(mine_lds + ((f * 4 + kg) * ROWS + t * 16 + r16) * 16) = acc[t][f];
  __syncthreads();
#pragma unroll
  for (int q = 0; q < NO; ++q) {
    const int o = tid + q * NT, row = m0 + o % ROWS, col = n0 + o / ROWS * 8;
    if (!has_output(o)) continue;
    float v[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < KW; ++w) {
      const char* p = lds + w * (S * SLOT) + (2 * (o / ROWS) * ROWS + o % ROWS) * 16;
      const f32x4v a = *reinterpret_cast<const f32x4v*>(p), b = *reinterpret_cast<const f32x4v*>(p + ROWS * 16);
#pragma unroll
      for (int e = 0; e < 4; ++e) { v[e] += a[e]; v[4 + e] += b[e]; }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] += (float)bias[q][e];
    bf16x8 y;
    if constexpr (MODE == EPI_QKV) {
      const int sel = (col >= ep.C) + (col >= 2 * ep.C), cf = col - sel * ep.C;   // C is a multiple of 64: eight features lie in one part and head
      const float qs = sel == 0 ? ep.q_scale : 1.0f;
#pragma unroll
      for (int e = 0; e < 8; ++e) y[e] = (bf16_t)(v[e] * qs);
      if (sel == 0) {
        *reinterpret_cast<bf16x8*>(ep.out + (int64_t)row * ep.ldo + cf) = y;
        continue;
      }
      int s;
      const int b = ep.image(row, s);
      if (s >= image_count(ep.k_rows, b, ep.k)) continue;  // slots past an image's keep count append nothing
      const int head = cf >> ep.dh_log2, d = cf & (ep.dh - 1);
      const int64_t bh = (int64_t)b * ep.heads + head;
      const int pos = image_prior(ep.kv_rows, b, ep.P) + s;
      if (sel == 1) {
        *reinterpret_cast<bf16x8*>(ep.kc + (bh * ep.cap + pos) * ep.dh + d) = y;
      } else {
        bf16_t* vp = ep.vc + (bh * ep.dh + d) * ep.cap + pos;
#pragma unroll
        for (int e = 0; e < 8; ++e) vp[(int64_t)e * ep.cap] = y[e];
      }
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if (MODE == EPI_GELU) v[e] = gelu_erf(v[e]);
        if (MODE == EPI_GELU_TANH) v[e] = gelu_tanh(v[e]);
        if (MODE == EPI_PLAIN) v[e] *= ep.q_scale;
        y[e] = (bf16_t)v[e];
      }
      if constexpr (HAS_RES) {
        if (ep.gate) {
#pragma unroll
          for (int e = 0; e < 8; ++e) y[e] = (bf16_t)fmaf((float)gate[q][e], v[e], (float)res[q][e]);
        } else {
#pragma unroll
          for (int e = 0; e < 8; ++e) y[e] = (bf16_t)(v[e] + (float)res[q][e]);
        }
      }
      *reinterpret_cast<bf16x8*>(ep.out + (int64_t)row * ep.ldo + col) = y;
    }
  }
}

template <int RG, int NG, int KW, int S, int MODE, bool NORM>
hipError_t go(hipStream_t st, const bf16_t* A, const bf16_t* W, int m_base, int M, int Nout, int K,
              const EpiParams<bf16_t>& ep) {
  const dim3 grid(Nout / (NG * 8), (M - m_base + RG * 8 - 1) / (RG * 8));
  const size_t lds = NORM ? gemm_norm_lds({RG, NG, KW, S}, K) : 0;
  gemm_rows_kernel<RG, NG, KW, S, MODE, NORM><<<grid, KW * 64, lds, st>>>(A, W, M, Nout, K, m_base, ep);
  return hipGetLastError();
}

template <int MODE>
hipError_t by_plan(hipStream_t st, const RowsPlan& p, const bf16_t* A, const bf16_t* W, int m_base, int M, int Nout, int K,
                   const EpiParams<bf16_t>& ep, bool norm) {
  constexpr bool TAKES_NORM = MODE == EPI_QKV || MODE == EPI_GELU || MODE == EPI_GELU_TANH || MODE == EPI_PLAIN;
#define GO(RG, NG, KW, S, FIT)                                                                                       \
  if (p.rg == RG && p.ng == NG && p.kw == KW && p.s == S) {                                                          \
    if constexpr (TAKES_NORM && RG <= kNormMaxGroups && RG * NG > 1)                                                 \
      if (norm) return go<RG, NG, KW, S, MODE, true>(st, A, W, m_base, M, Nout, K, ep);                              \
    return norm ? hipErrorInvalidValue : go<RG, NG, KW, S, MODE, false>(st, A, W, m_base, M, Nout, K, ep);           \
  }
  NOVA_ROWS_TILES(GO)
#undef GO
  return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_gemm_rows_bf16(hipStream_t st, const RowsPlan& p, int mode, const bf16_t* A, const bf16_t* W, int m_base,
                                 int M, int Nout, int K, const EpiParams<bf16_t>& ep, bool norm) {
  switch (mode) {
    case EPI_QKV: return by_plan<EPI_QKV>(st, p, A, W, m_base, M, Nout, K, ep, norm);
    case EPI_ATTN_OUT: return by_plan<EPI_ATTN_OUT>(st, p, A, W, m_base, M, Nout, K, ep, norm);
    case EPI_GELU: return by_plan<EPI_GELU>(st, p, A, W, m_base, M, Nout, K, ep, norm);
    case EPI_GELU_TANH: return by_plan<EPI_GELU_TANH>(st, p, A, W, m_base, M, Nout, K, ep, norm);
    case EPI_PLAIN: return by_plan<EPI_PLAIN>(st, p, A, W, m_base, M, Nout, K, ep, norm);
    case EPI_RESIDUAL: return by_plan<EPI_RESIDUAL>(st, p, A, W, m_base, M, Nout, K, ep, norm);
    default: return hipErrorInvalidValue;
  }
}
