// Building blocks of the entropy-guided token selection (Sec. 3.3, "Dual-Linkage Acceleration", final sentence: the
// lowest-entropy tokens are pruned; Sec. 3.2: the highest-entropy tokens are maintained), written over the number
// of threads of the workgroup that runs them.  Everything is integer work on order-preserving keys:
// the result equals a stable sort (entropy descending, index ascending) bit for bit.
#pragma once
#include "common.h"

namespace select_core {


// 32-bit key whose unsigned order is the required numeric order: NaN lowest, -0 == +0
__device__ __forceinline__ uint32_t sort_key(float h) {
  uint32_t b = __float_as_uint(h);
  if ((b & 0x7fffffffu) > 0x7f800000u) return 0u;       // NaN: below every number
  if (b == 0x80000000u) b = 0u;                         // -0 == +0
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);    // -inf -> 0x007fffff > 0
}

constexpr int kCopies = 32;              // counters per histogram bin: one per LDS bank

// LDS scratch of one workgroup of NT threads
template <int NT>
struct Scratch {
  uint32_t hist[256];
  uint32_t hist_banked[256 * kCopies];   // [bin][copy]: copy = lane % kCopies
  uint32_t wave_sums[NT / NOVA_WAVE];
  uint32_t bin, remaining;
};

// exclusive prefix sum of v over the block's threads, in thread order; total in *total
template <int NT>
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* wave_sums, uint32_t* total) {
  constexpr int kWaves = NT / NOVA_WAVE;
  const int lane = threadIdx.x & (NOVA_WAVE - 1);
  const int wave = threadIdx.x / NOVA_WAVE;
  uint32_t inc = v;
#pragma unroll
  for (int o = 1; o < NOVA_WAVE; o <<= 1) {
    uint32_t t = __shfl_up(inc, o, NOVA_WAVE);
    if (lane >= o) inc += t;
  }
  __syncthreads();                       // wave_sums may still be read from a previous scan
  if (lane == NOVA_WAVE - 1) wave_sums[wave] = inc;
  __syncthreads();
  uint32_t base = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kWaves; ++w) {
    uint32_t s = wave_sums[w];
    if (w < wave) base += s;
    tot += s;
  }
  *total = tot;
  return base + inc - v;
}

// The k-th largest of the N keys key_at(0..N-1), 0 < k < N, by a 4-pass, 8-bit MSB radix select on LDS histograms:
// returns the threshold key; *remaining_out = how many of the keys equal to it are kept (the first ones in index
// order).  Keys of one image share their leading bits, so in the first passes nearly all keys fall into one or two
// bins: a single histogram would serialise its atomics on one address.  Each bin therefore has kCopies counters and a
// lane adds to the counter of its own bank; the counters are summed (and cleared) after the pass.  Called by all NT
// threads of the workgroup.
template <int NT, typename KeyAt>
__device__ __forceinline__ uint32_t radix_select(KeyAt key_at, int N, int k, Scratch<NT>& sc, uint32_t* remaining_out) {
  static_assert(NT % 256 == 0 && NT <= 1024, "the counter sum below gives NT / 256 threads to every bin");
  constexpr int TPB = NT / 256;          // threads per bin in the counter sum
  const int tid = threadIdx.x;
  const int lane = tid & (NOVA_WAVE - 1);
  const int wave = tid / NOVA_WAVE;
  uint32_t prefix = 0, prefix_mask = 0, remaining = (uint32_t)k;
  for (int i = tid; i < 256 * kCopies; i += NT) sc.hist_banked[i] = 0;
  for (int shift = 24; shift >= 0; shift -= 8) {
    __syncthreads();
    for (int i = tid; i < N; i += NT) {
      uint32_t key = key_at(i);
      if ((key & prefix_mask) == prefix)
        atomicAdd(&sc.hist_banked[((key >> shift) & 255u) * kCopies + (lane & (kCopies - 1))], 1u);
    }
    __syncthreads();
    {
      // TPB threads per bin, kCopies / TPB counters each (walked from a bin-dependent start, so that the lanes of a
      // wave touch all banks); the counters are left at zero for the next pass
      constexpr int CPT = kCopies / TPB;
      const int bin = tid / TPB, q = tid % TPB;
      uint32_t s = 0;
#pragma unroll
      for (int j = 0; j < CPT; ++j) {
        const int c = bin * kCopies + q * CPT + ((j + bin) & (CPT - 1));
        s += sc.hist_banked[c];
        sc.hist_banked[c] = 0;
      }
#pragma unroll
      for (int o = 1; o < TPB; o <<= 1) s += __shfl_xor(s, o, NOVA_WAVE);
      if (q == 0) sc.hist[bin] = s;
    }
    __syncthreads();
    if (wave == 0) {
      uint32_t h0 = sc.hist[4 * lane], h1 = sc.hist[4 * lane + 1], h2 = sc.hist[4 * lane + 2], h3 = sc.hist[4 * lane + 3];
      uint32_t s = h0 + h1 + h2 + h3;
      uint32_t suf = s;                        // sum over lanes >= this one (higher bins)
#pragma unroll
      for (int o = 1; o < NOVA_WAVE; o <<= 1) {
        uint32_t t = __shfl_down(suf, o, NOVA_WAVE);
        if (lane + o < NOVA_WAVE) suf += t;
      }
      uint32_t above = suf - s;
      if (above < remaining && remaining <= suf) {       // exactly one lane
        uint32_t r = remaining - above;
        uint32_t bin;
        if (r <= h3) { bin = 3; }
        else { r -= h3; if (r <= h2) { bin = 2; } else { r -= h2; if (r <= h1) { bin = 1; } else { r -= h1; bin = 0; } } }
        sc.bin = 4u * lane + bin;
        sc.remaining = r;
      }
    }
    __syncthreads();
    prefix |= sc.bin << shift;
    prefix_mask |= 255u << shift;
    remaining = sc.remaining;
    // hist and bin / remaining are rewritten only behind further barriers of the next pass
  }
  *remaining_out = remaining;
  return prefix;
}

// Writes the ascending kept-index list and the mask of one image from the selection rule: every key above `thr` is
// kept, of the keys equal to it the first `remaining` in index order; all = keep everything, none = keep nothing.
// Two block-wide prefix sums over contiguous index ranges.  Entries [kept, pitch) of the index row are set to -1.
template <int NT, typename KeyAt>
__device__ __forceinline__ void compact(KeyAt key_at, int N, uint32_t thr, uint32_t remaining, bool all, bool none,
                                        int pitch, int32_t* __restrict__ out_idx, uint8_t* __restrict__ out_mask,
                                        uint32_t* wave_sums) {
  const int tid = threadIdx.x;
  const int ipt = (N + NT - 1) / NT;
  const int i0 = min(tid * ipt, N), i1 = min(i0 + ipt, N);
  uint32_t n_gt = 0, n_eq = 0;
  if (!none) {
    for (int i = i0; i < i1; ++i) {
      uint32_t key = key_at(i);
      n_gt += (all || key > thr);
      n_eq += (!all && key == thr);
    }
  }
  uint32_t tot;
  uint32_t eq_before = block_exclusive_scan<NT>(n_eq, wave_sums, &tot);
  uint32_t eq_take = 0;
  if (eq_before < remaining) eq_take = min(n_eq, remaining - eq_before);
  uint32_t pos = block_exclusive_scan<NT>(n_gt + eq_take, wave_sums, &tot);
  uint32_t eq_seen = eq_before;
  for (int i = i0; i < i1; ++i) {
    bool keep = false;
    if (!none) {
      uint32_t key = key_at(i);
      if (all || key > thr) keep = true;
      else if (key == thr) { keep = eq_seen < remaining; ++eq_seen; }
    }
    out_mask[i] = keep ? 1 : 0;
    if (keep && pos < (uint32_t)pitch) out_idx[pos++] = i;   // pos < k <= pitch by construction
  }
  // unused tail of the row's index list
  for (int i = (int)tot + tid; i < pitch; i += NT) out_idx[i] = -1;
}

// ---- rows whose keys fit the workgroup's registers ------------------------------------------------------------------
// Inclusive prefix sum over the wave's lanes on the DPP paths (shifts inside rows of 16, then the two row broadcasts).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ uint32_t dpp_or_zero(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROW_MASK, 0xF, false);
}
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v) {
  v += dpp_or_zero<0x111, 0xF>(v);          // row_shr:1
  v += dpp_or_zero<0x112, 0xF>(v);          // row_shr:2
  v += dpp_or_zero<0x114, 0xF>(v);          // row_shr:4
  v += dpp_or_zero<0x118, 0xF>(v);          // row_shr:8
  v += dpp_or_zero<0x142, 0xA>(v);          // row_bcast15 into rows 1 and 3
  v += dpp_or_zero<0x143, 0xC>(v);          // row_bcast31 into rows 2 and 3
  return v;
}
__device__ __forceinline__ uint32_t lane_value(uint32_t v, int lane) {      // lane: wave-uniform
  return (uint32_t)__builtin_amdgcn_readlane((int)v, lane);
}

constexpr int kBins = 2048, kBinBits = 11;

template <int NT, int KPT>
struct RowScratch {
  uint32_t hist[kBins];
  uint32_t lo[NT / NOVA_WAVE], hi[NT / NOVA_WAVE], sums[NT / NOVA_WAVE];
  uint32_t counts[KPT * NT / NOVA_WAVE];     // per chunk of NT tokens and wave: keys above | equal << 16
  uint32_t cand[NOVA_WAVE];
  uint32_t n_cand, bin, rank, in_bin, thr, remaining;
};

// The k-th largest, 0 < k < N, of the keys key[u] of tokens u * NT + tid < N; *remaining_out = how many of the keys equal
// to it are kept.  The keys of an image lie close together, so a histogram over leading bits has a few full bins;
// here the 2048 bins divide the range between the smallest and the largest key.  The bin that holds the k-th key has
// a handful of keys as a rule, which one wave ranks; if it has more than 64, its range is divided again (ties: down
// to a single key, at most three times in all).
template <int NT, int KPT>
__device__ __forceinline__ uint32_t range_select(const uint32_t (&key)[KPT], int N, int k, RowScratch<NT, KPT>& sc,
                                                 uint32_t* remaining_out) {
  constexpr int WAVES = NT / NOVA_WAVE, BPT = kBins / NT;
  const int tid = threadIdx.x, lane = tid & (NOVA_WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / NOVA_WAVE);
  uint32_t lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
  for (int u = 0; u < KPT; ++u)
    if (u * NT + tid < N) { lo = min(lo, key[u]); hi = max(hi, key[u]); }
#pragma unroll
  for (int o = 1; o < NOVA_WAVE; o <<= 1) {
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, NOVA_WAVE));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, o, NOVA_WAVE));
  }
  if (lane == 0) { sc.lo[wave] = lo; sc.hi[wave] = hi; }
#pragma unroll
  for (int i = 0; i < BPT; ++i) sc.hist[i * NT + tid] = 0;
  if (tid == 0) sc.n_cand = 0;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < WAVES; ++w) { lo = min(lo, sc.lo[w]); hi = max(hi, sc.hi[w]); }
  uint32_t base = lo, range = hi - lo, rank = (uint32_t)k;
  for (;;) {
    const int sh = max(32 - __clz((int)range) - kBinBits, 0);
    // keys base ... base + range (all of them the first time), 2048 bins of 2^sh keys
#pragma unroll
    for (int u = 0; u < KPT; ++u)
      if (u * NT + tid < N && key[u] - base <= range) atomicAdd(&sc.hist[(key[u] - base) >> sh], 1u);
    __syncthreads();
    // this thread's bins, the highest bins first in thread order; left at zero for the next time round
    uint32_t h[BPT], own = 0;
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
      const int b = kBins - 1 - (tid * BPT + i);
      h[i] = sc.hist[b];
      sc.hist[b] = 0;
      own += h[i];
    }
    const uint32_t inc = wave_inclusive_scan(own);
    if (lane == NOVA_WAVE - 1) sc.sums[wave] = inc;
    __syncthreads();
    uint32_t above = inc - own;
    {
      const uint32_t waves = wave_inclusive_scan(lane < WAVES ? sc.sums[lane] : 0u);
      if (wave > 0) above += lane_value(waves, wave - 1);
    }
    if (above < rank && rank <= above + own) {           // exactly one thread
      uint32_t r = rank - above;
#pragma unroll
      for (int i = 0; i < BPT; ++i) {
        if (r > 0 && r <= h[i]) {
          sc.bin = (uint32_t)(kBins - 1 - (tid * BPT + i));
          sc.rank = r;
          sc.in_bin = h[i];
          r = 0;
        } else if (r > 0) {
          r -= h[i];
        }
      }
    }
    __syncthreads();
    base += sc.bin << sh;
    range = sh > 0 ? (1u << sh) - 1u : 0u;
    rank = sc.rank;
    const uint32_t in_bin = sc.in_bin;
    if (sh == 0) { *remaining_out = rank; return base; }
    if (in_bin <= NOVA_WAVE) break;
  }
#pragma unroll
  for (int u = 0; u < KPT; ++u)
    if (u * NT + tid < N && key[u] - base <= range) sc.cand[atomicAdd(&sc.n_cand, 1u)] = key[u];
  __syncthreads();
  if (wave == 0) {
    const int n = (int)__builtin_amdgcn_readfirstlane(sc.n_cand);
    const uint32_t mine = lane < n ? sc.cand[lane] : 0u;
    uint32_t gt = 0, eq = 0;
    for (int j = 0; j < n; ++j) {
      const uint32_t other = lane_value(mine, j);
      gt += other > mine;
      eq += other == mine;
    }
    if (lane < n && gt < rank && rank <= gt + eq) {      // lanes with the same key write the same
      sc.thr = mine;
      sc.remaining = rank - gt;
    }
  }
  __syncthreads();
  *remaining_out = sc.remaining;
  return sc.thr;
}

// compact() for keys in registers: token u * NT + tid is chunk u, ballots count in front of a lane, and one scan over
// the chunks' and waves' counts of keys above and equal to the threshold gives every kept token its place.
template <int NT, int KPT>
__device__ __forceinline__ void range_compact(const uint32_t (&key)[KPT], int N, uint32_t thr, uint32_t remaining, bool all,
                                              bool none, int pitch, int32_t* __restrict__ out_idx,
                                              uint8_t* __restrict__ out_mask, RowScratch<NT, KPT>& sc) {
  constexpr int WAVES = NT / NOVA_WAVE, E = KPT * WAVES, EPL = (E + NOVA_WAVE - 1) / NOVA_WAVE;
  const int tid = threadIdx.x, lane = tid & (NOVA_WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / NOVA_WAVE);
  uint64_t gtm[KPT], eqm[KPT];
#pragma unroll
  for (int u = 0; u < KPT; ++u) {
    const bool in = u * NT + tid < N && !none;
    gtm[u] = __ballot(in && (all || key[u] > thr));
    eqm[u] = __ballot(in && !all && key[u] == thr);
    if (lane == 0) sc.counts[u * WAVES + wave] = (uint32_t)__popcll(gtm[u]) | (uint32_t)__popcll(eqm[u]) << 16;
  }
  __syncthreads();
  uint32_t c[EPL], own = 0;
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    const int e = lane * EPL + i;
    c[i] = e < E ? sc.counts[e] : 0u;
    own += c[i];
  }
  const uint32_t inc = wave_inclusive_scan(own);
  const uint32_t total = lane_value(inc, NOVA_WAVE - 1);
#pragma unroll
  for (int u = 0; u < KPT; ++u) {
    const int i = u * NT + tid;
    if (u * NT >= N) break;
    const int e = u * WAVES + wave;                      // counts in front of this wave's part of chunk u
    uint32_t before = lane_value(inc - own, e / EPL);
#pragma unroll
    for (int q = 0; q + 1 < EPL; ++q)
      if (q < e % EPL) before += lane_value(c[q], e / EPL);
    const uint64_t below = (1ull << lane) - 1;
    const uint32_t gt_before = (before & 0xFFFFu) + (uint32_t)__popcll(gtm[u] & below);
    const uint32_t eq_before = (before >> 16) + (uint32_t)__popcll(eqm[u] & below);
    const bool keep = (gtm[u] >> lane & 1) || ((eqm[u] >> lane & 1) && eq_before < remaining);
    if (i < N) out_mask[i] = keep ? 1 : 0;
    const uint32_t pos = gt_before + min(eq_before, remaining);
    if (keep && pos < (uint32_t)pitch) out_idx[pos] = i;
  }
  // unused tail of the row's index list
  const int kept = (int)((total & 0xFFFFu) + min(total >> 16, remaining));
  for (int i = kept + tid; i < pitch; i += NT) out_idx[i] = -1;
}

}  // namespace select_core
