// Attention of few kept queries (the small and middle scales): same operation, layouts and conventions as
// attention_bf16.hip (query rows arrive multiplied by score scale * log2 e; everything is computed transposed, a lane owns
// one query), other division of the work.
//
// The kernel there gives a workgroup 128 queries and walks all keys with a barrier per 64-key tile: right when there are
// thousands of queries, but with few of them the chip is nearly empty and what is left is a serial chain of tiles, one
// memory latency and one barrier each (205 queries, 629 keys, 16 heads: 32 workgroups and 10 tiles in a row).  Here a
// workgroup owns 32 queries of one (image, head) and its NW waves split the KEYS: wave w takes the key tiles w, w + NW, ...
// Every wave has its own K and V tile in LDS, filled by its own global -> LDS loads, so nobody waits for anybody until the
// waves' partial results (reference point, sum, unnormalised output) are merged through LDS at the end.  A tile's K half
// is refilled as soon as its score MFMAs have read it and lands behind softmax and P V; its V half is refilled behind
// P V and lands behind the next scores.  Tiles are 16 KB whatever the head size (64 keys at dh = 64, 32 at dh = 128), so
// that two workgroups of four waves fit a CU.
#include "common.h"
#include "nova_internal.h"

namespace {


#define WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(0x0F70 | ((n) & 15) | (((n) >> 4) << 14))

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// MFMA row i of a 32-key block reads this key, so that a lane ends up holding runs of eight consecutive keys, the
// operand layout of the second MFMA
__device__ __forceinline__ int key_of_mfma_row(int i) {
  const int base = i & 16, t = i & 15;
  return base + 8 * ((t >> 2) & 1) + 4 * (t >> 3) + (t & 3);
}

// byte offset of 16-byte chunk c of row r in a swizzled tile whose rows are ROWB bytes
template <int ROWB>
__device__ __forceinline__ int swz(int r, int c) {
  if (ROWB == 256) return r * 256 + ((c ^ (r & 15)) << 4);
  if (ROWB == 128) return r * 128 + ((c ^ ((r >> 1) & 7)) << 4);
  return r * 64 + ((c ^ ((r >> 2) & 3)) << 4);
}

constexpr int BQ = 32;               // queries per workgroup

template <int DH, int NW>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2))) void attention_few_kernel(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ kc, const bf16_t* __restrict__ vc, int k, int C, int heads,
    int cap, int kv_total_uniform, int nqb, uint32_t nqb_inv, uint32_t heads_inv, bf16_t* __restrict__ out,
    const int32_t* __restrict__ k_rows, const int32_t* __restrict__ kv_rows, int P, int self_keys) {
  constexpr int KT = 4096 / DH;                  // keys per tile
  constexpr int KB = KT / 32;                    // 32-key blocks per tile
  constexpr int KROWB = DH * 2, VROWB = KT * 2;  // bytes per row of the K tile (a key) and of the V tile (a channel)
  constexpr int KSTEPS = DH / 16, DB = DH / 32, KG = KT / 16;
  constexpr int LK = 8, LV = 8;                  // 1 KB load instructions per tile half
  constexpr int TILE = 16384;
  __shared__ __attribute__((aligned(1024))) char lds[NW * TILE];
  __shared__ float part_m[NW][BQ], part_l[NW][BQ];

  // all arguments in one round trip, not one per branch below that needs some
  asm volatile("" ::"s"(q), "s"(kc), "s"(vc), "s"(k), "s"(C), "s"(heads), "s"(cap), "s"(kv_total_uniform), "s"(nqb),
               "s"(nqb_inv), "s"(heads_inv), "s"(out), "s"(k_rows), "s"(kv_rows), "s"(P), "s"(self_keys));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int half = lane >> 5, col = lane & 31;
  // the query blocks of one (image, head) go to one XCD (workgroups are dealt to the 8 XCDs in turn): shared K / V in its L2
  const int n = gridDim.x, xcd = blockIdx.x & 7;
  const int item = xcd * (n >> 3) + min(xcd, n & 7) + (blockIdx.x >> 3);
  int qb, head;
  const int bh = div_by(item, nqb, nqb_inv, qb), b = div_by(bh, heads, heads_inv, head);
  const bf16_t* Kg = kc + (int64_t)bh * cap * DH;          // [cap][DH]
  const bf16_t* Vg = vc + (int64_t)bh * DH * (int64_t)cap; // [DH][cap]
  const int kq = image_count(k_rows, b, k);
  const int kv_total = self_keys && (k_rows || kv_rows) ? image_prior(kv_rows, b, P) + kq : kv_total_uniform;
  const int live = max(min(BQ, kq - qb * BQ), 0);          // live queries of this block
  bf16_t* ob = out + ((int64_t)b * k + qb * BQ) * C + head * DH;
  if (live < BQ)
    // slots past the image's keep count: zeros
    for (int i = tid; i < (min(BQ, k - qb * BQ) - live) * (DH / 8); i += NW * 64)
      *reinterpret_cast<u32x4*>(ob + (int64_t)(live + i / (DH / 8)) * C + i % (DH / 8) * 8) = u32x4{0u, 0u, 0u, 0u};
  if (live == 0) return;                                   // the whole workgroup, before any barrier

  const int ntiles = (kv_total + KT - 1) / KT;
  char* sk = lds + wave * TILE;
  char* sv = sk + TILE / 2;
  // byte offsets of the lanes' 16-byte chunks in load instruction i (rows i * 64 / chunks per row ..): the swizzle repeats
  // after KV_ / VV instructions, the rest of the address is wave-uniform
  constexpr int KC = KROWB / 16, VC = VROWB / 16;          // 16-byte chunks per row
  constexpr int KR = 64 / KC, VR = 64 / VC;                // rows per instruction
  constexpr int KV_ = KROWB == 256 ? 4 : 2, VV = VROWB == 128 ? 2 : 1;
  uint32_t koff[KV_], voff[VV];
  {
    const int kr = lane / KC, kp = lane % KC, vr = lane / VC, vp = lane % VC;
#pragma unroll
    for (int i = 0; i < KV_; ++i) koff[i] = swz<KROWB>(i * KR + kr, kp) - i * KR * KROWB;
#pragma unroll
    for (int i = 0; i < VV; ++i) voff[i] = (uint32_t)vr * (uint32_t)(2 * cap) + (swz<VROWB>(i * VR + vr, vp) - (i * VR + vr) * VROWB);
  }
  auto issue_k = [&](int t) {
    const bf16_t* Kt = Kg + (int64_t)t * KT * DH;
#pragma unroll
    for (int i = 0; i < LK; ++i) fill_lds(Kt, sk + i * 1024, koff[i % KV_], i * KR * KROWB);
  };
  auto issue_v = [&](int t) {
    const bf16_t* Vt = Vg + t * KT;
#pragma unroll
    for (int i = 0; i < LV; ++i) fill_lds(Vt, sv + i * 1024, voff[i % VV], (uint32_t)(i * VR) * (uint32_t)(2 * cap));
  };
  // query fragments first: the first score MFMA needs them together with the first K tile
  bf16x8 qf[KSTEPS];
  {
    const int qrow = min(qb * BQ + col, kq - 1);           // clamped past the last live query; never stored
    const bf16_t* qp = q + ((int64_t)b * k + qrow) * C + head * DH + half * 8;
#pragma unroll
    for (int t = 0; t < KSTEPS; ++t) qf[t] = *reinterpret_cast<const bf16x8*>(qp + t * 16);
  }
  asm volatile("" ::: "memory");
  if (wave < ntiles) { issue_k(wave); issue_v(wave); }

  f32x16 o[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) o[d][r] = 0.f;
  // softmax state per query (= per lane): reference point and this lane's sum against it, in log2 units
  float m_run = -INFINITY, l_run = 0.f;
  const int krow = key_of_mfma_row(col);

  for (int t = wave; t < ntiles; t += NW) {
    const bool more = t + NW < ntiles;
    WAIT_VMCNT(LV);                                        // this tile's K half has landed, its V half may be in flight
    asm volatile("" ::: "memory");
    bf16x8 kf[KB * KSTEPS];
#pragma unroll
    for (int f = 0; f < KB * KSTEPS; ++f)
      kf[f] = *reinterpret_cast<const bf16x8*>(sk + swz<KROWB>(f / KSTEPS * 32 + krow, f % KSTEPS * 2 + half));
    __builtin_amdgcn_sched_barrier(0);
    f32x16 s[KB];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[kb][r] = 0.f;
#pragma unroll
    for (int f = 0; f < KB * KSTEPS; ++f) s[f / KSTEPS] = mfma32(kf[f], qf[f % KSTEPS], s[f / KSTEPS]);
    __builtin_amdgcn_sched_barrier(0);
    if (more) {                                 // every fragment is in registers: the K half can be refilled
      asm volatile("" ::: "memory");
      issue_k(t + NW);
    }

    // register r of block kb is key t KT + kb 32 + 16 (r / 8) + 8 half + r % 8
    if ((t + 1) * KT > kv_total) {
#pragma unroll
      for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (t * KT + kb * 32 + 16 * (r >> 3) + 8 * half + (r & 7) >= kv_total) s[kb][r] = -INFINITY;
    }
    float tmax = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) tmax = fmaxf(tmax, s[kb][r]);
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32, NOVA_WAVE));   // -inf where every score of the tile is
    // the reference moves when some query's maximum lies above it (always on the wave's first tile)
    if (__any(tmax > m_run)) {
      const float m_new = fmaxf(m_run, tmax);
      const float alpha = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
      l_run *= alpha;
#pragma unroll
      for (int d = 0; d < DB; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[d][r] *= alpha;
      m_run = m_new;
    }
    // keys whose scores are all -inf weigh nothing: another wave may hold the finite ones
    const float m_ref = m_run == -INFINITY ? 0.f : m_run;
    bf16x8 p[KG];
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float e = __builtin_amdgcn_exp2f(s[kb][r] - m_ref);
        l_run += e;
        p[kb * 2 + (r >> 3)][r & 7] = (bf16_t)e;
      }

    // the V half has landed, the next tile's K half may be in flight
    if (more) { WAIT_VMCNT(LK); } else { WAIT_VMCNT(0); }
    asm volatile("" ::: "memory");
    bf16x8 vf[KG * DB];
#pragma unroll
    for (int f = 0; f < KG * DB; ++f)
      vf[f] = *reinterpret_cast<const bf16x8*>(sv + swz<VROWB>(f % DB * 32 + col, f / DB * 2 + half));
    __builtin_amdgcn_sched_barrier(0);
    if ((t + 1) * KT > kv_total) {
      // value columns past the last key must be zero (0 * garbage could be NaN)
#pragma unroll
      for (int kg = 0; kg < KG; ++kg) {
        const int valid = kv_total - t * KT - kg * 16 - half * 8;      // of the eight keys of this lane's fragments
        u32x4 keep;
#pragma unroll
        for (int w = 0; w < 4; ++w) keep[w] = valid >= 2 * w + 2 ? 0xffffffffu : valid == 2 * w + 1 ? 0xffffu : 0u;
#pragma unroll
        for (int d = 0; d < DB; ++d)
          vf[kg * DB + d] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, vf[kg * DB + d]) & keep);
      }
    }
#pragma unroll
    for (int f = 0; f < KG * DB; ++f) o[f % DB] = mfma32(vf[f], p[f / DB], o[f % DB]);
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    if (more) issue_v(t + NW);
  }

  // ---- merge of the waves' partial results --------------------------------------------------------------------
  const float l_tot = l_run + __shfl_xor(l_run, 32, NOVA_WAVE);
  if constexpr (NW == 1) {
    // nothing to merge: a lane holds four consecutive channels of its query per register group
    const float inv = 1.0f / l_tot;
    if (col < live) {
#pragma unroll
      for (int d = 0; d < DB; ++d)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          bf16x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = (bf16_t)(o[d][r4 * 4 + e] * inv);
          *reinterpret_cast<bf16x4*>(ob + (int64_t)col * C + d * 32 + r4 * 8 + half * 4) = v;
        }
    }
    return;
  }
  if (half == 0) { part_m[wave][col] = m_run; part_l[wave][col] = l_tot; }
  // [channel / 4][query] of four channels each, in the wave's own tile (nothing of it is in flight or unread any more)
#pragma unroll
  for (int d = 0; d < DB; ++d)
#pragma unroll
    for (int r4 = 0; r4 < 4; ++r4) {
      f32x4 v;
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = o[d][r4 * 4 + e];
      *reinterpret_cast<f32x4*>(sk + ((d * 8 + r4 * 2 + half) * BQ + col) * 16) = v;
    }
  __syncthreads();
#pragma unroll
  for (int i = tid; i < BQ * (DH / 8); i += NW * 64) {
    const int qr = i % BQ, d8 = i / BQ;
    if (qr >= live) continue;
    float m = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) m = fmaxf(m, part_m[w][qr]);
    float l = 0.f;
    f32x4 a0 = {0.f, 0.f, 0.f, 0.f}, a1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float f = __builtin_amdgcn_exp2f(part_m[w][qr] - m);     // a wave without a finite score: reference -inf, weight 0
      l = fmaf(f, part_l[w][qr], l);
      const char* pw = lds + w * TILE + (2 * d8 * BQ + qr) * 16;
      a0 += f * *reinterpret_cast<const f32x4*>(pw);
      a1 += f * *reinterpret_cast<const f32x4*>(pw + BQ * 16);
    }
    const float inv = 1.0f / l;
    bf16x8 r;
#pragma unroll
    for (int e = 0; e < 4; ++e) { r[e] = (bf16_t)(a0[e] * inv); r[4 + e] = (bf16_t)(a1[e] * inv); }
    *reinterpret_cast<bf16x8*>(ob + (int64_t)qr * C + d8 * 8) = r;
  }
}

}  // namespace

// Waves per workgroup (0: attention_bf16.hip is faster).  `slots` = CUs.
//  * One workgroup per CU at most: eight waves once there are more than four tiles to split, four otherwise.  Past 12 tiles
//    per wave the other kernel's key runs over several workgroups win (100 queries, dh = 128, 16 heads, K / V from HBM:
//    1600 keys 18.9 us there, 15.9 here; 3100 keys 25.9 / 25.5; 6100 keys 39.4 / 44.6).
//  * Up to two workgroups per CU: four waves, and only if that is at most three tiles each (102 queries of 8 images, 526
//    keys, dh = 64: 10.8 / 9.9 us; 400 of two images, 921 keys, dh = 128: 21.2 / 27.7): every workgroup fetches all keys
//    of its head for 32 queries, four times the traffic of the 128-query workgroups.
//  Measured (us, there / here): 16 heads of 64, one image: 64 queries, 155 keys 6.0 / 4.4; 135, 390 9.2 / 5.7;
//  205, 629 10.7 / 6.7; 8 images, 64 queries, 155 keys 6.1 / 4.6; dh = 128, 2 images, 256 queries, 521 keys 16.0 / 10.0.
int attention_few_waves(int slots, int dh, int B, int k, int heads, int kv_total) {
  const int64_t grid = (int64_t)B * heads * ((k + BQ - 1) / BQ);
  const int tiles = (kv_total + 4096 / dh - 1) / (4096 / dh);
  if (grid <= slots && tiles <= 8 * 12) return tiles > 4 ? 8 : tiles > 1 ? 4 : 1;
  return grid <= 2 * slots && tiles <= 4 * 3 ? 4 : 0;
}

hipError_t launch_attention_few_bf16(hipStream_t st, int waves, const void* q, const void* kc, const void* vc, int B, int k,
                                     int C, int heads, int cap, int kv_total, void* out, const int32_t* k_rows,
                                     const int32_t* kv_rows, int P, int self_keys) {
  const int nqb = (k + BQ - 1) / BQ, grid = nqb * heads * B;
  const bf16_t *qt = static_cast<const bf16_t*>(q), *kt = static_cast<const bf16_t*>(kc), *vt = static_cast<const bf16_t*>(vc);
  bf16_t* ot = static_cast<bf16_t*>(out);
#define GO(DH_, NW_)                                                                                                  \
  attention_few_kernel<DH_, NW_><<<grid, NW_ * 64, 0, st>>>(qt, kt, vt, k, C, heads, cap, kv_total, nqb, div_inv(nqb), \
                                                            div_inv(heads), ot, k_rows, kv_rows, P, self_keys)
  if (C / heads == 64) { if (waves == 8) GO(64, 8); else if (waves == 4) GO(64, 4); else GO(64, 1); }
  else { if (waves == 8) GO(128, 8); else if (waves == 4) GO(128, 4); else GO(128, 1); }
#undef GO
  return hipGetLastError();
}
