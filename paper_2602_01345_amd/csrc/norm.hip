// Row gather + LayerNorm (no affine, biased variance, eps 1e-6) feeding the block's
// two projections; optionally modulated per image, LN(x) (1 + scale[b]) + shift[b].  One wave64 per row; mean and
// variance are two separate fp32 passes over the row, which is read once and held in registers when it fits
// (else three reads, the second and third from the cache); the output is rounded once to the storage type.
// Bound by latency (2 ... 20 MB): the row, its image and its index are scalar, the sums stay off the LDS crossbar, and
// the kernel is made for the vectors a lane holds: 16 ... 256 rows of 1024 in a graph 3.6 -> 2.8 us, 1640 rows 4.35 -> 3.8.
#include "common.h"
#include "nova_internal.h"

namespace {

constexpr int kWavesPerBlock = 4;

// U: vectors per lane, a row of at most U * 64 vectors is kept in registers (every count up to eight has its kernel: with
// modulation eight vectors are 96 registers); 0: any row, three passes
template <typename T, int U>
__global__ __launch_bounds__(kWavesPerBlock* NOVA_WAVE) void gather_ln_kernel(
    const T* __restrict__ src, const int32_t* __restrict__ idx, int M, int k, uint32_t k_inv, int N, int C,
    const T* __restrict__ shift, const T* __restrict__ scale, int mod_pitch, T* __restrict__ dst,
    const int32_t* __restrict__ k_rows, const int32_t* __restrict__ kv_rows, int32_t* __restrict__ kv_next, int P) {
  using VT = Vec16<T>;
  constexpr int VN = VT::N;
  const int lane = threadIdx.x & (NOVA_WAVE - 1);
  // the row is the wave's: its image, its index and its count are scalar work
  const int m = blockIdx.x * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x / NOVA_WAVE);
  if (kv_next && blockIdx.x == 0) {
    // per-image cache lengths after this block: prior rows + kept rows.  Written by this launch (the second
    // LayerNorm: everything that reads the old lengths has run), so the output may be the input array.
    const int B = M / k;
    for (int b = threadIdx.x; b < B; b += kWavesPerBlock * NOVA_WAVE)
      kv_next[b] = image_prior(kv_rows, b, P) + image_count(k_rows, b, k);
  }
  if (m >= M) return;
  int slot;
  const int image = div_by(m, k, k_inv, slot);
  if (k_rows && slot >= image_count(k_rows, image, k)) {
    // a slot past its image's keep count: zeros, so that everything downstream of it stays finite
    VT z;
#pragma unroll
    for (int e = 0; e < VN; ++e) z.set(e, 0.0f);
    for (int vi = lane; vi < C / VN; vi += NOVA_WAVE) z.store(dst + (int64_t)m * C + vi * VN);
    return;
  }
  int64_t srow = m;
  if (idx) {
    const int t = min(max(idx[m], 0), N - 1);   // idx is [B, k] and m = b * k + s; clamped, never out of bounds
    srow = (int64_t)image * N + t;
  }
  const T* p = src + srow * C;
  T* q = dst + (int64_t)m * C;
  const int nvec = C / VN;

  if constexpr (U > 0) {
    // read once; the same sums in the same order as the three-pass form below
    VT v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int vi = u * NOVA_WAVE + lane;
      if (vi < nvec) v[u].load(p + vi * VN);
    }
    // the modulation vectors are requested with the row, not behind its sums
    VT a[U], g[U];
    if (shift) {
      const T* sh = shift + (int64_t)image * mod_pitch;
      const T* sc = scale + (int64_t)image * mod_pitch;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int vi = u * NOVA_WAVE + lane;
        if (vi < nvec) { a[u].load(sh + vi * VN); g[u].load(sc + vi * VN); }
      }
    }
    float sum = 0.f;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (u * NOVA_WAVE + lane < nvec) {
#pragma unroll
        for (int e = 0; e < VN; ++e) sum += v[u].get(e);
      }
    const float mean = wave_sum(sum) / (float)C;
    float sq = 0.f;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (u * NOVA_WAVE + lane < nvec) {
#pragma unroll
        for (int e = 0; e < VN; ++e) { float d = v[u].get(e) - mean; sq = fmaf(d, d, sq); }
      }
    const float rstd = 1.0f / sqrtf(wave_sum(sq) / (float)C + kNormEps);
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int vi = u * NOVA_WAVE + lane;
      if (vi < nvec) {
        VT o;
        if (shift) {
#pragma unroll
          for (int e = 0; e < VN; ++e) o.set(e, fmaf((v[u].get(e) - mean) * rstd, 1.0f + g[u].get(e), a[u].get(e)));
        } else {
#pragma unroll
          for (int e = 0; e < VN; ++e) o.set(e, (v[u].get(e) - mean) * rstd);
        }
        o.store(q + vi * VN);
      }
    }
    return;
  }

  float sum = 0.f;
  for (int vi = lane; vi < nvec; vi += NOVA_WAVE) {
    VT v; v.load(p + vi * VN);
#pragma unroll
    for (int e = 0; e < VN; ++e) sum += v.get(e);
  }
  const float mean = wave_sum(sum) / (float)C;
  float sq = 0.f;
  for (int vi = lane; vi < nvec; vi += NOVA_WAVE) {
    VT v; v.load(p + vi * VN);
#pragma unroll
    for (int e = 0; e < VN; ++e) { float d = v.get(e) - mean; sq = fmaf(d, d, sq); }
  }
  const float rstd = 1.0f / sqrtf(wave_sum(sq) / (float)C + kNormEps);
  if (shift) {          // modulation vectors of image m / k (both given or neither)
    const T* sh = shift + (int64_t)image * mod_pitch;
    const T* sc = scale + (int64_t)image * mod_pitch;
    for (int vi = lane; vi < nvec; vi += NOVA_WAVE) {
      VT v, o, a, g; v.load(p + vi * VN); a.load(sh + vi * VN); g.load(sc + vi * VN);
#pragma unroll
      for (int e = 0; e < VN; ++e) o.set(e, fmaf((v.get(e) - mean) * rstd, 1.0f + g.get(e), a.get(e)));
      o.store(q + vi * VN);
    }
    return;
  }
  for (int vi = lane; vi < nvec; vi += NOVA_WAVE) {
    VT v, o; v.load(p + vi * VN);
#pragma unroll
    for (int e = 0; e < VN; ++e) o.set(e, (v.get(e) - mean) * rstd);
    o.store(q + vi * VN);
  }
}

template <typename T>
void launch_t(hipStream_t st, const void* src, const int32_t* idx, int M, int k, int N, int C, const void* shift,
              const void* scale, int mod_pitch, void* dst, const int32_t* k_rows, const int32_t* kv_rows,
              int32_t* kv_next, int P) {
  const unsigned grid = (unsigned)((M + kWavesPerBlock - 1) / kWavesPerBlock);
  const int vecs = (C / Vec16<T>::N + NOVA_WAVE - 1) / NOVA_WAVE;      // per lane
  auto go = [&](auto kernel) {
    kernel<<<grid, kWavesPerBlock * NOVA_WAVE, 0, st>>>(static_cast<const T*>(src), idx, M, k, div_inv(k), N, C,
                                                        static_cast<const T*>(shift), static_cast<const T*>(scale),
                                                        mod_pitch, static_cast<T*>(dst), k_rows, kv_rows, kv_next, P);
  };
  switch (vecs) {
    case 1: return go(gather_ln_kernel<T, 1>);
    case 2: return go(gather_ln_kernel<T, 2>);
    case 3: return go(gather_ln_kernel<T, 3>);
    case 4: return go(gather_ln_kernel<T, 4>);
    case 5: return go(gather_ln_kernel<T, 5>);
    case 6: return go(gather_ln_kernel<T, 6>);
    case 7: return go(gather_ln_kernel<T, 7>);
    case 8: return go(gather_ln_kernel<T, 8>);
    default: return go(gather_ln_kernel<T, 0>);
  }
}

}  // namespace

hipError_t launch_gather_ln(hipStream_t st, int dtype, const void* src, const int32_t* idx, int M, int k,
                            int N, int C, const void* shift, const void* scale, int mod_pitch, void* dst,
                            const int32_t* k_rows, const int32_t* kv_rows, int32_t* kv_next, int P) {
  if (dtype == NOVA_BF16)
    launch_t<bf16_t>(st, src, idx, M, k, N, C, shift, scale, mod_pitch, dst, k_rows, kv_rows, kv_next, P);
  else
    launch_t<float>(st, src, idx, M, k, N, C, shift, scale, mod_pitch, dst, k_rows, kv_rows, kv_next, P);
  return hipGetLastError();
}
