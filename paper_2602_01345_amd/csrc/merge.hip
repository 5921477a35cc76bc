// Residual cache reuse (Sec. 3.3, "Residual Cache Reuse", second and third equations):
// kept tokens take the block's output; pruned tokens take their input plus the prior
// scale's residual cache interpolated to the current grid; the new residual cache is
// output minus input everywhere.
//
// Bandwidth-bound streaming kernel.  One wave64 owns one row of C channels and moves it in 16-byte vectors; all
// loads of a sweep are issued before the first use.  The launch has one wave per token (it serves the
// pruned tokens: a wave whose mask byte says "kept" leaves at once) followed by one wave per kept slot s, which
// copies row s of the block's output to token kept_idx[b, s] -- so nobody has to look up where in the kept
// list a token sits.  What a wave does is scalar work without a division (the quotients come from the host): with
// 64-bit divisions in every lane 9 rows of 1024 took 1.82 us in a graph, 1.70 without (a launch alone 1.57).  Per-image
// keep counts: slots past an image's count (or holding -1) leave at once.
// The bilinear taps (half-pixel centres) are wave-uniform and evaluated in fp32.  Other interpolation
// kernels (nearest cell, cubic convolution) go through a generic separable-taps kernel further down.
#include <algorithm>

#include "common.h"
#include "nova_internal.h"

namespace {

constexpr int kWavesPerBlock = 4;
constexpr int kUnroll = 4;

struct Taps {
  int i0, i1;
  float w1;
};

__device__ __forceinline__ Taps axis_taps(int dst, int n_in, float ratio) {
  float src = ((float)dst + 0.5f) * ratio - 0.5f;
  src = src < 0.0f ? 0.0f : src;
  int i0 = (int)floorf(src);
  i0 = i0 > n_in - 1 ? n_in - 1 : i0;
  Taps t;
  t.i0 = i0;
  t.i1 = i0 + 1 > n_in - 1 ? n_in - 1 : i0 + 1;
  t.w1 = src - (float)i0;
  return t;
}

// From this many tokens on the launch goes image by image, else the tokens of all images come first: the longer waves, they
// hide under the copies (bilinear, half kept, tokens first / by image: 4 x 256 rows of 1920 6.8 / 7.1 us, 16 x 256 of 2304
// 22.5 / 23.9; 8 x 1024 of 2304 38.7 / 38.6, nearest 37.0 / 35.8; 2 x 4096 of 2048 32.5 / 31.0).
constexpr int kImageTokens = 1024;

// Quotients made once on the host.
struct MergeGrid {
  int tok_blocks, slot_blocks;    // workgroups per image for its tokens / its kept slots
  int group_blocks, group_toks;   // per group of images, one or all: workgroups, those of them for tokens, which come first
  uint32_t group_inv, tok_inv, slot_inv, w_inv;   // div_inv of group_blocks, tok_blocks, slot_blocks, the grid's width
  float ry, rx;                   // (rows, columns of the prior grid) / (of this one)
  uint32_t ny_inv, nx_inv;        // nearest cell: div_inv of twice the rows / columns, 0 where its products need 64 bits
};

// The wave's job: a pruned token (tok >= 0, slot < 0), a kept slot (both >= 0), or nothing (tok < 0).
struct MergeItem {
  int b, tok;
  int64_t slot;      // row of y_kept, or -1
};
__device__ __forceinline__ MergeItem merge_item(const MergeGrid& g, int N, int k, const int32_t* __restrict__ idx,
                                                const uint8_t* __restrict__ mask, const int32_t* __restrict__ k_rows) {
  MergeItem it = {0, -1, -1};
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / NOVA_WAVE);
  int in_group, block;
  it.b = div_by(blockIdx.x, g.group_blocks, g.group_inv, in_group);
  if (in_group < g.group_toks) {
    it.b += div_by(in_group, g.tok_blocks, g.tok_inv, block);
    const int i = block * kWavesPerBlock + wave;
    // kept tokens are written by their slot's wave (with k == 0 there are no slots: every token takes this path)
    if (i < N && (!mask[(int64_t)it.b * N + i] || k == 0)) it.tok = i;
  } else {
    it.b += div_by(in_group - g.group_toks, g.slot_blocks, g.slot_inv, block);
    const int s = block * kWavesPerBlock + wave;
    const int64_t slot = (int64_t)it.b * k + s;
    const int t = s < image_count(k_rows, it.b, k) ? idx[slot] : -1;
    if (t >= 0 && t < N) { it.tok = t; it.slot = slot; }
  }
  // every lane has read the same bytes: what follows is scalar
  it.tok = __builtin_amdgcn_readfirstlane(it.tok);
  return it;
}

// kept token: the block's output, copied; residual = output - input
template <typename T>
__device__ __forceinline__ void merge_kept_row(const T* __restrict__ yr, const T* __restrict__ xr, T* __restrict__ outr,
                                               T* __restrict__ cnr, int nvec, int lane) {
  using VT = Vec16<T>;
  constexpr int VN = VT::N;
  for (int v0 = 0; v0 < nvec; v0 += kUnroll * NOVA_WAVE) {
    VT vy[kUnroll], vx[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      int vi = v0 + u * NOVA_WAVE + lane;
      if (vi < nvec) { vy[u].load(yr + vi * VN); vx[u].load(xr + vi * VN); }
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      int vi = v0 + u * NOVA_WAVE + lane;
      if (vi < nvec) {
        vy[u].store(outr + vi * VN);
        if (cnr) {
          VT c;
#pragma unroll
          for (int e = 0; e < VN; ++e) c.set(e, vy[u].get(e) - vx[u].get(e));
          c.store(cnr + vi * VN);
        }
      }
    }
  }
}

template <typename T>
__global__ __launch_bounds__(kWavesPerBlock* NOVA_WAVE) void merge_kernel(
    MergeGrid g, int C, int h, int w, int hp, int wp, int k, const T* __restrict__ x, const T* __restrict__ y,
    const int32_t* __restrict__ idx, const uint8_t* __restrict__ mask, const T* __restrict__ cache_prev,
    T* __restrict__ out, T* __restrict__ cache_new, const int32_t* __restrict__ k_rows) {
  using VT = Vec16<T>;
  constexpr int VN = VT::N;
  const int lane = threadIdx.x & (NOVA_WAVE - 1);
  const int N = h * w;
  const MergeItem it = merge_item(g, N, k, idx, mask, k_rows);
  if (it.tok < 0) return;
  const int b = it.b, i = it.tok;
  const int64_t row = (int64_t)b * N + i;
  const int nvec = C / VN;                                           // C % VN == 0 (checked by the host)
  const T* xr = x + row * C;
  T* outr = out + row * C;
  T* cnr = cache_new ? cache_new + row * C : nullptr;

  if (it.slot >= 0) {
    merge_kept_row<T>(y + it.slot * C, xr, outr, cnr, nvec, lane);
    return;
  }

  if (!cache_prev) {
    // no prior cache was given (legal only when every token is kept): a row the mask still
    // marks as pruned passes through unchanged with a zero residual
    for (int vi = lane; vi < nvec; vi += NOVA_WAVE) {
      VT v, z;
      v.load(xr + vi * VN);
#pragma unroll
      for (int e = 0; e < VN; ++e) z.set(e, 0.0f);
      v.store(outr + vi * VN);
      if (cnr) z.store(cnr + vi * VN);
    }
    return;
  }
  int ox;
  const int oy = div_by(i, w, g.w_inv, ox);
  const Taps ty = axis_taps(oy, hp, g.ry);
  const Taps tx = axis_taps(ox, wp, g.rx);
  const T* base = cache_prev + (int64_t)b * hp * wp * C;
  const T* c00 = base + ((int64_t)ty.i0 * wp + tx.i0) * C;
  const T* c01 = base + ((int64_t)ty.i0 * wp + tx.i1) * C;
  const T* c10 = base + ((int64_t)ty.i1 * wp + tx.i0) * C;
  const T* c11 = base + ((int64_t)ty.i1 * wp + tx.i1) * C;
  const float wy1 = ty.w1, wy0 = 1.0f - ty.w1, wx1 = tx.w1, wx0 = 1.0f - tx.w1;

  for (int v0 = 0; v0 < nvec; v0 += kUnroll * NOVA_WAVE) {
    VT vx[kUnroll], a00[kUnroll], a01[kUnroll], a10[kUnroll], a11[kUnroll];
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      int vi = v0 + u * NOVA_WAVE + lane;
      if (vi < nvec) {
        vx[u].load(xr + vi * VN);
        a00[u].load(c00 + vi * VN); a01[u].load(c01 + vi * VN);
        a10[u].load(c10 + vi * VN); a11[u].load(c11 + vi * VN);
      }
    }
#pragma unroll
    for (int u = 0; u < kUnroll; ++u) {
      int vi = v0 + u * NOVA_WAVE + lane;
      if (vi < nvec) {
        VT o, c;
#pragma unroll
        for (int e = 0; e < VN; ++e) {
          // rows first (y), then columns (x), as separable linear interpolation
          float top = a00[u].get(e) * wy0 + a10[u].get(e) * wy1;
          float bot = a01[u].get(e) * wy0 + a11[u].get(e) * wy1;
          float up = top * wx0 + bot * wx1;
          o.set(e, vx[u].get(e) + up);
          c.set(e, up);
        }
        o.store(outr + vi * VN);
        if (cnr) c.store(cnr + vi * VN);
      }
    }
  }
}

// ---- other interpolation kernels: NT taps per axis (1 = nearest cell, 4 = cubic convolution) -------------
template <int NT>
struct AxisTaps {
  int i[NT];
  float w[NT];
};

// nearest: the source cell that contains the output cell's centre, min(floor((dst + 1/2) n_in / n_out), n_in - 1),
// in integer arithmetic (centres on a cell boundary must not depend on rounding)
__device__ __forceinline__ AxisTaps<1> nearest_taps(int dst, int n_in, int n_out, uint32_t inv) {
  AxisTaps<1> t;
  int rem;
  const int64_t q = inv ? div_by((2 * dst + 1) * n_in, 2 * n_out, inv, rem) : ((int64_t)(2 * dst + 1) * n_in) / (2 * (int64_t)n_out);
  t.i[0] = (int)(q > n_in - 1 ? n_in - 1 : q);
  t.w[0] = 1.0f;
  return t;
}

// cubic convolution, kernel parameter a = -3/4, half-pixel centres, taps floor(src) - 1 .. floor(src) + 2
// clamped to the grid
__device__ __forceinline__ AxisTaps<4> cubic_taps(int dst, int n_in, float ratio) {
  constexpr float a = -0.75f;
  const float src = ((float)dst + 0.5f) * ratio - 0.5f;
  const float fl = floorf(src);
  const float t = src - fl;
  const int i0 = (int)fl;
  auto near = [](float d) { return ((a + 2.0f) * d - (a + 3.0f)) * d * d + 1.0f; };          // |d| <= 1
  auto far = [](float d) { return ((a * d - 5.0f * a) * d + 8.0f * a) * d - 4.0f * a; };     // 1 < |d| < 2
  AxisTaps<4> r;
  r.w[0] = far(t + 1.0f); r.w[1] = near(t); r.w[2] = near(1.0f - t); r.w[3] = far(2.0f - t);
#pragma unroll
  for (int j = 0; j < 4; ++j) r.i[j] = min(max(i0 - 1 + j, 0), n_in - 1);
  return r;
}

// Bicubic: three waves per SIMD, each with 17 rows in flight, not the six that fit (they fetch the shared taps again: 16 x 256
// rows of 1920, four of five kept, 22.7 -> 20.0 us)
template <typename T, int NT>
__global__ __launch_bounds__(kWavesPerBlock* NOVA_WAVE) __attribute__((amdgpu_waves_per_eu(NT == 4 ? 3 : 1, NT == 4 ? 3 : 8))) void
merge_taps_kernel(
    MergeGrid g, int C, int h, int w, int hp, int wp, int k, const T* __restrict__ x, const T* __restrict__ y,
    const int32_t* __restrict__ idx, const uint8_t* __restrict__ mask, const T* __restrict__ cache_prev,
    T* __restrict__ out, T* __restrict__ cache_new, const int32_t* __restrict__ k_rows) {
  using VT = Vec16<T>;
  constexpr int VN = VT::N;
  const int lane = threadIdx.x & (NOVA_WAVE - 1);
  const int N = h * w;
  const MergeItem it = merge_item(g, N, k, idx, mask, k_rows);
  if (it.tok < 0) return;
  const int b = it.b, i = it.tok;
  const int64_t row = (int64_t)b * N + i;
  const int nvec = C / VN;
  const T* xr = x + row * C;
  T* outr = out + row * C;
  T* cnr = cache_new ? cache_new + row * C : nullptr;

  if (it.slot >= 0) {
    merge_kept_row<T>(y + it.slot * C, xr, outr, cnr, nvec, lane);
    return;
  }
  if (!cache_prev) {              // legal only when every token is kept: pass through, zero residual
    for (int vi = lane; vi < nvec; vi += NOVA_WAVE) {
      VT v, z;
      v.load(xr + vi * VN);
#pragma unroll
      for (int e = 0; e < VN; ++e) z.set(e, 0.0f);
      v.store(outr + vi * VN);
      if (cnr) z.store(cnr + vi * VN);
    }
    return;
  }
  int ox;
  const int oy = div_by(i, w, g.w_inv, ox);
  AxisTaps<NT> ty, tx;
  if constexpr (NT == 1) { ty = nearest_taps(oy, hp, h, g.ny_inv); tx = nearest_taps(ox, wp, w, g.nx_inv); }
  else { ty = cubic_taps(oy, hp, g.ry); tx = cubic_taps(ox, wp, g.rx); }
  const T* base = cache_prev + (int64_t)b * hp * wp * C;
  for (int vi = lane; vi < nvec; vi += NOVA_WAVE) {
    VT vx, a[NT][NT];
#pragma unroll
    for (int jx = 0; jx < NT; ++jx)
#pragma unroll
      for (int jy = 0; jy < NT; ++jy) a[jx][jy].load(base + ((int64_t)ty.i[jy] * wp + tx.i[jx]) * C + vi * VN);
    vx.load(xr + vi * VN);
    // all of them before the first use: left alone the compiler waits for the last taps of sixteen one by one (bicubic, half
    // of the tokens kept: 2 x 1024 rows of 2048 11.9 us, so 9.8; 8 x 256 of 1920 12.8, 10.0)
    __builtin_amdgcn_sched_barrier(0);
    float up[VN];
#pragma unroll
    for (int e = 0; e < VN; ++e) up[e] = 0.0f;
#pragma unroll
    for (int jx = 0; jx < NT; ++jx) {
      float col[VN];                                     // rows first (y), then columns (x)
#pragma unroll
      for (int e = 0; e < VN; ++e) col[e] = 0.0f;
#pragma unroll
      for (int jy = 0; jy < NT; ++jy)
#pragma unroll
        for (int e = 0; e < VN; ++e) col[e] = fmaf(a[jx][jy].get(e), ty.w[jy], col[e]);
#pragma unroll
      for (int e = 0; e < VN; ++e) up[e] = fmaf(col[e], tx.w[jx], up[e]);
    }
    VT o, c;
#pragma unroll
    for (int e = 0; e < VN; ++e) { o.set(e, vx.get(e) + up[e]); c.set(e, up[e]); }
    o.store(outr + vi * VN);
    if (cnr) c.store(cnr + vi * VN);
  }
}

template <typename T>
hipError_t launch_t(hipStream_t st, int interp, int B, int C, int h, int w, int hp, int wp, int k, const void* x,
                    const void* y, const int32_t* idx, const uint8_t* mask, const void* cache_prev, void* out,
                    void* cache_new, const int32_t* k_rows) {
  MergeGrid g;
  g.tok_blocks = (int)(((int64_t)h * w + kWavesPerBlock - 1) / kWavesPerBlock);
  g.slot_blocks = (k + kWavesPerBlock - 1) / kWavesPerBlock;
  g.tok_inv = div_inv(g.tok_blocks);
  g.slot_inv = div_inv(g.slot_blocks);
  g.w_inv = div_inv(w);
  g.ry = (float)hp / (float)h;
  g.rx = (float)wp / (float)w;
  auto nearest_inv = [](int n_in, int n_out) {
    return 2 * (int64_t)n_out * n_in <= INT32_MAX && 2 * (int64_t)n_out <= INT32_MAX ? div_inv(2 * n_out) : 0u;
  };
  g.ny_inv = nearest_inv(hp, h);
  g.nx_inv = nearest_inv(wp, w);
  constexpr int threads = kWavesPerBlock * NOVA_WAVE;
  // a launch has fewer than 2^32 threads: images beyond that (from 8 million of up to four tokens on) take another one
  const int64_t per_image = (int64_t)g.tok_blocks + g.slot_blocks;
  const int most = (int)std::max<int64_t>(UINT32_MAX / threads / per_image, 1);
  const int64_t N = (int64_t)h * w, np = (int64_t)hp * wp;
  for (int b = 0; b < B; b += std::min(most, B - b)) {
    const int images = std::min(most, B - b);
    const unsigned grid = (unsigned)(images * per_image);
    const int group = N >= kImageTokens ? 1 : images;
    g.group_blocks = (int)(group * per_image);
    g.group_inv = div_inv(g.group_blocks);
    g.group_toks = group * g.tok_blocks;
    const T* xt = static_cast<const T*>(x) + b * N * C;
    const T* yt = y ? static_cast<const T*>(y) + (int64_t)b * k * C : nullptr;
    const T* ct = cache_prev ? static_cast<const T*>(cache_prev) + b * np * C : nullptr;
    T* ot = static_cast<T*>(out) + b * N * C;
    T* nt = cache_new ? static_cast<T*>(cache_new) + b * N * C : nullptr;
    const int32_t* it = idx ? idx + (int64_t)b * k : nullptr;
    const int32_t* kt = k_rows ? k_rows + b : nullptr;
    const uint8_t* mt = mask + b * N;
    if (interp == NOVA_INTERP_NEAREST)
      merge_taps_kernel<T, 1><<<grid, threads, 0, st>>>(g, C, h, w, hp, wp, k, xt, yt, it, mt, ct, ot, nt, kt);
    else if (interp == NOVA_INTERP_BICUBIC)
      merge_taps_kernel<T, 4><<<grid, threads, 0, st>>>(g, C, h, w, hp, wp, k, xt, yt, it, mt, ct, ot, nt, kt);
    else
      merge_kernel<T><<<grid, threads, 0, st>>>(g, C, h, w, hp, wp, k, xt, yt, it, mt, ct, ot, nt, kt);
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_merge(hipStream_t st, int dtype, int interp, int B, int C, int h, int w, int hp, int wp, int k,
                        const void* x, const void* y, const int32_t* idx, const uint8_t* mask,
                        const void* cache_prev, void* out, void* cache_new, const int32_t* k_rows) {
  if (dtype == NOVA_BF16)
    return launch_t<bf16_t>(st, interp, B, C, h, w, hp, wp, k, x, y, idx, mask, cache_prev, out, cache_new, k_rows);
  return launch_t<float>(st, interp, B, C, h, w, hp, wp, k, x, y, idx, mask, cache_prev, out, cache_new, k_rows);
}
