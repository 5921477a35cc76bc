// Token predictive entropy H = -sum_v p(v) ln p(v), p = softmax(logits)
// (Sec. 3.3, "Adaptive Acceleration Activation", entropy equation; the optional
// per-batch-row mean is the scale mean entropy of the same section).
//
// Bandwidth-bound: every logit is read from HBM exactly once.  One wave64 owns one row at a
// time and walks several rows.  A row is consumed in chunks of CH 16-byte vectors per lane; the
// next chunk (of this or the next row) is already in flight while the current one is reduced.
// Per chunk the wave agrees on a running maximum m, so all lanes accumulate against the same m
// and the final combine is a plain wave sum.
//
// With S = sum_v e^{x_v - m} and T = sum_v (m - x_v) e^{x_v - m}:  H = ln S + T / S.
// Both terms are non-negative, so nothing cancels.  To keep relative accuracy when H
// is tiny (one dominant logit) the elements equal to m are counted, not summed:
// S = cnt + R with R = sum over x_v < m, and H = log1p(R + cnt - 1) + T / (R + cnt).
#include <algorithm>

#include "common.h"
#include "entropy_core.h"
#include "nova_internal.h"

namespace {

using namespace entropy_core;

// The tensors of a launch, one set per blockIdx.y: a whole step's blocks go through one launch, since each of them alone
// is mostly launch, ramp and tail (a step of 16 blocks of 2048 rows of 4096 bf16 logits: 16 launches 105 us, one 67).
template <int NB>
struct EntropyBatch {
  const void* logits[NB];
  float* H[NB];
};
template <int NB>
struct MeanBatch {
  const float* H[NB];
  float* mean[NB];
};

// Any shape: one row per wave, lanes past the row's end masked.
template <typename T, int CH, int NB>
__global__ __launch_bounds__(kWavesPerBlock* NOVA_WAVE) void entropy_generic_kernel(
    EntropyBatch<NB> batch, int64_t rows, int V, int64_t stride, int vec_ok) {
  const T* __restrict__ logits = static_cast<const T*>(batch.logits[blockIdx.y]);
  float* __restrict__ H = batch.H[blockIdx.y];
  using VT = Vec16<T>;
  constexpr int VN = VT::N;
  const int lane = threadIdx.x & (NOVA_WAVE - 1);
  const int wave = threadIdx.x / NOVA_WAVE;
  const int64_t row = (int64_t)blockIdx.x * kWavesPerBlock + wave;
  if (row >= rows) return;                       // whole wave leaves together
  const T* p = logits + row * stride;

  Row st;
  st.init();

  int done = 0;
  if (vec_ok) {
    const int nvec = V / VN;                     // full 16-byte vectors in the row
    for (int v0 = 0; v0 < nvec; v0 += CH * NOVA_WAVE) {
      VT buf[CH];
      bool have[CH];
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        int vi = v0 + c * NOVA_WAVE + lane;
        have[c] = vi < nvec;
        if (have[c]) buf[c].load(p + (int64_t)vi * VN);
      }
      float cm = -INFINITY;
      bool unordered = false;                    // the maximum drops NaNs: they are caught here
#pragma unroll
      for (int c = 0; c < CH; ++c)
        if (have[c]) {
#pragma unroll
          for (int i = 0; i < VN; i += 2) {
            const float x0 = buf[c].get(i), x1 = buf[c].get(i + 1);
            cm = fmaxf(cm, fmaxf(x0, x1));
            unordered = unordered || __builtin_isunordered(x0, x1);
          }
        }
      if (__any(unordered)) st.nan = true;
      st.rebase(wave_max(cm));
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        // have[c] is false only in the last, partial sweep; keep ballots wave-wide
        if (__all(have[c])) {
#pragma unroll
          for (int i = 0; i < VN; ++i) st.add(buf[c].get(i));
        } else if (__any(have[c])) {
#pragma unroll
          for (int i = 0; i < VN; ++i) st.add_masked(have[c] ? buf[c].get(i) : 0.0f, have[c]);
        }
      }
    }
    done = nvec * VN;
  }
  // scalar tail (or the whole row when it is not 16-byte aligned)
  for (int e0 = done; e0 < V; e0 += NOVA_WAVE) {
    int ei = e0 + lane;
    bool valid = ei < V;
    float x = valid ? ld_f32(p + ei) : -INFINITY;
    st.rebase(wave_max(x));
    st.add_masked(valid ? x : 0.0f, valid);
  }

  float h = st.finish();
  if (lane == 0) H[row] = h;
}


// Regular rows: each wave walks rows  w, w + nwaves, ...  (entropy_core.h: walk_rows).
template <typename T, int CH, int NB>
__global__ __launch_bounds__(kWavesPerBlock* NOVA_WAVE) void entropy_kernel(EntropyBatch<NB> batch, int64_t rows, int nchunk,
                                                                             int64_t stride) {
  const T* __restrict__ logits = static_cast<const T*>(batch.logits[blockIdx.y]);
  float* __restrict__ H = batch.H[blockIdx.y];
  const int lane = threadIdx.x & (NOVA_WAVE - 1);
  const int64_t w0 = (int64_t)blockIdx.x * kWavesPerBlock + threadIdx.x / NOVA_WAVE;
  const int64_t nwaves = (int64_t)gridDim.x * kWavesPerBlock;
  if (w0 >= rows) return;                        // whole wave leaves together
  walk_rows<T, CH>(logits, w0, nwaves, (rows - w0 + nwaves - 1) / nwaves, nchunk, stride, lane,
                   [&](int64_t row, float h) { if (lane == 0) H[row] = h; });
}

// Scale mean entropy of one image per workgroup: mean[b] = (sum_i H[b, i]) / N with a fixed summation order
// (thread t adds elements t, t + 1024, ..., then a fixed tree over the threads), so the
// result is the same bits on every run: the layer-linkage ratio turns it into an integer keep count.  A NaN
// entropy gives NaN.  One latency for up to 4096 tokens: 256 threads that add contiguous shares one load after the
// other take 4.0 us for 4096, this 3.1.
constexpr int kMeanThreads = 1024;
template <int NB>
__global__ __launch_bounds__(kMeanThreads) void row_mean_kernel(MeanBatch<NB> batch, int64_t rows_per_batch) {
  __shared__ float part[kMeanThreads / NOVA_WAVE];
  const float* __restrict__ h = batch.H[blockIdx.y] + (int64_t)blockIdx.x * rows_per_batch;
  float s = 0.0f;
  for (int64_t i = threadIdx.x; i < rows_per_batch; i += 4 * kMeanThreads) {
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = i + u * kMeanThreads < rows_per_batch ? h[i + u * kMeanThreads] : 0.0f;
    s += (v[0] + v[1]) + (v[2] + v[3]);
  }
  s = wave_sum(s);
  if ((threadIdx.x & (NOVA_WAVE - 1)) == 0) part[threadIdx.x / NOVA_WAVE] = s;
  __syncthreads();
  if (threadIdx.x != 0) return;
  float t = 0.0f;
#pragma unroll
  for (int w = 0; w < kMeanThreads / NOVA_WAVE; ++w) t += part[w];
  batch.mean[blockIdx.y][blockIdx.x] = t / (float)rows_per_batch;
}

// Entropies and mean of images of a few regular rows in one launch: a workgroup per image, a wave per row, then the first
// wave takes the mean in row_mean_kernel's order, so its bits.  Of two launches most is start and end (bf16, V = 4096, us in a
// graph, two / one: 1 row 5.3 / 3.8, 8 images of 4 rows 6.1 / 4.2, 16 of 9 6.1 / 5.7; a call from the host 7.9 / 5.5), which
// entropy_core.h: one_launch decides by.
static_assert(kFewRows == kMeanThreads / NOVA_WAVE);
template <typename T, int CH>
__global__ __launch_bounds__(kMeanThreads) void entropy_few_rows_kernel(const T* __restrict__ logits, float* __restrict__ H,
                                                                        float* __restrict__ mean, int rows_per_batch, int nchunk,
                                                                        int64_t stride) {
  __shared__ float hs[kFewRows];
  const int lane = threadIdx.x & (NOVA_WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / NOVA_WAVE);   // the launch has a wave per row
  const int64_t row0 = (int64_t)blockIdx.x * rows_per_batch;
  walk_rows<T, CH>(logits, row0 + wave, (int64_t)1, (int64_t)1, nchunk, stride, lane, [&](int64_t row, float h) {
    if (lane == 0) { H[row] = h; hs[wave] = h; }
  });
  __syncthreads();
  if (wave != 0) return;
  const float s = wave_sum(lane < rows_per_batch ? hs[min(lane, kFewRows - 1)] : 0.0f);
  if (lane == 0) mean[blockIdx.x] = s / (float)rows_per_batch;
}

// Whether that kernel took the call
template <typename T>
bool launch_few_rows(hipStream_t st, int num_cus, const void* logits, int64_t rows_per_batch, int batch, int V, int64_t stride,
                     float* H, float* mean) {
  const int sweeps = regular_sweeps<T>(logits, V, stride);
  if (sweeps == 0 || !one_launch<T>(num_cus, rows_per_batch, batch, V)) return false;
  const int n = (int)rows_per_batch;
  const T* p = static_cast<const T*>(logits);
  if (sweeps % 4 == 0) entropy_few_rows_kernel<T, 4><<<batch, n * NOVA_WAVE, 0, st>>>(p, H, mean, n, sweeps / 4, stride);
  else if (sweeps % 2 == 0) entropy_few_rows_kernel<T, 2><<<batch, n * NOVA_WAVE, 0, st>>>(p, H, mean, n, sweeps / 2, stride);
  else entropy_few_rows_kernel<T, 1><<<batch, n * NOVA_WAVE, 0, st>>>(p, H, mean, n, sweeps, stride);
  return true;
}

// `n` tensors of the same shape and alignment, at most NB
template <typename T, int NB>
void launch_t(hipStream_t st, int num_cus, int n, const void* const* logits, int64_t rows, int V, int64_t stride, float* const* H) {
  EntropyBatch<NB> batch = {};
  for (int i = 0; i < n; ++i) { batch.logits[i] = logits[i]; batch.H[i] = H[i]; }
  const int64_t per_row = (rows + kWavesPerBlock - 1) / kWavesPerBlock;
  if (const int sweeps = regular_sweeps<T>(logits[0], V, stride)) {
    // at most kWavesPerSimd resident waves per SIMD over all tensors, each walking several rows
    const int64_t max_blocks = std::max<int64_t>((int64_t)num_cus * 4 * kWavesPerSimd / kWavesPerBlock / n, 1);
    const dim3 grid((unsigned)std::min<int64_t>(per_row, max_blocks), n);
    const int block = kWavesPerBlock * NOVA_WAVE;
    if (sweeps % 4 == 0) entropy_kernel<T, 4, NB><<<grid, block, 0, st>>>(batch, rows, sweeps / 4, stride);
    else if (sweeps % 2 == 0) entropy_kernel<T, 2, NB><<<grid, block, 0, st>>>(batch, rows, sweeps / 2, stride);
    else entropy_kernel<T, 1, NB><<<grid, block, 0, st>>>(batch, rows, sweeps, stride);
  } else {
    const int vec_ok = aligned_rows<T>(logits[0], stride);
    const dim3 grid((unsigned)per_row, n);
    entropy_generic_kernel<T, 8, NB><<<grid, kWavesPerBlock * NOVA_WAVE, 0, st>>>(batch, rows, V, stride, vec_ok);
  }
}

template <int NB>
void launch_mean(hipStream_t st, int n, const float* const* H, int64_t rows_per_batch, int batch_rows, float* const* mean) {
  MeanBatch<NB> batch = {};
  for (int i = 0; i < n; ++i) { batch.H[i] = H[i]; batch.mean[i] = mean[i]; }
  row_mean_kernel<NB><<<dim3(batch_rows, n), kMeanThreads, 0, st>>>(batch, rows_per_batch);
}

}  // namespace

hipError_t launch_row_mean(hipStream_t st, const float* H, int64_t rows_per_batch, int batch, float* mean) {
  launch_mean<1>(st, 1, &H, rows_per_batch, batch, &mean);
  return hipGetLastError();
}

hipError_t launch_entropy(hipStream_t st, int num_cus, int n, const void* const* logits, int dtype, int64_t rows_per_batch,
                          int batch, int V, int64_t stride, float* const* H, float* const* mean) {
  const int64_t rows = rows_per_batch * batch;
  for (int i = 0; i < n;) {
    // a run of tensors of one alignment: the kernel is chosen as for each of them alone
    int run = 1;
    const bool aligned = (reinterpret_cast<uintptr_t>(logits[i]) & 15) == 0;
    while (run < kMaxBatch && i + run < n && ((reinterpret_cast<uintptr_t>(logits[i + run]) & 15) == 0) == aligned) ++run;
    if (run == 1 && mean &&
        (dtype == NOVA_BF16 ? launch_few_rows<bf16_t>(st, num_cus, logits[i], rows_per_batch, batch, V, stride, H[i], mean[i])
                            : launch_few_rows<float>(st, num_cus, logits[i], rows_per_batch, batch, V, stride, H[i], mean[i]))) {
      ++i;
      continue;
    }
    auto go = [&](auto one, auto many) { run == 1 ? one() : many(); };
    if (dtype == NOVA_BF16)
      go([&] { launch_t<bf16_t, 1>(st, num_cus, 1, logits + i, rows, V, stride, H + i); },
         [&] { launch_t<bf16_t, kMaxBatch>(st, num_cus, run, logits + i, rows, V, stride, H + i); });
    else
      go([&] { launch_t<float, 1>(st, num_cus, 1, logits + i, rows, V, stride, H + i); },
         [&] { launch_t<float, kMaxBatch>(st, num_cus, run, logits + i, rows, V, stride, H + i); });
    if (mean)
      go([&] { launch_mean<1>(st, 1, H + i, rows_per_batch, batch, mean + i); },
         [&] { launch_mean<kMaxBatch>(st, run, H + i, rows_per_batch, batch, mean + i); });
    i += run;
  }
  return hipGetLastError();
}
