// Entropy-guided token selection: per batch row keep the k tokens that come first in
// the order (entropy descending, index ascending)  (Sec. 3.3, "Dual-Linkage
// Acceleration", final sentence; Sec. 3.2, the highest-entropy tokens are maintained).
//
// One workgroup per batch row.  Entropies are mapped to 32-bit keys whose unsigned order is the required numeric order
// (NaN lowest, -0 == +0), and the k-th largest key is found.  Every key above the threshold is kept; of the keys equal to
// it the first (k - #above) in index order are kept, which prefix sums turn into the ascending index list and the mask.
// Integer compares only: the result equals a stable sort bit for bit.
//
// Bound by latency (1 ... 32 KB per row): every barrier, LDS round trip and lane shuffle counts.  Rows of up to 8192
// tokens keep their keys in registers, divide the range of the keys that occur into 2048 bins, rank the few keys of
// the bin that matters in one wave, and need nine barriers; the radix select on LDS histograms with its four passes,
// 24 barriers, stays for longer rows.  Radix select / this (us): 8 rows of 256 8.5 / 4.6, one row of 256 in a
// graph 7.8 / 3.5, one of 1024 7.8 / 4.9, two of 4096 11.4 / 8.0.
#include <algorithm>

#include "common.h"
#include "nova_internal.h"
#include "select_core.h"

namespace {

using namespace select_core;

constexpr int kThreads = 1024;

__device__ __forceinline__ int row_count(int k_uniform, const int32_t* __restrict__ k_per_row, int b, int N, int pitch) {
  if (!k_per_row) return k_uniform;
  int k = k_per_row[b];
  k = k < 0 ? 0 : (k > N ? N : k);
  return k > pitch ? pitch : k;
}

// The rows of a launch, one set per blockIdx.y: a step's blocks select together (16 launches of eight rows of 256 62 us, one 5).
template <int NB>
struct SelectBatch {
  const float* H[NB];
  int32_t* idx[NB];
  uint8_t* mask[NB];
  int k[NB];
};

// N <= NT * KPT
template <int NT, int KPT, int NB>
__global__ __launch_bounds__(NT) void select_kernel(SelectBatch<NB> batch, int N, const int32_t* __restrict__ k_per_row) {
  __shared__ RowScratch<NT, KPT> sc;
  const int b = blockIdx.x, pitch = batch.k[blockIdx.y];
  const float* __restrict__ h = batch.H[blockIdx.y] + (int64_t)b * N;
  const int k = row_count(pitch, k_per_row, b, N, pitch);
  uint32_t key[KPT];
#pragma unroll
  for (int u = 0; u < KPT; ++u) key[u] = sort_key(h[min(u * NT + (int)threadIdx.x, N - 1)]);
  uint32_t thr = 0, remaining = 0;
  if (k > 0 && k < N) thr = range_select<NT, KPT>(key, N, k, sc, &remaining);
  range_compact<NT, KPT>(key, N, thr, remaining, k == N, k == 0, pitch, batch.idx[blockIdx.y] + (int64_t)b * pitch,
                         batch.mask[blockIdx.y] + (int64_t)b * N, sc);
}

// any N
template <int NB>
__global__ __launch_bounds__(kThreads) void select_long_kernel(SelectBatch<NB> batch, int N, const int32_t* __restrict__ k_per_row) {
  __shared__ Scratch<kThreads> sc;
  const int b = blockIdx.x, pitch = batch.k[blockIdx.y];
  const float* __restrict__ h = batch.H[blockIdx.y] + (int64_t)b * N;
  const int k = row_count(pitch, k_per_row, b, N, pitch);
  auto key_at = [&](int i) -> uint32_t { return sort_key(h[i]); };
  uint32_t thr = 0, remaining = 0;
  if (k > 0 && k < N) thr = radix_select<kThreads>(key_at, N, k, sc, &remaining);
  compact<kThreads>(key_at, N, thr, remaining, k == N, k == 0, pitch, batch.idx[blockIdx.y] + (int64_t)b * pitch,
                    batch.mask[blockIdx.y] + (int64_t)b * N, sc.wave_sums);
}

template <int NB>
void launch_t(hipStream_t st, int n, const float* const* H, int B, int N, const int* k, const int32_t* k_per_row,
              int32_t* const* idx, uint8_t* const* mask) {
  SelectBatch<NB> batch = {};
  for (int i = 0; i < n; ++i) { batch.H[i] = H[i]; batch.idx[i] = idx[i]; batch.mask[i] = mask[i]; batch.k[i] = k[i]; }
  auto go = [&](auto kernel, int threads) { kernel<<<dim3(B, n), threads, 0, st>>>(batch, N, k_per_row); };
  if (N <= 256) go(select_kernel<256, 1, NB>, 256);
  else if (N <= 1024) go(select_kernel<512, 2, NB>, 512);     // 8 rows of 1024: 256 / 512 / 1024 threads 4.9 / 4.2 / 4.3 us
  else if (N <= 2048) go(select_kernel<1024, 2, NB>, 1024);
  else if (N <= 4096) go(select_kernel<1024, 4, NB>, 1024);
  else if (N <= 8192) go(select_kernel<1024, 8, NB>, 1024);
  else go(select_long_kernel<NB>, kThreads);
}

}  // namespace

hipError_t launch_select(hipStream_t st, int n, const float* const* H, int B, int N, const int* k, const int32_t* k_per_row,
                         int32_t* const* idx, uint8_t* const* mask) {
  for (int i = 0; i < n;) {
    const int run = std::min(n - i, kMaxBatch);
    if (run == 1) launch_t<1>(st, 1, H + i, B, N, k + i, k_per_row, idx + i, mask + i);
    else launch_t<kMaxBatch>(st, run, H + i, B, N, k + i, k_per_row, idx + i, mask + i);
    i += run;
  }
  return hipGetLastError();
}
