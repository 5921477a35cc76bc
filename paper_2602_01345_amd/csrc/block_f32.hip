// fp32 path of the pruned block (Sec. 3.3, "Residual Cache Reuse", first equation,
// evaluated on the kept rows): plain, LDS-tiled fp32 kernels for small fp32 models.
// It exists for correctness at full fp32 precision; the matrix-core path is block_bf16.hip.
#include <algorithm>

#include "common.h"
#include "epilogue.h"
#include "nova_internal.h"

namespace {

constexpr int kTile = 16;
constexpr int kStepK = 64;                 // elements of K per step
constexpr int kPitch = kStepK + 4;         // 16-byte reads of sixteen rows hit all banks once
constexpr int kNormMaxK = 256;             // NORM: a thread holds a sixteenth of a row

// out[m][n] = sum_k A[m][k] * W[n][k]  (+ epilogue); A [M, K] row-major, W [Nout, K] row-major.
// One thread per output element, K in ascending order.  These launches are a few workgroups that wait for memory: the
// next 64 elements of K are requested before the current ones are used, so K = 256 costs one exposed latency and four
// pairs of barriers where steps of 16 cost sixteen of each (128 x 64, K = 256: 9.9 -> 5.4 us).
// NORM: the rows of A are normalised here (in mode EPI_QKV gathered through ep.idx as well), the sixteen threads of a row
// holding it, and lie in LDS whole.  Every workgroup of a row tile does it again, while its weights are on the way, which
// never cost as much as the norm's own launch: block and merge in a graph, us, C = 64, 128 / 512 rows 31.7 / 37.9 -> 27.3 /
// 32.2, C = 192, 128 / 1024 rows 43.7 / 101.7 -> 38.4 / 97.0, C = 256, 85 / 3900 / 15600 rows 47.6 / 468 / 1830 -> 42.8 / 464
// / 1787.
template <int MODE, bool NORM>
__global__ __launch_bounds__(kTile* kTile) void gemm_f32_kernel(const float* __restrict__ A,
                                                                const float* __restrict__ W, int M, int Nout,
                                                                int K, EpiParams<float> ep) {
  constexpr int PitchA = NORM ? kNormMaxK + 4 : kPitch;
  __shared__ __attribute__((aligned(16))) float As[kTile][PitchA];
  __shared__ __attribute__((aligned(16))) float Ws[kTile][kPitch];
  const int tx = threadIdx.x % kTile, ty = threadIdx.x / kTile;
  const int row = blockIdx.y * kTile + ty;
  const int col = blockIdx.x * kTile + tx;
  const int wr = blockIdx.x * kTile + ty;            // the weight row this thread loads for the tile
  const int m = min(row, M - 1), image = NORM ? m / ep.k : 0;
  const float* ap = A + (NORM && MODE == EPI_QKV ? (int64_t)image * ep.Ntok + min(max(ep.idx[m], 0), ep.Ntok - 1) : m) * (int64_t)K;
  const float* wp = W + (int64_t)min(wr, Nout - 1) * K;
  constexpr int NL = kStepK / kTile;
  float a[NL], w[NL];
  auto request = [&](int k0) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int kk = k0 + tx + i * kTile;
      if (!NORM) a[i] = kk < K ? ap[kk] : 0.f;
      w[i] = kk < K ? wp[kk] : 0.f;
    }
  };
  if constexpr (NORM) {
    // four vectors of a row per thread, summed as a wave of norm.hip does it, which has one per lane: the bits are its bits
    constexpr int NV = kNormMaxK / (4 * kTile);
    f32x4 x[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int at = (j * kTile + tx) * 4;
      x[j] = at < K ? *reinterpret_cast<const f32x4*>(ap + at) : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    request(0);
    float part[NV];
    auto row_sum = [&]() {
#pragma unroll
      for (int j = 0; j < NV; ++j) part[j] = row16_sum(part[j]);
      return (part[3] + part[2]) + (part[1] + part[0]);
    };
    static_assert(NV == 4, "as many as a wave has rows of sixteen lanes");
#pragma unroll
    for (int j = 0; j < NV; ++j) part[j] = ((x[j][0] + x[j][1]) + x[j][2]) + x[j][3];
    const float mean = row_sum() / (float)K;
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      part[j] = 0.f;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float d = (j * kTile + tx) * 4 < K ? x[j][e] - mean : 0.f;
        part[j] = fmaf(d, d, part[j]);
      }
    }
    const float rstd = 1.0f / sqrtf(row_sum() / (float)K + kNormEps);
    // zeros behind the row's end and in a slot past its image's keep count
    const bool live = m - image * ep.k < image_count(ep.k_rows, image, ep.k);
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const int at = (j * kTile + tx) * 4;
      f32x4 o;
#pragma unroll
      for (int e = 0; e < 4; ++e) o[e] = live && at < K ? (x[j][e] - mean) * rstd : 0.f;
      *reinterpret_cast<f32x4*>(&As[ty][at]) = o;
    }
    // per-image cache lengths after this block (the up-projection: everything that reads the old ones has run)
    if (ep.kv_next && blockIdx.x == 0 && blockIdx.y == 0)
      for (int b = threadIdx.x; b * ep.k < M; b += kTile * kTile)
        ep.kv_next[b] = image_prior(ep.kv_rows, b, ep.P) + image_count(ep.k_rows, b, ep.k);
  } else {
    request(0);
  }
  float acc = 0.f;
  for (int k0 = 0; k0 < K; k0 += kStepK) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      if (!NORM) As[ty][tx + i * kTile] = a[i];
      Ws[ty][tx + i * kTile] = w[i];
    }
    __syncthreads();
    if (k0 + kStepK < K) request(k0 + kStepK);
#pragma unroll
    for (int i = 0; i < kStepK; i += 4) {
      const f32x4 av = *reinterpret_cast<const f32x4*>(&As[ty][NORM ? k0 + i : i]), wv = *reinterpret_cast<const f32x4*>(&Ws[tx][i]);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = fmaf(av[e], wv[e], acc);
    }
    __syncthreads();
  }
  if (row < M && col < Nout) epilogue_store<float, MODE>(ep, row, col, acc);
}

// One workgroup per (query row m, head), its waves splitting the keys and then the channels.  Scores of all P+k cached
// keys are kept in LDS.  Bound by latency: with one wave per query and head 128 queries of 4 heads (dh = 16) over 552 keys
// took 31.9 us, one scalar load after the other; now 7.1 us.
constexpr int kAttnWaves = 4;
constexpr int kChannels = 4;               // channels of V a wave sums at a time

__global__ __launch_bounds__(kAttnWaves* NOVA_WAVE) void attention_f32_kernel(const float* __restrict__ q,
                                                                  const float* __restrict__ kc,
                                                                  const float* __restrict__ vc, int k, int C,
                                                                  int heads, int dh, int cap, int kv_total_uniform,
                                                                  float scale, float* __restrict__ out,
                                                                  const int32_t* __restrict__ k_rows,
                                                                  const int32_t* __restrict__ kv_rows, int P,
                                                                  int self_keys) {
  extern __shared__ float sc[];            // [kv_total] scores, then the waves' maxima and sums
  constexpr int NT = kAttnWaves * NOVA_WAVE;
  const int tid = threadIdx.x, lane = tid & (NOVA_WAVE - 1);
  const int wave = __builtin_amdgcn_readfirstlane(tid / NOVA_WAVE);
  const int m = blockIdx.x, head = blockIdx.y;
  const int b = m / k;
  // per-image keep counts: a slot past its image's count gets zeros; an image's keys are its own prior rows plus
  // its own kept rows (never more than the uniform total the LDS was sized for)
  const int kq = image_count(k_rows, b, k);
  if (m - b * k >= kq) {
    for (int d = tid; d < dh; d += NT) out[(int64_t)m * C + head * dh + d] = 0.0f;
    return;
  }
  const int kv_total = self_keys && (k_rows || kv_rows) ? image_prior(kv_rows, b, P) + kq : kv_total_uniform;
  float* red = sc + kv_total;
  const int64_t bh = (int64_t)b * heads + head;
  const float* K = kc + bh * cap * dh;
  const float* V = vc + bh * dh * (int64_t)cap;
  const float* qr = q + (int64_t)m * C + head * dh;      // the same for all threads: scalar loads
  float mx = -INFINITY;
  for (int j = tid; j < kv_total; j += NT) {
    const float* kr = K + (int64_t)j * dh;
    float s = 0.f;
    int d = 0;
    for (; d + 16 <= dh; d += 16) {
      float v[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) v[e] = kr[d + e];
#pragma unroll
      for (int e = 0; e < 16; ++e) s = fmaf(qr[d + e], v[e], s);
    }
    for (; d < dh; ++d) s = fmaf(qr[d], kr[d], s);
    s *= scale;
    sc[j] = s;
    mx = fmaxf(mx, s);
  }
  mx = wave_max(mx);
  if (lane == 0) red[wave] = mx;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kAttnWaves; ++w) mx = fmaxf(mx, red[w]);
  float z = 0.f;
  for (int j = tid; j < kv_total; j += NT) {
    const float e = expf(sc[j] - mx);
    sc[j] = e;
    z += e;
  }
  z = wave_sum(z);
  if (lane == 0) red[kAttnWaves + wave] = z;
  __syncthreads();
  z = 0.f;
#pragma unroll
  for (int w = 0; w < kAttnWaves; ++w) z += red[kAttnWaves + w];
  for (int d0 = wave * kChannels; d0 < dh; d0 += kAttnWaves * kChannels) {
    float a[kChannels] = {};
    const float* vr[kChannels];
#pragma unroll
    for (int c = 0; c < kChannels; ++c) vr[c] = V + (int64_t)min(d0 + c, dh - 1) * cap;
#pragma unroll 4
    for (int j = lane; j < kv_total; j += NOVA_WAVE) {
      const float p = sc[j];
#pragma unroll
      for (int c = 0; c < kChannels; ++c) a[c] = fmaf(p, vr[c][j], a[c]);
    }
#pragma unroll
    for (int c = 0; c < kChannels; ++c) {
      const float s = wave_sum(a[c]);
      if (lane == 0 && d0 + c < dh) out[(int64_t)m * C + head * dh + d0 + c] = s / z;
    }
  }
}

// LDS of attention_f32_kernel: the scores, and dh floats or what the waves exchange
size_t attention_f32_lds(int kv_total, int dh) { return (size_t)(kv_total + std::max(dh, 2 * kAttnWaves)) * sizeof(float); }

template <int MODE, bool NORM = false>
void gemm(hipStream_t st, const float* A, const float* W, int M, int Nout, int K, const EpiParams<float>& ep) {
  dim3 grid((Nout + kTile - 1) / kTile, (M + kTile - 1) / kTile);
  gemm_f32_kernel<MODE, NORM><<<grid, kTile * kTile, 0, st>>>(A, W, M, Nout, K, ep);
}

}  // namespace

hipError_t launch_block_f32(nova_ctx* ctx, hipStream_t st, const nova_block_shape& s, const nova_block_weights& w,
                            const nova_block_variant& var, const RowCounts& rc, const float* x, const int32_t* idx,
                            float* kc, float* vc, float* y, const BlockWorkspace& ws) {
  const int M = s.B * s.k, C = s.C, F = s.C * s.ffn_mult, dh = s.C / s.heads;
  float* u = reinterpret_cast<float*>(ws.u);
  float* q = reinterpret_cast<float*>(ws.q);
  float* attn = reinterpret_cast<float*>(ws.attn);
  float* x1 = reinterpret_cast<float*>(ws.x1);
  float* hid = reinterpret_cast<float*>(ws.hid);

  // per-image conditioning vectors [B, 6, C]: shift1, scale1, gate1, shift2, scale2, gate2
  const float* ada = static_cast<const float*>(var.ada);
  const int ada_pitch = 6 * C;
  auto ada_row = [&](int j) { return ada ? ada + (int64_t)j * C : nullptr; };

  EpiParams<float> ep = {};
  ep.C = C; ep.heads = s.heads; ep.dh = dh; ep.cap = s.kv_capacity; ep.P = s.kv_len; ep.k = s.k;
  ep.k_rows = rc.k_rows; ep.kv_rows = rc.kv_rows;
  ep.idx = idx; ep.Ntok = s.N;
  ep.gate_pitch = ada_pitch;

  hipError_t e = hipSuccess;
  // LayerNorm of src in front of a projection: short rows without modulation are the projection's, others go through u
  auto layer_norm = [&](int stage, const float* src, const int32_t* src_idx, const float* shift, const float* scale,
                        int32_t* kv_next) -> const float* {
    ep.kv_next = kv_next;
    if (!shift && C <= kNormMaxK) return src;
    StageTimer t(stage < 0 ? nullptr : ctx, st, stage);
    e = launch_gather_ln(st, NOVA_F32, src, src_idx, M, s.k, s.N, C, shift, scale, ada_pitch, u, rc.k_rows, rc.kv_rows, kv_next,
                         s.kv_len);
    return u;
  };
  const float* in = layer_norm(NOVA_STAGE_GATHER_LN, x, idx, ada_row(0), ada_row(1), nullptr);
  if (e != hipSuccess) return e;

  ep.bias = static_cast<const float*>(w.b_qkv); ep.out = q; ep.ldo = C; ep.kc = kc; ep.vc = vc;
  {
    StageTimer t(ctx, st, NOVA_STAGE_QKV);
    if (in != u) gemm<EPI_QKV, true>(st, in, static_cast<const float*>(w.w_qkv), M, 3 * C, C, ep);
    else gemm<EPI_QKV>(st, u, static_cast<const float*>(w.w_qkv), M, 3 * C, C, ep);
    if (var.qk_norm) {
      e = launch_qk_norm(st, NOVA_F32, q, kc, var.qk_scale, 1.0f, s.B, s.k, C, s.heads, s.kv_capacity, s.kv_len,
                         rc.k_rows, rc.kv_rows);
      if (e != hipSuccess) return e;
    }
  }

  const int kv_total = s.kv_len + s.k;
  const size_t lds = attention_f32_lds(kv_total, dh);
  {
    StageTimer t(ctx, st, NOVA_STAGE_ATTENTION);
    attention_f32_kernel<<<dim3(M, s.heads), kAttnWaves * NOVA_WAVE, lds, st>>>(q, kc, vc, s.k, C, s.heads, dh, s.kv_capacity,
                                                                   kv_total, var.qk_norm ? 1.0f : 1.0f / sqrtf((float)dh), attn,
                                                                   rc.k_rows, rc.kv_rows, s.kv_len, 1);
  }

  ep.bias = static_cast<const float*>(w.b_o); ep.out = x1; ep.ldo = C; ep.res = x; ep.gate = ada_row(2);
  {
    StageTimer t(ctx, st, NOVA_STAGE_OPROJ);
    gemm<EPI_ATTN_OUT>(st, attn, static_cast<const float*>(w.w_o), M, C, C, ep);
  }
  if (var.w_cq) {
    // cross-attention sub-layer over the condition tokens (see block_bf16.hip)
    in = layer_norm(-1, x1, nullptr, nullptr, nullptr, nullptr);
    if (e != hipSuccess) return e;
    ep.bias = static_cast<const float*>(var.b_cq); ep.out = q; ep.ldo = C; ep.gate = nullptr;
    if (in != u) gemm<EPI_PLAIN, true>(st, in, static_cast<const float*>(var.w_cq), M, C, C, ep);
    else gemm<EPI_PLAIN>(st, u, static_cast<const float*>(var.w_cq), M, C, C, ep);
    const size_t lds_t = attention_f32_lds(var.text_len, dh);
    attention_f32_kernel<<<dim3(M, s.heads), kAttnWaves * NOVA_WAVE, lds_t, st>>>(
        q, static_cast<const float*>(var.k_text), static_cast<const float*>(var.v_text), s.k, C, s.heads, dh,
        var.text_capacity, var.text_len, 1.0f / sqrtf((float)dh), attn, rc.k_rows, nullptr, 0, 0);
    ep.bias = static_cast<const float*>(var.b_co); ep.out = x1; ep.ldo = C; ep.res = x1;
    gemm<EPI_RESIDUAL>(st, attn, static_cast<const float*>(var.w_co), M, C, C, ep);
  }
  in = layer_norm(NOVA_STAGE_LN2, x1, nullptr, ada_row(3), ada_row(4), rc.kv_next);
  if (e != hipSuccess) return e;

  ep.bias = static_cast<const float*>(w.b_fc1); ep.out = hid; ep.ldo = F; ep.gate = nullptr;
  {
    StageTimer t(ctx, st, NOVA_STAGE_FFN1);
    const float* w1 = static_cast<const float*>(w.w_fc1);
    if (in != u && var.gelu_tanh) gemm<EPI_GELU_TANH, true>(st, in, w1, M, F, C, ep);
    else if (in != u) gemm<EPI_GELU, true>(st, in, w1, M, F, C, ep);
    else if (var.gelu_tanh) gemm<EPI_GELU_TANH>(st, u, w1, M, F, C, ep);
    else gemm<EPI_GELU>(st, u, w1, M, F, C, ep);
  }

  ep.bias = static_cast<const float*>(w.b_fc2); ep.out = y; ep.ldo = C; ep.res = x1; ep.gate = ada_row(5);
  {
    StageTimer t(ctx, st, NOVA_STAGE_FFN2);
    gemm<EPI_RESIDUAL>(st, hid, static_cast<const float*>(w.w_fc2), M, C, F, ep);
  }
  return hipGetLastError();
}
