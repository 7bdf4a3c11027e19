// logz_head.h - the log-Z head: per-prompt log-partition estimate from the prompt's hidden states.
//
//   pooled_p = mean of the prompt's hidden-state rows        logz_pool_kernel   (HBM-bound: reads the rows once)
//   a_p = W1 pooled_p + b1,  g_p = gelu(a_p)                 logz_hidden_kernel (HBM-bound: W1 streamed once per 16 prompts)
//   logZ_p = w2 . g_p + b2                                   logz_out_kernel, few units: by the last workgroup of the hidden layer
//   backward from d_logZ: db2, db1, dw2, dW1 = sum_p da_p pooled_p^T   logz_bwd_kernel (HBM-bound: writes dW1 once)
//
// The hidden states are constants here (no gradient into the language model).  Parameters and
// activations are f32; the hidden states come in the model's dtype.  With 16-32 prompts the layer is a matrix-vector product
// per prompt, bound by reading the hidden states and W1 and writing dW1 once (H = M = 3584, 16 prompts of 7050 rows: 153 MB,
// 32 us at the rate of a large copy), so every kernel moves 16 bytes per lane and keeps many loads in flight.
#pragma once
#include "gemm_nt.h"

namespace rlk {

__device__ inline float gelu_f(float a) { return 0.5f * a * (1.f + erff(a * 0.70710678118654752f)); }
__device__ inline float gelu_grad_f(float a) {
  return 0.5f * (1.f + erff(a * 0.70710678118654752f)) + a * expf(-0.5f * a * a) * 0.3989422804014327f;
}

// A piece of VEC consecutive elements of a row as f32.  VEC > 1: 16 bytes, for rows that are 16-byte aligned.
template <class T, int VEC> __device__ inline void logz_load(const T* p, float (&v)[VEC]) {
  if constexpr (VEC == 1) {
    v[0] = (float)p[0];
  } else {
    T e[VEC];
    const uint4 q = *reinterpret_cast<const uint4*>(p);
    __builtin_memcpy(e, &q, 16);
#pragma unroll
    for (int i = 0; i < VEC; ++i) v[i] = (float)e[i];
  }
}

// grid (P, ceil(H / (LANES VEC))): a workgroup of eight wavefronts pools LANES VEC columns of one prompt, 512 / LANES rows at a
// time, four pieces in flight per lane (eight: no faster, f32 at H 3584 64 prompts of 40 rows 10.6 us instead of 9.9); f32 sums, merged through LDS in a fixed order.
// (One element per lane, 64 columns per workgroup: 22 us on the shape above, 16 bytes per lane: 14 us.)
template <int VEC> constexpr int logz_pool_lanes() { return VEC == 1 ? 64 : 16; }
template <class T, int VEC>
__global__ __launch_bounds__(512) void logz_pool_kernel(const T* X, int64_t rows, int H, const int32_t* cu, float* pooled, int* done) {
  constexpr int LANES = logz_pool_lanes<VEC>(), SLICES = 512 / LANES;
  __shared__ float part[SLICES][LANES * VEC + 1];
  const int p = blockIdx.x, c = threadIdx.x % LANES, slice = threadIdx.x / LANES;
  const int h = (blockIdx.y * LANES + c) * VEC;
  if (blockIdx.y == 0 && p % 16 == 0 && threadIdx.x == 0) done[p / 16] = 0;
  int64_t a = cu[p], b = cu[p + 1];
  if (a < 0) a = 0;
  if (b > rows) b = rows;
  float s[4][VEC];
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int i = 0; i < VEC; ++i) s[u][i] = 0.f;
  if (h < H) {
    const T* x = X + h;
    int64_t r = a + slice;
    for (; r + 3 * SLICES < b; r += 4 * SLICES) {
      float v[4][VEC];
#pragma unroll
      for (int u = 0; u < 4; ++u) logz_load<T, VEC>(x + (r + SLICES * u) * H, v[u]);
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int i = 0; i < VEC; ++i) s[u][i] += v[u][i];
    }
    for (; r < b; r += SLICES) {
      float v[VEC];
      logz_load<T, VEC>(x + r * H, v);
#pragma unroll
      for (int i = 0; i < VEC; ++i) s[0][i] += v[i];
    }
  }
#pragma unroll
  for (int i = 0; i < VEC; ++i) part[slice][c * VEC + i] = (s[0][i] + s[1][i]) + (s[2][i] + s[3][i]);
  __syncthreads();
  if (threadIdx.x < LANES * VEC) {
    const int hh = blockIdx.y * LANES * VEC + threadIdx.x;
    if (hh < H) {
      float t = 0.f;
      for (int k = 0; k < SLICES; ++k) t += part[k][threadIdx.x];
      pooled[(int64_t)p * H + hh] = b > a ? t / (float)(b - a) : 0.f;
    }
  }
}

// Hidden layer.  grid (ceil(M / 16), ceil(P / 16)): a workgroup computes 16 units for 16 prompts with v_mfma_f32_16x16x4 (A = rows
// of W1, B = rows of the pooled states, both straight from memory in operand layout: lane l holds row l%16, four
// consecutive k of every 16), its eight wavefronts taking 16-wide k-steps in turn, eight in flight, into twelve
// accumulators: a chain adds at most H / 64 products, and few MFMAs wait for the one before them (one accumulator, H / 8 products: the layer's
// relative error at H = 3584 is 4.1e-7 against 1.5e-7, in the same time).  These are added in pairs, and so are the eight partial blocks,
// through LDS.  (Sixteen accumulators leave one workgroup per CU: 64 prompts at H = M = 5120 took 1.2 % longer.)  VEC: rows are
// 16-byte aligned (else element loads).  (The vector-FMA form with the pooled states in LDS was bound by its LDS reads: 94 us against
// 18 us on the shape above.)
// part_z != nullptr: log Z too.  A workgroup adds up its units' w2 g and the one that is last of its 16 prompts the workgroups', which it may read because the
// count that announces a sum is a release and an acquire at device scope, behind a barrier of the workgroup that wrote it.  That writes back what the L2 holds: forward + backward of 16 prompts, H 3584,
// M 1024 32.5 us, 32.2 with sums that go past the L2s and no more than a wait ahead of the count, 34.2 with the launch that this saves; one prompt of 20 rows,
// H 100, M 64 25.2 of 27.6 us, 4 of 800, H = M = 1024 24.8 of 27.2 (called from Python).  Many
// workgroups count one after the other: 40 prompts, H 300, M 3000 14.3 -> 17.6 (the forward), on the shape above no gain.  So up to kLogzSumUnits units and 16 prompts (33 prompts, M 500
// 30.1 -> 30.5).
constexpr int kLogzSumUnits = 1024;
constexpr int kLogzWaves = 8;
template <bool VEC>
__global__ __launch_bounds__(kLogzWaves * 64, 4) void logz_hidden_kernel(const float* W1, const float* b1, const float* pooled, int P, int H, int M,
                                                          float* a_out, float* g_out, const float* w2, const float* b2, float* part_z, int* done, float* log_z) {
  constexpr int WAVES = kLogzWaves, STEP = 16 * WAVES;
  __shared__ float part[WAVES][16][17];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, row = lane & 15, kq = lane >> 4;
  const int j0 = blockIdx.x * 16, p0 = blockIdx.y * 16, np = P < 16 ? P : 16;
  const int j = j0 + row < M ? j0 + row : M - 1, p = p0 + row < P ? p0 + row : P - 1;       // (rows past the end: not written)
  const float* w = W1 + (int64_t)j * H;
  const float* x = pooled + (int64_t)p * H;
  auto load = [&](const float* q, int k) __attribute__((always_inline)) {
    floatx4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = 0.f;
    if constexpr (VEC) { if (k < H) v = *reinterpret_cast<const floatx4*>(q + k); }          // (H % 4 == 0)
    else {
#pragma unroll
      for (int e = 0; e < 4; ++e) if (k + e < H) v[e] = q[k + e];
    }
    return v;
  };
  floatx4 acc[12];
#pragma unroll
  for (int u = 0; u < 12; ++u)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[u][e] = 0.f;
  for (int k0 = wave * 16; k0 < H; k0 += 8 * STEP) {
    floatx4 a[8], b[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) { a[u] = load(w, k0 + STEP * u + 4 * kq); b[u] = load(x, k0 + STEP * u + 4 * kq); }
#pragma unroll
    for (int u = 0; u < 8; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[2 * (u % 6) + (e & 1)] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][e], b[u][e], acc[2 * (u % 6) + (e & 1)], 0, 0, 0);
  }
#pragma unroll
  for (int u = 0; u < 6; ++u) acc[u] += acc[u + 6];
  acc[0] = ((acc[0] + acc[3]) + (acc[1] + acc[4])) + (acc[2] + acc[5]);
#pragma unroll
  for (int e = 0; e < 4; ++e) part[wave][row][4 * kq + e] = acc[0][e];                        // [prompt][unit]
  __syncthreads();
  if (threadIdx.x < 256) {
    const int u = threadIdx.x & 15, q = threadIdx.x >> 4;
    float s[WAVES];
#pragma unroll
    for (int k = 0; k < WAVES; ++k) s[k] = part[k][q][u];
#pragma unroll
    for (int o = 1; o < WAVES; o <<= 1)
#pragma unroll
      for (int k = 0; k < WAVES; k += 2 * o) s[k] += s[k + o];
    float z = 0.f;
    if (j0 + u < M && p0 + q < P) {
      const float v = s[0] + b1[j0 + u], gv = gelu_f(v);
      a_out[(int64_t)(p0 + q) * M + j0 + u] = v; g_out[(int64_t)(p0 + q) * M + j0 + u] = gv;
      if (part_z) z = w2[j0 + u] * gv;
    }
    if (part_z) {
#pragma unroll
      for (int o = 8; o > 0; o >>= 1) z += __shfl_xor(z, o);
      if (u == 0 && q < np) part_z[((int64_t)blockIdx.y * gridDim.x + blockIdx.x) * np + q] = z;
    }
  }
  if (!part_z) return;
  __shared__ int last;
  __syncthreads();
  if (threadIdx.x == 0) last = __hip_atomic_fetch_add(done + blockIdx.y, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == (int)gridDim.x - 1;
  __syncthreads();
  if (!last) return;
  const int q = threadIdx.x & 15, t = threadIdx.x >> 4;                                     // prompt; workgroups t, t + 4 WAVES, ...
  const float* z = part_z + (int64_t)blockIdx.y * gridDim.x * np + (q < np ? q : 0);
  float s = 0.f;
#pragma unroll 4
  for (int k = t; k < (int)gridDim.x; k += 4 * WAVES) s += z[(int64_t)k * np];
  s += __shfl_xor(s, 16); s += __shfl_xor(s, 32);
  if (lane < 16) part[wave][0][lane] = s;
  __syncthreads();
  if (threadIdx.x < 16 && p0 + q < P) {
    float v = 0.f;
#pragma unroll
    for (int k = 0; k < WAVES; ++k) v += part[k][0][q];
    log_z[p0 + q] = v + b2[0];
  }
}

// one workgroup per prompt: logZ_p = w2 . g_p + b2, where the hidden layer has not done it.  Latency only: many threads, their loads ahead of the additions.
constexpr int kLogzOutThreads = 1024;
__global__ __launch_bounds__(kLogzOutThreads) void logz_out_kernel(const float* g, const float* w2, const float* b2, int M, float* log_z) {
  __shared__ float sh[kLogzOutThreads / 64];
  const int p = blockIdx.x;
  float s = 0.f;
#pragma unroll 4
  for (int j = threadIdx.x; j < M; j += blockDim.x) s += w2[j] * g[(int64_t)p * M + j];
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x >= 64) return;
  s = threadIdx.x < blockDim.x / 64 ? sh[threadIdx.x] : 0.f;
  for (int o = kLogzOutThreads / 128; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if (threadIdx.x == 0) log_z[p] = s + b2[0];
}

// Backward: a workgroup takes eight units.  Per 32 prompts it forms da[p][j] = d_p w2_j gelu'(a[p][j]) in LDS, adds up
// db1_j and dw2_j, and accumulates dW1[j][h] = sum_p da[p][j] pooled[p][h], VEC columns x eight units per thread; workgroup 0
// also writes db2.  With more than 32 prompts or more than 256 VEC columns the da are formed again for every pass over
// the columns (a few hundred values).  grid (ceil(M / 8), ceil(H / (256 VEC))); the column blocks other than the first skip the sums.
// (da by a kernel of its own and single-element stores: 11 + 37 us on the shape above, fused with 16-byte stores: 16.5 us.)
// NT: the stores are non-temporal, where dW1 is whole lines of 128 bytes in every row and too large for the L2s to keep (logz_nontemporal): on buffers that no cache holds,
// forward + backward 57.9 -> 54.6 us, 64 prompts at H = M = 5120 227 -> 215; H 300, M 3000, rows of 1200 bytes, loses 0.8 of 11.1, and a dW1 of 4 MB gains nothing.
static inline bool logz_nontemporal(int M, int H, const float* dW1) { return H % 32 == 0 && reinterpret_cast<uintptr_t>(dW1) % 128 == 0 && (int64_t)M * H >= (1 << 21); }
template <int VEC, bool NT>
__global__ __launch_bounds__(256) void logz_bwd_kernel(const float* d, const float* a, const float* g, const float* w2, const float* pooled,
                                                       int P, int M, int H, float* dW1, float* db1, float* dw2, float* db2) {
  __shared__ float da[32][8], dg[32][8];
  const int t = threadIdx.x, j0 = blockIdx.x * 8, h = (blockIdx.y * 256 + t) * VEC;
  const bool first = blockIdx.y == 0;
  float s[8][VEC], sum = 0.f;
#pragma unroll
  for (int u = 0; u < 8; ++u)
#pragma unroll
    for (int i = 0; i < VEC; ++i) s[u][i] = 0.f;
  const int u8 = t & 7, q = t >> 3, j = j0 + u8;             // 32 prompts x 8 units
  for (int p0 = 0; p0 < P; p0 += 32) {
    __syncthreads();
    float v = 0.f, dw = 0.f;
    if (p0 + q < P && j < M) {
      const float dp = d[p0 + q];
      const int64_t at = (int64_t)(p0 + q) * M + j;
      v = dp * w2[j] * gelu_grad_f(a[at]);
      if (first) dw = dp * g[at];
    }
    da[q][u8] = v; dg[q][u8] = dw;
    __syncthreads();
    const int np = P - p0 < 32 ? P - p0 : 32;
    if (h < H)
#pragma unroll 4
      for (int p = 0; p < np; ++p) {
        float x[VEC];
        logz_load<float, VEC>(pooled + (int64_t)(p0 + p) * H + h, x);
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
          for (int i = 0; i < VEC; ++i) s[u][i] = fmaf(da[p][u], x[i], s[u][i]);
      }
    if (first && t < 16)                                     // threads 0..7: db1, 8..15: dw2, prompts in order
      for (int p = 0; p < np; ++p) sum += t < 8 ? da[p][t] : dg[p][t - 8];
  }
  if (h < H)
#pragma unroll
    for (int u = 0; u < 8; ++u)
      if (j0 + u < M) {
        float* o = dW1 + (int64_t)(j0 + u) * H + h;
        if constexpr (VEC == 4) { floatx4 v; v[0] = s[u][0]; v[1] = s[u][1]; v[2] = s[u][2]; v[3] = s[u][3]; if constexpr (NT) __builtin_nontemporal_store(v, reinterpret_cast<floatx4*>(o)); else *reinterpret_cast<floatx4*>(o) = v; }
        else o[0] = s[u][0];
      }
  if (first && t < 16 && j0 + (t & 7) < M) (t < 8 ? db1 : dw2)[j0 + (t & 7)] = sum;
  if (first && blockIdx.x == 0 && t == 16) { float b = 0.f; for (int p = 0; p < P; ++p) b += d[p]; db2[0] = b; }
}

struct LogzPlan { size_t off_pooled, off_a, off_g, off_part, total; };

static inline LogzPlan logz_plan(int P, int H, int M) {
  LogzPlan q; size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o += (bytes + 255) & ~(size_t)255; return at; };
  q.off_pooled = take(4 * (size_t)P * H); q.off_a = take(4 * (size_t)P * M); q.off_g = take(4 * (size_t)P * M);
  q.off_part = take(4 * (size_t)P * M);        // counts and partial sums of log Z (more than they need: the size is part of the interface)
  q.total = o;
  return q;
}

}  // namespace rlk
