// grads_small.h - dX and dW of a small f32 batch, straight from the logits that its forward kept.
//
//   dX[t][h] = sum_v dS[t][v] W[v][h]        dW[v][h] = sum_t dS[t][v] X[t][h]        dS[t][v] = zs c_t (1[v = y_t] - exp(zs z[v][t] - lse_t))
//
// A batch of a few hundred tokens of a small model is bound by latency: launches, and chains of load, barrier and MFMA.  So there is one launch
// (dS in memory, its transpose, W^T and X^T are not made) without LDS slabs: v_mfma_f32_16x16x4 takes one element of each operand per lane, and sixteen
// lanes reading sixteen consecutive elements of a row of W or X, or of z, is what its operands look like where the contracted index is the
// row.  A workgroup has one block of 16 x 16 NB outputs; its sixteen wavefronts share out the contracted index in pieces (32 vocabulary entries, 16 tokens), whose loads do not depend
// on each other, and their sums are added in order through LDS.  dS is formed in registers, in the arithmetic of kept_ds_f32_kernel, once per
// block of columns: H / 32 or H / 64 times for dX, H / 64 for dW.
// 356 tokens, H 128, V 1024: transposes, dS, the contractions in tiles of 64 x 16 through LDS and the sum of dX's slices took 27 us of a call of 50.6 us; this
// launch takes 7 of 28 (3.7 until its sums are formed, bound by the exponentials, 3 until the slowest wavefront's have been added).
#pragma once
#include "epilogues.h"

namespace rlk {

struct SmallGrads {
  KeptJob j; const float* kept; int64_t ld;             // kept logits [vocabulary][ld tokens], ld and the array multiples of 16 tokens / 16 bytes
  const float *X, *W; const int* row_map; int H;
  float *dX, *dW;
  int x_cols, dx_blocks;                                // dX: blocks of columns, workgroups
};
constexpr int kGradWaves = 16, kGradNBW = 4;

__device__ __attribute__((always_inline)) inline float small_ds(float z, bool target, float ct, float lse, float zs) {
  return ct * ((target ? 1.f : 0.f) - fast_exp<float>(z * zs - lse));
}

// sums of the wavefronts, in a fixed tree -> out(row, column, sum) of the block; a thread has one element at most, row small_row()
__device__ inline int small_row() { return (((int)threadIdx.x >> 6 & 3) << 2) + ((int)threadIdx.x & 3); }
template <int NB, class Out>
__device__ __attribute__((always_inline)) inline void small_reduce(const floatx4 (&acc)[NB], float* part, Out out) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, q = threadIdx.x;
#pragma unroll
  for (int j = 0; j < NB; ++j) *reinterpret_cast<floatx4*>(part + ((wave * NB + j) * 64 + lane) * 4) = acc[j];
  __syncthreads();
  if (q >= NB * 256) return;
  float s[kGradWaves];
#pragma unroll
  for (int w = 0; w < kGradWaves; ++w) s[w] = part[w * NB * 256 + q];
#pragma unroll
  for (int o = 1; o < kGradWaves; o <<= 1)
#pragma unroll
    for (int w = 0; w < kGradWaves; w += 2 * o) s[w] += s[w + o];
  out(small_row(), (q >> 8) * 16 + (q >> 2 & 15), s[0]);
}

// Workgroup `block` of the launch.  NBX: blocks of 16 columns of a dX workgroup; U: pieces whose loads go out together (two of 16 for dX, one for dW).
template <int NBX, int U>
__device__ __attribute__((always_inline)) inline void small_grads(const SmallGrads& s, int block) {
  __shared__ __attribute__((aligned(16))) float part[kGradWaves * kGradNBW * 256];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), r = lane & 15, g = lane >> 4;
  const int n_real = *s.j.n_real, V = s.j.V, H = s.H;
  const float zs = s.j.zs;
  if (block < s.dx_blocks) {                            // ---- 16 tokens x 16 NBX columns, K = vocabulary
    constexpr int NB = NBX, E = 8 * U;
    const int t0 = block / s.x_cols * 16, h0 = block % s.x_cols * 16 * NB;
    const int t = t0 + r, out_row = s.row_map[t0 + small_row()];        // (the token arrays have room past the last)
    const int yt = s.j.ids_c[t];
    const float lset = s.j.lse_c[t], cc = s.j.c_c[t];
    if (t0 >= n_real) return;
    const bool valid = t < n_real;
    const int y = valid ? yt : -1;
    const float lse = valid ? lset : 0.f, ct = valid ? cc * zs : 0.f;
    floatx4 acc[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int v0 = wave * 4 * E; v0 < V; v0 += kGradWaves * 4 * E) {
      float a[E], b[E][NB];
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int v = v0 + 16 * (e >> 2) + 4 * g + (e & 3);
        a[e] = v < V ? s.kept[(int64_t)v * s.ld + t] : 0.f;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          const int h = h0 + j * 16 + r;
          b[e][j] = v < V && h < H ? s.W[(int64_t)v * H + h] : 0.f;
        }
      }
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int v = v0 + 16 * (e >> 2) + 4 * g + (e & 3);
        const float ds = small_ds(a[e], v == y, ct, lse, zs), x = valid && v < V ? ds : 0.f;
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, b[e][j], acc[j], 0, 0, 0);
      }
    }
    small_reduce<NB>(acc, part, [&](int row, int col, float v) __attribute__((always_inline)) {
      if (t0 + row < n_real && h0 + col < H) s.dX[(int64_t)out_row * H + h0 + col] = v;
    });
  } else {                                              // ---- 16 vocabulary entries x 64 columns, K = tokens
    constexpr int NB = kGradNBW;
    const int cols = (H + 16 * NB - 1) / (16 * NB), q = block - s.dx_blocks;
    const int m0 = q / cols * 16, h0 = q % cols * 16 * NB, v = m0 + r;
    floatx4 acc[NB];
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[j] = floatx4{0.f, 0.f, 0.f, 0.f};
    for (int t0 = wave * 16; t0 < n_real; t0 += kGradWaves * 16 * U) {
      floatx4 z[U], lse[U], c[U];
      int4 y[U], row[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int tb = t0 + u * kGradWaves * 16, t = (tb < n_real ? tb : t0) + 4 * g;     // the lane's four tokens
        z[u] = *reinterpret_cast<const floatx4*>(s.kept + (int64_t)v * s.ld + t);
        lse[u] = *reinterpret_cast<const floatx4*>(s.j.lse_c + t); c[u] = *reinterpret_cast<const floatx4*>(s.j.c_c + t);
        y[u] = *reinterpret_cast<const int4*>(s.j.ids_c + t); row[u] = *reinterpret_cast<const int4*>(s.row_map + t);
      }
      float b[U][4][NB];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int t = t0 + u * kGradWaves * 16 + 4 * g, re[4] = {row[u].x, row[u].y, row[u].z, row[u].w};
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            const int h = h0 + j * 16 + r;
            b[u][e][j] = t + e < n_real && h < H ? s.X[(int64_t)re[e] * H + h] : 0.f;
          }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int t = t0 + u * kGradWaves * 16 + 4 * g, ye[4] = {y[u].x, y[u].y, y[u].z, y[u].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float ds = small_ds(z[u][e], v == ye[e], c[u][e] * zs, lse[u][e], zs), x = t + e < n_real && v < V ? ds : 0.f;
#pragma unroll
          for (int j = 0; j < NB; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(x, b[u][e][j], acc[j], 0, 0, 0);
        }
      }
    }
    small_reduce<NB>(acc, part, [&](int rr, int col, float x) __attribute__((always_inline)) {
      if (m0 + rr < V && h0 + col < H) s.dW[(int64_t)(m0 + rr) * H + h0 + col] = x;
    });
  }
}

}  // namespace rlk
