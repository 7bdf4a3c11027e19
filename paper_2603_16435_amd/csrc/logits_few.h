// logits_few.h - the logits of a few tokens (bf16), up to 128.
//
// What bounds it is reading W once.  The hot kernel has one workgroup per 256 vocabulary rows, 125 of them for V = 32000, two slabs in
// flight each, and multiplies 256 columns whatever the number of tokens.  Here a workgroup takes 128 rows (four wavefronts of 128 x BN / 4), and
// three slabs of 64 k are on their way while a fourth is computed on.  99 tokens, H 2048, V 32000 (131 MB: 26 us at the rate of a large
// copy): 46 us in the hot kernel, 32 here; 16 or 64 tokens 46 -> 27; 100 tokens, H 5120, V 1000 89 -> 65; H 512, V 10000 22 -> 11.
// Same MFMA and order of k as the hot kernel, and the softmax sums of a half tile are those of its wavefronts: lse_combine_kernel<true> merges two halves as
// that kernel's epilogue does, so that a token's log-prob does not depend on how many rows are scored with it.
#pragma once
#include "epilogues.h"

namespace rlk {

constexpr int kFewTokens = 128;

constexpr int kFewStages = 4;
template <int BN> constexpr int few_lds_bytes() { return kFewStages * (128 + BN) * kSlabBytes; }
// The work of workgroup `tile` of the launch, N tokens whose rows of X are in `rows`, their sampled tokens in `ids`.  BN: tokens per workgroup, 64 or 128.
// NT: W in non-temporal loads.  They stream faster (7.2 TB/s of a large array instead of 6.1), and leave nothing behind for a next call: for a W that the memory-side
// cache does not hold (few_streams_w).
template <int BN, bool NT>
__device__ __attribute__((always_inline)) inline void logits_few_tile(const bf16_t* __restrict__ W, const bf16_t* __restrict__ X, const GemmDims& d, const EpiFwd<bf16_t>& epi,
                                                                      int tile, int N, const int* rows, const int* ids, unsigned char* smem) {
  constexpr int BM = 128, BK = 64, MB = 8, NB = BN / 64, STAGES = kFewStages;
  constexpr int A_BYTES = BM * kSlabBytes, STAGE = A_BYTES + BN * kSlabBytes, LA = BM / 32, LB = BN / 32, LOADS = LA + LB;   // loads per slab and wavefront
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  if (N <= 0) return;
  const int K = d.K, nk = (K + BK - 1) / BK, m0 = tile * BM;

  const bf16_t* wbase = W + (int64_t)(m0 < d.M ? m0 : 0) * d.lda;       // (a half tile of nothing but padding: any rows)
  unsigned off[LOADS];
  int chunk[LOADS];
#pragma unroll
  for (int j = 0; j < LOADS; ++j) {
    const int lr = (j < LA ? wave * (BM / 4) + j * 8 : wave * (BN / 4) + (j - LA) * 8) + (lane >> 3);
    chunk[j] = (lane & 7) ^ ((lr >> 1) & 7);
    int r;
    if (j < LA) { const int last = (m0 < d.M ? d.M - m0 : d.M) - 1; r = lr < last ? lr : last; }
    else r = rows[lr < N ? lr : N - 1];
    off[j] = (unsigned)(((int64_t)r * (j < LA ? d.lda : d.ldb) + chunk[j] * 8) * 2);      // (128 rows of X: far below 4 GiB)
  }
  auto issue = [&](int kt) __attribute__((always_inline)) {
    const int k = kt < nk ? kt : nk - 1;                                // past the end: a harmless re-load keeps the count of loads
    unsigned char* stage = smem + (kt & (STAGES - 1)) * STAGE;
    const bool tail = (k + 1) * BK > K;
#pragma unroll
    for (int j = 0; j < LOADS; ++j) {
      unsigned char* dst = j < LA ? stage + (wave * (BM / 4) + j * 8) * kSlabBytes : stage + A_BYTES + (wave * (BN / 4) + (j - LA) * 8) * kSlabBytes;
      const bf16_t* base = (j < LA ? wbase : X) + (int64_t)k * BK;
      if (tail) load16_to_lds_lanes(k * BK + chunk[j] * 8 < K ? (const void*)((const unsigned char*)base + off[j]) : (const void*)&kZeroChunk, dst);
      else if (j < LA) load16_to_lds_uniform<NT>(base, off[j], dst);
      else load16_to_lds_uniform(base, off[j], dst);
    }
  };

  TileCtx c;
  c.m0 = m0; c.n0 = wave * (BN / 4);
  c.Mv = d.M; c.Nv = N; c.lane = lane; c.wm = 0; c.wn = wave; c.tile_m = tile; c.tile_n = 0; c.tid = tid; c.slice = 0; c.slices = 1;
  int y[NB];
#pragma unroll
  for (int bj = 0; bj < NB; ++bj) { const int n = c.n0 + Layout16::col(bj, lane); y[bj] = n < N ? ids[n] : -1; }

  floatx4 acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

  __builtin_amdgcn_s_waitcnt(0x0F70);       // vmcnt(0): what was fetched above is not among the loads counted below
#pragma unroll
  for (int s = 0; s < STAGES - 1; ++s) issue(s);
  const int frow = lane & 15, fq = lane >> 4, swz = (frow >> 1) & 7;
  constexpr int PEND = (STAGES - 2) * LOADS;
  for (int kt = 0; kt < nk; ++kt) {
    __builtin_amdgcn_s_waitcnt(0x0070 | (PEND & 15) | (PEND >> 4) << 14);       // all but the two slabs behind this one; lgkmcnt(0)
    __syncthreads();                        // ... in every wavefront, and the stage filled next has been read
    issue(kt + STAGES - 1);
    const unsigned char* stage = smem + (kt & (STAGES - 1)) * STAGE;
    u32x4_t fa[2][MB], fb[2][NB];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int slot = ((s * 4 + fq) ^ swz) << 4;
#pragma unroll
      for (int i = 0; i < MB; ++i) fa[s][i] = *reinterpret_cast<const u32x4_t*>(stage + (i * 16 + frow) * kSlabBytes + slot);
#pragma unroll
      for (int j = 0; j < NB; ++j) fb[s][j] = *reinterpret_cast<const u32x4_t*>(stage + A_BYTES + (wave * (BN / 4) + j * 16 + frow) * kSlabBytes + slot);
    }
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int i = 0; i < MB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, fa[s][i]), __builtin_bit_cast(bf16x8, fb[s][j]), acc[i][j], 0, 0, 0);
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);       // no load into LDS may be in flight when the workgroup gives its LDS back
  epi.half_tile<Layout16, MB, NB>(acc, c, y);
}

}  // namespace rlk
