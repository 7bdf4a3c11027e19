// gemm_f32.h - the f32 contraction kernel for 16-byte aligned operands (others take gemm_nt_kernel).
//
// 256 x 64 tile, four wavefronts of 128 x 32 (v_mfma_f32_32x32x2, 64 cycles each), two workgroups per CU.  What bounds it is the f32 MFMA
// rate (157 TFLOP/s at 2.4 GHz), and on this part vector instructions and MFMAs take turns on a SIMD: the register-staged loads of the
// general kernel, their addresses and their stores into LDS took a tenth of the time.  Here slabs (32 k) go straight from memory into
// LDS, addressed like those of the bf16 hot kernel (uniform base + lane offset, no vector operation in the loops of dX and dW; the gathered rows of the forward and dS take four 64-bit adds per two slabs), into two stages of
// 40 KiB.  A slab is four steps of 16 MFMAs, the order written is the order issued: the fragments of a step are read during the
// step before, the last step of a slab runs after the workgroup barrier and covers the first reads of the next slab, and the ten loads of a
// wavefront go out six in that last step and four in the first one, so that they have two steps to land.
// 2175 tokens, H 768, V 50257, us in the general kernel and here: forward 1464 -> 1230 (137 TFLOP/s), dS 1571 -> 1323, dX 1560 -> 1286, dW
// 1502 -> 1291; forward of 8 k tokens 5011 (its 256 x 256 tiles) -> 4393.
// The k of an eight-wide step are added in the order 0 4 1 5 2 6 3 7, like in every other f32 tile.
#pragma once
#include "gemm_nt.h"

namespace rlk {

constexpr int kF32StageBytes = (256 + 64) * kSlabBytes;

// KT: K need not be a multiple of 32 (only of 4): chunks past the end of a row are fetched from a zero block, in a copy of the loop body
// that the last slabs run in.
//
// KM: both operands are given K-major, element (m, k) at A[k * lda + m], (n, k) at B[k * ldb + n] with d.b_k_rows rows of B: dX contracts dS^T, which the
// dW contraction reads too, with W as it is stored, so that neither dS nor W^T has to be made (2175 tokens, H 768, V 50257: the contraction as long as before, 100 us less of dS and 78 of W^T, the call 4318 -> 4139 us).  An LDS row is then one k, of 256 m
// or 64 n, and a fragment four reads of 4 bytes that come in pairs; columns 32 apart are exchanged in every other four rows, so that the lanes' two halves, which
// read rows four apart, meet different banks.  Same products in the same order.  Rows of B past the last are read as the last one: A has zeros there.
template <class Epi, bool KT, bool KM = false>
__global__ __launch_bounds__(256, 2)
void gemm_nt_f32_kernel(const float* __restrict__ A, const float* __restrict__ B, GemmDims d, Epi epi) {
  constexpr int BM = 256, BN = 64, BK = 32, WM = 128, WN = 32, MB = 4, NB = 1;
  constexpr int A_BYTES = BM * kSlabBytes, LDA = 6, LDN = 10;          // loads per slab and wavefront: eight of A, two of B
  constexpr bool GB = Epi::kGatherB;
  static_assert(!KM || (!KT && !GB), "K-major operands: dX");
  typedef Layout32 L;
  __shared__ __attribute__((aligned(1024))) unsigned char stage0[kF32StageBytes];
  __shared__ __attribute__((aligned(1024))) unsigned char stage1[kF32StageBytes];

  const GeneralTile t = general_tile<BM, BN, BK>(d, blockIdx.x);
  if (!t.any) return;
  const int M = t.M, N = t.N, K = t.K;
  const int nk = __builtin_amdgcn_readfirstlane(t.nk), tm = __builtin_amdgcn_readfirstlane(t.tm), tn = __builtin_amdgcn_readfirstlane(t.tn);
  const int k_begin = __builtin_amdgcn_readfirstlane(t.k_begin);

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;

  // ---- slab staging: load j < 8 fills rows 64 w + 8 j .. + 7 of A, load 8 + j rows 16 w + 8 j .. + 7 of B
  // (KM: row 8 w + j of A, rows 8 w + 4 j .. + 3 of B)
  const float* abase = uniform_ptr(A + (KM ? (int64_t)tm * BM : (int64_t)tm * BM * d.lda));
  const float* bbase = uniform_ptr(B + (KM ? (int64_t)tn * BN : (int64_t)tn * BN * d.ldb));
  unsigned aoff[8], boff[2];
  const float* bp[2];
  int bcol[2];
  const int lchunk = lane & 7;
  int row[LDN];                                                       // (row of the slab, for the chunk's place in it)
#pragma unroll
  for (int j = 0; j < LDN; ++j) row[j] = (j < 8 ? wave * 64 + j * 8 : wave * 16 + (j - 8) * 8) + (lane >> 3);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if constexpr (KM) { const int k = wave * 8 + j; aoff[j] = (unsigned)(((int64_t)k * d.lda + ((lane * 4) ^ ((k & 4) << 3))) * 4); continue; }
    const int c = lchunk ^ ((row[j] >> 1) & 7);
    const int r = tm * BM + row[j] < M ? row[j] : M - 1 - tm * BM;
    aoff[j] = (unsigned)(((int64_t)r * d.lda + c * 4) * 4);
  }
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    if constexpr (KM) {
      const int n = ((lane & 15) * 4) ^ (j << 5), nl = d.N - 4 - tn * BN;       // (N % 4 == 0; columns past the last are not written)
      bcol[j] = n < nl ? n : nl;
      boff[j] = (unsigned)(((int64_t)(wave * 8 + j * 4 + (lane >> 4)) * d.ldb + bcol[j]) * 4);
      continue;
    }
    const int c = lchunk ^ ((row[8 + j] >> 1) & 7);
    int r = tn * BN + row[8 + j]; r = r < N ? r : N - 1;
    if constexpr (GB) bp[j] = B + (int64_t)d.b_rows[r] * d.ldb + c * 4;
    else boff[j] = (unsigned)(((int64_t)(r - tn * BN) * d.ldb + c * 4) * 4);
  }
  auto issue1 = [&](bool tail, int slab, unsigned char* stage, int j) __attribute__((always_inline)) {
    unsigned char* dst = j < 8 ? stage + (wave * 64 + j * 8) * kSlabBytes : stage + A_BYTES + (wave * 16 + (j - 8) * 8) * kSlabBytes;
    const int64_t k0 = (int64_t)(k_begin + slab) * BK;
    if constexpr (KM) {
      if (j < 8) load16_to_lds_uniform(abase + k0 * d.lda, aoff[j & 7], stage + (wave * 8 + j) * BM * 4);
      else {
        dst = stage + A_BYTES + (wave * 8 + (j - 8) * 4) * BN * 4;
        if (tail) {
          const int k = (int)k0 + wave * 8 + (j - 8) * 4 + (lane >> 4);
          load16_to_lds_lanes(bbase + (int64_t)(k < d.b_k_rows ? k : d.b_k_rows - 1) * d.ldb + bcol[j & 1], dst);
        } else load16_to_lds_uniform(bbase + k0 * d.ldb, boff[j & 1], dst);
      }
    } else if (KT && tail) {
      const int c = lchunk ^ ((row[j] >> 1) & 7);
      const float* g = j < 8 ? (const float*)((const unsigned char*)abase + aoff[j & 7]) + k0
                             : (GB ? bp[j & 1] : (const float*)((const unsigned char*)bbase + boff[j & 1])) + k0;
      load16_to_lds_lanes(k0 + c * 4 < K ? (const void*)g : (const void*)&kZeroChunk, dst);
    } else if (j < 8) {
      load16_to_lds_uniform(abase + k0, aoff[j & 7], dst);
    } else if constexpr (GB) {
      load16_to_lds_lanes(bp[j & 1] + k0, dst);
    } else {
      load16_to_lds_uniform(bbase + k0, boff[j & 1], dst);
    }
  };

  TileCtx c;
  c.m0 = tm * BM + wm * WM; c.n0 = tn * BN + wn * WN;
  c.Mv = M; c.Nv = N; c.lane = lane; c.wm = wm; c.wn = wn; c.tile_m = tm; c.tile_n = tn; c.tid = tid;
  c.slice = t.slice; c.slices = t.slices;
  const typename Epi::Pre pre = epi.template preload<L>(c, d);

  typename L::acc_t acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int e = 0; e < L::kRegs; ++e) acc[i][0][e] = 0.f;

  const int frow = lane & 31, fq = lane >> 5, swz = (frow >> 1) & 7;
  const int arow = (wm * WM + frow) * kSlabBytes, brow = A_BYTES + (wn * WN + frow) * kSlabBytes;
  u32x4_t fa[2][MB], fb[2];
  auto kof = [&](int k) __attribute__((always_inline)) { return k < nk ? k : nk - 1; };        // past the end: harmless re-load
  // KM: lane (l % 32, l / 32) holds column l % 32 of block i, rows 4 (l / 32) .. + 3 of the step's eight
  const int kcol[2] = {4 * fq * BM * 4 + (wm * WM + (fq << 5) + frow) * 4, 4 * fq * BM * 4 + (wm * WM + ((fq ^ 1) << 5) + frow) * 4};
  const int kbcol = A_BYTES + 4 * fq * BN * 4 + (((wn ^ fq) << 5) + frow) * 4;
  auto km_read = [&](int set, const unsigned char* fstage, int fs, int q) __attribute__((always_inline)) {      // 0 .. 7: half q % 2 of A block q / 2; 8, 9: of B
    const int e = (q & 1) * 2;
    const unsigned char* p = q < 8 ? fstage + kcol[(q >> 1) & 1] + (q >> 2) * 256 + (8 * fs + e) * BM * 4 : fstage + kbcol + (8 * fs + e) * BN * 4;
    u32x4_t& f = q < 8 ? fa[set][(q >> 1) & 3] : fb[set];
    f[e] = *reinterpret_cast<const unsigned*>(p);
    f[e + 1] = *reinterpret_cast<const unsigned*>(p + (q < 8 ? BM : BN) * 4);
  };
  // 16 MFMAs on fragment set `set`; meanwhile the fragments of step fs of fstage into the other set, and loads lo .. lo + n - 1 of a slab
  auto step = [&](bool tail, int set, const unsigned char* fstage, int fs, int slab, unsigned char* wstage, int lo, int n) __attribute__((always_inline)) {
    const int slot = ((fs * 2 + fq) ^ swz) << 4;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
      const int e = q >> 2, i = q & 3;
      acc[i][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(fa[set][i][e]), __uint_as_float(fb[set][e]), acc[i][0], 0, 0, 0);
      if constexpr (KM) { if (q < 10) km_read(set ^ 1, fstage, fs, q); }
      else if (q < 4) fa[set ^ 1][q] = *reinterpret_cast<const u32x4_t*>(fstage + arow + q * 32 * kSlabBytes + slot);
      else if (q == 4) fb[set ^ 1] = *reinterpret_cast<const u32x4_t*>(fstage + brow + slot);
      if (q >= 5 && (q & 1) && (q - 5) / 2 < n) issue1(tail, slab, wstage, lo + (q - 5) / 2);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto slab = [&](bool tail, unsigned char* cur, unsigned char* nxt, int kt) __attribute__((always_inline)) {
    step(tail, 0, cur, 1, kof(kt + 1), nxt, LDA, LDN - LDA);
    step(tail, 1, cur, 2, 0, nxt, 0, 0);
    step(tail, 0, cur, 3, 0, nxt, 0, 0);
    __builtin_amdgcn_s_waitcnt(0x0070);     // vmcnt(0) lgkmcnt(0)
    __syncthreads();
    step(tail, 1, nxt, 0, kof(kt + 2), cur, 0, LDA);
  };
  if (nk > 0) {
#pragma unroll
    for (int j = 0; j < LDN; ++j) issue1(true, 0, stage0, j);
    __builtin_amdgcn_s_waitcnt(0x0F70);     // vmcnt(0)
    __syncthreads();
#pragma unroll
    for (int j = 0; j < LDA; ++j) issue1(true, kof(1), stage1, j);
    if constexpr (KM) {
#pragma unroll
      for (int q = 0; q < 10; ++q) km_read(0, stage0, 0, q);
    } else {
      const int slot = (fq ^ swz) << 4;
#pragma unroll
      for (int i = 0; i < MB; ++i) fa[0][i] = *reinterpret_cast<const u32x4_t*>(stage0 + arow + i * 32 * kSlabBytes + slot);
      fb[0] = *reinterpret_cast<const u32x4_t*>(stage0 + brow + slot);
    }
    int kt = 0;
    // (the last slab's loads go out up to two slabs ahead; KM: K is B's rows rounded up to 256, eight slabs)
    constexpr int LAST = KM ? 10 : 3;
    const bool has_tail = KT || (KM && (k_begin + nk) * BK > d.b_k_rows);
    const int plain = has_tail ? (nk > LAST + 1 ? (nk - LAST) & ~1 : 0) : nk & ~1;
    for (; kt < plain; kt += 2) {
      slab(false, stage0, stage1, kt);
      slab(false, stage1, stage0, kt + 1);
    }
    if constexpr (KT || KM)
      for (; kt + 1 < nk; kt += 2) {
        slab(true, stage0, stage1, kt);
        slab(true, stage1, stage0, kt + 1);
      }
    if (kt < nk) slab(KT || KM, stage0, stage1, kt);
  }
  __builtin_amdgcn_s_waitcnt(0x0070);       // trailing re-loads must land before the epilogue reuses LDS
  __syncthreads();
  epi.template run<L, MB, NB, BM, BN, 2, 2, false>(acc, c, stage0, d, pre);
}

}  // namespace rlk
