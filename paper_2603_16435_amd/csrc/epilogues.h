// epilogues.h - what each contraction does with its accumulators while they are in registers.
//
// Orientation.  The logits contraction is run "vocab-major": A = W (rows = vocab entries),
// B = X (rows = tokens), so that in the MFMA accumulator layouts (see Layout32 / Layout16) a lane
// owns ONE token column per block and several vocab rows of it.  The softmax reductions over the
// vocabulary are then mostly in-register; the only cross-lane steps are between the lane groups
// that hold other rows of the same column (one or two shuffles), and the only cross-wavefront
// step is between the WAVES_M wavefronts stacked along the vocabulary.
#pragma once
#include "gemm_nt.h"

namespace rlk {

// 16-byte store of eight bf16 that nobody re-reads from cache (the chunk buffers are 10 GB): non-temporal,
// measured 26 % cheaper than a plain store in the tile-writing epilogues.
template <class T>
__device__ inline void store_stream(T* p, const bf16x8& v) { __builtin_nontemporal_store(v, reinterpret_cast<bf16x8*>(p)); }

template <class T> __device__ inline float fast_exp(float x);
template <> __device__ inline float fast_exp<bf16_t>(float x) { return __expf(x); }
template <> __device__ inline float fast_exp<float>(float x) { return expf(x); }

constexpr float kLog2e = 1.4426950408889634f;

// exp(zs z - m) for a raw logit z, the inverse temperature zs and a shift m given in tempered units, with
// m*log2(e) and zs*log2(e) precomputed: one fma and one v_exp for bf16 inputs, the accurate libm path for f32
template <class T> __device__ inline float exp_shifted(float z, float m, float m_l2e, float zs, float zs_l2e);
template <> __device__ inline float exp_shifted<bf16_t>(float z, float, float m_l2e, float, float zs_l2e) {
  return __builtin_amdgcn_exp2f(__builtin_fmaf(z, zs_l2e, -m_l2e));
}
template <> __device__ inline float exp_shifted<float>(float z, float m, float, float zs, float) { return expf(z * zs - m); }

// A lane's value and that of the lane OFF (16 or 32) away, lower lane first: the same pair in both lanes.
template <int OFF>
__device__ __attribute__((always_inline)) inline void lane_pair(float v, float& lo, float& hi) {
  const unsigned u = __float_as_uint(v);
  if constexpr (OFF == 16) { const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false); lo = __uint_as_float(r[0]); hi = __uint_as_float(r[1]); }
  else { const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false); lo = __uint_as_float(r[0]); hi = __uint_as_float(r[1]); }
}

// ---- forward: per-token partial (max m, s = sum exp(z-m), u = sum exp(z-m) z) over this tile's vocab
//      range + target gather; z_t[y_t] is written by the single lane that holds vocab row y_t of token t.
//      u feeds the entropy H_t = lse_t - u/s of the full distribution at no extra pass.
//      z is the tempered logit zs * (W x_t), zs = 1 / temperature; everything written is in tempered units.
//      KEEP: the raw logits W x_t leave as well, in f32, for a backward that forms dS from them (kept_ds_kernel); in the hot kernel in the
//      order of the accumulators (1 KiB per store), else vocabulary-major like dS^T.
// Where a lane's floatx4 of those goes in the hot kernel.  The tiles of the first 256 tokens come first, then those of the next, and
// blocks of 16 columns without a token are neither written nor read: a batch of many rows and few tokens touches little memory, all of it in one piece.
// (With the token tiles innermost and all columns written: 16 and 128 tokens in 2000 rows, H 512, V 152064, the whole call 411 and 420 us, where
// recomputed logits take 354 and 360; like this 272 and 304.  4741 tokens, H 1160, V 50257: dS out of kept logits 261 us, like this 245; 11.5 k at the 7B head 1933 and 1833.)
__device__ inline int64_t kept_index(int tile_m, int tile_n, int tiles_m, int wave, int bi, int bj, int lane) {
  return (((int64_t)(tile_n * tiles_m + tile_m) * 4 + wave) * 64 + bj * 8 + bi) * 64 + lane;
}
template <class T, bool KEEP = false>
struct EpiFwd {
  // sampled tokens of the lane's columns, fetched ahead of the main loop (one after the other in the epilogue they cost a memory
  // latency per column block: 7 us of a tile)
  struct Pre { int y[8]; };
  template <class L> __device__ Pre preload(const TileCtx& c, const GemmDims& d) const {
    Pre p;
#pragma unroll
    for (int bj = 0; bj < 8; ++bj) {
      const int n = c.n0 + L::col(bj, c.lane);
      const int y = ids_c[d.chunk_start + (n < c.Nv ? n : c.Nv - 1)];        // (no branch around a load)
      p.y[bj] = n < c.Nv ? y : -1;
    }
    return p;
  }
  static constexpr bool kSwap = false;
  static constexpr bool kSplit = false;
  static constexpr bool kPermute = false;
  static constexpr bool kGatherB = true;      // the B rows come through a row map (GemmDims::b_rows)
  __device__ void keep_alive() const { zy_c[0] = 0.f; }
  const int* ids_c;     // [chunk-global compact row] sampled token
  float* zy_c;          // [compact row] target logit
  float4* part;         // [tiles_m(V)][ldp] partial (m, s, u, -) per token
  int ldp;              // = chunk rows
  int V;
  float zs;             // inverse temperature
  int* ycol_c;          // [compact row] vocabulary row the target logit was taken from (the position of the accumulator read)
  float* kept;          // KEEP: logits of the chunk

  // one token column of one lane: the MB * kRegs logits it holds.  PAD: some of the sub-tile's rows are
  // vocabulary padding (only in the last tile row) and must not enter the sums.
  template <class L, int MB, int NB, bool AGPR, bool PAD>
  __device__ __attribute__((always_inline)) void column(typename L::acc_t (&acc)[MB][NB], int bj, int lane, int vleft, const TileCtx& c,
                                                        float& mx, float& sm, float& su) const {
    const float NEG = -__builtin_inff();
    float z[MB * L::kRegs];
    mx = NEG;
    if constexpr (KEEP && !AGPR) keep_column<L, MB, NB>(acc, bj, c);
#pragma unroll
    for (int bi = 0; bi < MB; ++bi)
#pragma unroll
      for (int i = 0; i < L::kRegs; ++i) {
        const float v = acc_read<AGPR>(acc[bi][bj], i);
        z[bi * L::kRegs + i] = v;
        mx = fmaxf(mx, (!PAD || L::row(bi, i, lane) < vleft) ? v : NEG);
      }
    if (KEEP && AGPR && c.n0 + bj * 16 < c.Nv) {
#pragma unroll
      for (int bi = 0; bi < MB; ++bi) {
        floatx4 q; q[0] = z[bi * 4]; q[1] = z[bi * 4 + 1]; q[2] = z[bi * 4 + 2]; q[3] = z[bi * 4 + 3];
        __builtin_nontemporal_store(q, reinterpret_cast<floatx4*>(kept) + kept_index(c.tile_m, c.tile_n, (V + 255) / 256, c.wm * 2 + c.wn, bi, bj, lane));
      }
    }
    const float ms = (mx == NEG) ? 0.f : mx * zs;             // zs > 0: the largest raw logit is the largest tempered one
    const float ms_l2e = ms * kLog2e, zs_l2e = zs * kLog2e;
    sm = 0.f; su = 0.f;
#pragma unroll
    for (int bi = 0; bi < MB; ++bi)
#pragma unroll
      for (int i = 0; i < L::kRegs; ++i) {
        const float v = z[bi * L::kRegs + i];
        float e = exp_shifted<T>(v, ms, ms_l2e, zs, zs_l2e);
        if (PAD && !(L::row(bi, i, lane) < vleft)) e = 0.f;
        sm += e;
        su = __builtin_fmaf(e, v, su);
      }
    mx *= zs; su *= zs;
  }

  // vocabulary-major (the rows and columns of a tile that do not exist have room: both extents are padded to 256)
  template <class L, int MB, int NB>
  __device__ __attribute__((always_inline)) void keep_column(typename L::acc_t (&acc)[MB][NB], int bj, const TileCtx& c) const {
    float* p = kept + c.n0 + L::col(bj, c.lane);
#pragma unroll
    for (int bi = 0; bi < MB; ++bi)
#pragma unroll
      for (int i = 0; i < L::kRegs; ++i) p[(int64_t)(c.m0 + L::row(bi, i, c.lane)) * ldp] = acc[bi][bj][i];
  }

  template <int OFF, int NB>
  __device__ __attribute__((always_inline)) void merge_lanes(float (&mx)[NB], float (&sm)[NB], float (&su)[NB]) const {
    const float NEG = -__builtin_inff();
#pragma unroll
    for (int bj = 0; bj < NB; ++bj) {
      float m1, m2, s1, s2, u1, u2;
      lane_pair<OFF>(mx[bj], m1, m2); lane_pair<OFF>(sm[bj], s1, s2); lane_pair<OFF>(su[bj], u1, u2);
      const float mm = fmaxf(m1, m2);
      const float mms = (mm == NEG) ? 0.f : mm;
      const float f1 = fast_exp<T>(m1 - mms), f2 = fast_exp<T>(m2 - mms);
      sm[bj] = s1 * f1 + s2 * f2;
      su[bj] = u1 * f1 + u2 * f2;
      mx[bj] = mm;
    }
  }

  // Narrow tile of the f32 kernel (256 x 16, WAVES wavefronts stacked along the vocabulary).  Its sums are those of the 256 x 64 tile to the bit,
  // so that a token's log-prob does not depend on how many rows are staged with it: there one lane adds up, in order, the 64 rows of a half tile
  // (128 rows) whose bit 2 is the lane's half of the wavefront.  Here such a chain is spread over two lane groups of several wavefronts, so
  // the exponentials are formed where the logits are, pass through LDS, and wavefront 0 adds up one chain per lane.
  template <class L, int MB, int WAVES>
  __device__ __attribute__((always_inline)) void narrow(typename L::acc_t (&acc)[MB][1], const TileCtx& c, unsigned char* smem, int vleft) const {
    static_assert(L::kBlk == 16 && MB * WAVES == 16 && WAVES % 2 == 0 && sizeof(T) == 4, "256 rows in blocks of 16 x 16");
    const float NEG = -__builtin_inff();
    float2* ev = reinterpret_cast<float2*>(smem);               // [position in the chain][chain: half of the lanes, half of the tile, column]
    float* mw = reinterpret_cast<float*>(smem + 64 * 64 * 8);   // [wavefront][half of the lanes, column] largest logit
    const int col = c.lane & 15, g = c.lane >> 4, hc = c.lane & 31;
    constexpr int HALF = WAVES / 2;                             // wavefronts of a half tile
    float mx = NEG;
#pragma unroll
    for (int bi = 0; bi < MB; ++bi)
#pragma unroll
      for (int i = 0; i < 4; ++i) mx = fmaxf(mx, L::row(bi, i, c.lane) < vleft ? acc[bi][0][i] : NEG);
    float m1, m2;
    lane_pair<32>(mx, m1, m2);
    if (c.lane < 32) mw[c.wm * 32 + hc] = fmaxf(m1, m2);
    __syncthreads();
    const int half = c.wm / HALF;
    auto half_max = [&](int hf, int at) __attribute__((always_inline)) {
      float m = mw[hf * HALF * 32 + at];
#pragma unroll
      for (int w = 1; w < HALF; ++w) m = fmaxf(m, mw[(hf * HALF + w) * 32 + at]);
      return m;
    };
    mx = half_max(half, hc);
    const float ms = (mx == NEG) ? 0.f : mx * zs;
    float2* my = ev + ((c.wm % HALF) * MB * 8 + (g >> 1) * 4) * 64 + (g & 1) * 32 + half * 16 + col;
#pragma unroll
    for (int bi = 0; bi < MB; ++bi)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float v = acc[bi][0][i];
        const float e = exp_shifted<T>(v, ms, 0.f, zs, 0.f);
        my[(bi * 8 + i) * 64] = make_float2(L::row(bi, i, c.lane) < vleft ? e : 0.f, v);
      }
    __syncthreads();
    if (c.wm != 0) return;
    float m[1], s[1] = {0.f}, u[1] = {0.f};
#pragma unroll 16
    for (int k = 0; k < 64; ++k) {
      const float2 x = ev[k * 64 + c.lane];
      s[0] += x.x;
      u[0] = __builtin_fmaf(x.x, x.y, u[0]);
    }
    m[0] = half_max(g & 1, (g >> 1) * 16 + col) * zs;           // the chain of this lane: half tile g & 1, lane half g >> 1
    u[0] *= zs;
    merge_lanes<32, 1>(m, s, u);
    merge_lanes<16, 1>(m, s, u);
    const int n = c.n0 + col;
    if (c.lane < 16 && n < c.Nv) part[(int64_t)c.tile_m * ldp + n] = make_float4(m[0], s[0], u[0], 0.f);
  }

  // target gather of token t, whose sampled token is y (-1: none): at most one lane of the whole grid holds row y of its column, so this branch
  // is almost never taken
  template <class L, int MB, int NB, bool AGPR>
  __device__ __attribute__((always_inline)) void target(typename L::acc_t (&acc)[MB][NB], int bj, const TileCtx& c, int y, int t) const {
    const int yrel = y >= 0 ? y - c.m0 : -1;
    if (yrel >= 0 && yrel < MB * L::kBlk && L::owns(yrel, c.lane)) {
      float zy = 0.f;
      int got = -1;
#pragma unroll
      for (int bi = 0; bi < MB; ++bi)
#pragma unroll
        for (int i = 0; i < L::kRegs; ++i) {
          const float v = acc_read<AGPR>(acc[bi][bj], i);
          if (L::row(bi, i, c.lane) == yrel) { zy = v; got = c.m0 + L::row(bi, i, c.lane); }
        }
      zy_c[t] = zy * zs;
      ycol_c[t] = got;
    }
  }

  // Half a 256-row tile by one wavefront (logits_few_kernel): the partials of its columns leave without the merge with the other half.
  template <class L, int MB, int NB>
  __device__ __attribute__((always_inline)) void half_tile(typename L::acc_t (&acc)[MB][NB], const TileCtx& c, const int (&y)[NB]) const {
    const int vleft = V - c.m0;
    float mx[NB], sm[NB], su[NB];
#pragma unroll
    for (int bj = 0; bj < NB; ++bj) {
      target<L, MB, NB, false>(acc, bj, c, y[bj], c.n0 + L::col(bj, c.lane));
      if (vleft < MB * L::kBlk) column<L, MB, NB, false, true>(acc, bj, c.lane, vleft, c, mx[bj], sm[bj], su[bj]);
      else column<L, MB, NB, false, false>(acc, bj, c.lane, vleft, c, mx[bj], sm[bj], su[bj]);
    }
    merge_lanes<16, NB>(mx, sm, su);
    merge_lanes<32, NB>(mx, sm, su);
#pragma unroll
    for (int bj = 0; bj < NB; ++bj) {
      const int n = c.n0 + L::col(bj, c.lane);
      if (c.lane < 16 && n < c.Nv) part[(int64_t)c.tile_m * ldp + n] = make_float4(mx[bj], sm[bj], su[bj], 0.f);
    }
  }
  // ... and that merge, as the epilogue of a whole tile does it
  __device__ static float4 merge_halves(float4 r, const float4& o) {
    const float NEG = -__builtin_inff();
    const float mm = fmaxf(r.x, o.x);
    const float mms = (mm == NEG) ? 0.f : mm;
    const float f1 = fast_exp<T>(r.x - mms), f2 = fast_exp<T>(o.x - mms);
    r.y = r.y * f1 + o.y * f2;
    r.z = r.z * f1 + o.z * f2;
    r.x = mm;
    return r;
  }

  template <class L, int MB, int NB, int BM, int BN, int WAVES_M, int WAVES_N, bool AGPR>
  __device__ __attribute__((always_inline)) void run(typename L::acc_t (&acc)[MB][NB], const TileCtx& c, unsigned char* smem, const GemmDims& d, const Pre& pre) const {
    float4* red = reinterpret_cast<float4*>(smem);              // [WAVES_M][BN]
    const float NEG = -__builtin_inff();
    const int vleft = V - c.m0;                                 // rows of this sub-tile below vleft are real vocabulary
    const bool pad = vleft < MB * L::kBlk;                      // wavefront-uniform
    static_assert(NB <= 8, "Pre holds eight columns");
    constexpr bool kNarrow = L::kBlk == 16 && !AGPR;
    float mx[NB], sm[NB], su[NB];
#pragma unroll
    for (int bj = 0; bj < NB; ++bj) {
      const int n = c.n0 + L::col(bj, c.lane);
      target<L, MB, NB, AGPR>(acc, bj, c, pre.y[bj], d.chunk_start + n);
      if constexpr (kNarrow) { if constexpr (KEEP) keep_column<L, MB, NB>(acc, bj, c); continue; }
      else if (pad) column<L, MB, NB, AGPR, true>(acc, bj, c.lane, vleft, c, mx[bj], sm[bj], su[bj]);
      else column<L, MB, NB, AGPR, false>(acc, bj, c.lane, vleft, c, mx[bj], sm[bj], su[bj]);
    }
    if constexpr (kNarrow) {
      static_assert(WAVES_N == 1, "the wavefronts of a column are stacked along the vocabulary");
      narrow<L, MB, WAVES_M>(acc, c, smem, vleft);
      return;
    } else {
    // merge with the lane groups that hold the other rows of these columns (row swaps at vector speed; the pair comes lower
    // lane first, which is the order the lanes whose result is kept add in)
    merge_lanes<L::kBlk, NB>(mx, sm, su);
    if constexpr (L::kBlk == 16) merge_lanes<32, NB>(mx, sm, su);
#pragma unroll
    for (int bj = 0; bj < NB; ++bj)
      if (c.lane < L::kBlk) red[c.wm * BN + (c.n0 + L::col(bj, c.lane) - c.tile_n * BN)] = make_float4(mx[bj], sm[bj], su[bj], 0.f);
    __syncthreads();
    if (c.tid < BN) {
      const int n = c.tile_n * BN + c.tid;
      if (n < c.Nv) {
        float4 r = red[c.tid];
#pragma unroll
        for (int w = 1; w < WAVES_M; ++w) {
          r = merge_halves(r, red[w * BN + c.tid]);
        }
        part[(int64_t)c.tile_m * ldp + n] = r;
      }
    }
    }
  }
};

// ---- forward that also keeps the chunk's unnormalised probabilities for a single-pass backward.
//      Every token has a reference ref_t close to its logsumexp, known before the contraction
//      (target logit minus the old policy's log-prob), so e = exp(z - ref_t) needs no running
//      maximum: the epilogue adds up s = sum e and u = sum e z per token and tile row, and
//      stores e itself in the input precision, token-major E[t][v] (16-byte stores through the same
//      relabelling as EpiDS; the weight-gradient contraction reads E as a K-major operand, so no
//      vocab-major copy is kept).  bf16 keeps f32's exponent range, so e is
//      stored at full relative precision whatever its size.  Later, with Z_t = sum_v e,
//      dS[t][v] = -(c_t / Z_t) (E[t][v] - Z_t 1[v = y_t]): the backward contractions run on E
//      directly, with the target entry patched and the factor applied per token.
template <class T>
struct EpiFwdStash {
  struct Pre { float rl[8]; };                            // ref_t * log2(e) of the lane's eight token columns
  template <class L> __device__ Pre preload(const TileCtx& c, const GemmDims& d) const {
    Pre p;
    const int cc = c.lane & 15;
#pragma unroll
    for (int bj = 0; bj < 8; ++bj) {
      const int n = c.n0 + perm_col(bj, cc);
      const float rl = ref_l2e[d.chunk_start + (n < c.Nv ? n : c.Nv - 1)];
      p.rl[bj] = n < c.Nv ? rl : __builtin_inff();                             // column without a token: e = exp2(-inf) = 0
    }
    return p;
  }
  static constexpr bool kSwap = false;
  static constexpr bool kSplit = false;
  static constexpr bool kPermute = true;
  static constexpr bool kGatherB = true;      // the B rows come through a row map (GemmDims::b_rows)
  __device__ void keep_alive() const { E[0] = (T)0.f; }
  const float* ref_l2e;   // [compact row] ref_t * log2(e)
  float2* part;           // [tiles_m(V)][ldp] partial (s, u) per token of the chunk
  int ldp;
  T* E;  int64_t ld_e;    // [chunk rows][Vp = ld_e], slab-tiled
  int V;
  float zs;               // inverse temperature: z = zs * (W x_t) is the logit that ref_t, s and u refer to

  // Exponentials, sums and the stores, in two rounds of four block rows (64 vocabulary entries = one 128-byte
  // line of a token's E row).  A lane holds 16 bytes of the first half of that line (block rows 4j, 4j+1) and 16 of
  // the second (4j+2, 4j+3), and its four lane groups make each half 64 bytes wide; lane pairs (token columns cc,
  // cc^1) swap one half each, so that one store instruction writes whole lines: the eight lanes of the even token's
  // line first, then the odd token's.
  template <class L, int MB, int NB, bool AGPR, bool PAD>
  __device__ __attribute__((always_inline)) void body(typename L::acc_t (&acc)[MB][NB], const TileCtx& c, int g, int cc, int vleft,
                                                      const float (&rl)[NB], float (&sm)[NB], float (&su)[NB]) const {
    const int p = cc & 1;
    const float zs_l2e = zs * kLog2e;
#pragma unroll
    for (int j = 0; j < MB / 4; ++j) {
#pragma unroll
      for (int bj = 0; bj < NB; ++bj) {
        bf16x8 half[2];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          const int mrel = (2 * j + kk) * 32 + g * 8;
#pragma unroll
          for (int i = 0; i < 8; ++i) {
            const float z = acc_read<AGPR>(acc[2 * (2 * j + kk) + (i >> 2)][bj], i & 3);
            float v = __builtin_amdgcn_exp2f(__builtin_fmaf(z, zs_l2e, -rl[bj]));
            if (PAD && !(mrel + i < vleft)) v = 0.f;
            sm[bj] += v;
            su[bj] = __builtin_fmaf(v, z, su[bj]);
            half[kk][i] = (bf16_t)v;
          }
        }
        const u32x4_t a = __builtin_bit_cast(u32x4_t, half[0]), b = __builtin_bit_cast(u32x4_t, half[1]);
        u32x4_t recv;
#pragma unroll
        for (int q = 0; q < 4; ++q)                         // swap with the neighbouring lane (quad_perm [1,0,3,2])
          recv[q] = (unsigned)__builtin_amdgcn_mov_dpp((int)(p ? a[q] : b[q]), 0xB1, 0xF, 0xF, true);
        const u32x4_t d_even = p ? recv : a, d_odd = p ? b : recv;
        const int v0 = c.m0 + j * 64 + p * 32 + g * 8;
        store_stream(E + tiled_index(c.n0 + perm_col(bj, cc & ~1), v0, ld_e), __builtin_bit_cast(bf16x8, d_even));
        store_stream(E + tiled_index(c.n0 + perm_col(bj, cc | 1), v0, ld_e), __builtin_bit_cast(bf16x8, d_odd));
      }
      __builtin_amdgcn_sched_barrier(0);                  // keep the two rounds apart
    }
  }

  template <class L, int MB, int NB, int BM, int BN, int WAVES_M, int WAVES_N, bool AGPR>
  __device__ __attribute__((always_inline)) void run(typename L::acc_t (&acc)[MB][NB], const TileCtx& c, unsigned char* smem, const GemmDims& d, const Pre& pre) const {
    static_assert(L::kBlk == 16 && MB == 8 && NB == 8 && sizeof(T) == 2, "hot kernel only");
    float2* red = reinterpret_cast<float2*>(smem);              // [WAVES_M][BN + BN / 32]
    constexpr int kRedRow = BN + BN / 32;
    const int g = c.lane >> 4, cc = c.lane & 15;
    float rl[NB], sm[NB], su[NB];
#pragma unroll
    for (int bj = 0; bj < NB; ++bj) { rl[bj] = pre.rl[bj]; sm[bj] = 0.f; su[bj] = 0.f; }
    const int vleft = V - c.m0;                            // sub-tile rows >= vleft are vocabulary padding
    if (vleft < MB * L::kBlk) body<L, MB, NB, AGPR, true>(acc, c, g, cc, vleft, rl, sm, su);   // wavefront-uniform
    else body<L, MB, NB, AGPR, false>(acc, c, g, cc, vleft, rl, sm, su);
#pragma unroll
    for (int bj = 0; bj < NB; ++bj) {
#pragma unroll
      for (int off = 16; off < 64; off <<= 1) { sm[bj] += __shfl_xor(sm[bj], off); su[bj] += __shfl_xor(su[bj], off); }
      // (one spare slot after every 32 columns: the sixteen lanes write columns 8 apart, 64 bytes, and would otherwise meet
      // in the LDS banks four at a time)
      if (c.lane < 16) {
        const int col = c.wn * (BN / WAVES_N) + perm_col(bj, cc);
        red[c.wm * kRedRow + col + (col >> 5)] = make_float2(sm[bj], su[bj] * zs);
      }
    }
    __syncthreads();
    if (c.tid < BN) {
      const int n = c.tile_n * BN + c.tid;
      if (n < c.Nv) {
        const int slot = c.tid + (c.tid >> 5);
        float2 r = red[slot];
#pragma unroll
        for (int w = 1; w < WAVES_M; ++w) { const float2 o2 = red[w * kRedRow + slot]; r.x += o2.x; r.y += o2.y; }
        part[(int64_t)c.tile_m * ldp + n] = r;
      }
    }
  }
};

// Four floats, four bf16 or 16 bytes in the caller's d_weight / d_hidden, which may start at any element (a parameter's slice of a flat
// gradient buffer): the device takes such accesses at any address, the types say that it must.
typedef float floatx4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef __bf16 bf16x4_any __attribute__((ext_vector_type(4), aligned(2)));
template <class T> struct Piece16;
template <> struct Piece16<float> { typedef unsigned type __attribute__((ext_vector_type(4), aligned(4))); };
template <> struct Piece16<bf16_t> { typedef unsigned type __attribute__((ext_vector_type(4), aligned(2))); };

template <class T> struct Pack4;
template <> struct Pack4<bf16_t> {
  __device__ static void store(bf16_t* p, float a, float b, float c, float d) {
    bf16x4 v; v[0] = (bf16_t)a; v[1] = (bf16_t)b; v[2] = (bf16_t)c; v[3] = (bf16_t)d;
    *reinterpret_cast<bf16x4*>(p) = v;
  }
};
template <> struct Pack4<float> {
  __device__ static void store(float* p, float a, float b, float c, float d) {
    *reinterpret_cast<float4*>(p) = make_float4(a, b, c, d);
  }
};

// ---- backward, stage 1: recomputed logits -> dS = zs c_t (1[v=y_t] - exp(z - lse_t)) (z the tempered
//      logit, zs = 1 / temperature the chain factor back to W x_t), formed in
//      f32 (subtraction and scaling before rounding) and stored in the input precision, token-major
//      dS[t][v] (operand of dX = dS W).  dW = dS^T X reads the same array as a K-major operand in the
//      bf16 hot kernel; f32 inputs (the kernel of gemm_f32.h, narrow tiles and unaligned operands the general one) also get the vocab-major
//      copy dST[v][t], or only that where dX reads it K-major.
//
//      In the hot kernel (16x16 blocks) the tile rows and columns are relabelled (kPermute, see
//      perm_row / perm_col in gemm_nt.h) such that a lane ends up holding eight consecutive
//      vocabulary entries of a token: the copy leaves in 16-byte stores with no staging through LDS.
template <class T>
struct EpiDS {
  struct Pre { int y[8]; float lse[8], ct[8]; };          // hot kernel: the lane's eight token columns, fetched ahead of the main loop
  template <class L> __device__ Pre preload(const TileCtx& c, const GemmDims& d) const {
    Pre p;
    if constexpr (sizeof(T) == 2 && L::kBlk == 16) {
#pragma unroll
      for (int bj = 0; bj < 8; ++bj) {
        const int n = c.n0 + perm_col(bj, c.lane & 15);
        const bool valid = n < c.Nv;
        const int t = d.chunk_start + (valid ? n : c.Nv - 1), y = ids_c[t];
        const float lse = lse_c[t], ct = c_c[t];
        p.y[bj] = valid ? y : -1;
        p.lse[bj] = valid ? lse : 3.0e38f;                // invalid token: p = exp(z - huge) = 0 and
        p.ct[bj] = valid ? ct : 0.f;                      // c = 0, so every dS entry becomes 0
      }
    }
    return p;
  }
  static constexpr bool kSwap = false;
  static constexpr bool kSplit = false;
  static constexpr bool kPermute = true;
  static constexpr bool kGatherB = true;      // the B rows come through a row map (GemmDims::b_rows)
  __device__ void keep_alive() const { dS[0] = (T)0.f; }
  const int* ids_c; const float* lse_c; const float* c_c;
  T* dS;  int64_t ld_ds;    // [chunk rows][Vp]; f32 inputs: nullptr where dX reads dS^T (gemm_f32.h, KM)
  T* dST; int64_t ld_dst;   // [Vp][chunk rows]; f32 inputs only
  int V;
  bool tiled;               // dS slab-tiled (always so for bf16: its consumer is the hot kernel)
  float zs;                 // inverse temperature

  template <class L, int MB, int NB, int BM, int BN, int WAVES_M, int WAVES_N, bool AGPR>
  __device__ __attribute__((always_inline)) void run(typename L::acc_t (&acc)[MB][NB], const TileCtx& c, unsigned char*, const GemmDims& d, const Pre& pre) const {
    if constexpr (AGPR) {                                  // hot kernel
      static_assert(MB == 8 && NB == 8 && sizeof(T) == 2, "the relabelling is written for 128x128 wavefront sub-tiles");
      const int g = c.lane >> 4, cc = c.lane & 15;
      int y[NB]; float lse[NB], lse_l2e[NB], ct[NB];
#pragma unroll
      for (int bj = 0; bj < NB; ++bj) {
        y[bj] = pre.y[bj] >= 0 ? pre.y[bj] - c.m0 : -1;   // relative to the sub-tile; -1 never matches
        lse[bj] = pre.lse[bj];
        ct[bj] = pre.ct[bj] * zs;
        lse_l2e[bj] = lse[bj] * kLog2e;
      }
      const float zs_l2e = zs * kLog2e;
      const int vleft = V - c.m0;                          // sub-tile rows >= vleft are vocabulary padding
      const int p = cc & 1;
#pragma unroll
      for (int j = 0; j < MB / 4; ++j) {                   // four block rows = 64 vocabulary entries = one 128-byte line of a dS row
        bf16_t o[NB][16];
#pragma unroll
        for (int bj = 0; bj < NB; ++bj)
#pragma unroll
          for (int r = 0; r < 16; ++r) {                   // r: entry of the round, vocab offset j*64 + (r/8)*32 + g*8 + r%8
            const int m = (2 * j + (r >> 3)) * 32 + g * 8 + (r & 7);
            const float pr = exp_shifted<T>(acc_read<AGPR>(acc[4 * j + (r >> 2)][bj], r & 3), lse[bj], lse_l2e[bj], zs, zs_l2e);
            const float ds = ct[bj] * ((m == y[bj] ? 1.f : 0.f) - pr);
            o[bj][r] = (bf16_t)(m < vleft ? ds : 0.f);
          }
        // token-major copy: lane pairs (token columns cc, cc^1) swap one half each, so that a store writes whole lines
#pragma unroll
        for (int bj = 0; bj < NB; ++bj) {
          bf16x8 h0, h1;
#pragma unroll
          for (int i = 0; i < 8; ++i) { h0[i] = o[bj][i]; h1[i] = o[bj][8 + i]; }
          const u32x4_t a = __builtin_bit_cast(u32x4_t, h0), b = __builtin_bit_cast(u32x4_t, h1);
          u32x4_t recv;
#pragma unroll
          for (int q = 0; q < 4; ++q) recv[q] = (unsigned)__builtin_amdgcn_mov_dpp((int)(p ? a[q] : b[q]), 0xB1, 0xF, 0xF, true);
          const u32x4_t d_even = p ? recv : a, d_odd = p ? b : recv;
          const int v0 = c.m0 + j * 64 + p * 32 + g * 8;
          store_stream(dS + tiled_index(c.n0 + perm_col(bj, cc & ~1), v0, ld_ds), __builtin_bit_cast(bf16x8, d_even));
          store_stream(dS + tiled_index(c.n0 + perm_col(bj, cc | 1), v0, ld_ds), __builtin_bit_cast(bf16x8, d_odd));
        }
      }
    } else {
#pragma unroll
      for (int bj = 0; bj < NB; ++bj) {
        const int n = c.n0 + L::col(bj, c.lane);
        const bool valid = n < c.Nv;
        const int g = d.chunk_start + n;
        const int y = valid ? ids_c[g] : -1;
        const float lse = valid ? lse_c[g] : 0.f;
        const float ct = valid ? c_c[g] * zs : 0.f;
#pragma unroll
        for (int bi = 0; bi < MB; ++bi)
#pragma unroll
          for (int q = 0; q < L::kRegs / 4; ++q) {
            const int m = c.m0 + L::row(bi, q * 4, c.lane);
            float o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float p = fast_exp<T>(acc_read<AGPR>(acc[bi][bj], q * 4 + e) * zs - lse);
              const float ds = ct * (((m + e) == y ? 1.f : 0.f) - p);
              o[e] = (valid && (m + e) < V) ? ds : 0.f;
            }
            if (sizeof(T) == 2 || dS) Pack4<T>::store(dS + operand_index(tiled, n, m, ld_ds), o[0], o[1], o[2], o[3]);
            if constexpr (sizeof(T) == 4) {
#pragma unroll
              for (int e = 0; e < 4; ++e) dST[operand_index(tiled, m + e, n, ld_dst)] = (T)o[e];
            }
          }
      }
    }
  }
};

// ---- backward, stage 1, of a batch that is one chunk: dS from the logits the forward kept (EpiFwd<T, true>), in the arithmetic of EpiDS.
//      A contraction of 2 T V H operations becomes a pass over memory: 4 bytes in and 2 out per logit in bf16; f32 reads dS^T's place, where
//      the logits are, and writes dS^T over them, and dS besides where dX needs it.
struct KeptJob {
  const int* ids_c; const float* lse_c; const float* c_c; const int* n_real;
  int V; float zs;
};

// bf16: a wavefront takes 16 tokens x 128 vocabulary entries of a tile; grid (4 x tiles of 256 x 256, 2).  Lane (g, cc) = (l / 16, l % 16)
// holds entries 16 bi + 4 g .. + 3 of token cc; a row swap makes that eight consecutive entries, and lane pairs swap halves, so that
// a store writes whole 128-byte lines (as in EpiDS).
__global__ __launch_bounds__(256) void kept_ds_kernel(const float* kept, KeptJob j, int tiles_m, bf16_t* dS, int64_t ld_ds) {
  const int sub = blockIdx.x & 3, tile = blockIdx.x >> 2, tile_n = tile / tiles_m, tile_m = tile - tile_n * tiles_m;
  const int n_real = *j.n_real;
  if (tile_n * 256 >= n_real) return;
  const int lane = threadIdx.x & 63, bj = blockIdx.y * 4 + (threadIdx.x >> 6), g = lane >> 4, cc = lane & 15, p = cc & 1;
  const int n16 = tile_n * 256 + (sub & 1) * 128 + bj * 16;
  floatx4 z[8];
#pragma unroll
  for (int bi = 0; bi < 8; ++bi) {
    z[bi] = floatx4{0.f, 0.f, 0.f, 0.f};
    if (n16 < n_real) z[bi] = __builtin_nontemporal_load(reinterpret_cast<const floatx4*>(kept) + kept_index(tile_m, tile_n, tiles_m, sub, bi, bj, lane));
  }
  const int n = n16 + cc, m0 = tile_m * 256 + (sub >> 1) * 128;
  const bool valid = n < n_real;
  const int y = valid ? j.ids_c[n] - m0 : -1;
  const float lse = valid ? j.lse_c[n] : 3.0e38f, ct = valid ? j.c_c[n] * j.zs : 0.f;       // no token: every entry becomes 0
  const float lse_l2e = lse * kLog2e, zs_l2e = j.zs * kLog2e;
  u32x2_t o[8];
#pragma unroll
  for (int bi = 0; bi < 8; ++bi) {
    bf16x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int m = bi * 16 + g * 4 + e;
      const float pr = exp_shifted<bf16_t>(z[bi][e], lse, lse_l2e, j.zs, zs_l2e);
      v[e] = (bf16_t)(m < j.V - m0 ? ct * ((m == y ? 1.f : 0.f) - pr) : 0.f);
    }
    o[bi] = __builtin_bit_cast(u32x2_t, v);
  }
  // after the swap of rows of blocks 2 k and 2 k + 1: lane group 0 / 2 has entries 0..7 / 8..15 of block 2 k, group 1 / 3 those of block 2 k + 1
  u32x4_t h[4];
#pragma unroll
  for (int k = 0; k < 4; ++k)
#pragma unroll
    for (int w = 0; w < 2; ++w) {
      const auto r = __builtin_amdgcn_permlane16_swap(o[2 * k][w], o[2 * k + 1][w], false, false);
      h[k][w] = r[0]; h[k][2 + w] = r[1];
    }
#pragma unroll
  for (int k = 0; k < 2; ++k) {                                  // 64 entries: one line of a token's row
    u32x4_t recv;
#pragma unroll
    for (int q = 0; q < 4; ++q) recv[q] = (unsigned)__builtin_amdgcn_mov_dpp((int)(p ? h[2 * k][q] : h[2 * k + 1][q]), 0xB1, 0xF, 0xF, true);
    const u32x4_t d_even = p ? recv : h[2 * k], d_odd = p ? h[2 * k + 1] : recv;
    const int v0 = m0 + k * 64 + p * 32 + (g & 1) * 16 + (g >> 1) * 8;
    store_stream(dS + tiled_index(n & ~1, v0, ld_ds), __builtin_bit_cast(bf16x8, d_even));
    store_stream(dS + tiled_index(n | 1, v0, ld_ds), __builtin_bit_cast(bf16x8, d_odd));
  }
}

// f32: 64 tokens x 64 vocabulary entries per workgroup (vocabulary fastest); dST holds the logits on entry.  Token columns up to the next multiple of 64 become 0.
__global__ __launch_bounds__(256) void kept_ds_f32_kernel(KeptJob j, float* dST, int64_t ld_dst, float* dS, int64_t ld_ds) {
  __shared__ float tile[64][65];
  const int vb = (int)(ld_ds / 64), n0 = (int)(blockIdx.x / vb) * 64, m0 = (int)(blockIdx.x % vb) * 64, n_real = *j.n_real;
  if (n0 >= n_real) return;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6, n = n0 + tx;
  const bool valid = n < n_real;
  const int y = valid ? j.ids_c[n] : -1;
  const float lse = valid ? j.lse_c[n] : 0.f, ct = valid ? j.c_c[n] * j.zs : 0.f;
  float z[16];
#pragma unroll
  for (int k = 0; k < 16; ++k) z[k] = dST[(int64_t)(m0 + ty + 4 * k) * ld_dst + n];
#pragma unroll
  for (int k = 0; k < 16; ++k) {
    const int m = m0 + ty + 4 * k;
    const float ds = ct * ((m == y ? 1.f : 0.f) - fast_exp<float>(z[k] * j.zs - lse));
    const float o = valid && m < j.V ? ds : 0.f;
    dST[(int64_t)m * ld_dst + n] = o;
    tile[ty + 4 * k][tx] = o;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < 16; ++k) dS[(int64_t)(n0 + ty + 4 * k) * ld_ds + m0 + tx] = tile[tx][ty + 4 * k];
}

// ... and without dS (gemm_f32.h, KM): 256 tokens x 32 vocabulary entries per workgroup, eight rows of 16 bytes in flight per lane (2175 tokens, V 50257: 238 -> 137 us).
// Token columns up to the next multiple of 16, which dW's K is rounded up to, become 0.
__global__ __launch_bounds__(256) void kept_ds_t_kernel(KeptJob j, float* dST, int64_t ld_dst, int rows) {
  const int vb = rows / 32, n = (int)(blockIdx.x / vb) * 256 + (threadIdx.x & 63) * 4, m0 = (int)(blockIdx.x % vb) * 32 + (threadIdx.x >> 6) * 8, n_real = *j.n_real;
  if (n >= ((n_real + 15) & ~15)) return;
  float* p = dST + (int64_t)m0 * ld_dst + n;
  floatx4 z[8];
#pragma unroll
  for (int k = 0; k < 8; ++k) z[k] = *reinterpret_cast<const floatx4*>(p + k * ld_dst);
  int y[4];
  float lse[4], ct[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int t = n + e < n_real ? n + e : n_real - 1;
    y[e] = j.ids_c[t]; lse[e] = j.lse_c[t]; ct[e] = j.c_c[t] * j.zs;
  }
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    floatx4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float ds = ct[e] * ((m0 + k == y[e] ? 1.f : 0.f) - fast_exp<float>(z[k][e] * j.zs - lse[e]));
      o[e] = n + e < n_real && m0 + k < j.V ? ds : 0.f;
    }
    *reinterpret_cast<floatx4*>(p + k * ld_dst) = o;
  }
}

// ---- backward, stage 2: dX tile -> rows scattered back to their original positions
template <class T>
struct EpiDX {
  typedef NoPre Pre;
  template <class L> __device__ Pre preload(const TileCtx&, const GemmDims&) const { return Pre(); }
  static constexpr bool kSwap = true;        // hot kernel: blocks transposed, a lane holds four consecutive columns of one row
  static constexpr bool kSplit = true;       // may be cut along K (split_k)
  static constexpr bool kPermute = false;
  static constexpr bool kGatherB = false;      // the B rows come through a row map (GemmDims::b_rows)
  __device__ void keep_alive() const { dX[0] = (T)0.f; }
  const int* row_map;   // compact row -> original row
  T* dX; int64_t ldx; int H;
  const float* row_scale;   // optional [chunk row]: factor applied to the whole row
  float* split_part;        // K slices: [slice][ceil(M / BM) * BM][H] partial tiles, added up by splitk_reduce_kernel

  // Hot kernel: lane (g, r) = (l / 16, l % 16) holds row 16 bi + r, columns 16 bj + 4 g .. + 3 of the sub-tile.  PART: to the partial
  // buffer in f32; EDGE: the sub-tile reaches past the last row or column (H is a multiple of 8: never inside a lane's four).
  template <int MB, int NB, bool PART, bool EDGE>
  __device__ __attribute__((always_inline)) void rows(floatx4 (&acc)[MB][NB], const TileCtx& c, const GemmDims& d, float* part) const {
    const int r = c.lane & 15, n = c.n0 + (c.lane >> 4) * 4;
#pragma unroll
    for (int bi = 0; bi < MB; ++bi) {
      const int m = c.m0 + bi * 16 + r;
      if (EDGE && m >= c.Mv) continue;
      const float f = !PART && row_scale ? row_scale[m] : 1.f;
      float* p = PART ? part + (int64_t)m * H + n : nullptr;
      T* o = PART ? nullptr : dX + (int64_t)row_map[d.chunk_start + m] * ldx + n;
#pragma unroll
      for (int bj = 0; bj < NB; ++bj) {
        floatx4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = f * acc_read<true>(acc[bi][bj], e);
        if (EDGE && n + bj * 16 >= H) continue;
        if constexpr (PART) *reinterpret_cast<floatx4*>(p + bj * 16) = v;
        else {
          static_assert(sizeof(T) == 2, "hot kernel");
          bf16x4_any b; b[0] = (T)v[0]; b[1] = (T)v[1]; b[2] = (T)v[2]; b[3] = (T)v[3];
          *reinterpret_cast<bf16x4_any*>(o + bj * 16) = b;
        }
      }
    }
  }

  template <class L, int MB, int NB, int BM, int BN, int WAVES_M, int WAVES_N, bool AGPR>
  __device__ __attribute__((always_inline)) void run(typename L::acc_t (&acc)[MB][NB], const TileCtx& c, unsigned char*, const GemmDims& d, const Pre&) const {
    if constexpr (AGPR) {
      const bool edge = c.m0 + MB * 16 > c.Mv || c.n0 + NB * 16 > H;
      if (c.slices > 1) {
        float* part = split_part + (int64_t)c.slice * ((c.Mv + BM - 1) / BM * BM) * H;
        if (edge) rows<MB, NB, true, true>(acc, c, d, part); else rows<MB, NB, true, false>(acc, c, d, part);
      } else {
        if (edge) rows<MB, NB, false, true>(acc, c, d, nullptr); else rows<MB, NB, false, false>(acc, c, d, nullptr);
      }
      return;
    }
    if (c.slices > 1) {
      float* p = split_part + (int64_t)c.slice * ((c.Mv + BM - 1) / BM * BM) * H;     // (H % 4 == 0)
#pragma unroll
      for (int bi = 0; bi < MB; ++bi)
#pragma unroll
        for (int i = 0; i < L::kRegs; ++i) {
          const int m = c.m0 + L::row(bi, i, c.lane);
          if (m >= c.Mv) continue;
#pragma unroll
          for (int bj = 0; bj < NB; ++bj) {
            const int n = c.n0 + L::col(bj, c.lane);
            if (n < H) p[(int64_t)m * H + n] = acc_read<AGPR>(acc[bi][bj], i);
          }
        }
      return;
    }
#pragma unroll
    for (int bi = 0; bi < MB; ++bi)
#pragma unroll
      for (int i = 0; i < L::kRegs; ++i) {
        const int m = c.m0 + L::row(bi, i, c.lane);
        if (m >= c.Mv) continue;
        const int64_t dst = row_map[d.chunk_start + m];
        const float f = row_scale ? row_scale[m] : 1.f;
#pragma unroll
        for (int bj = 0; bj < NB; ++bj) {
          const int n = c.n0 + L::col(bj, c.lane);
          if (n < H) dX[dst * ldx + n] = (T)(f * acc_read<AGPR>(acc[bi][bj], i));
        }
      }
  }
};

// The slices of a split dX contraction added up in order, scaled and scattered to the original rows (four columns per
// thread, H % 4 == 0; `step`: elements of K per step of the cut).  Works the number of slices out like the contraction itself; returns at once if there was one.
template <class T>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(GemmDims d, EpiDX<T> e, int bm, int bn, int step) {
  int M, N, K;
  if (!resolve_dims(d, M, N, K)) return;
  const int tiles_m = (M + bm - 1) / bm;
  const SplitK sk = split_k(tiles_m * ((d.N + bn - 1) / bn), (K + step - 1) / step, d.split_slots, fill_steps(d, M));
  if (sk.slices == 1) return;
  const int64_t stride = (int64_t)tiles_m * bm * e.H;
  const int h4 = e.H / 4;
  for (int64_t q = (int64_t)blockIdx.x * 256 + threadIdx.x; q < (int64_t)M * h4; q += (int64_t)gridDim.x * 256) {
    const int m = (int)(q / h4), n = (int)(q - (int64_t)m * h4) * 4;
    const float* p = e.split_part + (int64_t)m * e.H + n;
    floatx4 s = *reinterpret_cast<const floatx4*>(p);
    for (int k0 = 1; k0 < sk.slices; k0 += 8) {                  // eight loads in flight
      floatx4 v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) if (k0 + k < sk.slices) v[k] = *reinterpret_cast<const floatx4*>(p + (k0 + k) * stride);
#pragma unroll
      for (int k = 0; k < 8; ++k) if (k0 + k < sk.slices) s += v[k];
    }
    const float f = e.row_scale ? e.row_scale[m] : 1.f;
    T* o = e.dX + (int64_t)e.row_map[d.chunk_start + m] * e.ldx + n;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = (T)(f * s[i]);
  }
}

// ---- backward, stage 3: dW tile, f32, overwritten by the first chunk and accumulated after.
//      When accumulating, the old values of several blocks are fetched first (many loads in flight)
//      and only then added and stored: a load-add-store per element would pay the memory latency
//      256 times per tile.  Hot kernel: 16 bytes per lane, bounds looked at once per tile.
struct EpiDW {
  typedef NoPre Pre;
  template <class L> __device__ Pre preload(const TileCtx&, const GemmDims&) const { return Pre(); }
  static constexpr bool kSwap = true;        // hot kernel: blocks transposed, a lane holds four consecutive columns of one row
  static constexpr bool kSplit = false;
  static constexpr bool kPermute = false;
  static constexpr bool kGatherB = false;      // the B rows come through a row map (GemmDims::b_rows)
  __device__ void keep_alive() const { dW[0] = 0.f; }
  float* dW; int64_t ldw; int V, H; int accumulate;

  // Hot kernel.  A lane holds four columns of one row in each of two neighbouring blocks, a lane pair thus two rows: it swaps halves, so that a
  // store writes eight rows in whole lines of 128 bytes instead of sixteen in halves, and the lines leave in non-temporal stores (NT) where the array has
  // its rows on lines.  256 KB a tile, with few slabs a tile this is what it waits for: 747 tokens at the 7B head (twelve slabs), the whole call 2390 us, whole
  // lines 2316, non-temporal as well 2258 (non-temporal halves 2485); 11.5 k tokens 29.73 ms and 29.57.  Rows off the lines, H 1160: 1822 us, whole lines 1822, non-temporal 1829.
  template <int MB, int NB, bool ACC, bool EDGE, bool NT>
  __device__ __attribute__((always_inline)) void rows(floatx4 (&acc)[MB][NB], const TileCtx& c) const {
    const int r = c.lane & 15, p = r & 1, n = c.n0 + p * 16 + (c.lane >> 4) * 4;
#pragma unroll
    for (int bi = 0; bi < MB; ++bi) {
      const int m = c.m0 + bi * 16 + (r & ~1);                     // the pair's first row
      float* const q[2] = {dW + (int64_t)m * ldw + n, dW + (int64_t)(m + 1) * ldw + n};
      auto there = [&](int w, int k) __attribute__((always_inline)) { return !EDGE || (m + w < V && n + k * 32 < H); };
      floatx4 old[2][NB / 2];
      if (ACC) {
#pragma unroll
        for (int k = 0; k < NB / 2; ++k)
#pragma unroll
          for (int w = 0; w < 2; ++w) if (there(w, k)) old[w][k] = *reinterpret_cast<const floatx4_any*>(q[w] + k * 32);
      }
#pragma unroll
      for (int k = 0; k < NB / 2; ++k) {
        floatx4 v[2];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float a = acc_read<true>(acc[bi][2 * k], e), b = acc_read<true>(acc[bi][2 * k + 1], e);
          const float recv = __uint_as_float((unsigned)__builtin_amdgcn_mov_dpp((int)__float_as_uint(p ? a : b), 0xB1, 0xF, 0xF, true));
          v[0][e] = p ? recv : a; v[1][e] = p ? b : recv;
          if (ACC) { v[0][e] = old[0][k][e] + v[0][e]; v[1][e] = old[1][k][e] + v[1][e]; }
        }
#pragma unroll
        for (int w = 0; w < 2; ++w)
          if (there(w, k)) {
            if (NT) __builtin_nontemporal_store(v[w], reinterpret_cast<floatx4*>(q[w] + k * 32));
            else *reinterpret_cast<floatx4_any*>(q[w] + k * 32) = v[w];
          }
      }
    }
  }

  template <class L, int MB, int NB, int BM, int BN, int WAVES_M, int WAVES_N, bool AGPR>
  __device__ __attribute__((always_inline)) void run(typename L::acc_t (&acc)[MB][NB], const TileCtx& c, unsigned char*, const GemmDims&, const Pre&) const {
    if constexpr (AGPR) {
      const bool edge = c.m0 + MB * 16 > V || c.n0 + NB * 16 > H;
      const bool lines = ldw % 32 == 0 && (reinterpret_cast<uintptr_t>(dW) & 127) == 0;
      if (accumulate) {
        if (edge) rows<MB, NB, true, true, false>(acc, c); else if (lines) rows<MB, NB, true, false, true>(acc, c); else rows<MB, NB, true, false, false>(acc, c);
      } else {
        if (edge) rows<MB, NB, false, true, false>(acc, c); else if (lines) rows<MB, NB, false, false, true>(acc, c); else rows<MB, NB, false, false, false>(acc, c);
      }
      return;
    }
    constexpr int RUN = L::kRegs < 4 ? L::kRegs : 4;      // registers handled per round: 4 rows x NB columns
#pragma unroll
    for (int bi = 0; bi < MB; ++bi)
#pragma unroll
      for (int q = 0; q < L::kRegs / RUN; ++q) {
        float old[RUN][NB];
        if (accumulate) {
#pragma unroll
          for (int e = 0; e < RUN; ++e) {
            const int m = c.m0 + L::row(bi, q * RUN + e, c.lane);
#pragma unroll
            for (int bj = 0; bj < NB; ++bj) {
              const int n = c.n0 + L::col(bj, c.lane);
              old[e][bj] = (m < V && n < H) ? dW[(int64_t)m * ldw + n] : 0.f;
            }
          }
        }
#pragma unroll
        for (int e = 0; e < RUN; ++e) {
          const int m = c.m0 + L::row(bi, q * RUN + e, c.lane);
#pragma unroll
          for (int bj = 0; bj < NB; ++bj) {
            const int n = c.n0 + L::col(bj, c.lane);
            const float v = acc_read<AGPR>(acc[bi][bj], q * RUN + e);
            if (m < V && n < H) dW[(int64_t)m * ldw + n] = accumulate ? old[e][bj] + v : v;
          }
        }
      }
  }
};

}  // namespace rlk
