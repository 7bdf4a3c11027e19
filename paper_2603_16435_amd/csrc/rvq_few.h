// rvq_few.h - residual-VQ encode of a few vectors per codebook group (a decode step: one vector per sequence of the batch).
//
// The codes are those of rvq_encode.h (the float64 arg-min of the definition, lowest index on ties, bf16 residual between the
// stages); with up to 32 vectors of a group the work is reading the codebooks once (256 groups x 16 stages x 512 entries:
// 547 MB, 115 us at the rate of a large copy), and the kernel written for 256 and more vectors spends its time scoring copies
// of the few there are (324 us; this one: 137).  Here a workgroup takes 16 NV vectors of one group:
//  * Four scoring wavefronts share the entries of a stage (blocks of 16 in turn).  They read the codebook straight from memory
//    in MFMA operand layout (A = 16 entries, B = 16 vectors, -|c|^2/2 as the start of the accumulator), a round of 64 entries each at a
//    time (32 with 32 vectors: registers), and have two more rounds on their way, also across the end of a stage: the codebook does not depend on the codes.
//  * The scores of a stage stay in LDS.  When all are there, every lane compares its own with the vector's largest and lists the
//    entries within the margin (twice the bound on a float32 score's error, see rvq_encode.h); only those can be the exact arg-min.
//  * A fifth wavefront settles the stage: one entry listed is the code; several are evaluated in float64 from the stored values,
//    and if more were listed than the list holds, all entries are.  It also fetches the chosen entries for the
//    residual update.  It is a wavefront of its own because a wait for these loads would wait for all loads issued
//    before them too: the scoring wavefronts' loads of the next stage stay in flight meanwhile.
// Four workgroup barriers per stage, written out (lgkmcnt only) so that they do not wait for loads in flight.
// What bounds it: a CU takes in about 28 bytes a ns, 4.7 us a stage of 512 entries, and little more than 32 KB of loads wait in its queue: beyond that a wavefront
// stands still at the load it issues.  Settling a stage takes 2.8 us in which nobody would issue one.  So the last round of a stage is
// fetched again behind the second barrier, once the chosen entries' loads are out (the third), while they come in: of 111 us 102.  And the registers of a round are all
// read before its loads are issued: where the norms were used later, the compiler copied them, a wait for everything in flight in each round (136 us -> 111).
// Non-temporal loads, faster in a stream, lose here (119): a line is taken in two halves.  Other rounds, 64 / 32 entries: three of 32 for 16 vectors 109, of one block for 32 vectors
// 140 against 135.  256 groups, us before and now: 12 vectors of 16 stages of 512 entries 136 -> 102, of 56 of 1024 774 -> 663, 30 vectors 177 -> 135; 8 groups, 1 vector, 56 of 1024 639 -> 491.
#pragma once
#include "rvq_encode.h"

namespace rlk {

constexpr int kRvqFewScoreBytes = 128 * 1024;                     // scores of one stage: 64 NV bytes per entry
constexpr int kRvqFewList = 32;
__host__ __device__ constexpr int rvq_few_max_entries(int nv) { return kRvqFewScoreBytes / (64 * nv); }

__device__ __attribute__((always_inline)) inline void rvq_few_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// The code of a vector none of whose distances is below infinity (the vector, or the whole codebook, is not finite): the entry that
// the main pass of rvq_encode_kernel is left with, so that a vector's codes do not depend on how many others are encoded with it.
// That pass keeps the largest block maximum with the block's number in its low mantissa bits (which makes a NaN of an infinity, but
// for block 0) behind a finite stand-in; here the same steps run over the stage's scores in LDS.  All 64 lanes call it; lane group kq
// walks entries 4 kq .. 4 kq + 3 of every block.  sc: the lane's scores of block 0; the four blocks of a round are 64 apart, rounds `stride`.
// Out of line: inlined, its code cost a call that never needs it 1.4 % (256 groups, 12 vectors: 136.6 -> 138.4 us; this way 135.9).
__device__ __attribute__((noinline)) int rvq_unsettled_index(const floatx4* sc, int stride, int nblk, int kq) {
  const int nb = 32 - __builtin_clz((unsigned)(nblk - 1));
  const unsigned idmask = (1u << nb) - 1u;
  float best = __uint_as_float((__float_as_uint(-3.0e38f) & ~idmask) | idmask);
  floatx4 sv;
#pragma unroll
  for (int e = 0; e < 4; ++e) sv[e] = -3.0e38f;
#pragma unroll 1
  for (int blk = 0; blk < nblk; ++blk) {
    const floatx4 v = sc[(blk >> 2) * stride + (blk & 3) * 64];
    const bool last = blk == nblk - 1;
    float m3, mx;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(m3) : "v"(v[0]), "v"(v[1]), "v"(v[2]));
    asm("v_max_f32 %0, %1, %2" : "=v"(mx) : "v"(m3), "v"(v[3]));
    if (last) mx = fmaxf(m3, v[3]);
    const float m4 = __uint_as_float((__float_as_uint(mx) & ~idmask) | (unsigned)blk);
    const bool gt = m4 > best;
#pragma unroll
    for (int e = 0; e < 4; ++e) sv[e] = gt ? v[e] : sv[e];
    float raw = best;
    asm("v_max_f32 %0, %0, %1" : "+v"(raw) : "v"(m4));
    best = last ? fmaxf(best, m4) : raw;
  }
  int blk = (int)(__float_as_uint(best) & idmask);
  if (blk >= nblk) blk = 0;
  const float m = fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3]));
  int i = 16 * blk + 4 * kq + (sv[0] == m ? 0 : sv[1] == m ? 1 : sv[2] == m ? 2 : 3);
  unsigned a, b, ia, ib;
  rvq_pair<16>(__float_as_uint(best), a, b); rvq_pair<16>((unsigned)i, ia, ib);
  bool tb = __uint_as_float(b) > __uint_as_float(a) || (__uint_as_float(b) == __uint_as_float(a) && (int)ib < (int)ia);
  best = __uint_as_float(tb ? b : a); i = (int)(tb ? ib : ia);
  rvq_pair<32>(__float_as_uint(best), a, b); rvq_pair<32>((unsigned)i, ia, ib);
  tb = __uint_as_float(b) > __uint_as_float(a) || (__uint_as_float(b) == __uint_as_float(a) && (int)ib < (int)ia);
  return (int)(tb ? ib : ia);
}

// grid as for rvq_encode_kernel with 16 NV vectors per workgroup; S % 64 == 0, S <= rvq_few_max_entries(NV)
template <int NV>
__global__ __launch_bounds__(320, 1)
void rvq_few_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ cb, const float* __restrict__ cn,
                    int G, int L, int N, int S, int32_t* __restrict__ codes, bf16_t* __restrict__ residual, int32_t* __restrict__ stats) {
  constexpr int VECS = 16 * NV, U = NV == 1 ? 4 : 2, D = 2;       // U: blocks per scoring wavefront and round (four wavefronts of 64 entries, or of 32)
  __shared__ floatx4 score[kRvqFewScoreBytes / 16];               // [round][block of the wavefront][vector block][wavefront, lane]
  __shared__ u32x4_t bits[VECS][kRvqD / 8], rows[VECS][kRvqD / 8]; // the vectors as stored; the chosen entries
  __shared__ float top[4][VECS], cmx[4];
  __shared__ int count[VECS], cand[VECS][kRvqFewList];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int e16 = lane & 15, kq = lane >> 4;
  const int w = blockIdx.x, gx = (L + VECS - 1) / VECS;
  const int g = 8 * ((w >> 3) / gx) + (w & 7);
  if (g >= G) return;                                             // (the whole workgroup)
  const int v0 = ((w >> 3) % gx) * VECS;
  x += (int64_t)g * L * kRvqD; codes += (int64_t)g * L * N;
  cb += (int64_t)g * N * S * kRvqD; cn += (int64_t)g * N * S;
  if (residual) residual += (int64_t)g * L * kRvqD;

  const int nblk = S / 16, rounds = (nblk + 4 * U - 1) / (4 * U), total = N * rounds;
  const bool scoring = wave < 4;
  u32x4_t ra[NV][4];                                              // [vector block][k-step]: vector l%16, k = 32 ks + 8 (l/16) .. +7
  float rn2[NV];
  u32x4_t nx[D][U][4];                                            // the entries and squared norms of the next D rounds
  floatx4 nn[D][U];
  // the next round to be fetched, into buffer i: block 16 r + 4 u + wave of its stage (past the stage's end: its last block, not used)
  int f_stage = 0, f_r = 0;
  auto fetch = [&](int i) __attribute__((always_inline)) {
    const int st = f_stage < N ? f_stage : N - 1;                 // (past the end one block again and again, not used: no branch around the loads)
    const bf16_t* scb = cb + (int64_t)st * S * kRvqD;
    const float* scn = cn + (int64_t)st * S;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      int blk = f_r * 4 * U + u * 4 + wave; blk = f_stage == N ? 0 : blk < nblk ? blk : nblk - 1;
      const bf16_t* ent = scb + (int64_t)(blk * 16 + e16) * kRvqD + kq * 8;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) nx[i][u][ks] = *reinterpret_cast<const u32x4_t*>(ent + ks * 32);
      nn[i][u] = *reinterpret_cast<const floatx4*>(scn + blk * 16 + 4 * kq);
    }
    if (++f_r == rounds) { f_r = 0; f_stage = f_stage < N ? f_stage + 1 : N; }
  };
  if (scoring) {
    fetch(0);
#pragma unroll
    for (int b = 0; b < NV; ++b) {
      int v = v0 + b * 16 + e16; v = v < L ? v : L - 1;
      float a = 0.f;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        ra[b][ks] = *reinterpret_cast<const u32x4_t*>(x + (int64_t)v * kRvqD + ks * 32 + kq * 8);
        a = rvq_sumsq(ra[b][ks], a);
        if (wave == 0) bits[b * 16 + e16][ks * 4 + kq] = ra[b][ks];
      }
      rn2[b] = rvq_sum4(a);
    }
#pragma unroll
    for (int i = 1; i < D; ++i) fetch(i);
  }
  if (tid < VECS) count[tid] = 0;                                 // (the first append comes after the first barrier)

  const float NEG = -__builtin_inff();
  if (scoring) {
    float mx[NV], cm = 0.f;
#pragma unroll
    for (int b = 0; b < NV; ++b) mx[b] = NEG;
    int r = 0;
    auto round = [&](int i) __attribute__((always_inline)) {
      floatx4 acc[U][NV];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        floatx4 h;
#pragma unroll
        for (int e = 0; e < 4; ++e) { cm = fmaxf(cm, nn[i][u][e]); h[e] = -0.5f * nn[i][u][e]; }
#pragma unroll
        for (int b = 0; b < NV; ++b) {
          acc[u][b] = h;
#pragma unroll
          for (int ks = 0; ks < 4; ++ks)
            acc[u][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, nx[i][u][ks]), __builtin_bit_cast(bf16x8, ra[b][ks]), acc[u][b], 0, 0, 0);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (r * 4 * U + u * 4 + wave < nblk) {                    // (uniform)
#pragma unroll
          for (int b = 0; b < NV; ++b) {
            score[((r * U + u) * NV + b) * 256 + tid] = acc[u][b];
#pragma unroll
            for (int e = 0; e < 4; ++e) mx[b] = fmaxf(mx[b], acc[u][b][e]);
          }
        }
      const bool last = ++r == rounds;
      if (last) {
        r = 0;
#pragma unroll
        for (int b = 0; b < NV; ++b) {
          const float m = rvq_max4(mx[b]);
          if (kq == 0) top[wave][b * 16 + e16] = m;
          mx[b] = NEG;
        }
        cm = rvq_max4(cm);                                          // (the lanes of a group have the same norms)
        if (lane == 0) cmx[wave] = cm;
        rvq_few_barrier();
        // list the entries that come within the margin of the largest score
        const float cmax = fmaxf(fmaxf(cmx[0], cmx[1]), fmaxf(cmx[2], cmx[3]));
#pragma unroll
        for (int b = 0; b < NV; ++b) {
          const int v = b * 16 + e16;
          const float best = fmaxf(fmaxf(top[0][v], top[1][v]), fmaxf(top[2][v], top[3][v]));
          const float margin = kRvqGamma2 * (sqrtf(rn2[b] * 1.02f * cmax) + 0.5f * cmax);   // (1.02: rn2 is known to one part in 2^7)
          for (int q0 = 0; q0 < rounds * U; q0 += U) {
            floatx4 s[U];
#pragma unroll
            for (int u = 0; u < U; ++u) s[u] = score[((q0 + u) * NV + b) * 256 + tid];
#pragma unroll
            for (int u = 0; u < U; ++u) {
              const int blk = (q0 + u) * 4 + wave;
              bool in[4];
#pragma unroll
              for (int e = 0; e < 4; ++e) in[e] = blk < nblk && !(best - s[u][e] > margin);
              if (in[0] | in[1] | in[2] | in[3])
#pragma unroll
                for (int e = 0; e < 4; ++e)
                  if (in[e]) {
                    const int pos = atomicAdd(&count[v], 1);
                    if (pos < kRvqFewList) cand[v][pos] = blk * 16 + 4 * kq + e;
                  }
            }
          }
        }
        cm = 0.f;
        rvq_few_barrier();
        rvq_few_barrier();                                          // (the chosen entries' loads are on their way)
      }
      // into the registers just read: any of these read later would want copies, and a copy waits for all loads on their way
      asm volatile("" : "+v"(cm) :: "memory");
      __builtin_amdgcn_sched_barrier(0);
      fetch(i);
      __builtin_amdgcn_sched_barrier(0);
      if (!last) return;
      rvq_few_barrier();
#pragma unroll
      for (int b = 0; b < NV; ++b) {
        float a = 0.f;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          ra[b][ks] = rvq_sub_bf16(ra[b][ks], rows[b * 16 + e16][ks * 4 + kq], a);
          if (wave == 0) bits[b * 16 + e16][ks * 4 + kq] = ra[b][ks];       // (read again after two more barriers)
        }
        rn2[b] = rvq_sum4(a);
      }
    };
    int t = 0;
    for (; t + D <= total; t += D)
#pragma unroll
      for (int i = 0; i < D; ++i) round(i);
    if (t < total) round(0);
  } else {
    for (int stage = 0; stage < N; ++stage) {                     // settle the stage: lane v answers for vector v
      rvq_few_barrier();
      rvq_few_barrier();
      const bf16_t* stage_cb = cb + (int64_t)stage * S * kRvqD;
      const int v = lane < VECS ? lane : VECS - 1;
      const int n = count[v];
      int z = cand[v][0];                                         // (at least one is listed: neither the largest score nor one that is not a number can fail the test)
      unsigned long long open = __ballot(lane < VECS && v0 + lane < L && n != 1);
      if (stats && lane == 0 && open) atomicAdd(stats, __builtin_popcountll(open));
      while (open) {
        const int q = __builtin_ctzll(open);
        open &= open - 1;
        // a vector that is not finite has no finite distance: nothing to look at
        const unsigned two = reinterpret_cast<const unsigned*>(&bits[q][0])[lane];
        const bool finite = !__ballot((two & 0x7f80u) == 0x7f80u || (two & 0x7f800000u) == 0x7f800000u);
        const int listed = count[q], m = !finite ? 0 : listed > kRvqFewList ? S : listed;
        double dmin = __builtin_inf();
        int imin = 0x7fffffff;
        for (int i = 0; i < m; i += 4) {                          // four entries at a time, one per 16 lanes
          int ent = -1;
          if (i + kq < m) ent = listed > kRvqFewList ? i + kq : cand[q][i + kq];
          const double d = rvq_exact_distance16(&bits[q][0], stage_cb, ent, e16);
#pragma unroll
          for (int k = 0; k < 4; ++k) {
            const double dk = __shfl(d, 16 * k);
            const int ek = __shfl(ent, 16 * k);
            if (ek >= 0 && dk < __builtin_inf() && (dk < dmin || (dk == dmin && ek < imin))) { dmin = dk; imin = ek; }
          }
        }
        if (__builtin_expect(imin >= S, 0)) imin = rvq_unsettled_index(score + (q >> 4) * 256 + kq * 16 + (q & 15), NV * 256, nblk, kq);     // (whatever the order of the list)
        if (lane == q) z = imin;
      }
      if (lane < VECS) {
        count[lane] = 0;
        if (v0 + lane < L) codes[(int64_t)(v0 + lane) * N + stage] = z;
      }
      u32x4_t c[VECS / 4];                                        // a quarter of the wavefront per entry
#pragma unroll
      for (int i = 0; i < VECS / 4; ++i) {
        const int zi = __shfl(z, 4 * i + kq);
        c[i] = *reinterpret_cast<const u32x4_t*>(stage_cb + (int64_t)zi * kRvqD + 8 * e16);
      }
      __builtin_amdgcn_sched_barrier(0);
      rvq_few_barrier();
#pragma unroll
      for (int i = 0; i < VECS / 4; ++i) rows[4 * i + kq][e16] = c[i];
      rvq_few_barrier();
    }
  }
  if (residual && wave == 0) {
#pragma unroll
    for (int b = 0; b < NV; ++b) {
      const int v = v0 + b * 16 + e16;
      if (v < L) {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) *reinterpret_cast<u32x4_t*>(residual + (int64_t)v * kRvqD + ks * 32 + kq * 8) = ra[b][ks];
      }
    }
  }
}

}  // namespace rlk
