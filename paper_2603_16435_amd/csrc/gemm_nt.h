// gemm_nt.h - the contraction main loops of the library (gfx950 / CDNA4).
//
//   C[m,n] = sum_k A[m,k] * B[n,k]        A: [M,K] row-major, B: [N,K] row-major ("NT")
//
// Every contraction of the path is brought into this form (K contiguous in both operands)
// so that one MFMA main loop serves the forward logits, the recomputed logits, dX and dW;
// what differs is the epilogue functor that consumes the accumulators in registers.  One
// exception: the hot kernel can also take an operand K-major (the stored array is A^T or B^T, rows = k),
// read through transposing LDS loads; dW uses that to contract dS^T X out of dS itself, dX of smaller batches to read W as it is.
//
// Two kernels (and that of gemm_f32.h) share tile order, LDS layout and epilogues:
//  * gemm_nt_bf16_kernel  - the hot one (bf16, 16-byte aligned rows).  256x256 tile, four wavefronts of
//    128x128 each (256 accumulator registers per lane live in AGPRs, one wavefront per SIMD),
//    K walked in slabs of 64, MFMA shape 16x16x32 (measured on this part: at the power limit it
//    sustains about 15 % more flops than 32x32x16 on random data).  Slabs go from global memory
//    straight into LDS (global_load ... lds, 16 bytes per lane) into two static 64 KiB stages.  A
//    slab is four phases of 32 MFMAs; its loads are spread over three phases so that no burst
//    blocks the MFMA issue, the fragments of a phase are read from LDS during the phase before,
//    and the last phase of a slab runs after the workgroup barrier so that it hides the first
//    fragment reads of the next slab.  The MFMAs are inline asm and every one is fenced with
//    sched_barrier, so the interleaving in the source is the interleaving issued.  A light
//    software prefetch (one 4-byte load per 128-byte line, two slabs ahead, shared between the
//    workgroups of an XCD) pulls the next panels into that XCD's L2.
//  * gemm_nt_kernel       - general kernel (narrow f32 tiles, unaligned operands, logits of small hidden sizes off the grid of 128): tile size as
//    a parameter, register-staged loads with a K-tail predicate.
//
// LDS rows are 128 B = eight 16-byte chunks; chunk c of row r sits at slot c ^ ((r>>1)&7),
// which spreads both the 16-byte row-wise stores and the column-wise fragment loads over all
// 64 banks (measured: zero bank conflicts).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rlk {

typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned u32x2_t __attribute__((ext_vector_type(2)));

constexpr int kSlabBytes = 128;   // bytes of K per LDS row
constexpr int kXcds = 8;          // MI355X: 8 accelerator dies, workgroups dealt round-robin

template <class T> struct Elem;
template <> struct Elem<bf16_t> { static constexpr int kPerChunk = 8; static constexpr int kBK = 64; };
template <> struct Elem<float>  { static constexpr int kPerChunk = 4; static constexpr int kBK = 32; };
struct Layout32;
struct Layout16;
template <bool SMALL> struct GeneralLayout { typedef Layout32 L; typedef u32x4_t F; };       // general kernel: MFMA blocks, fragment of a k-step
template <> struct GeneralLayout<true> { typedef Layout16 L; typedef u32x2_t F; };

struct GemmDims {
  int M, N, K;            // upper bounds (static); the dynamic extent trims one of them
  int64_t lda, ldb;       // row strides in elements
  const int* a_rows;      // optional gather: logical row m of A lives at row a_rows[m]
  const int* b_rows;
  int64_t b_span;         // rows of B that b_rows picks from
  const int* n_real;      // device scalar: number of compacted rows in the whole batch
  int chunk_start;        // first compacted row of this chunk
  const int* chunk;       // if set, device pair {first compacted row, rows} of this chunk; replaces n_real / chunk_start,
                          // and the gather tables are then indexed from the chunk's first row
  int dyn;                // which extent is min(rows left in the chunk, bound): 0 none, 1 M, 2 N, 3 K (rounded up to k_round)
  int k_round;            // dyn == 3: rows beyond the chunk's last that the producers of both operands have zeroed, a power of two
  int zero_if_empty;      // dyn == 3 only: an empty chunk still runs the epilogue (with K = 0) instead of returning
  int group_m;            // tile-order parameter: M-tiles per band
  int split_slots;        // > 0: the contraction may be cut along K (see split_k); workgroups the chip runs at a time
  int b_k_rows;           // hot kernel, B operand given K-major: its rows (K is their number rounded up, with zeros in the other operand)
  int fill_tiles;         // tiles of another contraction over K = M in the same launch, which fill the CUs this one leaves
};

// Slab-tiled operand layout of the library's own bf16 work buffers: [row / 256][k / 64][256 rows][64 k].
// The 32 KiB that a workgroup loads per operand and slab are then contiguous in memory (one page, one DRAM
// row run) instead of 256 pieces of 128 bytes a whole matrix row apart; K is the buffer's full K extent.
__device__ __host__ inline int64_t tiled_index(int r, int k, int64_t K) {
  return (int64_t)(r >> 8) * (K * 256) + (int64_t)(k >> 6) * 16384 + ((r & 255) << 6) + (k & 63);
}
__device__ __host__ inline int64_t operand_index(bool tiled, int r, int k, int64_t ld) {
  return tiled ? tiled_index(r, k, ld) : (int64_t)r * ld + k;
}

// Apply the dynamic extent.  Returns false if this launch has nothing to do.
__device__ inline bool resolve_dims(GemmDims& d, int& M, int& N, int& K) {
  M = d.M; N = d.N; K = d.K;
  if (!d.dyn) return true;
  int left;
  if (d.chunk) {
    const int2 c = *reinterpret_cast<const int2*>(d.chunk);         // (8-byte aligned)
    const int cs = c.x;
    left = c.y;
    d.chunk_start = cs;
    if (d.a_rows) d.a_rows += cs;
    if (d.b_rows) d.b_rows += cs;
  } else {
    left = *d.n_real - d.chunk_start;
  }
  if (left <= 0) {
    if (d.dyn == 3 && d.zero_if_empty) K = 0; else return false;
  } else if (d.dyn == 1) M = left < M ? left : M;
  else if (d.dyn == 2) N = left < N ? left : N;
  else { const int k = (left + d.k_round - 1) & ~(d.k_round - 1); K = k < K ? k : K; }
  return true;
}

// Cutting a contraction along K.  dX = dS W has K = V and only (tokens / tile) x (H / tile) tiles: a few hundred tokens
// leave most of the chip idle behind a serial chain of thousands of slabs.  It is then cut into slices of `per` steps
// (a step is one slab, two in the hot kernel), each slice's tile goes to a partial buffer in f32 and splitk_reduce_kernel
// adds the slices in order.  The number of slices minimises the time in steps, for `slots` workgroups at a time: the
// rounds of workgroups times (steps per slice + what a workgroup spends outside its main loop), but no less than all
// the work, `fill` steps of the other contraction of the launch included, spread over the slots.  A partial tile costs
// more outside the loop (it is written and read again in f32), and no more than 2 slots workgroups are made, which bounds
// the partial buffer.  The number of tokens is only known on the device, so every workgroup works the cut out for itself:
// lane s of a wavefront prices s + 1 slices.  (747 tokens at the 7B head, H 3584, V 152064: 42 tiles of 2376 slabs; dX + dW in one launch
// 3.84 ms, cut into three slices 2.24, and 1.72 since the tiles leave in 16-byte stores.)
constexpr int kMaxSplit = 64, kSplitMinSteps = 4;
struct SplitK { int slices, per; };
__device__ __host__ inline int64_t split_cost(int tiles, int nk, int want, int slots, int64_t fill, SplitK& k) {
  if ((int64_t)tiles * want > 2 * slots) want = 1;
  int per = (nk + want - 1) / want;
  if (per < kSplitMinSteps) per = nk < kSplitMinSteps ? (nk > 0 ? nk : 1) : kSplitMinSteps;
  k.per = per;
  k.slices = nk > 0 ? (nk + per - 1) / per : 1;
  const int64_t each = per + (k.slices > 1 ? 6 : 2), n = (int64_t)tiles * k.slices;
  const int64_t rounds = (n + slots - 1) / slots * each, spread = (n * each + fill) / slots;
  return rounds > spread ? rounds : spread;
}
inline SplitK split_k_host(int tiles, int nk, int slots, int64_t fill) {       // the same on the host
  SplitK best{1, nk}, k;
  int64_t c0 = split_cost(tiles, nk, 1, slots, fill, best);
  for (int s = 2; s <= kMaxSplit; ++s) {
    const int64_t c = split_cost(tiles, nk, s, slots, fill, k);
    if (c < c0) { c0 = c; best = k; }
  }
  return best;
}
__device__ inline SplitK split_k(int tiles, int nk, int slots, int64_t fill) {       // every lane of the wavefront must call it
  SplitK k;
  const int64_t c = split_cost(tiles, nk, (int)(threadIdx.x & 63) + 1, slots, fill, k);
  int64_t m = (c << 8) | (threadIdx.x & 63);
  for (int o = 32; o > 0; o >>= 1) { const int64_t x = __shfl_xor(m, o); m = x < m ? x : m; }
  split_cost(tiles, nk, __builtin_amdgcn_readfirstlane((int)(m & 63)) + 1, slots, fill, k);
  k.slices = __builtin_amdgcn_readfirstlane(k.slices); k.per = __builtin_amdgcn_readfirstlane(k.per);     // (uniform, and known to be)
  return k;
}
// steps of the filling contraction of the hot kernel (two slabs each): its K is the M rows here, rounded up to 256; 3 per tile for its epilogue
__device__ inline int64_t fill_steps(const GemmDims& d, int M) { return (int64_t)d.fill_tiles * ((M + 255) / 256 * 2 + 3); }

// Workgroup -> tile.  Workgroups are dealt to the 8 XCDs round-robin (workgroup id % 8), and each XCD has
// its own L2.  Tiles are walked in bands of group_m M-tiles by all N-tiles, M fastest inside a band column,
// so that the workgroups resident on one XCD at a time (about group_m M-tiles by 32 / group_m N-tiles)
// share their A and B panels through its L2.  Two ways of giving each XCD its part of that sequence:
//
//  * runs (by_share = false): the sequence is cut into eight equal runs.  The XCDs are then at unrelated
//    N positions, which spreads their B-panel reads over the memory channels.  Best where the B panels
//    are short or few enough to live in the memory-side cache (logits: K = H; dW: B = X^T chunk).
//  * shares (by_share = true): an XCD owns a contiguous share of the M-tiles that exist (after dynamic
//    trimming; shares differ by at most one tile) and all XCDs are at the same N-tiles at the same
//    time, so a B panel comes out of memory once and reaches the other XCDs through the memory-side
//    cache.  Needed for dX, where both operands stream from memory over a very long K (B = W^T, a
//    1 GB panel set per sweep): equal runs there are 7 % slower unless they happen to start on band
//    boundaries, and with shares a partly filled chunk is spread over all XCDs instead of the first few.
//
// The launch has launch_tiles() workgroups of the static bounds; the ones without a tile get false.
__device__ __host__ inline int launch_tiles(int tiles_m, int tiles_n) {
  return (tiles_m + kXcds - 1) / kXcds * kXcds * tiles_n;
}
__device__ __host__ inline bool tile_of_block(int pid, int tiles_m, int tiles_n, int group_m, bool by_share, int& tm, int& tn) {
  const int xcd = pid % kXcds, q = pid / kXcds;
  int t, first = 0, rows = tiles_m;                // position in the band sequence of `rows` M-tiles starting at `first`
  if (by_share) {
    const int base = tiles_m / kXcds, rem = tiles_m % kXcds;
    rows = base + (xcd < rem ? 1 : 0);
    first = xcd * base + (xcd < rem ? xcd : rem);
    if (q >= rows * tiles_n) return false;
    t = q;
  } else {
    const int total = tiles_m * tiles_n;
    if (pid >= total) return false;
    const int per = total / kXcds, rem = total % kXcds;
    t = xcd * per + (xcd < rem ? xcd : rem) + q;
  }
  const int band = group_m * tiles_n;
  const int g = t / band;
  const int first_m = g * group_m;
  const int gsz = (rows - first_m < group_m) ? (rows - first_m) : group_m;
  const int r = t - g * band;
  tm = first + first_m + r % gsz;
  tn = r / gsz;
  return true;
}

// Equal runs of `total` work items, one run per XCD: item of workgroup pid, or false.  (Any launch of at least `total`
// workgroups rounded up to a multiple of the XCD count covers them all.)
__device__ __host__ inline bool run_of_block(int pid, int total, int& t) {
  const int xcd = pid % kXcds, q = pid / kXcds, per = total / kXcds, rem = total % kXcds;
  if (q >= per + (xcd < rem ? 1 : 0)) return false;
  t = xcd * per + (xcd < rem ? xcd : rem) + q;
  return true;
}

__device__ inline int lds_off(int row, int chunk) {           // byte offset inside one operand slab
  return row * kSlabBytes + ((chunk ^ ((row >> 1) & 7)) << 4);
}

// Coordinates handed to an epilogue: everything it needs to map acc[bi][bj][i] to (m,n).
struct TileCtx {
  int m0, n0;        // first row / col of this wavefront's sub-tile
  int Mv, Nv;        // valid extents (after dynamic trimming)
  int lane, wm, wn;  // lane id, wavefront coordinates inside the workgroup
  int tile_m, tile_n;// workgroup tile indices
  int tid;
  int slice, slices; // K slice of this workgroup and how many there are (1: the tile is complete)
};
struct NoPre {};      // epilogue with nothing to fetch ahead of the main loop

// Accumulator layouts: where register i of block (bi, bj) of a lane sits inside the wavefront's
// sub-tile.  Registers come in runs of four consecutive rows of one column.
struct Layout32 {   // 32x32 MFMA blocks, 16 registers per block: row = 8*(i/4) + 4*(l/32) + i%4, col = l%32
  typedef floatx16 acc_t;
  static constexpr int kBlk = 32, kRegs = 16;
  __device__ static int row(int bi, int i, int lane) { return bi * 32 + ((i >> 2) << 3) + ((lane >> 5) << 2) + (i & 3); }
  __device__ static int col(int bj, int lane) { return bj * 32 + (lane & 31); }
  __device__ static bool owns(int r, int lane) { return ((r >> 2) & 1) == (lane >> 5); }   // does this lane hold row r of its columns?
};
struct Layout16 {   // 16x16 MFMA blocks, 4 registers per block: row = 4*(l/16) + i, col = l%16
  typedef floatx4 acc_t;
  static constexpr int kBlk = 16, kRegs = 4;
  __device__ static int row(int bi, int i, int lane) { return bi * 16 + ((lane >> 4) << 2) + i; }
  __device__ static int col(int bj, int lane) { return bj * 16 + (lane & 15); }
  __device__ static bool owns(int r, int lane) { return ((r >> 2) & 3) == (lane >> 4); }
};

// Reading one accumulator element in an epilogue.  In the hot kernel the 256 accumulators of a lane
// live in AGPRs; left to itself the compiler copies all of them to VGPRs at loop exit and spills
// most of them to scratch (tens of GB of extra HBM traffic per launch).  Reading each element
// through an explicit v_accvgpr_read at its point of use keeps them where they are.
template <bool AGPR, class V>
__device__ inline float acc_read(const V& v, int i) {
  if constexpr (AGPR) {
    float r;
    const float e = v[i];
    asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(r) : "a"(e));
    return r;
  } else {
    return v[i];
  }
}

// Narrow tiles of logits (`there` columns of the tiles_n of the static bounds exist): whether equal runs over the static grid put two on some CUs and three on none.  Workgroups that
// start together like this stay in step; they do best with the static runs and when each waits for its loads as soon as they are out (HOLD = false, below) and the other
// computes meanwhile.  In a run there are whole bands and part of one.  (Static grids of more than four workgroups a CU: those that do not exist make room, and the rest are not in step.)
// Scoring in f32, us, so and with held loads over the tiles that exist: 12 rows of tiles x 23, H 3916 213 and 230, 4 x 70, H 3072 161 and 168.  Others: one tile a CU at the most,
// 8 x 32, H 3072 127 and 98, 40 x 5 165 and 115; several on some, 12 x 33 302 and 180, 8 x 65 302 and 259; 100 x 4 206 and 177.  (The host asks for both forms where the bounds and K
// leave it open, may_be_two_a_cu: the second one costs short tiles 0.7 of 28 us.)
__device__ inline bool two_a_cu(int tiles_m, int tiles_n, int there, int group_m) {
  const int n = tiles_m * there, run = (tiles_m * tiles_n + kXcds - 1) / kXcds;
  if (n <= 32 * kXcds || n > 64 * kXcds || run > 128) return false;         // (ahead of the divisions)
  const int rows = tiles_m < group_m ? tiles_m : group_m, band = rows * tiles_n, part = run % band;
  return run / band * rows * there + (part < rows * there ? part : rows * there) <= 64;
}

// Tile, and slice of K, of a workgroup of the general and the f32 kernel.
struct GeneralTile { bool any, two; int M, N, K, nk, tm, tn, k_begin, slice, slices; };       // nk slabs of BK from slab k_begin on; two: two_a_cu
template <int BM, int BN, int BK, bool TWO = false>      // TWO: ask two_a_cu
__device__ inline GeneralTile general_tile(GemmDims& d, int pid) {
  GeneralTile t{};
  if (!resolve_dims(d, t.M, t.N, t.K)) return t;
  t.nk = (t.K + BK - 1) / BK; t.slices = 1;
  // dynamic M (dX): XCD shares of the M-tiles that exist; otherwise equal runs, of narrow tiles with dynamic N (logits) over those that exist: dealt over the static grid, which
  // is rounded up to 256 rows, they came two to a CU of one XCD while others had none (f32 scoring, us: 125 tokens, H 3816, V 4792 202 -> 154, 600, H 3072, V 3000 302 -> 181)
  const bool by_share = d.dyn == 1;
  const int tiles_m = ((by_share ? t.M : d.M) + BM - 1) / BM;
  int tiles_n = (d.N + BN - 1) / BN;
  if (d.dyn == 2 && BN == 16) {
    const int there = (t.N + BN - 1) / BN;
    t.two = TWO && two_a_cu(tiles_m, tiles_n, there, d.group_m);
    if (!t.two) tiles_n = there;
  }
  if (d.split_slots > 0) {
    const SplitK sk = split_k(tiles_m * tiles_n, t.nk, d.split_slots, 0);
    t.slices = sk.slices;
    int q;
    if (!run_of_block(pid, tiles_m * tiles_n * t.slices, q)) return t;      // slice after slice, M fastest inside one
    t.slice = q / (tiles_m * tiles_n);
    q -= t.slice * (tiles_m * tiles_n);
    t.tn = q / tiles_m; t.tm = q - t.tn * tiles_m;
    t.k_begin = t.slice * sk.per;
    t.nk = t.nk - t.k_begin < sk.per ? t.nk - t.k_begin : sk.per;
  } else if (!tile_of_block(pid, tiles_m, tiles_n, d.group_m, by_share, t.tm, t.tn)) return t;
  t.any = t.tm * BM < t.M && t.tn * BN < t.N;
  return t;
}

// General kernel: BM x BN tile, WAVES_M x WAVES_N wavefronts.  A slab is 128 bytes of K, staged global -> registers ->
// LDS (any alignment, K tail zeroed) into two LDS stages; one barrier per slab.
// Blocks of 32x32 (f32: v_mfma_f32_32x32x2), or of 16x16 where the tile is narrower than 32 (f32 only, 16x16x4).  Both add the k of an
// eight-wide step in the order 0 4 1 5 2 6 3 7, so that an f32 logit does not depend on the tile it came from: in the
// 16x16 form lane group g supplies element g/2, then g/2 + 2, of chunk g%2 - one 8-byte read, the chunks being stored in the
// order 0 2 1 3 for it.
//
// KG > 1: KG groups of such wavefronts share a tile, each taking every KG-th slab through LDS stages of its own; their accumulators are added in
// order at the end (for tiles that are few and have a long K; a step of a K cut is then KG slabs).
//
// HOLD (16x16 blocks): a slab's loads are waited for where it is stored, behind the MFMAs of the one before.  By itself the compiler exchanges the middle elements where the two kinds of load
// meet, ahead of the MFMAs, and waits for the loads there.  us without and with: scoring in f32, 2630 tokens, H 1024, V 1000 111 and 98; 13 tokens, H 3072, V 16 k 152 and 114; loss of 14 k tokens,
// H 64, V 2000 318 and 285.  (More slabs on their way: no faster anywhere, 160 tokens and tiles of sixteen wavefronts, H 3072 101 with four against 97.)
template <class T, int BM, int BN, int KG> constexpr int general_lds_bytes() { return KG * 2 * (BM + BN) * kSlabBytes; }
template <class T, class Epi, int BM, int BN, int WAVES_M, int WAVES_N, int KG, bool HOLD>
__device__ __attribute__((always_inline)) inline void gemm_nt_general_tile(const T* __restrict__ A, const T* __restrict__ B, const GemmDims& d, const GeneralTile& t,
                                                                           const Epi& epi, unsigned char* smem_all) {
  constexpr int NT = WAVES_M * WAVES_N * 64;
  constexpr int BK = Elem<T>::kBK;
  constexpr int EPC = Elem<T>::kPerChunk;
  constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
  constexpr bool SMALL = WN < 32;
  static_assert(!SMALL || sizeof(T) == 4, "16x16 blocks: f32 only");
  typedef typename GeneralLayout<SMALL>::L L;
  constexpr int MB = WM / L::kBlk, NB = WN / L::kBlk;
  constexpr int ROWS_PER_PASS = NT / 8;
  constexpr int PA = BM / ROWS_PER_PASS, PB = (BN + ROWS_PER_PASS - 1) / ROWS_PER_PASS;
  static_assert(BM % ROWS_PER_PASS == 0 && (BN % ROWS_PER_PASS == 0 || BN < ROWS_PER_PASS), "tile vs threads");
  constexpr int A_BYTES = BM * kSlabBytes, B_BYTES = BN * kSlabBytes;

  const int M = t.M, N = t.N, K = t.K, nk = t.nk, tm = t.tm, tn = t.tn;

  const int group = KG > 1 ? (int)threadIdx.x / NT : 0;
  const int tid = threadIdx.x - group * NT, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WAVES_N, wn = wave % WAVES_N;
  unsigned char* smem = smem_all + group * 2 * (A_BYTES + B_BYTES);
  const int k_begin = t.k_begin * KG + group;                        // first slab of the group; then every KG-th

  // ---- global -> register staging: thread owns chunk (tid&7) of rows (tid>>3) + p*ROWS_PER_PASS
  const int lchunk = tid & 7, lrow = tid >> 3;
  const T* ap[PA];
  const T* bp[PB];
#pragma unroll
  for (int p = 0; p < PA; ++p) {
    int r = tm * BM + lrow + p * ROWS_PER_PASS;
    r = r < M ? r : M - 1;
    if (d.a_rows) r = d.a_rows[r];
    ap[p] = A + (int64_t)r * d.lda + lchunk * EPC;
  }
#pragma unroll
  for (int p = 0; p < PB; ++p) {
    int r = tn * BN + lrow + p * ROWS_PER_PASS;
    r = r < N ? r : N - 1;
    if (d.b_rows) r = d.b_rows[r];
    bp[p] = B + (int64_t)r * d.ldb + lchunk * EPC;
  }
  uint4 ra[PA], rb[PB];
  auto gload = [&](int k0) __attribute__((always_inline)) {
    if (k0 + BK <= K) {                              // a whole slab
#pragma unroll
      for (int p = 0; p < PA; ++p) ra[p] = *reinterpret_cast<const uint4*>(ap[p] + k0);
#pragma unroll
      for (int p = 0; p < PB; ++p) rb[p] = *reinterpret_cast<const uint4*>(bp[p] + k0);
    } else {
      const bool ok = (k0 + lchunk * EPC) < K;
#pragma unroll
      for (int p = 0; p < PA; ++p) ra[p] = ok ? *reinterpret_cast<const uint4*>(ap[p] + k0) : make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int p = 0; p < PB; ++p) rb[p] = ok ? *reinterpret_cast<const uint4*>(bp[p] + k0) : make_uint4(0, 0, 0, 0);
    }
  };
  auto stored = [](uint4 v) __attribute__((always_inline)) {
    if (!SMALL) return v;
    if constexpr (HOLD) asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w));
    return make_uint4(v.x, v.z, v.y, v.w);
  };
  auto lstore = [&](int buf) __attribute__((always_inline)) {
    unsigned char* as = smem + buf * (A_BYTES + B_BYTES);
    unsigned char* bs = as + A_BYTES;
#pragma unroll
    for (int p = 0; p < PA; ++p) *reinterpret_cast<uint4*>(as + lds_off(lrow + p * ROWS_PER_PASS, lchunk)) = stored(ra[p]);
#pragma unroll
    for (int p = 0; p < PB; ++p)
      if (BN % ROWS_PER_PASS == 0 || lrow < BN) *reinterpret_cast<uint4*>(bs + lds_off(lrow + p * ROWS_PER_PASS, lchunk)) = stored(rb[p]);
  };

  typename L::acc_t acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < L::kRegs; ++e) acc[i][j][e] = 0.f;

  if (nk > 0) {
    gload(k_begin * BK);
    lstore(0);
  }
  __syncthreads();
  const int frow = lane & (L::kBlk - 1), fq = lane / L::kBlk;
  for (int kt = 0; kt < nk; ++kt) {
    const int cur = kt & 1;
    if (kt + 1 < nk) gload((k_begin + (kt + 1) * KG) * BK);
    const unsigned char* as = smem + cur * (A_BYTES + B_BYTES);
    const unsigned char* bs = as + A_BYTES;
    typedef typename GeneralLayout<SMALL>::F F;
#pragma unroll
    for (int s = 0; s < 4; ++s) {                  // four 32-byte k-steps per slab; in a step the blocks take turns, so that
      F a[MB], b[NB];                              // consecutive MFMAs do not wait for each other's accumulators
#pragma unroll
      for (int i = 0; i < MB; ++i)
        a[i] = *reinterpret_cast<const F*>(as + lds_off(wm * WM + i * L::kBlk + frow, s * 2 + (fq & 1)) + (fq >> 1) * 8);
#pragma unroll
      for (int j = 0; j < NB; ++j)
        b[j] = *reinterpret_cast<const F*>(bs + lds_off(wn * WN + j * L::kBlk + frow, s * 2 + (fq & 1)) + (fq >> 1) * 8);
#pragma unroll
      for (int e = 0; e < (sizeof(T) == 2 ? 1 : SMALL ? 2 : 4); ++e)
#pragma unroll
        for (int i = 0; i < MB; ++i)
#pragma unroll
          for (int j = 0; j < NB; ++j) {
            if constexpr (SMALL)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[i][e]), __uint_as_float(b[j][e]), acc[i][j], 0, 0, 0);
            else if constexpr (sizeof(T) == 4)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[i][e]), __uint_as_float(b[j][e]), acc[i][j], 0, 0, 0);
            else
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[i]), __builtin_bit_cast(bf16x8, b[j]), acc[i][j], 0, 0, 0);
          }
    }
    if (kt + 1 < nk) lstore(cur ^ 1);
    __syncthreads();
  }

  if constexpr (KG > 1) {                            // (the epilogues used with it need no barrier)
    static_assert(MB == 1 && NB == 1, "one block per wavefront");
    typename L::acc_t* part = reinterpret_cast<typename L::acc_t*>(smem_all);
    if (group > 0) part[(group - 1) * NT + tid] = acc[0][0];
    __syncthreads();
    if (group > 0) return;
#pragma unroll
    for (int g = 1; g < KG; ++g) acc[0][0] += part[(g - 1) * NT + tid];
  }
  TileCtx c;
  c.m0 = tm * BM + wm * WM; c.n0 = tn * BN + wn * WN;
  c.Mv = M; c.Nv = N; c.lane = lane; c.wm = wm; c.wn = wn; c.tile_m = tm; c.tile_n = tn; c.tid = tid;
  c.slice = t.slice; c.slices = t.slices;
  const typename Epi::Pre pre = epi.template preload<L>(c, d);
  epi.template run<L, MB, NB, BM, BN, WAVES_M, WAVES_N, false>(acc, c, smem, d, pre);
}
template <class T, class Epi, int BM, int BN, int WAVES_M, int WAVES_N, int KG = 1, bool TWO = false>
__global__ __launch_bounds__(WAVES_M * WAVES_N * KG * 64, WAVES_M * WAVES_N * KG > 8 ? 1 : 2)
void gemm_nt_kernel(const T* __restrict__ A, const T* __restrict__ B, GemmDims d, Epi epi) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[general_lds_bytes<T, BM, BN, KG>()];
  const GeneralTile t = general_tile<BM, BN, Elem<T>::kBK * KG, TWO>(d, blockIdx.x);
  if (!t.any) return;
  if constexpr (TWO)
    if (t.two) {
      gemm_nt_general_tile<T, Epi, BM, BN, WAVES_M, WAVES_N, KG, false>(A, B, d, t, epi, smem);
      return;
    }
  gemm_nt_general_tile<T, Epi, BM, BN, WAVES_M, WAVES_N, KG, true>(A, B, d, t, epi, smem);
}
// Two f32 contractions in tiles of 64 x 16 with four K groups in one launch: workgroups [0, n1) work on the first, the rest on the second.
template <class Epi1, class Epi2>
__global__ __launch_bounds__(1024)
void gemm_nt_small_pair_kernel(const float* __restrict__ A1, const float* __restrict__ B1, GemmDims d1, Epi1 epi1, int n1,
                               const float* __restrict__ A2, const float* __restrict__ B2, GemmDims d2, Epi2 epi2) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[general_lds_bytes<float, 64, 16, 4>()];
  if ((int)blockIdx.x < n1) {
    const GeneralTile t = general_tile<64, 16, Elem<float>::kBK * 4>(d1, blockIdx.x);
    if (t.any) gemm_nt_general_tile<float, Epi1, 64, 16, 4, 1, 4, true>(A1, B1, d1, t, epi1, smem);
  } else {
    const GeneralTile t = general_tile<64, 16, Elem<float>::kBK * 4>(d2, (int)blockIdx.x - n1);
    if (t.any) gemm_nt_general_tile<float, Epi2, 64, 16, 4, 1, 4, true>(A2, B2, d2, t, epi2, smem);
  }
}

// ------------------------------------------------------------------ bf16 hot kernel
typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef const __attribute__((address_space(1))) void* glb_ptr_t;

// The same load with its address given as a wavefront-uniform base (two scalar registers) plus a 32-bit lane offset in
// bytes: no vector operation goes into the address.  Written as inline assembly because the compiler, given base + offset,
// folds the offset into a per-lane 64-bit pointer outside the loop and adds the slab's stride to it with a vector add per
// load.  It keeps no count of such a load: the waits that cover it are the ones written out in the main loop.
// NT: non-temporal.
template <bool NT = false>
__device__ __attribute__((always_inline)) inline void load16_to_lds_uniform(const void* base, unsigned lane_bytes, void* l) {
  const unsigned lds = (unsigned)(size_t)(lds_ptr_t)l;      // uniform
  if constexpr (NT) asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" :: "v"(lane_bytes), "s"(base), "s"(lds) : "memory");
  else asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" :: "v"(lane_bytes), "s"(base), "s"(lds) : "memory");
}
// ... and with a 64-bit address per lane, for rows that span 4 GiB or more and for the last slabs of an operand.  (Every load of the hot kernel's main loop is
// one of these two, so that the compiler itself never sets M0 there.)
__device__ __attribute__((always_inline)) inline void load16_to_lds_lanes(const void* g, void* l) {
  const unsigned lds = (unsigned)(size_t)(lds_ptr_t)l;      // uniform
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" :: "v"(g), "s"(lds) : "memory");
}

__device__ inline void load16_to_lds(const void* g, void* l) {   // 64 lanes x 16 B -> 1 KiB of LDS at l
  __builtin_amdgcn_global_load_lds((glb_ptr_t)g, (lds_ptr_t)l, 16, 0, 0);
}

// A wavefront-uniform pointer the compiler may have computed in vector registers, in scalar ones.
template <class P> __device__ inline P* uniform_ptr(P* p) {
  const uint64_t v = (uint64_t)p;
  const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)v), hi = __builtin_amdgcn_readfirstlane((unsigned)(v >> 32));
  return (P*)(((uint64_t)hi << 32) | lo);
}

// Optional relabelling of the tile's rows and columns in the hot kernel (epilogues with kPermute).
// Which matrix row an LDS row holds is free to choose as long as the epilogue uses the same map.
// Inside each 128-row half of the tile, LDS row 16*b + 4*g + e (block b, lane group g, register e)
// holds matrix row 32*(b/2) + 8*g + 4*(b%2) + e, and LDS column-row 16*b + c holds matrix column
// 8*c + b: a lane (g, c) then owns runs of eight consecutive rows and of eight consecutive columns.
__device__ inline int perm_row(int b, int g, int e) { return ((b >> 1) << 5) + (g << 3) + ((b & 1) << 2) + e; }
__device__ inline int perm_col(int b, int c) { return (c << 3) + b; }
__device__ inline int perm_lds_row_a(int lr) { return (lr & 128) + perm_row((lr >> 4) & 7, (lr >> 2) & 3, lr & 3); }
__device__ inline int perm_lds_row_b(int lr) { return (lr & 128) + perm_col((lr >> 4) & 7, lr & 15); }

// One 16x16x32 bf16 MFMA, accumulator in place.  Written as inline asm so that the 64 accumulator
// blocks of a lane are pinned to the 256 AGPRs for the whole kernel: with the builtin the register
// allocator splits them between the two register files and fills the main loop with copies.  The
// compiler therefore does not know these are MFMAs: the required wait states before the epilogue
// reads the accumulators are inserted by hand (mfma_drain).
__device__ __attribute__((always_inline)) inline void mfma16(floatx4& acc, const u32x4_t& a, const u32x4_t& b) {
  asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
__device__ __attribute__((always_inline)) inline void mfma_drain() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); }

// Tune::kPfd: L2 prefetch distance in slabs (0 = none).  kPfWait: the prefetch goes out ahead of the slab's loads and is waited for with them.
// kVmg / kVmo: inside a phase of 32 MFMAs the slab loads are issued after MFMA number kVmo, kVmo + kVmg, ...  kLdA / kLdB: how many of
// a slab's 16 loads go into the phase after the barrier and into the first phase of the next slab (the rest into its second phase);
// the earlier they go, the longer they have to land before the next barrier.
constexpr int kHotStageBytes = (256 + 256) * kSlabBytes;      // one LDS stage of the hot kernel: a slab of A and of B

// Transposing LDS read (ds_read_b64_tr_b16).  Within each group of 16 lanes, the four 16-bit values that lane
// 4e + j/4 fetched (8 bytes at its own address) are dealt to lanes 4(j/4).. : lane j receives, as element e,
// value j%4 of the piece fetched by lane 4e + j/4.  With lanes 4e..4e+3 pointing at sixteen consecutive m of
// k-row e, lane j ends up with (m = j, k = 0..3): an MFMA operand read out of a K-major slab.
typedef short tr16x4_t __attribute__((ext_vector_type(4)));
__device__ __attribute__((always_inline)) inline u32x2_t lds_read_tr16(const unsigned char* p) {
  typedef __attribute__((address_space(3))) tr16x4_t* lds_ptr;
  return __builtin_bit_cast(u32x2_t, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p)));
}

// The work of one workgroup of the hot kernel: tile number `pid` of the contraction (A, B, d) into epi.
// stage0 / stage1 are the caller's two LDS stages; they must be separate objects so that the compiler
// can tell the stage being filled by the DMA loads from the stage the fragments are read from and
// does not serialise them with a vmcnt(0).
//
// ATR: the A operand is given K-major, element (m, k) at tiled_index(k, m, d.lda) (the slab-tiled layout of its
// transpose, whose rows are k): C = A^T-stored x B without a transposed copy of A in memory.  Its LDS slab is
// 64 k-rows of 256 m (512 bytes a row, 32-byte pieces XOR-swizzled by a function of the row such that the eight
// rows a half-wavefront's transposing read touches fall into different banks) and its fragments come from two
// transposing reads each.
//
// BTR: the B operand is given K-major and row-major, element (n, k) at B[k * d.ldb + n] with d.b_k_rows rows (dX contracts dS with W
// as it is stored, without a W^T in memory); same slab layout and reads as ATR.  Rows past the last are read as the last
// one: the A operand has zeros there.
//
// KT: K need not be a multiple of 128 (only of 8): 16-byte chunks past the end of a row are fetched from a zero block.
//
// FAR: the gathered B rows span 4 GiB or more, so that 32 bits do not hold a row's offset.
//
// Both have slabs whose load addresses are not those of the plain loop, at the end of K; the last six slabs (KT: three or four) run in a copy of the
// loop body that works them out per lane (`tail`), so that the plain loop needs no vector operation for its load addresses.  (With BTR
// it has others: the 16-bit offset of the transposing reads does not reach B's part of the second stage, 32 address adds per two slabs.)
__device__ const uint4 kZeroChunk = {0u, 0u, 0u, 0u};
template <class Epi, class Tune, bool ATR = false, bool BTR = false, bool KT = false, bool FAR = false>
__device__ __attribute__((always_inline)) inline void gemm_nt_bf16_tile(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, GemmDims d,
                                                                        const Epi& epi, int pid, unsigned char* stage0, unsigned char* stage1) {
  constexpr int PFD = Tune::kPfd, VMG = Tune::kVmg, VMO = Tune::kVmo, LDA = Tune::kLdA, LDB = Tune::kLdB;
  constexpr int BM = 256, BN = 256, BK = 64, WAVES_M = 2, WAVES_N = 2;
  constexpr int WM = 128, WN = 128, MB = 8, NB = 8;             // 8 x 8 blocks of 16 x 16 per wavefront
  constexpr int DSG = 2;                                        // one fragment read per DSG MFMAs
  constexpr int A_BYTES = BM * kSlabBytes, B_BYTES = BN * kSlabBytes, STAGE = A_BYTES + B_BYTES;
  constexpr int LDC = 16 - LDA - LDB;
  constexpr int LDMAX = LDA > LDB ? (LDA > LDC ? LDA : LDC) : (LDB > LDC ? LDB : LDC);
  static_assert(LDA >= 0 && LDB >= 0 && LDC >= 0 && VMO < VMG && (LDMAX - 1) * VMG + VMO < 32,
                "the slab loads of the fullest phase must fit into its 32 MFMAs");
  static_assert(STAGE == kHotStageBytes, "stage size");
  static_assert(!ATR || !Epi::kPermute, "the K-major A path loads rows in natural order");
  static_assert(!BTR || (!ATR && !KT && !Epi::kGatherB), "K-major B: dX");
  static_assert(!KT || !ATR, "K tail: row-wise operands");
  static_assert(!Epi::kSplit || (!ATR && !Epi::kGatherB), "a slice starts at a slab offset of both row-wise operands");

  int M, N, K;
  if (!resolve_dims(d, M, N, K)) return;
  int nk = KT ? (K + BK - 1) / BK : K / BK;
  // dynamic M (dX): XCD shares of the M-tiles that exist; otherwise equal runs over the static grid
  const bool by_share = d.dyn == 1;
  const int tiles_m = ((by_share ? M : d.M) + BM - 1) / BM, tiles_n = (d.N + BN - 1) / BN;
  int tm, tn, slice = 0, slices = 1, k_first = 0;                 // first slab
  if constexpr (Epi::kSplit) {
    const SplitK sk = split_k(tiles_m * tiles_n, nk / 2, d.split_slots, fill_steps(d, M));
    slices = sk.slices;
    if (slices > 1) {                                             // slice after slice, M fastest inside one: an XCD works on few
      int t;                                                      // slices, whose panels of both operands its L2 then holds
      if (!run_of_block(pid, tiles_m * tiles_n * slices, t)) return;
      slice = t / (tiles_m * tiles_n);
      t -= slice * (tiles_m * tiles_n);
      tn = t / tiles_m; tm = t - tn * tiles_m;
      k_first = slice * sk.per * 2;
      nk = nk - k_first < sk.per * 2 ? nk - k_first : sk.per * 2;
    }
  }
  if (slices == 1 && !tile_of_block(pid, tiles_m, tiles_n, d.group_m, by_share, tm, tn)) return;
  if constexpr (Epi::kSplit) {                                    // (all uniform; said so, because the slab loads want scalar addresses)
    nk = __builtin_amdgcn_readfirstlane(nk); k_first = __builtin_amdgcn_readfirstlane(k_first); tm = __builtin_amdgcn_readfirstlane(tm); tn = __builtin_amdgcn_readfirstlane(tn);
  }
  if (tm * BM >= M || tn * BN >= N) return;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);     // uniform: LDS addresses stay scalar
  const int wm = wave >> 1, wn = wave & 1;

  // ---- slab staging.  Wavefront w fills rows [64w, 64w+64) of A and of B: eight loads of eight
  // rows each.  A load writes lane l's 16 bytes to LDS offset 16*l of its 1 KiB target, i.e. row
  // l/8, slot l%8; the swizzle is therefore applied on the global side (which chunk a lane fetches).
  // Both operands are addressed as a wavefront-uniform base plus a 32-bit lane offset: the address of a load is then a scalar add per
  // slab and no vector operation (vector operations and MFMAs take turns on a SIMD).  All rows of a tile lie within
  // 256 rows of the tile's first, so the offsets fit; the hidden states, whose rows come through the row map, are addressed from their
  // first row, where they span less than 4 GiB (FAR otherwise: an address per lane; forward of 67 k tokens at the 7B head 56.4 ms that way, 55.8
  // with offsets, scoring of 10 k 8.22 and 8.06).
  // The rows that are gathered are all fetched before anything is done with one, and nothing in the way asks at run time how an operand is laid out: a
  // branch between the loads makes eight memory latencies of them, 1.3 us of a tile.
  constexpr bool GB = Epi::kGatherB;
  constexpr bool TILED = !GB;                                   // dX and dW contract the library's buffers, slab-tiled, the logits the caller's rows
  const bf16_t* ap[8];
  const bf16_t* bp[8];
  unsigned aoff[8], boff[8];
  int brow_of[8], pf_row = tn * BN + 32 * (tm & 7) + (lane & 31);
  pf_row = pf_row < N ? pf_row : N - 1;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int lr = wave * 64 + j * 8 + (lane >> 3), r = tn * BN + (Epi::kPermute ? perm_lds_row_b(lr) : lr);
    brow_of[j] = r < N ? r : N - 1;
    if constexpr (GB) brow_of[j] = d.b_rows[brow_of[j]];
  }
  if constexpr (GB && PFD > 0) pf_row = d.b_rows[pf_row];
  const bf16_t* abase = ATR ? A + tiled_index(0, tm * BM, d.lda)
                                  : A + (TILED ? tiled_index(tm * BM, 0, d.K) : (int64_t)(tm * BM) * d.lda);
  const bf16_t* bbase = BTR ? B + tn * BN : B + (TILED ? tiled_index(tn * BN, 0, d.K) : (int64_t)(tn * BN) * d.ldb);
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const int lr = wave * 64 + j * 8 + (lane >> 3);
    const int c = (lane & 7) ^ ((lr >> 1) & 7);
    if constexpr (ATR) {
      const int p = (wave * 8 + j) * 64 + lane;                  // 16-byte unit of the A slab this lane fills
      const int row = p >> 5, u = p & 31;                        // k-row of the slab, unit inside the row
      const int f = (row & 3) | (((row >> 3) & 1) << 2);
      const int m = tm * BM + (((u >> 1) ^ f) << 4) + ((u & 1) << 3);
      ap[j] = A + tiled_index(row, m, d.lda);
    } else {
      int r = tm * BM + (Epi::kPermute ? perm_lds_row_a(lr) : lr); r = r < M ? r : M - 1;
      ap[j] = A + (TILED ? tiled_index(r, 0, d.K) : (int64_t)r * d.lda) + c * 8;
    }
    if constexpr (BTR) {
      const int p = (wave * 8 + j) * 64 + lane;
      const int row = p >> 5, u = p & 31;
      const int f = (row & 3) | (((row >> 3) & 1) << 2);
      int n = tn * BN + (((u >> 1) ^ f) << 4) + ((u & 1) << 3); n = n < N ? n : N - 8;       // (N % 8 == 0)
      bp[j] = B + (int64_t)row * d.ldb + n;
    } else {
      bp[j] = B + (TILED ? tiled_index(brow_of[j], 0, d.K) : (int64_t)brow_of[j] * d.ldb) + c * 8;
    }
    aoff[j] = (unsigned)(ap[j] - abase) * 2u;                   // in bytes
    boff[j] = (unsigned)(bp[j] - (GB ? B : bbase)) * 2u;
  }
  const int a_ks = TILED ? 16384 : BK;                                    // elements from one slab to the next
  const int64_t b_ks = BTR ? (int64_t)BK * d.ldb : TILED ? 16384 : BK;
  if constexpr (Epi::kSplit) { abase = uniform_ptr(abase + (int64_t)k_first * a_ks); bbase = uniform_ptr(bbase + (int64_t)k_first * b_ks); }
  // K-major A: slab s is k-rows [64 s, 64 s + 64), i.e. quarter s%4 of row block s/4 of the tiled layout
  auto a_slab = [&](int slab) __attribute__((always_inline)) -> int64_t {
    return ATR ? (int64_t)(slab >> 2) * (d.lda * 256) + (slab & 3) * 4096 : (int64_t)slab * a_ks;
  };
  // load j of the 16 per slab (0..7 = A rows, 8..15 = B rows)
  // (the pointers are uniform, but behind a cut along K and a prefetch the compiler does not see it)
  auto uni = [&](const bf16_t* p) __attribute__((always_inline)) { if constexpr (Epi::kSplit && PFD > 0) return (const bf16_t*)uniform_ptr(p); else return p; };
  auto issue1 = [&](bool tail, int slab, unsigned char* stage, int j) __attribute__((always_inline)) {
    unsigned char* as = stage + wave * 64 * kSlabBytes;
    unsigned char* dst = j < 8 ? as + j * 8 * kSlabBytes : as + A_BYTES + (j - 8) * 8 * kSlabBytes;
    if (KT && tail) {
      const int c = (lane & 7) ^ ((4 * j + (lane >> 4)) & 7);         // the lane's chunk of the slab (row lr = 64 wave + 8 j + lane/8)
      const bf16_t* g = j < 8 ? ap[j & 7] + a_slab(slab) : bp[j & 7] + (int64_t)slab * b_ks;
      load16_to_lds_lanes(slab * BK + c * 8 < K ? (const void*)g : (const void*)&kZeroChunk, dst);
    } else if (j < 8) {
      load16_to_lds_uniform(uni(abase + a_slab(slab)), aoff[j], dst);      // (the hot kernel is not launched with gathered A rows)
    } else if (BTR && tail) {
      const int last = (d.b_k_rows - 1) >> 6, s_abs = k_first + slab, sc = s_abs < last ? s_abs : last;       // a slab that has rows
      const int row = ((wave * 8 + j - 8) * 64 + lane) >> 5, left = d.b_k_rows - 1 - sc * BK;
      load16_to_lds_lanes(bp[j - 8] + (int64_t)(sc * BK + (row < left ? row : left) - row) * d.ldb, dst);
    } else if constexpr (GB && FAR) {
      load16_to_lds_lanes(bp[j - 8] + (int64_t)slab * b_ks, dst);
    } else {
      load16_to_lds_uniform(uni((GB ? B : bbase) + (int64_t)slab * b_ks), boff[j - 8], dst);
    }
  };

  // ---- L2 prefetch.  The workgroups resident on one XCD at a time form (about) a block of 8 M-tiles
  // by 4 N-tiles that walks K in lock-step.  Wavefront 0 touches one quarter of the A panel rows,
  // wavefront 1 one eighth of the B panel rows, PFD slabs ahead, one 4-byte load per 128-byte line:
  // between them the block's workgroups cover every line once.  Wavefronts 2 and 3 execute the same
  // instruction on one fixed line (no divergent control flow around the accumulators).  The load goes out behind the slab's own loads
  // and is the one that the wait at the slab's end leaves in flight (loads come back in order; prefetch() says what holds it in its place): waited for there, a line that had to come from
  // memory held the slab up, which is what the prefetch is to avoid (67 k tokens at the 7B head: forward 56.4 -> 54.8 ms; 36 k tokens, H 2048,
  // V 32000: 3.81 -> 3.62, dX + dW 7.25 -> 6.77).  But the wait also keeps the workgroups of a block in step, so that a line is fetched once
  // for all of them: where a launch has very many rounds of tiles it stays (kPfWait), and in the slabs of a K tail, which do not run far enough
  // to drift and whose loads go out later for the work on their addresses (forward of 16 k tokens, V 50257, waited for or not: H 328, all six slabs 831 and
  // 842 us, H 392 892 and 909, H 504 956 and 981, H 1160 1796 and 1801).
  const unsigned char* pf_ptr;
  int pf_stride;
  const bool pf_atr = ATR && wave == 0;
  if (pf_atr) {                                    // K-major A: the slab's 256 lines are (k-row, 64-m block); a quarter per N-tile
    const int q = 64 * (tn & 3) + lane;
    pf_ptr = reinterpret_cast<const unsigned char*>(A + tiled_index(q >> 2, tm * BM + 64 * (q & 3), d.lda));
    pf_stride = 0;
  } else if (wave == 0) {
    int r = tm * BM + 64 * (tn & 3) + lane; r = r < M ? r : M - 1;
    pf_ptr = reinterpret_cast<const unsigned char*>(A + (TILED ? tiled_index(r, 0, d.K) : (int64_t)r * d.lda));
    pf_stride = a_ks * 2;
  } else if (BTR && PFD > 0 && wave == 1) {                   // K-major B: likewise, an eighth per M-tile
    const int q = 32 * (tm & 7) + (lane & 31);
    int n = tn * BN + 64 * (q & 3); n = n < N ? n : N - 8;
    pf_ptr = reinterpret_cast<const unsigned char*>(B + (int64_t)(q >> 2) * d.ldb + n);
    pf_stride = (int)b_ks * 2;
  } else if (wave == 1) {
    pf_ptr = reinterpret_cast<const unsigned char*>(B + (TILED ? tiled_index(pf_row, 0, d.K) : (int64_t)pf_row * d.ldb));
    pf_stride = (int)b_ks * 2;
  } else {
    pf_ptr = reinterpret_cast<const unsigned char*>(A);
    pf_stride = 0;
  }
  int pf_last = KT ? (K - 1) / BK : nk - 1;            // (a row has no lines past its end)
  if constexpr (BTR && PFD > 0) {
    const int whole = (d.b_k_rows >> 6) - 1 - k_first; // last slab of B all of whose rows exist
    if (wave == 1 && whole < pf_last) pf_last = whole;
    if (wave == 1 && whole < 0) { pf_ptr = reinterpret_cast<const unsigned char*>(B); pf_stride = 0; pf_last = 0; }
  }
  if constexpr (Epi::kSplit && PFD > 0) pf_ptr += (int64_t)k_first * pf_stride;
  unsigned pf0 = 0, pf1 = 0, pf_sink = 0;
  auto prefetch = [&](unsigned& slot, int kt) __attribute__((always_inline)) {
    if (PFD > 0) {
      pf_sink ^= slot;                                   // fetched two slabs ago: long since back
      const int k = kt + PFD < pf_last ? kt + PFD : pf_last;
      typedef const __attribute__((address_space(1))) unsigned* line_ptr;
      line_ptr p = (line_ptr)(pf_ptr + (int64_t)k * pf_stride + (pf_atr ? a_slab(k) * 2 : 0));
      asm volatile("" : "+v"(p));                        // not ahead of the slab's loads, volatile assembly like this ...
      slot = *p;
      asm volatile("" ::: "memory");                     // ... and not past the wait behind this, for all that is known of where p points
    }
  };

  TileCtx c;
  c.m0 = tm * BM + wm * WM; c.n0 = tn * BN + wn * WN;
  c.Mv = M; c.Nv = N; c.lane = lane; c.wm = wm; c.wn = wn; c.tile_m = tm; c.tile_n = tn; c.tid = tid;
  c.slice = slice; c.slices = slices;
  // what the epilogue needs from memory per column or row (a few registers): fetched now, used after the main loop
  const typename Epi::Pre pre = epi.template preload<Layout16>(c, d);

  floatx4 acc[MB][NB];
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

  // ---- fragments.  Operand of a 16x16x32 MFMA: lane l holds row l%16, k = 8*(l/16) .. +7 of the
  // 32-wide k-step, i.e. 16-byte chunk 4*s + l/16 of its row in the slab.  A k-step is consumed in
  // two phases (all eight A blocks against B blocks 0..3, then against B blocks 4..7), so the
  // register sets are: A two sets of eight, B two sets of four.
  const int frow = lane & 15, fq = lane >> 4;
  const int arow = (wm * WM + frow) * kSlabBytes, brow = A_BYTES + (wn * WN + frow) * kSlabBytes;
  const int swz = (frow >> 1) & 7;                 // the other row blocks are 16 rows apart: same swizzle
  u32x4_t fa[2][MB], fb[2][NB / 2];
  // K-major A: byte offset, in the slab, of the 8-byte piece this lane points a transposing read of block bi at:
  // k-row 8 (l/16) + (l%16)/4 of the k-step, 32-byte chunk (8 wm + bi) ^ f(row), piece l%4
  int atr_base[MB];
  if constexpr (ATR) {
    const int f = ((frow >> 2) & 3) | ((fq & 1) << 2);
#pragma unroll
    for (int i = 0; i < MB; ++i) atr_base[i] = (8 * fq + (frow >> 2)) * 512 + (((wm * 8 + i) ^ f) << 5) + ((frow & 3) << 3);
  }
  int btr_base[NB];                                // the same for a K-major B
  if constexpr (BTR) {
    const int f = ((frow >> 2) & 3) | ((fq & 1) << 2);
#pragma unroll
    for (int i = 0; i < NB; ++i) btr_base[i] = A_BYTES + (8 * fq + (frow >> 2)) * 512 + (((wn * 8 + i) ^ f) << 5) + ((frow & 3) << 3);
  }
  auto read_b_tr = [&](u32x4_t& dst, const unsigned char* fstage, int i, int fs, int h) __attribute__((always_inline)) {
    const u32x2_t v = lds_read_tr16(fstage + btr_base[i] + (32 * fs + 4 * h) * 512);
    dst[2 * h] = v[0]; dst[2 * h + 1] = v[1];
  };
  // half h (k = 0..3 or 4..7 of the lane's eight) of A block i of k-step fs
  auto read_a_tr = [&](u32x4_t& dst, const unsigned char* fstage, int i, int fs, int h) __attribute__((always_inline)) {
    const u32x2_t v = lds_read_tr16(fstage + atr_base[i] + (32 * fs + 4 * h) * 512);
    dst[2 * h] = v[0]; dst[2 * h + 1] = v[1];
  };
  auto kof = [&](int k) __attribute__((always_inline)) { return k < nk ? k : nk - 1; };   // slab number; past the end: harmless re-load

  // One phase = 32 MFMAs on (fa[aset], fb[bset]) into column half `half`, with, at fixed places between them,
  //  * fragment reads for the next phase, one per DSG MFMAs.  kind 4: fb[bset^1] <- B blocks 4..7 of
  //    k-step fs in fstage; kind 12: fa[aset^1], fb[bset^1] <- A blocks 0..7 and B blocks 0..3 of k-step fs
  //  * slab loads lo .. lo+nvm-1 of the slab at k0 into wstage.
  // Every MFMA (with what follows it) is fenced off, so the order below is the order issued.
  auto phase = [&](bool tail, int aset, int bset, int half, int kind, const unsigned char* fstage, int fs,
                   int k0, unsigned char* wstage, int lo, int nvm) __attribute__((always_inline)) {
    const int slot = ((fs * 4 + fq) ^ swz) << 4;
#pragma unroll
    for (int q = 0; q < 32; ++q) {
      // The B blocks are walked forth and back, so that from MFMA to MFMA only one operand changes: at the power limit that pays.  dX + dW of
      // 67 k tokens at the 7B head 108.4 ms without, 107.2 with it (holding a B block for all eight A blocks: 108.7 where the walk takes
      // 107.7); the forward 56.9 and 56.4.  kSwap: the operands' layouts are alike; exchanged, they give the transposed block with the same sums.
      const int w = (q >> 2) & 1 ? 3 - (q & 3) : q & 3;
      if constexpr (Epi::kSwap) mfma16(acc[q >> 2][half * 4 + w], fb[bset][w], fa[aset][q >> 2]);
      else mfma16(acc[q >> 2][half * 4 + w], fa[aset][q >> 2], fb[bset][w]);
      if (ATR && kind == 12) {                          // sixteen half-reads of A, one per MFMA, then the four of B
        if (q < 16) read_a_tr(fa[aset ^ 1][q >> 1], fstage, q >> 1, fs, q & 1);
        else if (q % DSG == 0 && q < 24) fb[bset ^ 1][(q - 16) / DSG] = *reinterpret_cast<const u32x4_t*>(fstage + brow + ((q - 16) / DSG) * 16 * kSlabBytes + slot);
      } else if (BTR) {                                 // B blocks in two half-reads each: eight for half of B, after the eight of A
        if (kind == 12 && q < 16) {
          if (q % DSG == 0) fa[aset ^ 1][q / DSG] = *reinterpret_cast<const u32x4_t*>(fstage + arow + (q / DSG) * 16 * kSlabBytes + slot);
        } else if (kind == 12 && q < 24) {
          read_b_tr(fb[bset ^ 1][(q - 16) >> 1], fstage, (q - 16) >> 1, fs, q & 1);
        } else if (kind == 4 && q < 8) {
          read_b_tr(fb[bset ^ 1][q >> 1], fstage, 4 + (q >> 1), fs, q & 1);
        }
      } else if (q % DSG == 0 && q / DSG < kind) {
        const int f = q / DSG;
        if (kind == 4) fb[bset ^ 1][f] = *reinterpret_cast<const u32x4_t*>(fstage + brow + (4 + f) * 16 * kSlabBytes + slot);
        else if (f < 8) fa[aset ^ 1][f] = *reinterpret_cast<const u32x4_t*>(fstage + arow + f * 16 * kSlabBytes + slot);
        else fb[bset ^ 1][f - 8] = *reinterpret_cast<const u32x4_t*>(fstage + brow + (f - 8) * 16 * kSlabBytes + slot);
      }
      if (q % VMG == VMO && q / VMG < nvm) issue1(tail, k0, wstage, lo + q / VMG);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // Slab kt sits in `cur`.  On entry fa[0] / fb[0] hold its k-step 0 (A all, B blocks 0..3) and loads
  // 0..LDA-1 of slab kt+1 are in flight towards `nxt`.  The last phase runs from registers after the
  // workgroup barrier, so it covers the first fragment reads of slab kt+1 and the first loads of kt+2.
  auto slab = [&](bool tail, unsigned char* cur, unsigned char* nxt, int kt, unsigned& pfslot) __attribute__((always_inline)) {
    const bool early = Tune::kPfWait || (KT && tail);
    if (early) prefetch(pfslot, kt);
    phase(tail, 0, 0, 0, 4, cur, 0, kof(kt + 1), nxt, LDA, LDB);
    phase(tail, 0, 1, 1, 12, cur, 1, kof(kt + 1), nxt, LDA + LDB, LDC);
    if (!early) prefetch(pfslot, kt);
    phase(tail, 1, 0, 0, 4, cur, 1, 0, nxt, 0, 0);
    // vmcnt(0), or 1: all but the prefetch; lgkmcnt(0): own loads have landed, own fragment reads are done
    if (PFD > 0 && !early) __builtin_amdgcn_s_waitcnt(0x0071); else __builtin_amdgcn_s_waitcnt(0x0070);
    __syncthreads();                        // ... and so have everybody else's: `nxt` is complete, `cur` is free
    phase(tail, 1, 1, 1, 12, nxt, 0, kof(kt + 2), cur, 0, LDA);
  };

  if (nk > 0) {
#pragma unroll
    for (int j = 0; j < 16; ++j) issue1(true, 0, stage0, j);
  }
  // (the accumulators are cleared while these are on their way: left to itself the compiler does it when they have landed, half a microsecond)
#pragma unroll
  for (int i = 0; i < MB; ++i)
#pragma unroll
    for (int j = 0; j < NB; ++j) asm volatile("" : "+a"(acc[i][j]));
  if (nk > 0) {
    __builtin_amdgcn_s_waitcnt(0x0F70);     // vmcnt(0)
    __syncthreads();
#pragma unroll
    for (int j = 0; j < LDA; ++j) issue1(true, kof(1), stage1, j);
    {
      const int slot = (fq ^ swz) << 4;
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        if constexpr (ATR) { read_a_tr(fa[0][i], stage0, i, 0, 0); read_a_tr(fa[0][i], stage0, i, 0, 1); }
        else fa[0][i] = *reinterpret_cast<const u32x4_t*>(stage0 + arow + i * 16 * kSlabBytes + slot);
      }
#pragma unroll
      for (int j = 0; j < NB / 2; ++j) {
        if constexpr (BTR) { read_b_tr(fb[0][j], stage0, j, 0, 0); read_b_tr(fb[0][j], stage0, j, 0, 1); }
        else fb[0][j] = *reinterpret_cast<const u32x4_t*>(stage0 + brow + j * 16 * kSlabBytes + slot);
      }
    }
    // nk is even but with KT (K is a multiple of 128).  Slabs that reach past the end of an operand are among the
    // last four (b_k_rows), or the last (KT), and loads run up to two slabs ahead: the last six slabs, or three.
    const bool has_tail = KT || (BTR && (k_first + nk) * BK > d.b_k_rows);
    constexpr int LAST = KT ? 3 : 6;
    const int plain = !has_tail ? nk : nk > LAST ? (nk - LAST) & ~1 : 0;
    int kt = 0;
    for (; kt < plain; kt += 2) {
      slab(false, stage0, stage1, kt, pf0);
      slab(false, stage1, stage0, kt + 1, pf1);
    }
    if constexpr (KT || BTR)
      for (; kt + 1 < nk; kt += 2) {
        slab(true, stage0, stage1, kt, pf0);
        slab(true, stage1, stage0, kt + 1, pf1);
      }
    if constexpr (KT)
      if (kt < nk) slab(true, stage0, stage1, kt, pf0);
  }
  __builtin_amdgcn_s_waitcnt(0x0070);       // trailing re-loads must land before the epilogue reuses LDS
  __syncthreads();
  mfma_drain();

  epi.template run<Layout16, MB, NB, BM, BN, WAVES_M, WAVES_N, true>(acc, c, stage0, d, pre);
  if (PFD > 0 && (pf_sink ^ pf0 ^ pf1) == 0x9E3779B9u && K < 0) epi.keep_alive();   // never true: keeps the prefetch loads
}

template <class Epi, class Tune, bool KT = false, bool FAR = false>
__global__ __launch_bounds__(256)
void gemm_nt_bf16_kernel(const bf16_t* __restrict__ A, const bf16_t* __restrict__ B, GemmDims d, Epi epi) {
  __shared__ __attribute__((aligned(1024))) unsigned char stage0[kHotStageBytes];
  __shared__ __attribute__((aligned(1024))) unsigned char stage1[kHotStageBytes];
  gemm_nt_bf16_tile<Epi, Tune, false, false, KT, FAR>(A, B, d, epi, blockIdx.x, stage0, stage1);
}

// Two independent contractions in one launch: workgroups [0, n1) work on the first, the rest on the
// second.  Used where one of them alone has too few tiles to fill the last round of the 256 CUs: the
// other's workgroups then fill the tail.  n1 = launch_tiles() of the first (a multiple of the XCD count).
// BTR1: the first contraction's B operand is given K-major; the second's A operand always is (see gemm_nt_bf16_tile).
// min_rows / max_rows: the launch is for chunks of more / of at most so many rows only (0: any); its twin does the others.
template <class Epi1, class Tune1, class Epi2, class Tune2, bool BTR1>
__global__ __launch_bounds__(256)
void gemm_nt_bf16_pair_kernel(const bf16_t* __restrict__ A1, const bf16_t* __restrict__ B1, GemmDims d1, Epi1 epi1, int n1,
                              const bf16_t* __restrict__ A2, const bf16_t* __restrict__ B2, GemmDims d2, Epi2 epi2, int min_rows, int max_rows) {
  if (min_rows | max_rows) {
    const int rows = d1.chunk ? d1.chunk[1] : *d1.n_real - d1.chunk_start;
    if ((min_rows && rows <= min_rows) || (max_rows && rows > max_rows)) return;
  }
  __shared__ __attribute__((aligned(1024))) unsigned char stage0[kHotStageBytes];
  __shared__ __attribute__((aligned(1024))) unsigned char stage1[kHotStageBytes];
  if ((int)blockIdx.x < n1)
    gemm_nt_bf16_tile<Epi1, Tune1, false, BTR1>(A1, B1, d1, epi1, blockIdx.x, stage0, stage1);
  else
    gemm_nt_bf16_tile<Epi2, Tune2, true>(A2, B2, d2, epi2, (int)blockIdx.x - n1, stage0, stage1);
}

}  // namespace rlk
