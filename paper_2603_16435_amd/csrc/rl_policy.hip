// rl_policy.hip - kernels of the O(T) stages and the C ABI of the library.
//
// Pipeline of rl_policy_loss_fwd_bwd (all on the caller's stream, no host sync):
//   prep      : row outputs cleared, group mean / std of the rewards -> A_i; per-sequence counts; scan and ordered
//               compaction of the rows that count (row_map, ids_c), chunk records
//   forward   : per chunk of compacted rows: logits tiles (MFMA) -> partial (max,sumexp) per
//               vocab tile + target logit -> combine -> lse_t, logp_t
//   loss      : one workgroup per sequence: length-normalised sums, loss_i, c_t; final reduce
//   backward  : masked rows of dX zeroed, W^T once (f32, and bf16 beyond 32768 rows); per chunk: X^T, recomputed logits, or those that the
//               forward of a batch of one chunk kept -> dS (input precision; f32 inputs also dS^T), dX = dS W (scattered to original rows; cut along K when its tiles are few),
//               dW (+)= dS^T X (bf16: dS read as a K-major operand, same launch as dX)
// The number of real rows is only known on the device, so grids are sized for the upper
// bound R and every kernel trims itself against the device-side count.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include <string.h>

#include <mutex>
#include <type_traits>
#include <utility>
#include <vector>

#include "../../include/rl_policy.h"
#include "../../include/rl_policy_diag.h"
#include "epilogues.h"
#include "logz_head.h"
#include "rvq_encode.h"
#include "rvq_few.h"
#include "gemm_nt.h"
#include "gemm_f32.h"
#include "grads_small.h"
#include "logits_few.h"

namespace rlk {

constexpr int kDefaultChunkRows = 32768;        // recompute mode: 128 x 14 dX tiles = 7 full rounds of 256 CUs on the 7B shape
constexpr int kDefaultChunkRowsStash = 40960;   // single-pass mode: the step time is flat (+-0.7 %) from 24576 to 65536 rows
constexpr int kBM = 256, kBN = 256;
// f32: tiles of 256 x 64 (four wavefronts of 128 x 32, two workgroups per CU; gemm_f32.h, operands that are not 16-byte aligned the general
// kernel), or 256 x 16 where the large ones would leave CUs without work.  MFMA-bound: 128-141 TFLOP/s, 102-109 in the general kernel, whose
// loads and addresses take a tenth of the issue slots.  Loss and gradients of 2175 tokens, H 768, V 50257, with dX cut along K and the logits
// recomputed: 5.25 ms, 6.2 in the general kernel; with its 256 x 256 tiles 17.9 (27 dX
// tiles of K = 50432: 12.5).  356 tokens, H 128, V 1024: 51 us (27 since small batches have a backward of their own, grads_small.h), 557 with 256 x 256 tiles (32-wide narrow ones took 7 % longer).
constexpr int kF32BN = 64, kF32SmallBN = 16, kF32Slots = 512;

// Batches of up to this many rows contract dX with W as it is stored (K-major operand of the hot kernel) instead of a transposed copy.
// The copy costs 2 x 2 V H bytes a call (7B head: 410 us); its contiguous slabs save up to 1 % of the two
// contractions.  747 tokens at the 7B head: 3274 us with the copy, 2860 without; 11.5 k tokens (16 k rows): 38.65 / 38.37 ms; 67 k tokens
// (131 k rows): 163.5 / 163.4; 36 k tokens at H 2048, V 32000 (65 k rows): 11.39 / 11.47.
constexpr int64_t kKMajorRows = 32768;

// Keeping the logits between forward and backward (recompute mode, batch of one chunk) turns the dS contraction into a pass over memory, for
// 4 bytes more per logit in the forward.  f32 always does (the logits wait in dS^T's place): 2175 tokens, H 768, V 50257 1323 -> 137 us, forward
// 1230 -> 1274.  bf16 in the default mode, with room of its own (4 bytes per row and vocabulary entry), if the workspace has it: batches of up to
// kKeepRows rows, padding included, since only the device knows the tokens.  At the 7B head that room is 10 GB, as much as the dS of the largest
// chunk, at V 32000 2 GB: the line is one of memory and drawn for large vocabularies.  Hidden sizes from kKeepH on: the general kernel, which keeps nothing
// in bf16, had the forward up to 448 when it was drawn; with its limit of 320 (small_k) keeping gains 2 to 9 % from 328 on too.  dS + forward in us, recomputed
// and kept: 11.5 k tokens at the 7B head 10019 + 9589, 1833 + 9904; 4741 tokens, H 1160, V 50257 663 + 609, 245 + 659; the whole call at H 456:
// 430 and 1350 tokens, V 50257 266 -> 238, 433 -> 402, 4600 tokens, V 152064 3509 -> 3249; H 512 258 -> 233, 438 -> 415, 3191 -> 3005.
constexpr int64_t kKeepRows = 16384;
constexpr int kKeepH = 456;
constexpr int64_t kFarBytes = (int64_t)1 << 32;      // hidden states that span this much are addressed per lane (FAR)

constexpr int kHotSlots = 256, kHotStep = 128;   // hot kernel: one workgroup per CU, a step of a K cut is two slabs
// Per-contraction tuning of the hot kernel, from sweeps on the 7B-shaped workload:
// tile-order band height (M-tiles per band), L2 prefetch distance in slabs (0 = off), where in a
// phase of 32 MFMAs the slab loads are issued (after MFMA kVmo, kVmo + kVmg, ...) and how many of a slab's 16 loads
// go into the phase after the barrier / the next phase (kLdA / kLdB; the rest into the phase after that).
// Measured on the 7B shape: dX, dW and the logits want the prefetch two slabs ahead, three is a little worse (dX without it: 4741 tokens, H 1160,
// V 50257 913 us instead of 848), dW is best with one M-tile per band (its A panel, the stored
// probabilities, then leaves memory once for all 14 N-tiles).
// dX, whose operands both stream from memory, waits 17 % of its loop time for its slab loads with the 6/5/5 placement and
// 5 % with 8/8/0 (all loads at least two phases before the barrier); at the power limit that is worth 0.8 % of dX+dW.
// The other two gain nothing from 8/8/0.
// dX and dW in very many rounds of the chip (step_prefetch): dX without prefetch, dW's waited for.  Otherwise the workgroups drift apart over
// the launch and fetch lines again that they would have found in L2: 38.5 k tokens at the 7B head fetch 233 GB instead of 174, which takes
// fewer cycles (95 M against 102 M) at a lower clock: at the power limit (1.60 GHz against 1.75) dX + dW take 62.4 ms instead of 59.9, and
// the 286 k tokens of 16 prompts 438 instead of 433 (on another box 459 and 439).
struct TuneLogits { static constexpr int kBand = 8, kPfd = 2, kVmg = 5, kVmo = 3, kLdA = 6, kLdB = 5; static constexpr bool kPfWait = false; };
struct TuneDX     { static constexpr int kBand = 8, kPfd = 2, kVmg = 4, kVmo = 1, kLdA = 8, kLdB = 8; static constexpr bool kPfWait = false; };
struct TuneDW     { static constexpr int kBand = 1, kPfd = 2, kVmg = 4, kVmo = 1, kLdA = 6, kLdB = 5; static constexpr bool kPfWait = false; };
struct TuneDXStep : TuneDX { static constexpr int kPfd = 0; };
struct TuneDWStep : TuneDW { static constexpr bool kPfWait = true; };

// dW tiles in a row (tn) and in all, of a chunk of at most M rows: more than 24 rounds, in rows that are not of whole blocks of four tiles (the
// lines of a panel are shared out among four), or longer than 20.  ms of dX + dW, prefetches not waited for / as above, 36, 38.5 and
// 40.5 k tokens:
//   V 152064, 128256 from 24 tiles on       10 tiles 39.2 42.2 44.9 / 39.8 42.5 44.6      11 45.2 48.7 50.9 / 44.8 47.5 50.2      12 47.0 50.5 54.0 / 48.2 50.1 53.9
//   13 54.1 57.2 60.3 / 51.6 55.5 57.8      14 55.8 60.3 63.4 / 55.9 58.6 61.7            15 62.7 65.9 70.7 / 60.9 63.4 68.6      16 62.1 66.9 69.2 / 63.5 68.4 70.6
//   18 73.7 78.0 82.6 / 71.9 75.7 79.9      20 78.5 84.6 89.3 / 80.0 84.9 92.2            24 83.9 88.8 93.0 / 82.1 86.3 90.4      28 98.4 107 112 / 98.1 103 109
//   14 tiles in 21, 14, 7 rounds (V 100000, 65536, 32000): 37.2 40.0 41.0 / 37.2 39.4 40.6, 24.0 26.6 27.7 / 24.5 26.3 27.5, 11.8 13.2 13.6 / 12.3 13.6 13.9
//   8 tiles in 18 rounds, 16 in 16 (V 152064, 65536): 31.1 32.9 34.1 / 31.3 33.3 34.8, 26.8 29.2 29.7 / 27.8 29.9 31.0
// A chunk with fewer tokens, which only the device knows, does not drift far enough: 14 tiles, 28 k, 33 k, 34 k tokens 41.3 50.6 53.9 / 42.2 51.7 52.8.  So
// such a launch goes out in both forms, and the one that the chunk is not for returns at once (20 us, of some 50 ms).
static bool step_prefetch(int M, int tn, int64_t tiles) { return M > kKMajorRows && tiles > 24 * kHotSlots && (tn % 4 || tn > 20); }
constexpr int kStepRows = 33280;

struct Ctrl {            // device control block at the head of the workspace
  int n_real;
  int too_long;          // single-pass backward: some sequence has more rows than the caller promised / a chunk holds
  int overflow;          // single-pass backward: rows whose stored probabilities left the range of the staging precision
  int done;              // sequences whose loss is formed: the last one finishes the call's loss
  int pad[12];
};

struct ChunkDesc {       // device record of one sequence-aligned chunk (single-pass backward)
  int row_start, rows;   // compacted rows [row_start, row_start + rows)
  int seq_begin, seq_end;// sequences [seq_begin, seq_end) lie wholly inside
};

// ------------------------------------------------------------------ optional launch timing
// When enabled (benchmarks only), each group of launches is bracketed by a pair of HIP events
// on the caller's stream; rl_profile_read() folds the elapsed times per class.
struct ProfRec { hipEvent_t a, b; int cls; };
struct Profiler {
  bool on = false;
  std::vector<ProfRec> recs;
  std::vector<std::pair<hipEvent_t, hipEvent_t>> pool;
};
static Profiler g_prof;

struct ProfScope {
  hipStream_t s; hipEvent_t a{}, b{}; int cls; bool live;
  ProfScope(int cls_, hipStream_t s_) : s(s_), cls(cls_), live(g_prof.on) {
    if (!live) return;
    if (!g_prof.pool.empty()) { a = g_prof.pool.back().first; b = g_prof.pool.back().second; g_prof.pool.pop_back(); }
    else { if (hipEventCreate(&a) != hipSuccess || hipEventCreate(&b) != hipSuccess) { live = false; return; } }
    (void)hipEventRecord(a, s);
  }
  ~ProfScope() {
    if (!live) return;
    (void)hipEventRecord(b, s);
    g_prof.recs.push_back({a, b, cls});
  }
};

// ------------------------------------------------------------------ small utilities
__device__ inline int wave_prefix_count(bool flag, int lane, int& total) {
  const unsigned long long b = __ballot(flag);
  total = __popcll(b);
  return __popcll(b & ((1ull << lane) - 1ull));
}

__device__ inline double block_sum(double v, double* sh) {   // blockDim.x multiple of 64, <= 1024
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double r = 0.0;
  const int nw = blockDim.x >> 6;
  for (int i = 0; i < nw; ++i) r += sh[i];                   // same order in every thread
  return r;
}

// ------------------------------------------------------------------ prep
// Everything the call needs cleared or worked out before the rows are looked at, in one launch (a call on a few hundred tokens is
// bound by its launches: nine fills, the advantages and the running maximum were 11 of 27).
//   workgroup 0:     inclusive running maximum of the sequence offsets, hi[i] = max(cu[0..i]) for i < B.  A sequence keeps its rows
//                    only if its first offset is not below any earlier offset: the kept row ranges are then pairwise disjoint
//                    whatever the offsets are, so no row can count twice and the compacted rows never exceed R.
//   the next adv.blocks:  group advantages
//   the rest:        row outputs to zero / -1
struct RowFill { int32_t* p[8]; int v[8]; };       // arrays of R words and the value of each (NULL: skipped)
struct AdvJob {
  int blocks; const float* rewards; const int32_t* group_idx; int P; float adv_eps; int ddof;
  float* adv; int32_t* group_count;
};
constexpr int kInitThreads = 256;

__device__ inline void fill_rows(const RowFill& f, int64_t R, int block, int blocks) {
  const int64_t step = (int64_t)blocks * kInitThreads;
  for (int64_t r = (int64_t)block * kInitThreads + threadIdx.x; r < R; r += step)
#pragma unroll
    for (int k = 0; k < 8; ++k) if (f.p[k]) f.p[k][r] = f.v[k];
}

// Wavefront per prompt p: mean and std of the rewards of its members, then A_i for each member (lane l takes sequences l, l + 64, ...; the
// sums are merged in a fixed tree).  Sequences that name no prompt get 0.  (A thread per prompt that walks all sequences: 128 sequences
// 42 us with the rest of the preparation, 1600 sequences 409.)
__device__ inline double wave_sum(double v) { for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o); return v; }
__device__ inline void advantages_of_prompt(int p, int B, const AdvJob& a, const int32_t* group_idx, const float* rewards) {
  const int lane = threadIdx.x & 63;
  int n = 0; double s = 0.0, q = 0.0;
  for (int i0 = 0; i0 < B; i0 += 64) {
    const int i = i0 + lane, g = i < B ? group_idx[i] : -1;
    const bool mine = i < B && g == p;
    n += __popcll(__ballot(mine));
    if (mine) s += (double)rewards[i];
    if (p == 0 && i < B && (g < 0 || g >= a.P)) a.adv[i] = 0.f;
  }
  const double mu = n ? wave_sum(s) / n : 0.0;
  for (int i = lane; i < B; i += 64)
    if (group_idx[i] == p) { const double d = (double)rewards[i] - mu; q += d * d; }
  q = wave_sum(q);
  const double inv = n - a.ddof > 0 ? 1.0 / (sqrt(q / (n - a.ddof)) + (double)a.adv_eps) : 0.0;
  for (int i = lane; i < B; i += 64)
    if (group_idx[i] == p) a.adv[i] = (float)(((double)rewards[i] - mu) * inv);
  if (lane == 0 && a.group_count) a.group_count[p] = n;
}

__global__ __launch_bounds__(kInitThreads) void prep_init_kernel(const int32_t* cu, int B, int64_t R, int32_t* hi, RowFill f, AdvJob adv, rl_stats* stats) {
  __shared__ int sh_i[kInitThreads / 64];
  const int t = threadIdx.x;
  if (blockIdx.x == 0) {
    if (stats && t < (int)(sizeof(rl_stats) / 4)) reinterpret_cast<int32_t*>(stats)[t] = 0;
    const int lane = t & 63, w = t >> 6;
    int carry = INT32_MIN;
    for (int base = 0; base < B; base += kInitThreads) {
      const int i = base + t;
      int x = i < B ? cu[i] : INT32_MIN;
      for (int o = 1; o < 64; o <<= 1) { const int y = __shfl_up(x, o); if (lane >= o) x = max(x, y); }
      if (lane == 63) sh_i[w] = x;
      __syncthreads();
      int all = carry;
      for (int k = 0; k < kInitThreads / 64; ++k) { if (k < w) x = max(x, sh_i[k]); all = max(all, sh_i[k]); }
      if (i < B) hi[i] = max(x, carry);
      carry = all;
      __syncthreads();
    }
  } else if ((int)blockIdx.x <= adv.blocks) {
    const int p = ((int)blockIdx.x - 1) * (kInitThreads / 64) + (t >> 6);
    if (p < adv.P) advantages_of_prompt(p, B, adv, adv.group_idx, adv.rewards);
  } else {
    fill_rows(f, R, blockIdx.x - 1 - adv.blocks, gridDim.x - 1 - adv.blocks);
  }
}
__global__ __launch_bounds__(kInitThreads) void row_fill_kernel(int64_t R, RowFill f) { fill_rows(f, R, blockIdx.x, gridDim.x); }

// One workgroup per sequence: validate its row range and group index, count rows that count.
__global__ void seq_count_kernel(const uint8_t* mask, const int32_t* ids, const int32_t* cu, const int32_t* cu_hi,
                                 const int32_t* group_idx, int64_t R, int V, int P,
                                 int32_t* seq_len, rl_stats* stats) {
  const int i = blockIdx.x;
  __shared__ int sh_cnt, sh_bad;
  if (threadIdx.x == 0) { sh_cnt = 0; sh_bad = 0; }
  __syncthreads();
  const int64_t a = cu[i], b = cu[i + 1];
  const bool seq_ok = (a >= 0 && a <= b && b <= R && a >= cu_hi[i]);
  const bool grp_ok = (group_idx == nullptr) || (group_idx[i] >= 0 && group_idx[i] < P);
  int cnt = 0, bad = 0;
  if (seq_ok && grp_ok) {
    for (int64_t r = a + threadIdx.x; r < b; r += blockDim.x) {
      if (mask[r]) {
        const int y = ids[r];
        if (y >= 0 && y < V) ++cnt; else ++bad;
      }
    }
  }
  for (int o = 32; o > 0; o >>= 1) { cnt += __shfl_down(cnt, o); bad += __shfl_down(bad, o); }
  if ((threadIdx.x & 63) == 0) { atomicAdd(&sh_cnt, cnt); atomicAdd(&sh_bad, bad); }
  __syncthreads();
  if (threadIdx.x == 0) {
    seq_len[i] = sh_cnt;
    if (stats) {
      if (sh_bad) atomicAdd(&stats->n_bad_token, sh_bad);
      if (!seq_ok) atomicAdd(&stats->n_bad_seq, 1);
      if (!grp_ok) atomicAdd(&stats->n_bad_group, 1);
    }
  }
}

// Exclusive scan of seq_len over sequences (single workgroup of 1024).  Up to kScanInline sequences every workgroup of the
// compaction adds up the lengths before its own instead, which saves a launch.
constexpr int kScanInline = 1024;
__global__ void seq_scan_kernel(const int32_t* seq_len, int B, int32_t* cstart) {
  __shared__ int wsum[16];
  __shared__ int carry;
  if (threadIdx.x == 0) carry = 0;
  __syncthreads();
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int base = 0; base < B; base += 1024) {
    const int i = base + threadIdx.x;
    const int v = i < B ? seq_len[i] : 0;
    int x = v;
    for (int o = 1; o < 64; o <<= 1) { const int y = __shfl_up(x, o); if (lane >= o) x += y; }
    if (lane == 63) wsum[w] = x;
    __syncthreads();
    int woff = 0;
    for (int k = 0; k < w; ++k) woff += wsum[k];
    if (i < B) cstart[i] = carry + woff + x - v;
    __syncthreads();
    if (threadIdx.x == 1023) carry += woff + x;
    __syncthreads();
  }
  if (threadIdx.x == 0) cstart[B] = carry;
}

// sum of seq_len[0 .. n) (n <= kScanInline = blockDim.x), the same in every thread
__device__ inline int block_count(const int32_t* seq_len, int n, int* wsum) {
  int x = (int)threadIdx.x < n ? seq_len[threadIdx.x] : 0;
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = x;
  __syncthreads();
  x = 0;
  for (int k = 0; k < (int)(blockDim.x >> 6); ++k) x += wsum[k];
  __syncthreads();
  return x;
}

// Single-pass backward: greedy packing of whole sequences into chunks of at most Tc compacted rows (one thread; the lengths pass
// through LDS).  Two consecutive chunks together hold more than Tc rows, so n_desc = 2 ceil(R / Tc) + 1 records
// always suffice; unused records are empty.  A sequence longer than max_len (<= Tc) raises the flag.
struct ChunkJob { ChunkDesc* desc; int n_desc, Tc, max_len; };
__device__ inline void build_chunks(const int32_t* seq_len, int B, const ChunkJob& c, Ctrl* ctrl, rl_stats* stats, int* sh) {
  ChunkDesc* desc = c.desc;
  int k = 0, start = 0, rows = 0, sb = 0, bad = 0;
  for (int base = 0; base < B; base += blockDim.x) {
    __syncthreads();
    if (base + (int)threadIdx.x < B) sh[threadIdx.x] = seq_len[base + threadIdx.x];
    __syncthreads();
    if (threadIdx.x != 0) continue;
    const int m = B - base < (int)blockDim.x ? B - base : (int)blockDim.x;
    for (int i = 0; i < m; ++i) {
      const int n = sh[i];
      if (n > c.max_len) ++bad;
      if (rows > 0 && rows + n > c.Tc && k < c.n_desc - 1) {
        desc[k].row_start = start; desc[k].rows = rows; desc[k].seq_begin = sb; desc[k].seq_end = base + i;
        ++k; start += rows; rows = 0; sb = base + i;
      }
      rows += n;
    }
  }
  if (threadIdx.x != 0) return;
  desc[k].row_start = start; desc[k].rows = rows; desc[k].seq_begin = sb; desc[k].seq_end = B;
  for (int j = k + 1; j < c.n_desc; ++j) { desc[j].row_start = start + rows; desc[j].rows = 0; desc[j].seq_begin = B; desc[j].seq_end = B; }
  ctrl->too_long = bad ? 1 : 0;
  if (bad && stats) stats->n_seq_too_long = bad;
}

// Ordered compaction, one workgroup per sequence: the k-th counting row of sequence i becomes
// compact row cstart[i]+k.  cpos[r] = compact position of original row r (left at -1 otherwise).  One workgroup more writes the
// control block (number of rows, flags) and the chunk records.
__global__ __launch_bounds__(1024) void compact_kernel(const uint8_t* mask, const int32_t* ids, const int32_t* cu, const int32_t* seq_len, int B,
                               int32_t* cstart, bool scanned, int V, int32_t* row_map, int32_t* ids_c, int32_t* cpos, int32_t* row_map_out,
                               Ctrl* ctrl, ChunkJob chunks, rl_stats* stats) {
  const int i = blockIdx.x;
  __shared__ int wsum[16];
  __shared__ int carry;
  __shared__ int sh_len[1024];
  const int first = scanned ? cstart[i] : block_count(seq_len, i, wsum);        // (cstart[B] = all rows)
  if (i == B) {
    if (threadIdx.x == 0) {
      cstart[B] = first;
      ctrl->n_real = first; ctrl->too_long = 0; ctrl->overflow = 0; ctrl->done = 0;
      if (stats) stats->n_tokens = first;
    }
    if (chunks.desc) build_chunks(seq_len, B, chunks, ctrl, stats, sh_len);
    return;
  }
  if (threadIdx.x == 0) { cstart[i] = first; carry = first; }
  if (seq_len[i] == 0) return;
  __syncthreads();
  const int64_t a = cu[i], b = cu[i + 1];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int64_t base = a; base < b; base += blockDim.x) {
    const int64_t r = base + threadIdx.x;
    int y = 0;
    bool f = false;
    if (r < b && mask[r]) { y = ids[r]; f = (y >= 0 && y < V); }
    int tot;
    const int pre = wave_prefix_count(f, lane, tot);
    if (lane == 0) wsum[w] = tot;
    __syncthreads();
    int woff = 0, all = 0;
    for (int k = 0; k < nw; ++k) { if (k < w) woff += wsum[k]; all += wsum[k]; }
    if (f) {
      const int c = carry + woff + pre;
      row_map[c] = (int)r; ids_c[c] = y; cpos[r] = c;
      if (row_map_out) row_map_out[c] = (int)r;
    }
    __syncthreads();
    if (threadIdx.x == 0) carry += all;
    __syncthreads();
  }
}

// All of the preparation in one launch of one workgroup, for small batches: three launches of mostly latency become one.  The rows are read
// once, all at a time, into bit masks in LDS (counting rows, rows dropped for their token id) with the ids beside them, and everything after
// that looks at those: the rows of a sequence are a difference of two ranks.  The whole call of a scoring or loss-only batch at H 64, V 300, three launches and
// one, us: scoring 128, 1024, 4096 rows of 8 sequences 22.2 22.5 23.1 / 18.0 18.6 21.0; 32 sequences 22.2 22.5 22.9 / 18.8 19.4 21.3; 64 sequences 22.3 22.6 22.9 /
// 20.2 20.8 22.1 (3072 rows 22.8 / 23.0); 128 sequences 22.3 22.6 22.9 / 23.3 23.8 25.3.  Loss of 1024 rows: 8 prompts 30.4 / 26.8, 32 prompts 31.6 / 30.1, 64 (four for a
// wavefront, one after the other) 32.5 / 35.1.
constexpr int kSmallRows = 4096, kSmallSeqs = 64, kSmallPrompts = 32;
struct SmallPrep {
  const uint8_t* mask; const int32_t *ids, *cu, *group_idx;
  int R, V, P, B;
  int32_t *seq_len, *cstart, *row_map, *ids_c, *cpos, *row_map_out;
  Ctrl* ctrl; ChunkJob chunks; rl_stats* stats;
};
// inclusive, over the first n lanes (fewer steps for few)
__device__ inline int wave_scan_max(int x, int n) { for (int o = 1; o < 64 && o < n; o <<= 1) { const int y = __shfl_up(x, o); if ((int)(threadIdx.x & 63) >= o) x = max(x, y); } return x; }
__device__ inline int wave_scan_sum(int x, int n) { for (int o = 1; o < 64 && o < n; o <<= 1) { const int y = __shfl_up(x, o); if ((int)(threadIdx.x & 63) >= o) x += y; } return x; }
template <int NT, int ROWS>       // threads of the workgroup, most rows
__device__ inline void prep_small(const SmallPrep& s, const RowFill& f, const AdvJob& adv) {
  constexpr int kWords = ROWS / 64, kPer = (ROWS + NT - 1) / NT, W = NT / 64;
  __shared__ unsigned long long good[kWords], bad[kWords];
  __shared__ int good_before[kWords + 1], bad_before[kWords + 1];        // rows in the words before a word
  __shared__ int sh_y[kPer * NT];
  __shared__ int sh_g[kSmallSeqs], sh_cu[kSmallSeqs + 1], sh_len[NT], sh_at[kSmallSeqs + 1];
  __shared__ float sh_r[kSmallSeqs];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  int y[kPer];
  bool on[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {                             // (all loads in flight together)
    const int r = k * NT + t;
    on[k] = false; y[k] = -1;
    if (r < s.R) { on[k] = s.mask[r]; y[k] = s.ids[r]; }
  }
  if (t <= s.B) sh_cu[t] = s.cu[t];
  if (t < s.B) {
    sh_g[t] = s.group_idx ? s.group_idx[t] : 0;
    if (adv.blocks) sh_r[t] = adv.rewards[t];
  }
  if (s.stats && t < (int)(sizeof(rl_stats) / 4)) reinterpret_cast<int32_t*>(s.stats)[t] = 0;
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int r = k * NT + t;
    if (r - lane >= s.R) continue;
    const bool ok = y[k] >= 0 && y[k] < s.V;
    const unsigned long long gm = __ballot(on[k] && ok), bm = __ballot(on[k] && !ok);
    if (lane == 0) { good[r >> 6] = gm; bad[r >> 6] = bm; }
    sh_y[r] = y[k];
    if (r < s.R)
#pragma unroll
      for (int q = 0; q < 8; ++q) if (f.p[q]) f.p[q][r] = f.v[q];
  }
  __syncthreads();
  if (w == W / 2 || w == W / 2 + 1) {
    static_assert(kWords <= 64, "a word per lane");
    const int words = (s.R + 63) / 64, n = wave_scan_sum(lane < words ? __popcll(w == W / 2 ? good[lane] : bad[lane]) : 0, words);
    int* before = w == W / 2 ? good_before : bad_before;
    if (lane < kWords) before[lane + 1] = n;
    if (lane == 0) before[0] = 0;
  }
  // sequences: a valid range at or behind every earlier offset (see prep_init_kernel), of a valid prompt
  static_assert(kSmallSeqs == 64, "a sequence per lane");
  const int hi = w == 0 ? wave_scan_max(t < s.B ? sh_cu[t] : INT32_MIN, s.B) : 0;
  __syncthreads();
  auto rank = [&](const unsigned long long* m, const int* before, int r) { return before[r >> 6] + (r & 63 ? __popcll(m[r >> 6] & ((1ull << (r & 63)) - 1ull)) : 0); };
  if (t < s.B) {
    const int a = sh_cu[t], b = sh_cu[t + 1];
    const bool seq_ok = a >= 0 && a <= b && b <= s.R && a >= hi;
    const bool grp_ok = !s.group_idx || (sh_g[t] >= 0 && sh_g[t] < s.P);
    int cnt = 0, nb = 0;
    if (seq_ok && grp_ok) {
      cnt = rank(good, good_before, b) - rank(good, good_before, a);
      nb = rank(bad, bad_before, b) - rank(bad, bad_before, a);
    }
    sh_len[t] = cnt; s.seq_len[t] = cnt;
    if (s.stats) {
      if (nb) atomicAdd(&s.stats->n_bad_token, nb);
      if (!seq_ok) atomicAdd(&s.stats->n_bad_seq, 1);
      if (!grp_ok) atomicAdd(&s.stats->n_bad_group, 1);
    }
  }
  if (w == 0) {
    const int at = wave_scan_sum(t < s.B ? sh_len[t] : 0, s.B);         // (its own)
    if (t < s.B) { sh_at[t + 1] = at; s.cstart[t + 1] = at; }
    if (t == 0) { sh_at[0] = 0; s.cstart[0] = 0; }
    if (t == s.B - 1) {
      s.ctrl->n_real = at; s.ctrl->too_long = 0; s.ctrl->overflow = 0; s.ctrl->done = 0;
      if (s.stats) s.stats->n_tokens = at;
    }
  }
  __syncthreads();
  const int sub = s.B < W ? W / s.B : 1;                     // wavefronts per sequence, 64 rows in turn
  for (int u = w; u < s.B * sub; u += W) {
    const int i = u / sub;
    if (sh_len[i] == 0) continue;
    const int a = sh_cu[i], b = sh_cu[i + 1], at = sh_at[i] - rank(good, good_before, a);
    for (int r0 = (a & ~63) + 64 * (u - i * sub); r0 < b; r0 += 64 * sub) {
      unsigned long long m = good[r0 >> 6];
      if (r0 + 64 > b) m &= ~0ull >> (64 - (b - r0));
      const int r = r0 + lane;
      if (r >= a && (m >> lane & 1)) {
        const int c = at + good_before[r0 >> 6] + __popcll(m & ((1ull << lane) - 1ull));
        s.row_map[c] = r; s.ids_c[c] = sh_y[r]; s.cpos[r] = c;
        if (s.row_map_out) s.row_map_out[c] = r;
      }
    }
  }
  if (adv.blocks)
    for (int p = w; p < adv.P; p += W) advantages_of_prompt(p, s.B, adv, sh_g, sh_r);
  if constexpr (ROWS == kSmallRows)
    if (s.chunks.desc) build_chunks(s.seq_len, s.B, s.chunks, s.ctrl, s.stats, sh_len);
}

__global__ __launch_bounds__(1024) void prep_small_kernel(SmallPrep s, RowFill f, AdvJob adv) { prep_small<1024, kSmallRows>(s, f, adv); }

// The preparation inside the launch of the logits (logits_small_kernel, logits_few_kernel), for batches of so few rows that every workgroup can work out for itself
// which ones count: workgroup 0 does the above, for the launches that follow, the others go by their own list in LDS (2 us, about what the two
// dependent loads of the row map took).  A launch is saved: scoring of 99 tokens, H 2048, V 32000 46.7 -> 42.4 us; f32 loss of 356 tokens, H 128, V 1024 35.1 -> 30.3.
template <int ROWS> struct LocalRows { int n, rows[ROWS], ids[ROWS], count[ROWS / 64]; };
template <int NT, int ROWS>
__device__ inline void local_rows(const SmallPrep& s, LocalRows<ROWS>& l) {
  constexpr int kPer = (ROWS + NT - 1) / NT;
  const int t = threadIdx.x, lane = t & 63;
  int y[kPer];
  bool on[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int r = k * NT + t;
    on[k] = false; y[k] = -1;
    if (r < s.R) { on[k] = s.mask[r]; y[k] = s.ids[r]; }
  }
  // A lane of every wavefront has a sequence (as there: a valid range at or behind every earlier offset, of a valid prompt), and the lanes put together which of
  // the wavefront's 64 rows are in one: no barrier, and no walk over the sequences (60 of them, 947 rows, V 114 in f32 25.6 us that way).
  int a = INT32_MIN, b = 0, g = 0;
  if (lane < s.B) { a = s.cu[lane]; b = s.cu[lane + 1]; if (s.group_idx) g = s.group_idx[lane]; }
  const int hi = wave_scan_max(a, s.B);
  if (!(lane < s.B && a >= 0 && a <= b && b <= s.R && a >= hi && (!s.group_idx || (g >= 0 && g < s.P)))) a = b = 0;
  unsigned long long m[kPer];
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int r = k * NT + t, r0 = r - lane, lo = min(max(a - r0, 0), 64), up = min(max(b - r0, 0), 64);
    unsigned long long in = up > lo ? ~0ull >> (64 - (up - lo)) << lo : 0ull;
    for (int o = 1; o < 64 && o < s.B; o <<= 1) in |= __shfl_xor(in, o);
    in = __shfl(in, 0);
    m[k] = __ballot((in >> lane & 1) && on[k] && y[k] >= 0 && y[k] < s.V);
    if (lane == 0 && r < ROWS) l.count[r >> 6] = __popcll(m[k]);
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < kPer; ++k) {
    const int r = k * NT + t;
    int at = 0;
    for (int q = 0; q < (r >> 6) && q < ROWS / 64; ++q) at += l.count[q];       // (the kept sequences are in the order of their rows)
    if (m[k] >> lane & 1) {
      const int c = at + __popcll(m[k] & ((1ull << lane) - 1ull));
      l.rows[c] = r; l.ids[c] = y[k];
    }
  }
  if (t == 0) { int n = 0; for (int q = 0; q < ROWS / 64; ++q) n += l.count[q]; l.n = n; }
  __syncthreads();
}

// Logits of a few tokens (bf16), see logits_few.h.  PREP: with the preparation.
template <int BN, bool PREP, bool NT>
__global__ __launch_bounds__(256, 1)
void logits_few_kernel(const bf16_t* __restrict__ W, const bf16_t* __restrict__ X, GemmDims d, EpiFwd<bf16_t> epi, SmallPrep s, RowFill f, AdvJob adv) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[few_lds_bytes<BN>()];
  if constexpr (PREP) {
    if (blockIdx.x == 0) { prep_small<256, kFewTokens>(s, f, adv); return; }
    __shared__ LocalRows<kFewTokens> l;
    local_rows<256>(s, l);
    logits_few_tile<BN, NT>(W, X, d, epi, (int)blockIdx.x - 1, l.n, l.rows, l.ids, smem);
  } else {
    const int left = *d.n_real;
    logits_few_tile<BN, NT>(W, X, d, epi, blockIdx.x, left < d.N ? left : d.N, d.b_rows, epi.ids_c, smem);
  }
}

// Logits of a small f32 batch with the preparation: the general kernel's narrow tiles by sixteen wavefronts.  (A's loads ahead of local_rows
// as well: 29.0 us of that call instead of 27.9.)
constexpr int kLocalRows = 1024;
template <class Epi>
__global__ __launch_bounds__(1024)
void logits_small_kernel(const float* __restrict__ W, const float* __restrict__ X, GemmDims d, Epi epi, SmallPrep s, RowFill f, AdvJob adv) {
  __shared__ __attribute__((aligned(1024))) unsigned char smem[general_lds_bytes<float, kBM, kF32SmallBN, 1>()];
  if (blockIdx.x == 0) { prep_small<1024, kLocalRows>(s, f, adv); return; }
  __shared__ LocalRows<kLocalRows> l;
  local_rows<1024>(s, l);
  d.n_real = &l.n; d.b_rows = l.rows; epi.ids_c = l.ids;
  const GeneralTile t = general_tile<kBM, kF32SmallBN, Elem<float>::kBK>(d, (int)blockIdx.x - 1);
  if (t.any) gemm_nt_general_tile<float, Epi, kBM, kF32SmallBN, 16, 1, 1, true>(W, X, d, t, epi, smem);
}

// one wavefront per row; rows that count are left alone (the dX epilogue writes them)
template <class T>
__device__ inline void zero_masked_row(int64_t r, const int32_t* cpos, T* dX, int64_t R, int H) {
  if (r >= R || cpos[r] >= 0) return;
  const int lane = threadIdx.x & 63;
  typename Piece16<T>::type* p = reinterpret_cast<typename Piece16<T>::type*>(dX + r * H);
  const int n16 = H * (int)sizeof(T) / 16;
  for (int k = lane; k < n16; k += 64) p[k] = 0u;
}
template <class T>
__global__ void zero_masked_rows_kernel(const int32_t* cpos, T* dX, int64_t R, int H) {
  zero_masked_row((int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6), cpos, dX, R, H);
}

// ------------------------------------------------------------------ single-pass backward: references
// Single-pass backward, one wavefront per original row: a row that does not count has its dX row zeroed; for one that does, at
// compact position t, the target logit zy_t = x_t . W[y_t] (f32 accumulation of bf16 products)
// (times the inverse temperature) and the reference of the stored probabilities, ref_t = zy_t - old_t, which is
// the logsumexp of the row up to the (small) drift between the old and the current policy (NaN-free for any finite old_t).
__global__ void target_logit_kernel(const bf16_t* X, const bf16_t* W, int64_t R, int H, const int32_t* cpos, const int32_t* ids_c,
                                    const float* old_lp, float inv_tau, bf16_t* dX, float* zy, float* ref_l2e, int32_t* ycol) {
  const int64_t r = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6);
  if (r >= R) return;
  const int lane = threadIdx.x & 63;
  const int t = cpos[r];
  if (t < 0) {
    Piece16<bf16_t>::type* p = reinterpret_cast<Piece16<bf16_t>::type*>(dX + r * H);
    for (int k = lane; k < H / 8; k += 64) p[k] = 0u;
    return;
  }
  const uint4* x = reinterpret_cast<const uint4*>(X + r * H);
  const int y = ids_c[t];
  const uint4* w = reinterpret_cast<const uint4*>(W + (int64_t)y * H);
  float acc = 0.f;
  for (int k = lane; k < H / 8; k += 64) {
    const uint4 a = x[k], b = w[k];
    const unsigned av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      acc = fmaf(__uint_as_float(av[j] << 16), __uint_as_float(bv[j] << 16), acc);
      acc = fmaf(__uint_as_float(av[j] & 0xffff0000u), __uint_as_float(bv[j] & 0xffff0000u), acc);
    }
  }
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o);
  if (lane == 0) {
    // the old log-prob only steers the reference; clamped to [-40, 0] a wild value costs range, not correctness:
    // exp(z - ref) stays representable for current log-probs between about -120 and 0
    const float o = fminf(fmaxf(old_lp[r], -40.f), 0.f);
    acc *= inv_tau;
    zy[t] = acc; ref_l2e[t] = (acc - o) * 1.4426950408889634f;
    ycol[t] = y;                                   // the row of W the target logit was read from
  }
}

// Per-tile-row partial sums (s, u) of a chunk -> lse, logp, entropy and Z_t = sum_v exp(z - ref_t).
// A workgroup handles 16 rows (a line of 128 bytes) x 64 slices of the tile range (1024 threads: the sums are chains of dependent f64 adds,
// so it takes many short chains to keep the memory system busy), merged through LDS in a fixed order.  (64 rows x 16 slices: few workgroups, which a CU's 28 bytes a ns held up, 747
// tokens, 594 tiles 22 us instead of 10, 67 k 101 instead of 83.)
constexpr int kSumRows = 16, kSumSlices = 64;
__global__ __launch_bounds__(kSumRows * kSumSlices) void lse_sum_kernel(const float2* part, int ldp, int tiles_v, const float* zy_c, const float* ref_l2e,
                               const int32_t* row_map, const ChunkDesc* desc, const int32_t* ycol_c, Ctrl* ctrl, rl_stats* stats,
                               float* lse_c, float* logp_c, float* zsum_c, float* lse_out, float* logp_out, float* ent_out,
                               float* zy_out, int32_t* ycol_out) {
  __shared__ double ss[kSumSlices][kSumRows], su[kSumSlices][kSumRows];
  const int left = desc->rows, chunk_start = desc->row_start;
  if ((int)blockIdx.x * kSumRows >= left) return;
  const int col = threadIdx.x % kSumRows, slice = threadIdx.x / kSumRows;
  const int n = blockIdx.x * kSumRows + col;
  double s = 0.0, u = 0.0;
  if (n < left)
    for (int t0 = slice; t0 < tiles_v; t0 += 8 * kSumSlices) {       // eight loads in flight, added in order
      float2 v[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) { const int t = t0 + k * kSumSlices; v[k] = t < tiles_v ? part[(int64_t)t * ldp + n] : make_float2(0.f, 0.f); }
#pragma unroll
      for (int k = 0; k < 8; ++k) { s += (double)v[k].x; u += (double)v[k].y; }
    }
  ss[slice][col] = s; su[slice][col] = u;
  __syncthreads();
  if (threadIdx.x >= 64) return;
  double S = 0.0, U = 0.0;                                           // four lanes per row, sixteen slices each
#pragma unroll
  for (int k = 0; k < kSumSlices / 4; ++k) { S += ss[slice * (kSumSlices / 4) + k][col]; U += su[slice * (kSumSlices / 4) + k][col]; }
#pragma unroll
  for (int o = kSumRows; o < 64; o <<= 1) { S += __shfl_xor(S, o); U += __shfl_xor(U, o); }
  if (slice == 0 && n < left) {
    const int g = chunk_start + n;
    const double lse_d = (double)ref_l2e[g] * 0.6931471805599453 + log(S);
    const float lse = (float)lse_d;
    const float lp = zy_c[g] - lse;
    lse_c[g] = lse; logp_c[g] = lp; zsum_c[g] = (float)S;
    // Z_t = exp(lse_t - ref_t) is of order one when the old log-prob is anywhere near the current one.  A row whose
    // sum left [1e-30, 1e30] (or is not a number) had stored probabilities outside the staging precision's range:
    // counted, and the loss of the call comes back NaN.
    if (!(S >= 1e-30 && S <= 1e30)) { atomicAdd(&ctrl->overflow, 1); if (stats) atomicAdd(&stats->n_overflow_rows, 1); }
    const int r = row_map[g];
    if (lse_out) lse_out[r] = lse;
    if (logp_out) logp_out[r] = lp;
    if (ent_out) ent_out[r] = (float)fmax(lse_d - U / S, 0.0);
    if (zy_out) zy_out[r] = zy_c[g];
    if (ycol_out) ycol_out[r] = ycol_c[g];
  }
}

// After the loss: per row of the chunk the factor -c_t / (tau Z_t) of the backward contractions (1 / tau: from the
// tempered logit back to W x_t), and the target entry of the stored probabilities replaced by e_y - Z_t (so that
// the factor times the stored row is dS).
template <class T>
__global__ void stash_patch_kernel(const ChunkDesc* desc, const int32_t* ids_c, const float* zy_c, const float* ref_l2e,
                                   const float* zsum_c, const float* c_c, float inv_tau, float* row_scale,
                                   T* E, int64_t ld_e) {
  const int n = blockIdx.x * blockDim.x + threadIdx.x;
  if (n >= desc->rows) return;
  const int g = desc->row_start + n;
  const float Z = zsum_c[g];
  row_scale[n] = -c_c[g] * inv_tau / Z;
  const float ey = exp2f(fmaf(zy_c[g], 1.4426950408889634f, -ref_l2e[g]));
  const T v = (T)(ey - Z);
  const int y = ids_c[g];
  E[tiled_index(n, y, ld_e)] = v;
}

// ------------------------------------------------------------------ forward combine
// Fold the per-vocab-tile partials (max, sumexp) of a chunk into lse, logp.  A workgroup handles 16 or 64
// compact rows x SLICES slices of the tile range: one online (rescaling) pass per thread, coalesced
// along the rows, sums in f64, then the slices are scaled to the row's maximum, one exponential per thread, and added through LDS in order.
// Few rows are all latency and want many slices, many rows of few tiles pay for the exponential of every slice.  32768 rows, 4, 8, 16 slices, us: 4 tiles
// 4.3 - 4.6, 16 tiles 4.8 4.7 5.9, 63 tiles 9.0 8.3 11.3; 96 rows: 4 tiles 3.0 - 3.6, 16 tiles 3.8 3.5 4.2, 63 tiles 8.4 5.6 5.2, 125 tiles 8.8 - 6.7.  (By the
// vocabulary alone: a token's bits must not depend on the batch.)
constexpr int combine_slices(int tiles_v) { return tiles_v <= 8 ? 4 : tiles_v <= 64 ? 8 : 16; }
// Rows of a workgroup: 64 (above), 16 where the partials of a row are many and few workgroups would wait for what a CU takes in (28 bytes a ns): scoring of 99 tokens, V 32000
// 36.6 -> 35.7 us, of 25 30.6 -> 29.4; with four slices and many rows 64 are the better ones (48 k rows, V 1000 79.0 against 80.7).  Same bits.
constexpr int combine_rows(int slices) { return slices == 16 ? 16 : 64; }
// HALVES: the partials are those of half tiles (logits_few_kernel), two of which make one.
template <bool HALVES, int SLICES>
__global__ __launch_bounds__(combine_rows(SLICES) * SLICES) void lse_combine_kernel(const float4* part, int ldp, int tiles_v, const float* zy_c,
                                   const int32_t* row_map, const Ctrl* ctrl, int chunk_start, int chunk_rows, const int32_t* ycol_c,
                                   float* lse_c, float* logp_c, float* lse_out, float* logp_out, float* ent_out,
                                   float* zy_out, int32_t* ycol_out) {
  constexpr int ROWS = combine_rows(SLICES);
  __shared__ float sm[SLICES][ROWS];
  __shared__ double ss[SLICES][ROWS], su[SLICES][ROWS];
  int left = ctrl->n_real - chunk_start;
  if (left > chunk_rows) left = chunk_rows;
  if ((int)blockIdx.x * ROWS >= left) return;
  const int col = threadIdx.x % ROWS, slice = threadIdx.x / ROWS;
  const int n = blockIdx.x * ROWS + col;
  const float NEG = -__builtin_inff();
  float m = NEG;
  double s = 0.0, u = 0.0;
  if (n < left) {
    for (int t0 = slice; t0 < tiles_v; t0 += 8 * SLICES) {             // eight loads in flight, folded in order
      float4 q[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int t = t0 + SLICES * k;
        q[k] = make_float4(NEG, 0.f, 0.f, 0.f);
        if (t < tiles_v) {
          if constexpr (HALVES) q[k] = EpiFwd<bf16_t>::merge_halves(part[(int64_t)(2 * t) * ldp + n], part[(int64_t)(2 * t + 1) * ldp + n]);
          else q[k] = part[(int64_t)t * ldp + n];
        }
      }
      float mm = m;
#pragma unroll
      for (int k = 0; k < 8; ++k) mm = fmaxf(mm, q[k].x);
      if (mm == NEG) continue;
      const double f0 = (double)expf(m - mm);
      s *= f0; u *= f0;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        if (t0 + SLICES * k >= tiles_v) break;
        const double f = (double)expf(q[k].x - mm);
        s += (double)q[k].y * f; u += (double)q[k].z * f;
      }
      m = mm;
    }
  }
  sm[slice][col] = m;
  __syncthreads();
  float M = sm[0][col];
#pragma unroll
  for (int k = 1; k < SLICES; ++k) M = fmaxf(M, sm[k][col]);
  {
    const double f = m != NEG ? exp((double)(m - M)) : 0.0;
    ss[slice][col] = s * f; su[slice][col] = u * f;
  }
  __syncthreads();
  if (slice == 0 && n < left) {
    double S = 0.0, U = 0.0;
#pragma unroll
    for (int k = 0; k < SLICES; ++k) { S += ss[k][col]; U += su[k][col]; }
    const double lse_d = (double)M + log(S);
    const float lse = (float)lse_d;
    const int g = chunk_start + n;
    const float lp = zy_c[g] - lse;
    lse_c[g] = lse; logp_c[g] = lp;
    const int r = row_map[g];
    if (lse_out) lse_out[r] = lse;
    if (logp_out) logp_out[r] = lp;
    if (ent_out) ent_out[r] = (float)fmax(lse_d - U / S, 0.0);     // H = lse - sum_v p_v z_v
    if (zy_out) zy_out[r] = zy_c[g];
    if (ycol_out) ycol_out[r] = ycol_c[g];
  }
}

// ------------------------------------------------------------------ loss
struct LossOpts {
  float clip_lo, clip_hi;   // ratio / weight kept inside [1 - clip_lo, 1 + clip_hi]
  float kl_coef, beta;
  int token_agg;            // GRPO: loss = (1/T) sum of all token terms instead of the mean of per-sequence means
  int seq_ratio;            // GRPO: one ratio per sequence, exp(mean_t (logp - old))
  int w_mean;               // FLOW: weight from the mean instead of the sum of the token log-ratios
};

// The combine of a batch of few rows and tiles inside its loss launch (fold_combine): a thread takes a token.
struct CombineJob {
  const float4* part; int ldp, tiles_v; const float* zy_c; const int32_t *row_map, *ycol_c;
  float *lse_c, *logp_c, *lse_out, *logp_out, *ent_out, *zy_out; int32_t* ycol_out;
};

struct LossJob {
  int objective; const float *logp_c, *old_lp, *ref_lp; const int32_t *row_map, *cstart; const float* adv;
  const int32_t* group_idx; const float* log_z; int B, P; LossOpts o; Ctrl* ctrl;
  float *seq_loss, *gterm, *c_c, *coeff_out; rl_stats* stats;
  const ChunkDesc* desc;                // only the sequences of this chunk
  float* adv_out; int32_t* seq_len_out;
  float *loss, *d_log_z, *seq_loss_out;
  CombineJob comb;                      // loss_fold_kernel
  int finish_later;                     // a workgroup of the next launch adds the sequences up (small_grads_kernel)
};
// Up to kFinishSeqs sequences, the workgroup that forms the last one's loss adds them up as well; with more, the release that every workgroup
// then owes the others costs as much as a launch or more (256 sequences 16 us against 15, 20000 469 against 46).
constexpr int kLossThreads = 256, kFinishSeqs = 64;

// loss = (1/B) sum_i seq_loss_i
__device__ inline void add_up_loss(const LossJob& j) {
  __shared__ double sh[16];
  double acc = 0.0;
#pragma unroll 8
  for (int i = threadIdx.x; i < j.B; i += blockDim.x) {
    const float v = j.seq_loss[i];
    acc += (double)v;
    if (j.seq_loss_out) j.seq_loss_out[i] = v;
  }
  const double tot = block_sum(acc, sh);
  // a sequence longer than the caller promised: the single-pass backward dropped rows, say so loudly
  // ... or stored probabilities that left the representable range: the gradients of those rows are not numbers
  if (threadIdx.x == 0) *j.loss = (j.ctrl->too_long || j.ctrl->overflow) ? __builtin_nanf("") : (float)(tot / j.B);
}
// ... and d_logZ_p = sum over members of gterm (0 for an empty sequence), in order
__device__ inline void finish_loss(const LossJob& j) {
  __shared__ int sh_g[kFinishSeqs];
  __shared__ float sh_t[kFinishSeqs];
  add_up_loss(j);
  if (!j.d_log_z) return;
  for (int i = threadIdx.x; i < j.B; i += blockDim.x) { sh_g[i] = j.group_idx[i]; sh_t[i] = j.gterm[i]; }
  __syncthreads();
  for (int p = threadIdx.x; p < j.P; p += blockDim.x) {
    double s = 0.0;
    if (j.objective == RL_OBJ_FLOW)
#pragma unroll 8
      for (int k = 0; k < j.B; ++k) s += sh_g[k] == p ? (double)sh_t[k] : 0.0;
    j.d_log_z[p] = (float)s;
  }
}
// The same for more sequences, in a launch of its own: workgroup 0 the loss, a wavefront per prompt d_log_z.
__global__ __launch_bounds__(1024) void finalize_kernel(LossJob j) {
  if (blockIdx.x == 0) { add_up_loss(j); return; }
  const int p = ((int)blockIdx.x - 1) * 16 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (p >= j.P) return;
  double s = 0.0;
  if (j.objective == RL_OBJ_FLOW) {
#pragma unroll 8
    for (int i = lane; i < j.B; i += 64) s += j.group_idx[i] == p ? (double)j.gterm[i] : 0.0;
    s = wave_sum(s);
  }
  if (lane == 0) j.d_log_z[p] = (float)s;
}

// What lse_combine_kernel<false, 4> does for token g, to the bit: its four slices one after the other (at most two tiles each), then their sum.
constexpr int kFoldTiles = 8, kFoldRows = 1024;
__device__ inline void combine_token(const CombineJob& c, int g) {
  const float NEG = -__builtin_inff();
  float4 q[kFoldTiles];
#pragma unroll
  for (int t = 0; t < kFoldTiles; ++t) q[t] = t < c.tiles_v ? c.part[(int64_t)t * c.ldp + g] : make_float4(NEG, 0.f, 0.f, 0.f);
  const float zy = c.zy_c[g];
  const int r = c.row_map[g], ycol = c.ycol_c[g];
  float m[4];
  double s[4], u[4];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    m[k] = fmaxf(q[k].x, q[k + 4].x); s[k] = 0.0; u[k] = 0.0;
    if (m[k] == NEG) continue;
    const double f0 = (double)expf(q[k].x - m[k]);
    s[k] += (double)q[k].y * f0; u[k] += (double)q[k].z * f0;
    if (k + 4 < c.tiles_v) {
      const double f1 = (double)expf(q[k + 4].x - m[k]);
      s[k] += (double)q[k + 4].y * f1; u[k] += (double)q[k + 4].z * f1;
    }
  }
  const float M = fmaxf(fmaxf(m[0], m[1]), fmaxf(m[2], m[3]));
  double S = 0.0, U = 0.0;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const double f = m[k] != NEG ? exp((double)(m[k] - M)) : 0.0;
    double sf = s[k] * f, uf = u[k] * f;
    asm volatile("" : "+v"(sf), "+v"(uf));                  // rounded, as on their way through LDS: no fused multiply-add
    S += sf; U += uf;
  }
  const double lse_d = (double)M + log(S);
  const float lse = (float)lse_d, lp = zy - lse;
  c.lse_c[g] = lse; c.logp_c[g] = lp;
  if (c.lse_out) c.lse_out[r] = lse;
  if (c.logp_out) c.logp_out[r] = lp;
  if (c.ent_out) c.ent_out[r] = (float)fmax(lse_d - U / S, 0.0);
  if (c.zy_out) c.zy_out[r] = zy;
  if (c.ycol_out) c.ycol_out[r] = ycol;
}

// One workgroup per sequence over its compact rows [cstart[i], cstart[i+1]).  The caller's advantages and lengths leave here, when the
// rewards and the offsets have been read everywhere: an output may take the place of an input.
template <bool FOLD>
__device__ inline void sequence_loss(const LossJob& j, int i) {
  const float *logp_c = j.logp_c, *old_lp = j.old_lp, *ref_lp = j.ref_lp, *log_z = j.log_z;
  const int32_t *row_map = j.row_map, *group_idx = j.group_idx;
  const int objective = j.objective, B = j.B;
  const LossOpts& o = j.o;
  float *seq_loss = j.seq_loss, *gterm = j.gterm, *c_c = j.c_c, *coeff_out = j.coeff_out;
  rl_stats* stats = j.stats;
  __shared__ double sh[16];
  __shared__ int sh_hi, sh_lo;
  const int a = j.cstart[i], b = j.cstart[i + 1], n = b - a;
  const float A = j.adv[i];
  if (threadIdx.x == 0) {
    sh_hi = 0; sh_lo = 0;
    if (j.adv_out) j.adv_out[i] = A;
    if (j.seq_len_out) j.seq_len_out[i] = n;
  }
  if (n <= 0) {
    if (threadIdx.x == 0) { seq_loss[i] = 0.f; gterm[i] = 0.f; }
    return;
  }
  if constexpr (FOLD)
    for (int k = a + threadIdx.x; k < b; k += blockDim.x) combine_token(j.comb, k);        // (read back below by the thread that wrote them)
  const double Ad = (double)A;
  const double inv_bn = 1.0 / ((double)B * (double)n);
  const double lo_c = 1.0 - (double)o.clip_lo, hi_c = 1.0 + (double)o.clip_hi;
  if (objective == RL_OBJ_GRPO && !o.seq_ratio) {
    // weight of a token term in the loss: 1/(B n_i) (mean of per-sequence means) or 1/T (mean over all tokens)
    const double wt = o.token_agg ? 1.0 / (double)j.ctrl->n_real : inv_bn;
    double acc = 0.0; int hi = 0, lo = 0;
    for (int k = a + threadIdx.x; k < b; k += blockDim.x) {
      const int r = row_map[k];
      // per-token terms in f64: e^d - d - 1 cancels to ~d^2/2 and would lose digits in f32
      const double lp = (double)logp_c[k];
      const double rho = exp(lp - (double)old_lp[r]);
      const double dd = (double)ref_lp[r] - lp;
      const double ed = exp(dd);
      const double rc = fmin(fmax(rho, lo_c), hi_c);
      const double l = -fmin(rho * Ad, rc * Ad) + (double)o.kl_coef * (ed - dd - 1.0);
      const bool chi = (A > 0.f) && (rho > hi_c);
      const bool clo = (A < 0.f) && (rho < lo_c);
      hi += chi; lo += clo;
      const double g = ((chi || clo) ? 0.0 : -Ad * rho) + (double)o.kl_coef * (1.0 - ed);
      const float ct = (float)(g * wt);
      c_c[k] = ct;
      if (coeff_out) coeff_out[r] = ct;
      acc += l;
    }
    const double tot = block_sum(acc, sh);
    for (int q = 32; q > 0; q >>= 1) { hi += __shfl_down(hi, q); lo += __shfl_down(lo, q); }
    if ((threadIdx.x & 63) == 0) { if (hi) atomicAdd(&sh_hi, hi); if (lo) atomicAdd(&sh_lo, lo); }
    __syncthreads();
    if (threadIdx.x == 0) {
      // token aggregation reports (B/T) sum_t l_t, so that loss = mean_i seq_loss_i in both aggregations
      seq_loss[i] = (float)(o.token_agg ? tot * wt * (double)B : tot / n); gterm[i] = 0.f;
      if (stats) { if (sh_hi) atomicAdd(&stats->n_clip_hi, sh_hi); if (sh_lo) atomicAdd(&stats->n_clip_lo, sh_lo); }
    }
  } else if (objective == RL_OBJ_GRPO) {
    // sequence-level ratio s = exp(mean_t (logp - old)): first the mean and the KL sum, then the coefficients
    double s_old = 0.0, s_kl = 0.0;
    for (int k = a + threadIdx.x; k < b; k += blockDim.x) {
      const int r = row_map[k];
      const double lp = (double)logp_c[k];
      const double dd = (double)ref_lp[r] - lp;
      s_old += lp - (double)old_lp[r];
      s_kl += exp(dd) - dd - 1.0;
    }
    const double t_old = block_sum(s_old, sh);
    const double t_kl = block_sum(s_kl, sh);
    const double sr = exp(t_old / n);
    const double rc = fmin(fmax(sr, lo_c), hi_c);
    const bool chi = (A > 0.f) && (sr > hi_c);
    const bool clo = (A < 0.f) && (sr < lo_c);
    const double ds = (chi || clo) ? 0.0 : -Ad * sr;               // d(-surrogate)/d(mean log-ratio)
    for (int k = a + threadIdx.x; k < b; k += blockDim.x) {
      const int r = row_map[k];
      const double dd = (double)ref_lp[r] - (double)logp_c[k];
      const float ct = (float)((ds + (double)o.kl_coef * (1.0 - exp(dd))) * inv_bn);
      c_c[k] = ct;
      if (coeff_out) coeff_out[r] = ct;
    }
    if (threadIdx.x == 0) {
      seq_loss[i] = (float)(-fmin(sr * Ad, rc * Ad) + (double)o.kl_coef * t_kl / n); gterm[i] = 0.f;
      if (stats) { if (chi) atomicAdd(&stats->n_clip_hi, 1); if (clo) atomicAdd(&stats->n_clip_lo, 1); }
    }
  } else {
    double s_ref = 0.0, s_old = 0.0;
    for (int k = a + threadIdx.x; k < b; k += blockDim.x) {
      const int r = row_map[k];
      const float lp = logp_c[k];
      s_ref += (double)(lp - ref_lp[r]);
      s_old += (double)(lp - old_lp[r]);
    }
    const double t_ref = block_sum(s_ref, sh);
    double t_old = block_sum(s_old, sh);
    if (o.w_mean) t_old /= n;
    const double lo_b = log1p(-(double)o.clip_lo), hi_b = log1p((double)o.clip_hi);
    const double w = exp(fmin(fmax(t_old, lo_b), hi_b));
    const double delta = (double)log_z[group_idx[i]] + t_ref / n - (double)o.beta * Ad;
    const float ct = (float)(2.0 * w * delta * inv_bn);
    for (int k = a + threadIdx.x; k < b; k += blockDim.x) {
      c_c[k] = ct;
      if (coeff_out) coeff_out[row_map[k]] = ct;
    }
    if (threadIdx.x == 0) {
      seq_loss[i] = (float)(w * delta * delta);
      gterm[i] = (float)(2.0 * w * delta / (double)B);
      if (stats) { if (t_old > hi_b) atomicAdd(&stats->n_clip_hi, 1); if (t_old < lo_b) atomicAdd(&stats->n_clip_lo, 1); }
    }
  }
}

// ... and the workgroup that is the last of the call to get here adds the sequences up (a launch of its own took 2 to 5 us, 16 with
// 64 sequences and the flow objective, whose prompts a thread each walked all sequences for).
template <bool FOLD>
__device__ inline void sequence_loss_and_finish(const LossJob& j, int i) {
  __shared__ int sh_last;
  if (j.desc) {
    i += j.desc->seq_begin;
    if (i >= j.desc->seq_end) return;
  }
  sequence_loss<FOLD>(j, i);
  if (j.B > kFinishSeqs || j.finish_later) return;
  if (threadIdx.x == 0) {                 // (it wrote the sequence's terms)
    __threadfence();
    sh_last = atomicAdd(&j.ctrl->done, 1) == j.B - 1;
  }
  __syncthreads();
  if (!sh_last) return;
  __threadfence();
  finish_loss(j);
}
__global__ __launch_bounds__(kLossThreads) void seq_loss_kernel(LossJob j) { sequence_loss_and_finish<false>(j, blockIdx.x); }

// ------------------------------------------------------------------ transposes (K-contiguous operands)
// dst[c][r] = src[row_of(r)][c] for r < rows_valid, 0 for rows_valid <= r < ld_dst rows covered by the grid.
template <class T>
struct TransposeJob {
  const T* src; int64_t ld_src; int rows, cols; const int32_t* row_idx;
  const Ctrl* ctrl; int chunk_start, dyn_rows; const ChunkDesc* desc; const float* row_scale;
  T* dst; int64_t ld_dst; int rows_padded; bool dst_tiled;
};
template <class T>
__device__ inline void transpose_block(const TransposeJob<T>& j, int bx, int by, T (&tile)[64][65]) {
  int rv = j.rows, chunk_start = j.chunk_start;
  if (j.dyn_rows) {
    int left;
    if (j.desc) { chunk_start = j.desc->row_start; left = j.desc->rows; } else left = j.ctrl->n_real - chunk_start;
    if (left <= 0) return;
    rv = left < j.rows ? left : j.rows;
  }
  const int r0 = bx * 64, c0 = by * 64;
  if (j.dyn_rows && r0 >= ((rv + 255) & ~255)) return;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;        // 256 threads: 4 rows per pass
#pragma unroll 4
  for (int k = ty; k < 64; k += 4) {
    const int r = r0 + k, c = c0 + tx;
    T v = (T)0.f;
    if (r < rv && c < j.cols) {
      const int64_t sr = j.row_idx ? (int64_t)j.row_idx[chunk_start + r] : (int64_t)r;
      v = j.src[sr * j.ld_src + c];
      if (j.row_scale) v = (T)((float)v * j.row_scale[r]);
    }
    tile[k][tx] = v;
  }
  __syncthreads();
  for (int k = ty; k < 64; k += 4) {
    const int c = c0 + k, r = r0 + tx;
    if (c < j.cols && r < j.rows_padded) j.dst[operand_index(j.dst_tiled, c, r, j.ld_dst)] = tile[tx][k];
  }
}
template <class T>
__global__ void transpose_kernel(TransposeJob<T> j) {
  __shared__ T tile[64][65];
  transpose_block(j, blockIdx.x, blockIdx.y, tile);
}
// The loss with W^T, X^T of the only chunk and the zeroing of the rows that do not count beside it in one launch (f32: a small call is bound by
// its launches): workgroups [0, B) form the loss, [B, B + nw) and the next nx transpose, the rest zero four rows each.
__global__ __launch_bounds__(kLossThreads) void loss_prep_kernel(LossJob j, TransposeJob<float> w, int wx, int nw, TransposeJob<float> x, int xx, int nx,
                                                                 const int32_t* cpos, float* dX, int64_t R, int H) {
  __shared__ float tile[64][65];
  int b = blockIdx.x;
  if (b < j.B) { sequence_loss_and_finish<false>(j, b); return; }
  b -= j.B;
  if (b < nw) { transpose_block(w, b % wx, b / wx, tile); return; }
  b -= nw;
  if (b < nx) { transpose_block(x, b % xx, b / xx, tile); return; }
  zero_masked_row((int64_t)(b - nx) * 4 + (threadIdx.x >> 6), cpos, dX, R, H);
}

// Combine, loss and that zeroing (dX != nullptr) in one launch: fold_combine().
__global__ __launch_bounds__(kLossThreads) void loss_fold_kernel(LossJob j, const int32_t* cpos, float* dX, int64_t R, int H) {
  const int b = blockIdx.x;
  if (b < j.B) { sequence_loss_and_finish<true>(j, b); return; }
  zero_masked_row((int64_t)(b - j.B) * 4 + (threadIdx.x >> 6), cpos, dX, R, H);
}

// The backward of such a batch, see grads_small.h; workgroup 0 adds up the loss (as the last workgroup of the loss launch did at the cost of 3 us).  U = 2: for launches that leave a CU to each workgroup.
template <int NBX, int U>
__global__ __launch_bounds__(kGradWaves * 64, U == 1 ? 8 : 4) void small_grads_kernel(SmallGrads s, LossJob j) {
  if (blockIdx.x == 0) { if (j.finish_later) finish_loss(j); return; }
  small_grads<NBX, U>(s, (int)blockIdx.x - 1);
}

// The same for bf16 with 16-byte accesses on both sides (cols % 8 == 0, 16-byte aligned rows; rows_padded % 8 == 0, tiled
// destination): a thread loads two 16-byte pieces of source rows and stores two 16-byte pieces of destination rows, each
// gathered from eight consecutive source rows of one column in LDS (row stride 33 dwords: the gather is conflict-free).
__global__ __launch_bounds__(256)
void transpose_bf16_kernel(const bf16_t* src, int64_t ld_src, int rows, int cols, const int32_t* row_idx,
                           const Ctrl* ctrl, int chunk_start, int dyn_rows, const ChunkDesc* desc, const float* row_scale,
                           bf16_t* dst, int64_t ld_dst, int rows_padded) {
  __shared__ unsigned tile[64][33];
  int rv = rows;
  if (dyn_rows) {
    int left;
    if (desc) { chunk_start = desc->row_start; left = desc->rows; } else left = ctrl->n_real - chunk_start;
    if (left <= 0) return;
    rv = left < rows ? left : rows;
  }
  const int r0 = blockIdx.x * 64, c0 = blockIdx.y * 64;
  if (dyn_rows && r0 >= ((rv + 255) & ~255)) return;
  const int ch = threadIdx.x & 7, k0 = threadIdx.x >> 3;
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int k = k0 + 32 * p, r = r0 + k, c = c0 + 8 * ch;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (r < rv && c < cols) {
      const int64_t sr = row_idx ? (int64_t)row_idx[chunk_start + r] : (int64_t)r;
      v = *reinterpret_cast<const uint4*>(src + sr * ld_src + c);
      if (row_scale) {
        const float f = row_scale[r];
        bf16x8 e = __builtin_bit_cast(bf16x8, v);
#pragma unroll
        for (int i = 0; i < 8; ++i) e[i] = (bf16_t)((float)e[i] * f);
        v = __builtin_bit_cast(uint4, e);
      }
    }
    tile[k][4 * ch] = v.x; tile[k][4 * ch + 1] = v.y; tile[k][4 * ch + 2] = v.z; tile[k][4 * ch + 3] = v.w;
  }
  __syncthreads();
  const unsigned short* t16 = reinterpret_cast<const unsigned short*>(&tile[0][0]);
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    const int k = k0 + 32 * p, c = c0 + k, r = r0 + 8 * ch;
    if (c < cols && r < rows_padded) {
      unsigned w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        w[i] = (unsigned)t16[(8 * ch + 2 * i) * 66 + k] | ((unsigned)t16[(8 * ch + 2 * i + 1) * 66 + k] << 16);
      *reinterpret_cast<uint4*>(dst + tiled_index(c, r, ld_dst)) = make_uint4(w[0], w[1], w[2], w[3]);
    }
  }
}

// Host side: the 16-byte kernel where its conditions hold (always, for the library's own bf16 buffers and 16-byte aligned inputs).
template <class T>
static void launch_transpose(dim3 grid, hipStream_t s, const T* src, int64_t ld_src, int rows, int cols, const int32_t* row_idx,
                             const Ctrl* ctrl, int chunk_start, int dyn_rows, const ChunkDesc* desc, const float* row_scale,
                             T* dst, int64_t ld_dst, int rows_padded, bool dst_tiled) {
  if constexpr (sizeof(T) == 2) {
    if (dst_tiled && cols % 8 == 0 && ld_src % 8 == 0 && rows_padded % 8 == 0 && reinterpret_cast<uintptr_t>(src) % 16 == 0) {
      transpose_bf16_kernel<<<grid, 256, 0, s>>>(src, ld_src, rows, cols, row_idx, ctrl, chunk_start, dyn_rows, desc, row_scale,
                                                 dst, ld_dst, rows_padded);
      return;
    }
  }
  transpose_kernel<T><<<grid, 256, 0, s>>>(TransposeJob<T>{src, ld_src, rows, cols, row_idx, ctrl, chunk_start, dyn_rows, desc, row_scale,
                                                           dst, ld_dst, rows_padded, dst_tiled});
}

// ------------------------------------------------------------------ MFMA ceiling probe (benchmark aid)
__global__ __launch_bounds__(256) void mfma_peak_kernel(float* out, int iters, long long* clk) {
  // the hot kernel's own instruction and register blocking: 8 x 8 blocks of v_mfma_f32_16x16x32_bf16
  floatx4 acc[64];
#pragma unroll
  for (int i = 0; i < 64; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc[i][e] = 0.f;
  // operands: pseudo-random bf16 values in (-1,1) (constant or small-integer operands let the part hold
  // 2.4 GHz; real data does not: it is the values that cost power)
  bf16x8 a[8], b[8];
  unsigned h = (blockIdx.x * 256u + threadIdx.x) * 2654435761u + 12345u;
#pragma unroll
  for (int k = 0; k < 8; ++k)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      h = h * 1664525u + 1013904223u; a[k][e] = (bf16_t)(((int)(h >> 8) & 0xffff) * (1.f / 32768.f) - 1.f);
      h = h * 1664525u + 1013904223u; b[k][e] = (bf16_t)(((int)(h >> 8) & 0xffff) * (1.f / 32768.f) - 1.f);
    }
  const long long t0 = clock64(), w0 = wall_clock64();
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int i = 0; i < 64; ++i) acc[i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i >> 3], b[i & 7], acc[i], 0, 0, 0);
  }
  const long long t1 = clock64(), w1 = wall_clock64();
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < 64; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) s += acc[i][e];
  out[blockIdx.x * blockDim.x + threadIdx.x] = s;
  if (threadIdx.x == 0) { clk[blockIdx.x * 2] = t1 - t0; clk[blockIdx.x * 2 + 1] = w1 - w0; }
}

// ------------------------------------------------------------------ host side
struct Plan {
  int64_t R; int H, V, B, P; int dtype; size_t esz;
  int Tc, Vp, tiles_v, n_chunks;
  bool bwd;
  bool tiled;            // bf16: the work buffers dS/E, W^T, X^T are slab-tiled (hot kernel operands)
  bool k_major_w;        // dX reads W as it is stored: no W^T is made (f32: dS^T too, no dS)
  bool small_pair;       // f32: dX and dW in tiles of 64 x 16, in one launch, out of dS, W^T, dS^T and X^T
  bool small_grads;      // f32: the whole backward in one launch, out of the kept logits, W and X (grads_small.h)
  bool stash;            // single-pass backward (forward keeps each chunk's unnormalised probabilities)
  bool keep;             // recompute mode, one chunk: the forward keeps the logits, dS is formed from them
  int n_desc, max_len;   // stash: number of chunk records, promised bound on rows per sequence
  float inv_tau;         // 1 / temperature
  size_t off_ctrl, off_seq_len, off_cstart, off_row_map, off_ids_c, off_cpos, off_zy, off_lse_c, off_logp_c,
      off_c_c, off_adv, off_seq_loss, off_gterm, off_part, off_wt, off_xt, off_ds, off_dst, off_split, off_kept,
      off_desc, off_ref, off_zsum, off_scale, off_ycol, least, total;       // total: with room for kept logits; least: what the calls accept
};

static inline size_t up256(size_t x) { return (x + 255) & ~(size_t)255; }

// Width of the f32 tiles of an M x N contraction over K.  (Bounds: the real extents may be smaller.)
static int f32_tile_n(int M, int N, int K, bool split) {
  const int64_t big = (int64_t)((M + kBM - 1) / kBM) * ((N + kF32BN - 1) / kF32BN);
  const int nk = (K + 31) / 32, most = split ? (nk / kSplitMinSteps < kMaxSplit ? nk / kSplitMinSteps : kMaxSplit) : 1;
  return big * (most > 1 ? most : 1) < kF32Slots ? kF32SmallBN : kF32BN;
}

// Tile rows (slices x M-tiles) of the partial buffer of a contraction of at most tm x tn tiles and `steps` steps of K that may be cut:
// at most kMaxSplit slices of at least kSplitMinSteps steps, at most 2 slots workgroups.
static int64_t split_tile_rows(int tm, int tn, int steps, int slots) {
  int64_t slices = (steps + kSplitMinSteps - 1) / kSplitMinSteps;
  if (slices > kMaxSplit) slices = kMaxSplit;
  const int64_t rows = tm * slices, most = 2 * slots / tn;
  return rows < most ? rows : most;
}
static size_t split_bytes(int M, int N, int K, int bn, int step, int slots) {
  return (size_t)split_tile_rows((M + kBM - 1) / kBM, (N + bn - 1) / bn, (K + step - 1) / step, slots) * kBM * (size_t)N * 4;
}

// dX (and dW beside it) in tiles of 64 x 16 with four K groups: one round of them at most.
static bool small_dx(int M, int N, int K) {
  return f32_tile_n(M, N, K, false) == kF32SmallBN && (int64_t)((M + 63) / 64) * ((N + kF32SmallBN - 1) / kF32SmallBN) <= kHotSlots;
}

// The launch of grads_small.h: blocks of 16 columns of a dX workgroup (two where those of dX are one round of the CUs at most, else four), workgroups of dX and of dX and dW.
static int small_dx_cols(int tc, int H) { return tc / 16 * ((H + 31) / 32) <= kHotSlots ? 2 : 4; }
static int small_dx_blocks(int tc, int H) { const int w = 16 * small_dx_cols(tc, H); return tc / 16 * ((H + w - 1) / w); }
static int small_grads_blocks(int tc, int H, int V) { return small_dx_blocks(tc, H) + (V + 15) / 16 * ((H + 16 * kGradNBW - 1) / (16 * kGradNBW)); }

// whether two arrays of so many bytes share memory
static bool meets(const void* a, size_t a_bytes, const void* b, size_t b_bytes) {
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return a && b && x < y + b_bytes && y < x + a_bytes;
}

// out: where the call's outputs go, nullptr where only the size of the workspace is asked for (which no choice that depends on them changes)
static rl_status make_plan(const rl_batch* b, const rl_params* prm, bool bwd, Plan& p, const rl_outputs* out = nullptr) {
  if (!b) return RL_ERR_NULL;
  if (b->R < 1 || b->R >= ((int64_t)1 << 31) - (1 << 16) || b->H < 1 || b->V < 1 || b->B < 1 || b->P < 1) return RL_ERR_SHAPE;
  if (b->dtype != RL_F32 && b->dtype != RL_BF16) return RL_ERR_DTYPE;
  if (b->dtype == RL_BF16 && (b->H % 8)) return RL_ERR_SHAPE;
  if (b->dtype == RL_F32 && (b->H % 4)) return RL_ERR_SHAPE;
  p.R = b->R; p.H = b->H; p.V = b->V; p.B = b->B; p.P = b->P; p.dtype = b->dtype;
  p.esz = b->dtype == RL_BF16 ? 2 : 4;
  p.inv_tau = 1.f;
  if (prm && prm->temperature != 0.f) {
    if (!(prm->temperature > 0.f) || !(prm->temperature <= 3.0e38f)) return RL_ERR_RANGE;
    p.inv_tau = 1.f / prm->temperature;
  }
  if (prm && prm->chunk_rows < 0) return RL_ERR_SHAPE;
  const int mode = prm ? prm->backward_mode : RL_BWD_AUTO;
  if (mode != RL_BWD_AUTO && mode != RL_BWD_RECOMPUTE && mode != RL_BWD_STASH) return RL_ERR_RANGE;
  if (prm && prm->max_seq_len < 0) return RL_ERR_RANGE;
  // Single-pass backward: bf16 hot-kernel shapes only, and only when the caller bounds the sequence length by a chunk.
  const int64_t rp = (b->R + 255) & ~(int64_t)255;
  auto chunk_rows = [&](int dflt) { int t = (prm && prm->chunk_rows > 0) ? prm->chunk_rows : dflt; t = (t + 255) & ~255; return t > rp ? (int)rp : t; };
  const bool stash_kernels = b->dtype == RL_BF16 && (b->H % 128 == 0) &&
                             ((reinterpret_cast<uintptr_t>(b->hidden) | reinterpret_cast<uintptr_t>(b->weight)) % 16 == 0);
  const bool stash_asked = bwd && prm && prm->max_seq_len > 0 && mode != RL_BWD_RECOMPUTE && prm->max_seq_len <= chunk_rows(kDefaultChunkRowsStash);
  const bool can_stash = stash_asked && stash_kernels;
  if (mode == RL_BWD_STASH && !stash_kernels) return RL_ERR_UNIMPLEMENTED;
  if (mode == RL_BWD_STASH && !can_stash) return RL_ERR_RANGE;
  const int tc = chunk_rows(can_stash ? kDefaultChunkRowsStash : kDefaultChunkRows);
  p.Tc = tc;
  p.Vp = (b->V + kBM - 1) / kBM * kBM;
  p.tiles_v = p.Vp / kBM;
  p.n_chunks = (int)((b->R + tc - 1) / tc);
  p.bwd = bwd;
  p.tiled = (b->dtype == RL_BF16);
  p.k_major_w = p.tiled && reinterpret_cast<uintptr_t>(b->weight) % 16 == 0 && b->R <= kKMajorRows;
  p.small_pair = b->dtype == RL_F32 && bwd && small_dx(tc, b->H, p.Vp) && small_dx(b->V, b->H, tc);
  // A gradient may take the place of an input.  dX, then dW are contracted from copies, in that order; a launch that writes one while it reads the inputs themselves is
  // not taken where they share memory.
  const size_t x_bytes = p.esz * (size_t)b->R * b->H, w_bytes = p.esz * (size_t)b->V * b->H;
  auto on_gradients = [&](const void* in, size_t bytes) { return out && (meets(out->d_hidden, x_bytes, in, bytes) || meets(out->d_weight, 4 * (size_t)b->V * b->H, in, bytes)); };
  if (b->dtype == RL_F32)          // (256 x 64 tiles of gemm_f32.h: their dX reads dS^T and W K-major.  A dX cut along K may count as so many tiles and still be small_pair's.)
    p.k_major_w = bwd && !p.small_pair && reinterpret_cast<uintptr_t>(b->weight) % 16 == 0 && tc < (1 << 22) && b->H < (1 << 22) && f32_tile_n(tc, b->H, p.Vp, true) == kF32BN &&
                  !(out && meets(out->d_hidden, x_bytes, b->weight, w_bytes));
  p.stash = can_stash;
  p.max_len = p.stash ? prm->max_seq_len : 0;
  // chunk records: two consecutive chunks hold more than Tc rows, and every chunk but the last more than Tc - max_len
  // (a batch of no more rows than a chunk holds is one chunk)
  p.n_desc = p.n_chunks == 1 ? 1 : 2 * p.n_chunks + 1;
  if (p.stash && p.max_len < tc) {
    const int64_t alt = (b->R + (tc - p.max_len)) / (tc - p.max_len + 1) + 1;
    if (alt < p.n_desc) p.n_desc = (int)alt;
  }
  // (room is set aside by shape, not alignment: a workspace serves a weight of any alignment)
  const bool keep_room = bwd && p.n_chunks == 1 && (b->dtype == RL_F32 || (mode == RL_BWD_AUTO && b->R <= kKeepRows && b->H >= kKeepH && b->R * b->H * 2 < kFarBytes &&
                                                                           !(stash_asked && b->H % 128 == 0)));
  p.keep = keep_room && (b->dtype == RL_F32 || (reinterpret_cast<uintptr_t>(b->hidden) | reinterpret_cast<uintptr_t>(b->weight)) % 16 == 0);
  // The whole backward of a small f32 batch in one launch, see grads_small.h.  What it gains is launches; a workgroup of dX walks the whole vocabulary by itself, so a
  // large one takes longer than they did.  us of the call, former launches / this one, 16, 400, 2000 rows: H 16, V 1000 43 46 73 / 28 31 51, V 2000 40 48 84 / 34 39 61,
  // V 4000 41 54 99 / 48 56 78, V 16000 47 87 212 / 120 143 185; H 128, V 300 42 47 77 / 28 31 57, V 2000 45 59 113 / 40 47 88; H 512, V 500 55 68 - / 40 50 -.
  // It is to be one round of two workgroups a CU, or of a small vocabulary: us likewise, H 4, V 1000 6000, 8000, 16000 rows 135 149 283 / 116 173 337; V 700 8000, 16000 rows 140 270 / 133 267.
  // (It adds up the loss as well, out of group_idx.)
  p.small_grads = p.small_pair && p.keep && b->V <= 2048 && (b->V <= 3 * kBM || small_grads_blocks(tc, b->H, b->V) <= 2 * kHotSlots) && !on_gradients(b->hidden, x_bytes) && !on_gradients(b->weight, w_bytes) && !on_gradients(b->group_idx, 4 * (size_t)b->B);
  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o += up256(bytes); return at; };
  const size_t Rp = (size_t)rp + 256;
  p.off_ctrl = take(sizeof(Ctrl));
  p.off_seq_len = take(sizeof(int32_t) * (size_t)b->B);
  p.off_cstart = take(sizeof(int32_t) * ((size_t)b->B + 1));
  p.off_row_map = take(4 * Rp); p.off_ids_c = take(4 * Rp); p.off_cpos = take(4 * Rp);
  p.off_zy = take(4 * Rp); p.off_lse_c = take(4 * Rp); p.off_logp_c = take(4 * Rp); p.off_c_c = take(4 * Rp);
  p.off_ycol = take(4 * Rp);
  p.off_adv = take(4 * (size_t)b->B); p.off_seq_loss = take(4 * (size_t)b->B); p.off_gterm = take(4 * (size_t)b->B);
  p.off_part = take(sizeof(float4) * (size_t)p.tiles_v * (size_t)tc);
  p.off_wt = p.off_xt = p.off_ds = p.off_dst = p.off_split = p.off_kept = 0;
  if (bwd) {
    const size_t Hp = ((size_t)b->H + 255) & ~(size_t)255;   // tiled layouts come in blocks of 256 rows
    p.off_wt = take(p.esz * Hp * (size_t)p.Vp);            // (also where an aligned W is read as it is: the size holds for a W of any alignment)
    p.off_xt = take(p.esz * Hp * (size_t)tc);
    p.off_ds = take(p.esz * (size_t)tc * (size_t)p.Vp);
    if (b->dtype == RL_F32) {
      p.off_dst = take(p.esz * (size_t)p.Vp * (size_t)tc);   // bf16: dW reads dS / E itself
      p.off_split = take(split_bytes(tc, b->H, p.Vp, f32_tile_n(tc, b->H, p.Vp, true), 32, kF32Slots));
    } else {
      p.off_split = take(split_bytes(tc, b->H, p.Vp, kBN, kHotStep, kHotSlots));
    }
  }
  p.off_desc = p.off_ref = p.off_zsum = p.off_scale = 0;
  if (p.stash) {
    p.off_desc = take(sizeof(ChunkDesc) * (size_t)p.n_desc);
    p.off_ref = take(4 * Rp); p.off_zsum = take(4 * Rp); p.off_scale = take(4 * (size_t)tc);
  }
  p.least = o;
  if (keep_room && b->dtype == RL_BF16) p.off_kept = take(4 * (size_t)tc * (size_t)p.Vp);      // last: without room for them they are recomputed
  p.total = o;
  return RL_OK;
}

// bf16 contractions take the hot kernel but for logits whose operands are not 16-byte aligned, and those of small hidden sizes off its
// grid of 128 (small_k).
template <class Epi>
static void launch_generic(const bf16_t* A, const bf16_t* B, const GemmDims& d, const Epi& epi, int tiles, hipStream_t s) {
  gemm_nt_kernel<bf16_t, Epi, kBM, kBN, 2, 4><<<tiles, 512, 0, s>>>(A, B, d, epi);
}

// Workgroups of a launch that may be split.
static int split_launch(int tiles_m, int tiles_n, int slots) {
  const int64_t t = launch_tiles(tiles_m, tiles_n);
  return (int)(t > 2 * slots ? t : 2 * slots);
}

// Logits of small hidden sizes off the grid of 128 that take the general kernel: with few slabs the shorter prologue and epilogue of its
// smaller wavefronts count for more than the main loop.  V 50257, 16 k tokens, forward: H 136 724 us in the hot kernel, 584 in the general one;
// 200 747 / 682; 320 855 / 780; 328 878 / 898; 392 969 / 966 and 440 981 / 983, with 200 tokens 24 / 27; 520 1119 / 1184.  The same holds from 96 tokens on
// (H 136 46.5 / 43.7, 328 49.9 / 49.7).  The dS epilogue, whose tiles the general kernel writes in pieces of 8 bytes, tips over earlier (with the backward: H 192
// 2502 / 2397, 200 2510 / 2621).  (By H alone: a token's bits must not depend on the batch.)
template <class Epi> constexpr bool small_k(int) { return false; }
template <> constexpr bool small_k<EpiFwd<bf16_t>>(int K) { return K % 128 && K <= 320; }
template <> constexpr bool small_k<EpiDS<bf16_t>>(int K) { return K % 128 && K <= 192; }

template <class Tune, class Epi>
static void launch_gemm(const bf16_t* A, const bf16_t* B, const GemmDims& d, const Epi& epi, hipStream_t s) {
  const int tiles = launch_tiles((d.M + kBM - 1) / kBM, (d.N + kBN - 1) / kBN);
  const bool fast = (d.lda % 8 == 0) && (d.ldb % 8 == 0) && (d.K % 8 == 0) &&
                    ((reinterpret_cast<uintptr_t>(A) | reinterpret_cast<uintptr_t>(B)) % 16 == 0) &&
                    !d.a_rows && (d.b_rows != nullptr) == Epi::kGatherB &&     // (how the hot kernel addresses its operands)
                    !small_k<Epi>(d.K);
  // (two epilogues are written for the hot kernel, one of them for K on its grid, the other for rows that span less than 4 GiB: make_plan sees to it)
  constexpr bool stash = std::is_same_v<Epi, EpiFwdStash<bf16_t>>, keep = std::is_same_v<Epi, EpiFwd<bf16_t, true>>;
  if constexpr (!stash && !keep)
    if (!fast) { launch_generic(A, B, d, epi, tiles, s); return; }
  const bool far = d.b_rows && d.b_span * d.ldb * 2 >= kFarBytes;
  if constexpr (!keep)
    if (far) {
      if constexpr (!stash)
        if (d.K % 128) { gemm_nt_bf16_kernel<Epi, Tune, true, true><<<tiles, 256, 0, s>>>(A, B, d, epi); return; }
      gemm_nt_bf16_kernel<Epi, Tune, false, true><<<tiles, 256, 0, s>>>(A, B, d, epi);
      return;
    }
  if constexpr (!stash)
    if (d.K % 128) { gemm_nt_bf16_kernel<Epi, Tune, true><<<tiles, 256, 0, s>>>(A, B, d, epi); return; }
  gemm_nt_bf16_kernel<Epi, Tune><<<tiles, 256, 0, s>>>(A, B, d, epi);
}

// Whether an M x N f32 contraction has so few tiles of 64 x 16 that four groups of wavefronts share one, each taking every fourth slab (dW of
// 2048 tokens, H 64, V 1024: 47 us; with dX in the same launch 17 + 47 -> 36; 16 k tokens, V 2000 435 -> 193; 356 tokens, H 128, V 1024, both 29 -> 22).
static bool few_small_tiles(int M, int N) { return (int64_t)((M + 63) / 64) * ((N + kF32SmallBN - 1) / kF32SmallBN) <= kF32Slots; }

// f32 logits in so few tiles of 256 x 16 that each has a CU to itself: sixteen wavefronts share one instead of four
static bool few_forward_tiles(int M, int N, int K) {
  return f32_tile_n(M, N, K, false) == kF32SmallBN && (int64_t)((M + kBM - 1) / kBM) * ((N + kF32SmallBN - 1) / kF32SmallBN) <= kHotSlots;
}

template <class Epi> constexpr bool kIsForward = false;
template <bool KEEP> constexpr bool kIsForward<EpiFwd<float, KEEP>> = true;
// f32 logits in narrow tiles of which two may come to share a CU (two_a_cu), over more than eight slabs
static bool may_be_two_a_cu(int tiles, int K) { return tiles > kHotSlots && tiles <= 4 * kHotSlots && K > 256; }
template <class Tune, class Epi>
static void launch_gemm(const float* A, const float* B, const GemmDims& d, const Epi& epi, hipStream_t s) {
  const int bn = f32_tile_n(d.M, d.N, d.K, d.split_slots > 0);
  const int tm = (d.M + kBM - 1) / kBM, tn = (d.N + bn - 1) / bn;
  const int tiles = d.split_slots > 0 ? split_launch(tm, tn, d.split_slots) : launch_tiles(tm, tn);
  const bool fast = (reinterpret_cast<uintptr_t>(A) | reinterpret_cast<uintptr_t>(B)) % 16 == 0 && d.lda % 4 == 0 && d.ldb % 4 == 0 && d.K % 4 == 0 && d.lda < (1 << 22) && d.ldb < (1 << 22) &&
                    !d.a_rows && (d.b_rows != nullptr) == Epi::kGatherB;                  // (how the kernel of gemm_f32.h addresses its operands)
  if constexpr (std::is_same_v<Epi, EpiDW>) {
    // dW has no per-tile partials and no padding to write, which ask for 256 rows: 64 x 16 tiles where the others would leave most CUs idle
    // (356 tokens, H 128, V 1024: 128 workgroups instead of 32, 21.7 -> 11.2 us), in four K groups where even these are few.
    if (bn == kF32SmallBN && tm * tn < kHotSlots) {
      const int n = launch_tiles((d.M + 63) / 64, tn);
      if (few_small_tiles(d.M, d.N)) gemm_nt_kernel<float, Epi, 64, kF32SmallBN, 4, 1, 4><<<n, 1024, 0, s>>>(A, B, d, epi);
      else gemm_nt_kernel<float, Epi, 64, kF32SmallBN, 4, 1><<<n, 256, 0, s>>>(A, B, d, epi);
      return;
    }
  }
  if constexpr (kIsForward<Epi>) {
    // The logits of unaligned operands in 256 x 256 tiles (eight wavefronts) where these come in ten rounds of the chip or more and fill them as
    // well (aligned ones: 256 x 64 tiles of the other kernel are the faster ones there too, 8 k tokens, H 768, V 50257 5041 -> 4497 us): each reads its operands fewer times over (8 k tokens: H 768, V 50257 5251 -> 5056 us, H 1536, V 30000 6176 -> 5909), but with
    // few rounds the last one, of a batch with fewer tokens than rows, costs more than that (1040 tokens, V 50257: 784 -> 843).  Same
    // bits (EpiFwd).
    const int64_t square = (int64_t)tm * ((d.N + 255) / 256), rounds = (square + kHotSlots - 1) / kHotSlots;
    const int64_t halves = ((int64_t)tm * tn + kF32Slots - 1) / kF32Slots;          // rounds of 256 x 64 tiles, half as long
    if (!fast && bn == kF32BN && rounds >= 10 && 100 * rounds <= 51 * halves) {
      gemm_nt_kernel<float, Epi, kBM, 256, 2, 4><<<launch_tiles(tm, (d.N + 255) / 256), 512, 0, s>>>(A, B, d, epi);
      return;
    }
  }
  if constexpr (kIsForward<Epi>) {
    if (few_forward_tiles(d.M, d.N, d.K)) {
      gemm_nt_kernel<float, Epi, kBM, kF32SmallBN, 16, 1><<<tiles, 1024, 0, s>>>(A, B, d, epi);
      return;
    }
    if (bn == kF32SmallBN && may_be_two_a_cu(tm * tn, d.K)) {
      gemm_nt_kernel<float, Epi, kBM, kF32SmallBN, 4, 1, 1, true><<<tiles, 256, 0, s>>>(A, B, d, epi);
      return;
    }
  }
  if constexpr (std::is_same_v<Epi, EpiDX<float>>)
    if (d.b_k_rows) { gemm_nt_f32_kernel<Epi, false, true><<<tiles, 256, 0, s>>>(A, B, d, epi); return; }        // (k_major_w)
  if (bn == kF32BN && fast) {
    // (K of dW, a number of tokens, is a multiple of 16 only; K of dX, the padded vocabulary, one of 256)
    constexpr bool tail = std::is_same_v<Epi, EpiDW>, whole = std::is_same_v<Epi, EpiDX<float>>;
    if (!whole && (tail || d.K % 32)) { if constexpr (!whole) gemm_nt_f32_kernel<Epi, true><<<tiles, 256, 0, s>>>(A, B, d, epi); }
    else if constexpr (!tail) gemm_nt_f32_kernel<Epi, false><<<tiles, 256, 0, s>>>(A, B, d, epi);
  } else if (bn == kF32BN) gemm_nt_kernel<float, Epi, kBM, kF32BN, 2, 2><<<tiles, 256, 0, s>>>(A, B, d, epi);
  else gemm_nt_kernel<float, Epi, kBM, kF32SmallBN, 4, 1><<<tiles, 256, 0, s>>>(A, B, d, epi);
}

// dX = diag(f) dS W  (A = dS or E' [Tc][Vp], B = W^T [H][Vp]) and dW (+)= dS^T (diag(f) X)  (A = the same array read as a K-major
// operand, B = X^T [H][Tc]) of a bf16 chunk in one launch: dX alone has few (long) tiles, whose last round would leave CUs
// idle; the dW tiles fill them.  dX is cut along K where its tiles are fewer still.
static void launch_dx_dw(const bf16_t* E, const bf16_t* W, const bf16_t* WT, GemmDims dx, EpiDX<bf16_t> ex, const bf16_t* XT, const GemmDims& dw,
                         const EpiDW& ew, hipStream_t s) {
  const int tn = (dx.N + kBN - 1) / kBN;
  dx.split_slots = kHotSlots; dx.fill_tiles = (dw.M + kBM - 1) / kBM * tn;
  const int n1 = split_launch((dx.M + kBM - 1) / kBM, tn, kHotSlots);
  const int n2 = launch_tiles((dw.M + kBM - 1) / kBM, tn);
  if (WT) {
    const bool both = step_prefetch(dx.M, tn, dx.fill_tiles);
    gemm_nt_bf16_pair_kernel<EpiDX<bf16_t>, TuneDX, EpiDW, TuneDW, false><<<n1 + n2, 256, 0, s>>>(E, WT, dx, ex, n1, E, XT, dw, ew, 0, both ? kStepRows : 0);
    if (both) gemm_nt_bf16_pair_kernel<EpiDX<bf16_t>, TuneDXStep, EpiDW, TuneDWStep, false><<<n1 + n2, 256, 0, s>>>(E, WT, dx, ex, n1, E, XT, dw, ew, kStepRows, 0);
  } else {
    dx.ldb = dx.N; dx.b_k_rows = dw.M;
    gemm_nt_bf16_pair_kernel<EpiDX<bf16_t>, TuneDX, EpiDW, TuneDW, true><<<n1 + n2, 256, 0, s>>>(E, W, dx, ex, n1, E, XT, dw, ew, 0, 0);
  }
  splitk_reduce_kernel<bf16_t><<<512, 256, 0, s>>>(dx, ex, kBM, kBN, kHotStep);
}

// The combine of a small f32 batch inside its loss launch, also where no gradients are asked for: up to 1024 rows, which are four tokens of a thread at most.
static bool fold_combine(const Plan& p) { return p.dtype == RL_F32 && p.n_chunks == 1 && p.tiles_v <= kFoldTiles && p.Tc <= kFoldRows && (!p.bwd || p.small_grads); }

struct Ptrs {
  Ctrl* ctrl; int32_t *seq_len, *cstart, *row_map, *ids_c, *cpos;
  float *zy, *lse_c, *logp_c, *c_c, *adv, *seq_loss, *gterm; float4* part;
  void *wt, *xt, *ds, *dst; float *split, *kept;
  ChunkDesc* desc; float *ref, *zsum, *scale;
  int32_t* ycol;
};

static Ptrs carve(void* ws, const Plan& p) {
  unsigned char* w = static_cast<unsigned char*>(ws);
  Ptrs q;
  q.ctrl = (Ctrl*)(w + p.off_ctrl); q.seq_len = (int32_t*)(w + p.off_seq_len); q.cstart = (int32_t*)(w + p.off_cstart);
  q.row_map = (int32_t*)(w + p.off_row_map); q.ids_c = (int32_t*)(w + p.off_ids_c); q.cpos = (int32_t*)(w + p.off_cpos);
  q.zy = (float*)(w + p.off_zy); q.lse_c = (float*)(w + p.off_lse_c); q.logp_c = (float*)(w + p.off_logp_c);
  q.c_c = (float*)(w + p.off_c_c); q.adv = (float*)(w + p.off_adv); q.seq_loss = (float*)(w + p.off_seq_loss);
  q.gterm = (float*)(w + p.off_gterm); q.part = (float4*)(w + p.off_part);
  q.wt = w + p.off_wt; q.xt = w + p.off_xt; q.ds = w + p.off_ds;
  q.dst = p.off_dst ? w + p.off_dst : nullptr;          // f32 inputs only
  q.split = (float*)(w + p.off_split);
  q.kept = p.dtype == RL_F32 ? (float*)q.dst : (float*)(w + p.off_kept);
  q.desc = (ChunkDesc*)(w + p.off_desc); q.ref = (float*)(w + p.off_ref); q.zsum = (float*)(w + p.off_zsum);
  q.scale = (float*)(w + p.off_scale);
  q.ycol = (int32_t*)(w + p.off_ycol);
  return q;
}

// whether an output (of `size` bytes) shares memory with what the preparation reads
static bool on_prep_inputs(const rl_batch* b, const Plan& p, const void* out, size_t size) {
  auto on = [&](const void* in, size_t bytes) { return meets(out, size, in, bytes); };
  return on(b->token_ids, 4 * (size_t)p.R) || on(b->mask, (size_t)p.R) || on(b->cu_seqlens, 4 * ((size_t)p.B + 1)) || on(b->group_idx, 4 * (size_t)p.B);
}

// The preparation as the launch of the logits does it, if it does (on).
struct PrepJob { bool on; SmallPrep s; RowFill f; AdvJob adv; };

// bf16 logits in tiles of 128 rows, see logits_few.h, where their rounds of 256 CUs are worth less than those of the 256-row tiles: an odd number of
// rounds.  100 tokens, H 2048: V 40000 (313 tiles, two rounds against one of twice their length) 57 us in the hot kernel, 67 in the other; V 80000 124 and 111,
// V 100000 (four against two) 142 and 142; 30 tokens at the 7B head 294 and 224, 128 tokens, H 4096, V 151936 335 and 324.  (H by the same rule
// as there, so that a token's bits do not depend on the batch.)
static bool few_tokens(const rl_batch* b, const Plan& p) {
  return p.dtype == RL_BF16 && !p.stash && !p.keep && p.R <= kFewTokens && (p.tiles_v + 127) / 128 % 2 && !small_k<EpiFwd<bf16_t>>(p.H) &&
         (reinterpret_cast<uintptr_t>(b->weight) | reinterpret_cast<uintptr_t>(b->hidden)) % 16 == 0;
}
// ... with W in non-temporal loads where it is larger than the 256 MB of the memory-side cache, so that a next call finds nothing of it in any case, and its rows lie on lines of 128
// bytes.  us without and with, scored again and again: 5 tokens, H 3584, V 83705 (600 MB) 128 and 118; 60 tokens, H 2048, V 80566 (330 MB) 99 and 93; 40 at H 4096, V 151936 291 and 266;
// behind 1 GB of other stores 30 to 80 us less.  A W of 131 MB (H 2048, V 32000) 25 tokens 30.7 and 37.8, 110 tokens 36.9 and 40.2; rows off the lines, each of which is then taken
// twice: 5 tokens, H 2040, V 142262 152 and 169, H 3592, V 152064 241 and 259.
static bool few_streams_w(const rl_batch* b, const Plan& p) { return (int64_t)p.V * p.H * 2 > (int64_t)256 << 20 && p.H % 64 == 0 && reinterpret_cast<uintptr_t>(b->weight) % 128 == 0; }
// ... and the preparation in the same launch where it is one to three rounds of workgroups, each of which works out the rows: us in the launch and ahead of it, 99 tokens, V 32000
// 35.5 and 38.1, 120 tokens, H 512, V 68000 40.4 and 42.2; five rounds, 38 tokens in as many sequences, H 128, V 153761 41.7 and 39.6, 110 tokens at the 7B head 246 and 241.
static bool few_prepare(const Plan& p) { return p.tiles_v <= 3 * 128; }
template <bool NT> static auto few_kernel(int64_t rows, bool prep) {
  return prep ? (rows <= 64 ? logits_few_kernel<64, true, NT> : logits_few_kernel<128, true, NT>) : rows <= 64 ? logits_few_kernel<64, false, NT> : logits_few_kernel<128, false, NT>;
}
static bool small_logits(const Plan& p) { return p.dtype == RL_F32 && p.n_chunks == 1 && p.R <= kLocalRows && few_forward_tiles(p.V, p.Tc, p.H); }

// prep: row outputs cleared (rows that do not count read 0 / -1), advantages, counts, compaction, chunk records
static void run_prep(const rl_batch* b, const Plan& p, const Ptrs& q, const int32_t* group_idx, const rl_outputs& out, const AdvJob& adv,
                     PrepJob& job, hipStream_t s) {
  ProfScope ps(RL_PROF_PREP, s);
  job.on = false;
  RowFill f{};
  int nf = 0;
  auto clear = [&](void* a, int v) { f.p[nf] = static_cast<int32_t*>(a); f.v[nf++] = v; };
  // (the last three may take the place of what the compaction reads, e.g. target_col that of token_ids: they are then cleared after it)
  const size_t rows4 = 4 * (size_t)p.R;
  const bool late = on_prep_inputs(b, p, out.target_col, rows4) || on_prep_inputs(b, p, out.entropy, rows4) || on_prep_inputs(b, p, out.target_logit, rows4);
  auto clear_last = [&]() { clear(out.target_col, -1); clear(out.entropy, 0); clear(out.target_logit, 0); };
  clear(q.cpos, -1); clear(out.row_map, -1);
  clear(out.logprob, 0); clear(out.lse, 0); clear(out.coeff, 0);
  if (!late) clear_last();
  if (!late && p.R <= kSmallRows && p.B <= kSmallSeqs && (!adv.blocks || p.P <= kSmallPrompts)) {
    job = PrepJob{small_logits(p) || (few_tokens(b, p) && few_prepare(p)),
                  SmallPrep{b->mask, b->token_ids, b->cu_seqlens, group_idx, (int)p.R, p.V, p.P, p.B, q.seq_len, q.cstart, q.row_map, q.ids_c, q.cpos, out.row_map, q.ctrl,
                            ChunkJob{p.stash ? q.desc : nullptr, p.n_desc, p.Tc, p.max_len}, out.stats}, f, adv};
    // (there, outputs are cleared while other workgroups still read the inputs: with one in the place of another the preparation goes first)
    for (const void* o : {(const void*)out.row_map, (const void*)out.logprob, (const void*)out.lse, (const void*)out.coeff})
      if (on_prep_inputs(b, p, o, rows4)) job.on = false;
    if (on_prep_inputs(b, p, out.stats, sizeof(rl_stats)) || on_prep_inputs(b, p, out.group_count, 4 * (size_t)p.P)) job.on = false;
    if (!job.on) prep_small_kernel<<<1, 1024, 0, s>>>(job.s, f, adv);
    return;
  }
  const int64_t fill = (p.R + kInitThreads - 1) / kInitThreads;
  // the running maximum of the offsets borrows cstart until the compaction overwrites it with the compacted starts
  prep_init_kernel<<<1 + adv.blocks + (int)(fill < 2048 ? fill : 2048), kInitThreads, 0, s>>>(b->cu_seqlens, p.B, p.R, q.cstart, f, adv, out.stats);
  seq_count_kernel<<<p.B, 256, 0, s>>>(b->mask, b->token_ids, b->cu_seqlens, q.cstart, group_idx, p.R, p.V, p.P, q.seq_len, out.stats);
  const bool scan = p.B > kScanInline;
  if (scan) seq_scan_kernel<<<1, 1024, 0, s>>>(q.seq_len, p.B, q.cstart);
  compact_kernel<<<p.B + 1, 1024, 0, s>>>(b->mask, b->token_ids, b->cu_seqlens, q.seq_len, p.B, q.cstart, scan, p.V, q.row_map, q.ids_c, q.cpos,
                                          out.row_map, q.ctrl, ChunkJob{p.stash ? q.desc : nullptr, p.n_desc, p.Tc, p.max_len}, out.stats);
  if (late) {
    f = RowFill{}; nf = 0;
    clear_last();
    row_fill_kernel<<<(int)(fill < 2048 ? fill : 2048), kInitThreads, 0, s>>>(p.R, f);
  }
}

template <class T>
static void run_forward(const rl_batch* b, const Plan& p, const Ptrs& q, float* logp_out, float* lse_out, float* ent_out,
                        float* zy_out, int32_t* ycol_out, bool fold, const PrepJob& prep, hipStream_t s) {
  const T* X = static_cast<const T*>(b->hidden);
  const T* W = static_cast<const T*>(b->weight);
  for (int ch = 0; ch < p.n_chunks; ++ch) {
    const int c0 = ch * p.Tc;
    GemmDims d{};
    d.M = p.V; d.N = p.Tc; d.K = p.H; d.lda = p.H; d.ldb = p.H;
    d.a_rows = nullptr; d.b_rows = q.row_map + c0; d.b_span = p.R; d.n_real = &q.ctrl->n_real; d.chunk_start = c0; d.dyn = 2; d.group_m = TuneLogits::kBand;
    bool few = false;
    {
      ProfScope ps(RL_PROF_GEMM_FWD, s);
      if constexpr (sizeof(T) == 2) {
        few = few_tokens(b, p);
        if (few) {
          const EpiFwd<T> e{q.ids_c, q.zy, q.part, kFewTokens, p.V, p.inv_tau, q.ycol, nullptr};
          auto kern = few_streams_w(b, p) ? few_kernel<true>(p.R, prep.on) : few_kernel<false>(p.R, prep.on);
          kern<<<2 * p.tiles_v + (prep.on ? 1 : 0), 256, 0, s>>>(W, X, d, e, prep.s, prep.f, prep.adv);
        }
      } else if (prep.on) {
        d.b_rows = nullptr; d.n_real = nullptr;                // (lists of the workgroups)
        const int tiles = launch_tiles(p.tiles_v, (p.Tc + kF32SmallBN - 1) / kF32SmallBN);
        if (p.keep) logits_small_kernel<<<tiles + 1, 1024, 0, s>>>(W, X, d, EpiFwd<T, true>{nullptr, q.zy, q.part, p.Tc, p.V, p.inv_tau, q.ycol, q.kept}, prep.s, prep.f, prep.adv);
        else logits_small_kernel<<<tiles + 1, 1024, 0, s>>>(W, X, d, EpiFwd<T>{nullptr, q.zy, q.part, p.Tc, p.V, p.inv_tau, q.ycol, nullptr}, prep.s, prep.f, prep.adv);
      }
      if (few || prep.on) {}
      else if (p.keep) launch_gemm<TuneLogits>(W, X, d, EpiFwd<T, true>{q.ids_c, q.zy, q.part, p.Tc, p.V, p.inv_tau, q.ycol, q.kept}, s);
      else launch_gemm<TuneLogits>(W, X, d, EpiFwd<T>{q.ids_c, q.zy, q.part, p.Tc, p.V, p.inv_tau, q.ycol, nullptr}, s);
    }
    if (fold) continue;
    ProfScope ps(RL_PROF_COMBINE, s);
    const int slices = combine_slices(p.tiles_v);
    auto kern = slices == 4 ? (few ? lse_combine_kernel<true, 4> : lse_combine_kernel<false, 4>)
                : slices == 8 ? (few ? lse_combine_kernel<true, 8> : lse_combine_kernel<false, 8>) : few ? lse_combine_kernel<true, 16> : lse_combine_kernel<false, 16>;
    const int rows = combine_rows(slices);
    kern<<<((few ? kFewTokens : p.Tc) + rows - 1) / rows, rows * slices, 0, s>>>(q.part, few ? kFewTokens : p.Tc, p.tiles_v, q.zy, q.row_map, q.ctrl, c0, p.Tc,
                                                                               q.ycol, q.lse_c, q.logp_c, lse_out, logp_out, ent_out, zy_out, ycol_out);
  }
}

template <class T>
static void run_backward(const rl_batch* b, const Plan& p, const Ptrs& q, void* d_hidden, float* d_weight, bool xt_done, const LossJob& loss, hipStream_t s) {
  const T* X = static_cast<const T*>(b->hidden);
  const T* W = static_cast<const T*>(b->weight);
  T* WT = static_cast<T*>(q.wt); T* XT = static_cast<T*>(q.xt);
  T* dS = static_cast<T*>(q.ds); T* dST = static_cast<T*>(q.dst);
  T* dX = static_cast<T*>(d_hidden);
  // masked rows of dX are zero; rows that count are written by the dX epilogue.  W^T [H][Vp] with zero padding columns, once per
  // call unless dX reads W as it is (k_major_w).  xt_done: those that are needed, and X^T of the only chunk, are there (loss_prep_kernel; a batch whose gradients come in one launch needs none).
  const dim3 gw((p.Vp + 63) / 64, (p.H + 63) / 64), gx((p.Tc + 63) / 64, (p.H + 63) / 64);
  if (!xt_done) {
    ProfScope ps(RL_PROF_TRANSPOSE, s);
    zero_masked_rows_kernel<T><<<(unsigned)((p.R + 3) / 4), 256, 0, s>>>(q.cpos, dX, p.R, p.H);
    if (!p.k_major_w) launch_transpose<T>(gw, s, W, p.H, p.V, p.H, nullptr, q.ctrl, 0, 0, nullptr, nullptr, WT, p.Vp, p.Vp, p.tiled);
  }
  if constexpr (sizeof(T) == 4)
    if (p.small_grads) {
      ProfScope ps(RL_PROF_GEMM_BWD, s);
      const int nbx = small_dx_cols(p.Tc, p.H), xc = (p.H + 16 * nbx - 1) / (16 * nbx), nx = small_dx_blocks(p.Tc, p.H), n = small_grads_blocks(p.Tc, p.H, p.V);
      auto kern = nbx == 4 ? small_grads_kernel<4, 1> : n <= kHotSlots ? small_grads_kernel<2, 2> : small_grads_kernel<2, 1>;
      kern<<<n + 1, kGradWaves * 64, 0, s>>>(
          SmallGrads{{q.ids_c, q.lse_c, q.c_c, &q.ctrl->n_real, p.V, p.inv_tau}, q.kept, p.Tc, X, W, q.row_map, p.H, dX, d_weight, xc, nx}, loss);
      return;
    }
  for (int ch = 0; ch < p.n_chunks; ++ch) {
    const int c0 = ch * p.Tc;
    if (!xt_done) {  // X^T chunk [H][Tc], gathered through row_map, zero beyond the valid rows
      ProfScope ps(RL_PROF_TRANSPOSE, s);
      launch_transpose<T>(gx, s, X, p.H, p.Tc, p.H, q.row_map, q.ctrl, c0, 1, nullptr, nullptr, XT, p.Tc, p.Tc, p.tiled);
    }
    if (p.keep) {
      ProfScope ps(RL_PROF_GEMM_DS, s);
      const KeptJob j{q.ids_c, q.lse_c, q.c_c, &q.ctrl->n_real, p.V, p.inv_tau};
      if constexpr (sizeof(T) == 4) {
        if (p.k_major_w) kept_ds_t_kernel<<<(unsigned)((int64_t)(p.Vp / 32) * (p.Tc / 256)), 256, 0, s>>>(j, dST, p.Tc, p.Vp);
        else kept_ds_f32_kernel<<<(unsigned)((int64_t)(p.Vp / 64) * (p.Tc / 64)), 256, 0, s>>>(j, dST, p.Tc, dS, p.Vp);
      } else kept_ds_kernel<<<dim3((unsigned)(4 * p.tiles_v * (p.Tc / 256)), 2), 256, 0, s>>>(q.kept, j, p.tiles_v, dS, p.Vp);
    } else {  // recompute logits, form dS (and dS^T for f32 inputs)
      GemmDims d{};
      d.M = p.V; d.N = p.Tc; d.K = p.H; d.lda = p.H; d.ldb = p.H;
      d.b_rows = q.row_map + c0; d.b_span = p.R; d.n_real = &q.ctrl->n_real; d.chunk_start = c0; d.dyn = 2; d.group_m = TuneLogits::kBand;
      EpiDS<T> e{q.ids_c, q.lse_c, q.c_c, sizeof(T) == 4 && p.k_major_w ? nullptr : dS, p.Vp, dST, p.Tc, p.V, p.tiled, p.inv_tau};
      ProfScope ps(RL_PROF_GEMM_DS, s);
      launch_gemm<TuneLogits>(W, X, d, e, s);
    }
    // dX = dS W: A = dS [Tc][Vp], B = W^T [H][Vp]
    GemmDims dx{};
    dx.M = p.Tc; dx.N = p.H; dx.K = p.Vp; dx.lda = p.Vp; dx.ldb = p.Vp;
    dx.n_real = &q.ctrl->n_real; dx.chunk_start = c0; dx.dyn = 1; dx.group_m = TuneDX::kBand;
    EpiDX<T> ex{q.row_map, dX, p.H, p.H, nullptr, q.split};
    // dW (+)= dS^T X: B = X^T [H][Tc]; A = dS^T, for bf16 read out of dS itself as a K-major operand (K = Tc is a multiple of 256
    // and the workspace is aligned: always the hot kernel), for f32 the stored copy [Vp][Tc]
    GemmDims dw{};
    dw.M = p.V; dw.N = p.H; dw.K = p.Tc; dw.lda = p.tiled ? p.Vp : p.Tc; dw.ldb = p.Tc;
    dw.n_real = &q.ctrl->n_real; dw.chunk_start = c0; dw.dyn = 3; dw.k_round = p.tiled ? 256 : kF32SmallBN; dw.group_m = TuneDW::kBand;
    dw.zero_if_empty = (ch == 0);
    EpiDW ew{d_weight, p.H, p.V, p.H, ch > 0 ? 1 : 0};
    if constexpr (sizeof(T) == 2) {
      ProfScope ps(RL_PROF_GEMM_BWD, s);
      launch_dx_dw(dS, W, p.k_major_w ? nullptr : WT, dx, ex, XT, dw, ew, s);
    } else {
      dx.split_slots = kF32Slots;
      if (p.small_pair) {
        ProfScope ps(RL_PROF_GEMM_BWD, s);
        const int n1 = split_launch((dx.M + 63) / 64, (dx.N + kF32SmallBN - 1) / kF32SmallBN, kF32Slots);
        gemm_nt_small_pair_kernel<<<n1 + launch_tiles((dw.M + 63) / 64, (dw.N + kF32SmallBN - 1) / kF32SmallBN), 1024, 0, s>>>(dS, WT, dx, ex, n1, dST, XT, dw, ew);
        splitk_reduce_kernel<T><<<512, 256, 0, s>>>(dx, ex, 64, kF32SmallBN, 128);
        continue;
      }
      {
        ProfScope ps(RL_PROF_GEMM_DX, s);
        if (p.k_major_w) { dx.lda = p.Tc; dx.ldb = p.H; dx.b_k_rows = p.V; }
        launch_gemm<TuneDX>(p.k_major_w ? dST : dS, p.k_major_w ? W : WT, dx, ex, s);
        splitk_reduce_kernel<T><<<512, 256, 0, s>>>(dx, ex, kBM, f32_tile_n(dx.M, dx.N, dx.K, true), 32);
      }
      ProfScope ps(RL_PROF_GEMM_DW, s);
      launch_gemm<TuneDW>(dST, XT, dw, ew, s);
    }
  }
}

// f32 batch of one chunk: the loss and what the backward needs prepared, in one launch.  False if the launch would be too large.
static bool run_loss_prep(const rl_batch* b, const Plan& p, const Ptrs& q, const LossJob& j, float* dX, hipStream_t s) {
  const float *X = static_cast<const float*>(b->hidden), *W = static_cast<const float*>(b->weight);
  float *WT = static_cast<float*>(q.wt), *XT = static_cast<float*>(q.xt);
  const int wx = (p.Vp + 63) / 64, xx = (p.Tc + 63) / 64, hy = (p.H + 63) / 64;
  const bool small = p.small_grads;                     // (reads W and X as they are)
  const int64_t nw = small || p.k_major_w ? 0 : (int64_t)wx * hy, nx = small ? 0 : (int64_t)xx * hy, n = p.B + nw + nx + (p.R + 3) / 4;
  if (p.dtype != RL_F32 || p.n_chunks != 1 || n >= (1 << 24)) return false;        // (2^32 threads a launch)
  loss_prep_kernel<<<(unsigned)n, kLossThreads, 0, s>>>(
      j, TransposeJob<float>{W, p.H, p.V, p.H, nullptr, q.ctrl, 0, 0, nullptr, nullptr, WT, p.Vp, p.Vp, false}, wx, (int)nw,
      TransposeJob<float>{X, p.H, p.Tc, p.H, q.row_map, q.ctrl, 0, 1, nullptr, nullptr, XT, p.Tc, p.Tc, false}, xx, (int)nx, q.cpos, dX, p.R, p.H);
  return true;
}

static LossOpts loss_opts(const rl_params* prm) {
  LossOpts o;
  o.clip_lo = prm->clip_eps;
  o.clip_hi = prm->clip_eps_high > 0.f ? prm->clip_eps_high : prm->clip_eps;
  o.kl_coef = prm->kl_coef; o.beta = prm->beta;
  o.token_agg = prm->aggregation == RL_AGG_TOKEN;
  o.seq_ratio = prm->ratio_level == RL_RATIO_SEQUENCE;
  o.w_mean = prm->flow_weight_norm == RL_WNORM_MEAN;
  return o;
}

static void run_finalize(const LossJob& j, hipStream_t s) {
  if (j.B > kFinishSeqs) finalize_kernel<<<1 + (j.d_log_z ? (j.P + 15) / 16 : 0), 1024, 0, s>>>(j);
}
static LossJob loss_job(const rl_batch* b, const rl_params* prm, int objective, const Plan& p, const Ptrs& q, const rl_outputs* out,
                        const ChunkDesc* desc) {
  return LossJob{objective, q.logp_c, b->old_logprob, b->ref_logprob, q.row_map, q.cstart, q.adv, b->group_idx, b->log_z, p.B, p.P, loss_opts(prm),
                 q.ctrl, q.seq_loss, q.gterm, q.c_c, out->coeff, out->stats, desc, out->advantages, out->seq_len, out->loss, out->d_log_z, out->seq_loss, CombineJob{}, 0};
}

// Single-pass variant of forward + loss + backward (bf16 hot kernels): chunks are made of whole
// sequences, so each chunk's loss coefficients are known as soon as its forward is; the forward
// keeps the chunk's unnormalised probabilities E and the backward contractions run on
// them directly: dX = diag(-c/Z) E' W and dW += E'^T diag(-c/Z) X, E' = E with the target entry
// patched (E' is the row-major A operand of the first and the K-major A operand of the second).  Three contractions per chunk instead of four; T x V is still never held, only Tc x V.
static void run_fused(const rl_batch* b, const rl_params* prm, int objective, const Plan& p, const Ptrs& q,
                      const rl_outputs* out, hipStream_t s) {
  typedef bf16_t T;
  const T* X = static_cast<const T*>(b->hidden);
  const T* W = static_cast<const T*>(b->weight);
  T* WT = static_cast<T*>(q.wt); T* XT = static_cast<T*>(q.xt);
  T* E = static_cast<T*>(q.ds);
  T* dX = static_cast<T*>(out->d_hidden);
  if (!p.k_major_w) {
    ProfScope ps(RL_PROF_TRANSPOSE, s);
    dim3 g((p.Vp + 63) / 64, (p.H + 63) / 64);
    launch_transpose<T>(g, s, W, p.H, p.V, p.H, nullptr, q.ctrl, 0, 0, nullptr, nullptr, WT, p.Vp, p.Vp, p.tiled);
  }
  {
    ProfScope ps(RL_PROF_PREP, s);
    target_logit_kernel<<<(unsigned)((p.R + 3) / 4), 256, 0, s>>>(X, W, p.R, p.H, q.cpos, q.ids_c, b->old_logprob, p.inv_tau, dX, q.zy, q.ref, q.ycol);
  }
  float2* part = reinterpret_cast<float2*>(q.part);
  for (int k = 0; k < p.n_desc; ++k) {
    const ChunkDesc* dk = q.desc + k;
    const int* chunk = &dk->row_start;
    {  // forward: partial sums + E
      GemmDims d{};
      d.M = p.V; d.N = p.Tc; d.K = p.H; d.lda = p.H; d.ldb = p.H;
      d.b_rows = q.row_map; d.b_span = p.R; d.chunk = chunk; d.dyn = 2; d.group_m = TuneLogits::kBand;
      EpiFwdStash<T> e{q.ref, part, p.Tc, E, p.Vp, p.V, p.inv_tau};
      ProfScope ps(RL_PROF_GEMM_FWD, s);
      launch_gemm<TuneLogits>(W, X, d, e, s);
    }
    {
      ProfScope ps(RL_PROF_COMBINE, s);
      lse_sum_kernel<<<(p.Tc + kSumRows - 1) / kSumRows, kSumRows * kSumSlices, 0, s>>>(part, p.Tc, p.tiles_v, q.zy, q.ref, q.row_map, dk, q.ycol, q.ctrl, out->stats,
                                                      q.lse_c, q.logp_c, q.zsum, out->lse, out->logprob, out->entropy,
                                                      out->target_logit, out->target_col);
    }
    {
      ProfScope ps(RL_PROF_LOSS, s);
      seq_loss_kernel<<<p.B, kLossThreads, 0, s>>>(loss_job(b, prm, objective, p, q, out, dk));
      stash_patch_kernel<T><<<(p.Tc + 255) / 256, 256, 0, s>>>(dk, q.ids_c, q.zy, q.ref, q.zsum, q.c_c, p.inv_tau, q.scale, E, p.Vp);
    }
    {  // X^T chunk scaled by -c/Z, zero beyond the valid rows
      ProfScope ps(RL_PROF_TRANSPOSE, s);
      dim3 g((p.Tc + 63) / 64, (p.H + 63) / 64);
      launch_transpose<T>(g, s, X, p.H, p.Tc, p.H, q.row_map, q.ctrl, 0, 1, dk, q.scale, XT, p.Tc, p.Tc, true);
    }
    {  // dX = diag(-c/Z) E' W and dW (+)= E'^T (diag(-c/Z) X)
      GemmDims dx{};
      dx.M = p.Tc; dx.N = p.H; dx.K = p.Vp; dx.lda = p.Vp; dx.ldb = p.Vp;
      dx.chunk = chunk; dx.dyn = 1; dx.group_m = TuneDX::kBand;
      EpiDX<T> ex{q.row_map, dX, p.H, p.H, q.scale, q.split};
      GemmDims dw{};
      dw.M = p.V; dw.N = p.H; dw.K = p.Tc; dw.lda = p.Vp; dw.ldb = p.Tc;
      dw.chunk = chunk; dw.dyn = 3; dw.k_round = 256; dw.zero_if_empty = (k == 0); dw.group_m = TuneDW::kBand;
      EpiDW ew{out->d_weight, p.H, p.V, p.H, k > 0 ? 1 : 0};
      ProfScope ps(RL_PROF_GEMM_BWD, s);
      launch_dx_dw(E, W, p.k_major_w ? nullptr : WT, dx, ex, XT, dw, ew, s);
    }
  }
  ProfScope ps(RL_PROF_LOSS, s);
  run_finalize(loss_job(b, prm, objective, p, q, out, nullptr), s);
}

static rl_status check_ws(void* ws, size_t bytes, Plan& p) {
  if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255) || bytes < p.least) return RL_ERR_WORKSPACE;
  if (bytes < p.total) p.keep = false;
  return RL_OK;
}

}  // namespace rlk

using namespace rlk;

extern "C" {

const char* rl_status_string(int32_t s) {
  switch (s) {
    case RL_OK: return "ok";
    case RL_ERR_NULL: return "a required pointer is NULL";
    case RL_ERR_SHAPE: return "a size is non-positive, too large or misaligned";
    case RL_ERR_DTYPE: return "unknown dtype";
    case RL_ERR_RANGE: return "objective or a coefficient is out of range";
    case RL_ERR_WORKSPACE: return "workspace is NULL, misaligned or too small";
    case RL_ERR_HIP: return "a HIP launch failed";
    case RL_ERR_UNIMPLEMENTED: return "this build has no kernel for the request (single-pass backward needs bf16 inputs and H % 128 == 0)";
    default: return "unknown status";
  }
}

void rl_profile_enable(int32_t on) { g_prof.on = (on != 0); }

rl_status rl_profile_read(rl_profile* out) {
  if (!out) return RL_ERR_NULL;
  memset(out, 0, sizeof(*out));
  rl_status st = RL_OK;
  for (const ProfRec& r : g_prof.recs) {
    float ms = 0.f;
    if (hipEventSynchronize(r.b) != hipSuccess || hipEventElapsedTime(&ms, r.a, r.b) != hipSuccess) st = RL_ERR_HIP;
    else if (r.cls >= 0 && r.cls < RL_PROF_CLASSES) { out->ms[r.cls] += (double)ms; out->launches[r.cls] += 1; }
    g_prof.pool.push_back({r.a, r.b});
  }
  g_prof.recs.clear();
  return st;
}

int32_t rl_version(void) { return 107; }
int32_t rl_default_chunk_rows(void) { return kDefaultChunkRows; }
int32_t rl_default_chunk_rows_single_pass(void) { return kDefaultChunkRowsStash; }

rl_status rl_measure_mfma_peak(int32_t millis, void* scratch, size_t scratch_bytes, void* stream,
                               double* tflops, double* shader_mhz) {
  if (!scratch || !tflops || !shader_mhz) return RL_ERR_NULL;
  if (millis < 1 || millis > 5000) return RL_ERR_RANGE;
  constexpr int kBlocks = 1024;                                   // 4 workgroups of 4 wavefronts per CU
  if (scratch_bytes < (size_t)kBlocks * 256 * 4 + (size_t)kBlocks * 16 || (reinterpret_cast<uintptr_t>(scratch) & 15)) return RL_ERR_WORKSPACE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  float* out = static_cast<float*>(scratch);
  long long* clk = reinterpret_cast<long long*>(out + kBlocks * 256);
  // one launch of `iters` rounds of 64 MFMAs per wavefront: ~16 cycles per MFMA, 4 workgroups share a CU
  const double cycles_per_round = 64.0 * 16.0 * 4.0;
  int iters = (int)(millis * 1e-3 * 2.0e9 / cycles_per_round);
  if (iters < 16) iters = 16;
  hipEvent_t e0, e1;
  if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) return RL_ERR_HIP;
  mfma_peak_kernel<<<kBlocks, 256, 0, s>>>(out, 16, clk);        // warm-up
  (void)hipEventRecord(e0, s);
  mfma_peak_kernel<<<kBlocks, 256, 0, s>>>(out, iters, clk);
  (void)hipEventRecord(e1, s);
  rl_status st = RL_OK;
  float ms = 0.f;
  if (hipEventSynchronize(e1) != hipSuccess || hipEventElapsedTime(&ms, e0, e1) != hipSuccess || ms <= 0.f) st = RL_ERR_HIP;
  long long h[2] = {0, 0};
  if (st == RL_OK && hipMemcpy(h, clk, sizeof(h), hipMemcpyDeviceToHost) != hipSuccess) st = RL_ERR_HIP;
  (void)hipEventDestroy(e0); (void)hipEventDestroy(e1);
  if (st != RL_OK) return st;
  *tflops = (double)kBlocks * 4.0 * iters * 64.0 * 16384.0 / (ms * 1e-3) / 1e12;
  *shader_mhz = h[1] > 0 ? 100.0 * (double)h[0] / (double)h[1] : 0.0;   // wall clock ticks at 100 MHz
  return RL_OK;
}

rl_status rl_debug_tile_order(int32_t tiles_m, int32_t tiles_n, int32_t group_m, int32_t by_share,
                              int32_t* workgroups, int32_t* tile) {
  if (!workgroups) return RL_ERR_NULL;
  if (tiles_m < 1 || tiles_n < 1 || group_m < 1 || (int64_t)tiles_m * tiles_n > (1 << 24)) return RL_ERR_SHAPE;
  const int n = launch_tiles(tiles_m, tiles_n);
  *workgroups = n;
  if (!tile) return RL_OK;
  for (int w = 0; w < n; ++w) {
    int tm = -1, tn = -1;
    if (!tile_of_block(w, tiles_m, tiles_n, group_m, by_share != 0, tm, tn)) tm = tn = -1;
    tile[2 * w] = tm; tile[2 * w + 1] = tn;
  }
  return RL_OK;
}

rl_status rl_debug_split_k(int32_t tiles_m, int32_t tiles_n, int32_t steps, int32_t slots, int64_t fill, int32_t* slices, int32_t* per,
                           int32_t* tile_rows) {
  if (!slices || !per || !tile_rows) return RL_ERR_NULL;
  if (tiles_m < 1 || tiles_n < 1 || (int64_t)tiles_m * tiles_n > (1 << 24) || steps < 0 || slots < 1 || fill < 0) return RL_ERR_SHAPE;
  const SplitK k = split_k_host(tiles_m * tiles_n, steps, slots, fill);
  *slices = k.slices; *per = k.per;
  *tile_rows = (int32_t)split_tile_rows(tiles_m, tiles_n, steps, slots);
  return RL_OK;
}

rl_status rl_workspace_bytes(const rl_batch* batch, const rl_params* params, int32_t want_backward, size_t* bytes) {
  if (!batch || !bytes) return RL_ERR_NULL;
  Plan p;
  rl_status st = make_plan(batch, params, want_backward != 0, p);
  if (st != RL_OK) return st;
  *bytes = p.total;
  return RL_OK;
}

rl_status rl_token_logprob(const rl_batch* b, float* logprob, float* lse, void* ws, size_t ws_bytes, void* stream) {
  return rl_token_logprob_tempered(b, 1.f, logprob, lse, ws, ws_bytes, stream);
}

rl_status rl_token_logprob_tempered(const rl_batch* b, float temperature, float* logprob, float* lse,
                                    void* ws, size_t ws_bytes, void* stream) {
  if (!b) return RL_ERR_NULL;
  if (!b->hidden || !b->weight || !b->token_ids || !b->mask || !b->cu_seqlens) return RL_ERR_NULL;
  if (!logprob && !lse) return RL_ERR_NULL;
  if (!(temperature > 0.f) || !(temperature <= 3.0e38f)) return RL_ERR_RANGE;
  Plan p;
  rl_status st = make_plan(b, nullptr, false, p);
  if (st != RL_OK) return st;
  p.inv_tau = 1.f / temperature;
  st = check_ws(ws, ws_bytes, p);
  if (st != RL_OK) return st;
  hipStream_t s = static_cast<hipStream_t>(stream);
  (void)hipGetLastError();
  Ptrs q = carve(ws, p);
  rl_outputs out{};
  out.logprob = logprob; out.lse = lse;
  PrepJob prep;
  run_prep(b, p, q, nullptr, out, AdvJob{}, prep, s);
  if (p.dtype == RL_BF16) run_forward<bf16_t>(b, p, q, logprob, lse, nullptr, nullptr, nullptr, false, prep, s);
  else run_forward<float>(b, p, q, logprob, lse, nullptr, nullptr, nullptr, false, prep, s);
  return hipGetLastError() == hipSuccess ? RL_OK : RL_ERR_HIP;
}

rl_status rl_policy_loss_fwd_bwd(const rl_batch* b, const rl_params* prm, int32_t objective, const rl_outputs* out,
                                 void* ws, size_t ws_bytes, void* stream) {
  if (!b || !prm || !out) return RL_ERR_NULL;
  if (!b->hidden || !b->weight || !b->token_ids || !b->mask || !b->cu_seqlens || !b->group_idx || !b->rewards ||
      !b->old_logprob || !b->ref_logprob || !out->loss)
    return RL_ERR_NULL;
  if (objective != RL_OBJ_GRPO && objective != RL_OBJ_FLOW) return RL_ERR_RANGE;
  if (objective == RL_OBJ_FLOW && !b->log_z) return RL_ERR_NULL;
  if (!(prm->clip_eps > 0.f && prm->clip_eps < 1.f)) return RL_ERR_RANGE;
  if (prm->adv_std_ddof != 0 && prm->adv_std_ddof != 1) return RL_ERR_RANGE;
  if (!(prm->adv_eps >= 0.f)) return RL_ERR_RANGE;
  if (!(prm->clip_eps_high >= 0.f)) return RL_ERR_RANGE;
  if ((prm->aggregation != RL_AGG_SEQUENCE && prm->aggregation != RL_AGG_TOKEN) ||
      (prm->ratio_level != RL_RATIO_TOKEN && prm->ratio_level != RL_RATIO_SEQUENCE) ||
      (prm->flow_weight_norm != RL_WNORM_SUM && prm->flow_weight_norm != RL_WNORM_MEAN))
    return RL_ERR_RANGE;
  if (prm->ratio_level == RL_RATIO_SEQUENCE && prm->aggregation == RL_AGG_TOKEN) return RL_ERR_RANGE;
  const bool bwd = out->d_hidden || out->d_weight;
  if (bwd && (!out->d_hidden || !out->d_weight)) return RL_ERR_NULL;
  Plan p;
  rl_status st = make_plan(b, prm, bwd, p, out);
  if (st != RL_OK) return st;
  st = check_ws(ws, ws_bytes, p);
  if (st != RL_OK) return st;
  hipStream_t s = static_cast<hipStream_t>(stream);
  (void)hipGetLastError();
  Ptrs q = carve(ws, p);

  const AdvJob adv{(p.P + kInitThreads / 64 - 1) / (kInitThreads / 64), b->rewards, b->group_idx, p.P, prm->adv_eps, prm->adv_std_ddof, q.adv, out->group_count};
  PrepJob prep;
  run_prep(b, p, q, b->group_idx, *out, adv, prep, s);

  if (p.stash) {
    run_fused(b, prm, objective, p, q, out, s);
    return hipGetLastError() == hipSuccess ? RL_OK : RL_ERR_HIP;
  }
  const bool fold = fold_combine(p);
  if (p.dtype == RL_BF16) run_forward<bf16_t>(b, p, q, out->logprob, out->lse, out->entropy, out->target_logit, out->target_col, false, prep, s);
  else run_forward<float>(b, p, q, out->logprob, out->lse, out->entropy, out->target_logit, out->target_col, fold, prep, s);

  bool prep_done = false;
  LossJob j = loss_job(b, prm, objective, p, q, out, nullptr);
  {
    ProfScope ps(RL_PROF_LOSS, s);
    j.finish_later = p.small_grads && p.B <= kFinishSeqs;
    if (fold) {
      j.comb = CombineJob{q.part, p.Tc, p.tiles_v, q.zy, q.row_map, q.ycol, q.lse_c, q.logp_c, out->lse, out->logprob, out->entropy, out->target_logit, out->target_col};
      loss_fold_kernel<<<p.B + (bwd ? (p.R + 3) / 4 : 0), kLossThreads, 0, s>>>(j, q.cpos, static_cast<float*>(out->d_hidden), p.R, p.H);
      prep_done = bwd;
    } else {
      prep_done = bwd && run_loss_prep(b, p, q, j, static_cast<float*>(out->d_hidden), s);
      if (!prep_done) seq_loss_kernel<<<p.B, kLossThreads, 0, s>>>(j);
    }
    run_finalize(j, s);
  }
  if (bwd) {
    if (p.dtype == RL_BF16) run_backward<bf16_t>(b, p, q, out->d_hidden, out->d_weight, prep_done, j, s);
    else run_backward<float>(b, p, q, out->d_hidden, out->d_weight, prep_done, j, s);
  }
  return hipGetLastError() == hipSuccess ? RL_OK : RL_ERR_HIP;
}

// ------------------------------------------------------------------ scoring call that allocates nothing
// The forward-only call with its workspace in a file-scope device array instead of a caller's buffer.  Every GPU the
// library runs on holds its own copy of the array at its own address; the host-side name of the array is only a handle
// for hipGetSymbolAddress, never a device address, so the address is looked up once per device and kept.
static __device__ __align__(256) unsigned char scratch[RL_STATIC_SCRATCH_BYTES];
constexpr int kMaxDevices = 64;
static void* g_scratch_ptr[kMaxDevices];
static std::mutex g_scratch_mutex;

static rl_status static_scratch(void** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return RL_ERR_HIP;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return RL_ERR_HIP;
    g_scratch_ptr[dev] = p;
  }
  *out = g_scratch_ptr[dev];
  return RL_OK;
}

rl_status rl_token_logprob_static(const rl_batch* b, float temperature, float* logprob, float* lse, void* stream) {
  if (!b) return RL_ERR_NULL;
  if (!b->hidden || !b->weight || !b->token_ids || !b->mask || !b->cu_seqlens) return RL_ERR_NULL;
  if (!logprob && !lse) return RL_ERR_NULL;
  if (!(temperature > 0.f) || !(temperature <= 3.0e38f)) return RL_ERR_RANGE;
  // the largest chunk (a power of two times 256 rows) whose plan fits the array; none fits: the batch is beyond the limit
  Plan p;
  bool fits = false;
  for (int tc = kDefaultChunkRows; tc >= 256 && !fits; tc >>= 1) {
    rl_params prm{};
    prm.chunk_rows = tc;
    const rl_status st = make_plan(b, &prm, false, p);
    if (st != RL_OK) return st;
    fits = p.total <= (size_t)RL_STATIC_SCRATCH_BYTES;
  }
  if (!fits) return RL_ERR_WORKSPACE;
  p.inv_tau = 1.f / temperature;
  void* ws = nullptr;
  const rl_status st = static_scratch(&ws);
  if (st != RL_OK) return st;
  hipStream_t s = static_cast<hipStream_t>(stream);
  (void)hipGetLastError();
  Ptrs q = carve(ws, p);
  rl_outputs out{};
  out.logprob = logprob; out.lse = lse;
  PrepJob prep;
  run_prep(b, p, q, nullptr, out, AdvJob{}, prep, s);
  if (p.dtype == RL_BF16) run_forward<bf16_t>(b, p, q, logprob, lse, nullptr, nullptr, nullptr, false, prep, s);
  else run_forward<float>(b, p, q, logprob, lse, nullptr, nullptr, nullptr, false, prep, s);
  return hipGetLastError() == hipSuccess ? RL_OK : RL_ERR_HIP;
}

// ------------------------------------------------------------------ log-Z head
static rl_status logz_check(int32_t P, int32_t H, int32_t M) {
  if (P < 1 || H < 1 || M < 1 || P > (1 << 20) || (int64_t)((M + 7) / 8) > 65535) return RL_ERR_SHAPE;
  return RL_OK;
}

rl_status rl_logz_head_workspace_bytes(int32_t P, int32_t H, int32_t M, size_t* bytes) {
  if (!bytes) return RL_ERR_NULL;
  rl_status st = logz_check(P, H, M);
  if (st != RL_OK) return st;
  *bytes = logz_plan(P, H, M).total;
  return RL_OK;
}

rl_status rl_logz_head_forward(const void* prompt_hidden, int32_t dtype, int64_t rows, int32_t H,
                               const int32_t* cu_prompt, int32_t P, const float* W1, const float* b1,
                               const float* w2, const float* b2, int32_t M, float* log_z,
                               void* ws, size_t ws_bytes, void* stream) {
  if (!prompt_hidden || !cu_prompt || !W1 || !b1 || !w2 || !b2 || !log_z) return RL_ERR_NULL;
  if (dtype != RL_F32 && dtype != RL_BF16) return RL_ERR_DTYPE;
  rl_status st = logz_check(P, H, M);
  if (st != RL_OK) return st;
  if (rows < 0) return RL_ERR_SHAPE;
  const LogzPlan q = logz_plan(P, H, M);
  if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255) || ws_bytes < q.total) return RL_ERR_WORKSPACE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  (void)hipGetLastError();
  unsigned char* w = static_cast<unsigned char*>(ws);
  float* pooled = (float*)(w + q.off_pooled); float* a = (float*)(w + q.off_a); float* g = (float*)(w + q.off_g);
  // (one float per prompt and workgroup of the hidden layer, of the P M there are; with fewer than 32 units the counts might not fit)
  int* done = (int*)(w + q.off_part); float* part_z = P <= 16 && M >= 32 && M <= kLogzSumUnits ? (float*)(w + q.off_part) + (P + 15) / 16 : nullptr;
  const bool vec_x = H % (dtype == RL_BF16 ? 8 : 4) == 0 && reinterpret_cast<uintptr_t>(prompt_hidden) % 16 == 0;
  auto pool = [&](auto kern, auto* X, int cols) { kern<<<dim3(P, (H + cols - 1) / cols), 512, 0, s>>>(X, rows, H, cu_prompt, pooled, done); };
  if (dtype == RL_BF16) {
    const bf16_t* X = static_cast<const bf16_t*>(prompt_hidden);
    if (vec_x) pool(logz_pool_kernel<bf16_t, 8>, X, 128); else pool(logz_pool_kernel<bf16_t, 1>, X, 64);
  } else {
    const float* X = static_cast<const float*>(prompt_hidden);
    if (vec_x) pool(logz_pool_kernel<float, 4>, X, 64); else pool(logz_pool_kernel<float, 1>, X, 64);
  }
  const dim3 gh((M + 15) / 16, (P + 15) / 16);
  if (H % 4 == 0 && reinterpret_cast<uintptr_t>(W1) % 16 == 0) logz_hidden_kernel<true><<<gh, 64 * kLogzWaves, 0, s>>>(W1, b1, pooled, P, H, M, a, g, w2, b2, part_z, done, log_z);
  else logz_hidden_kernel<false><<<gh, 64 * kLogzWaves, 0, s>>>(W1, b1, pooled, P, H, M, a, g, w2, b2, part_z, done, log_z);
  if (!part_z) logz_out_kernel<<<P, M > kLogzOutThreads ? kLogzOutThreads : 256, 0, s>>>(g, w2, b2, M, log_z);
  return hipGetLastError() == hipSuccess ? RL_OK : RL_ERR_HIP;
}

rl_status rl_logz_head_backward(const float* d_log_z, int32_t P, int32_t H, int32_t M, const float* w2,
                                float* dW1, float* db1, float* dw2, float* db2,
                                void* ws, size_t ws_bytes, void* stream) {
  if (!d_log_z || !w2 || !dW1 || !db1 || !dw2 || !db2) return RL_ERR_NULL;
  rl_status st = logz_check(P, H, M);
  if (st != RL_OK) return st;
  const LogzPlan q = logz_plan(P, H, M);
  if (!ws || (reinterpret_cast<uintptr_t>(ws) & 255) || ws_bytes < q.total) return RL_ERR_WORKSPACE;
  hipStream_t s = static_cast<hipStream_t>(stream);
  (void)hipGetLastError();
  unsigned char* w = static_cast<unsigned char*>(ws);
  float* pooled = (float*)(w + q.off_pooled); float* a = (float*)(w + q.off_a); float* g = (float*)(w + q.off_g);
  if (H % 4 == 0 && reinterpret_cast<uintptr_t>(dW1) % 16 == 0)
    (logz_nontemporal(M, H, dW1) ? logz_bwd_kernel<4, true> : logz_bwd_kernel<4, false>)<<<dim3((M + 7) / 8, (H + 1023) / 1024), 256, 0, s>>>(d_log_z, a, g, w2, pooled, P, M, H, dW1, db1, dw2, db2);
  else
    logz_bwd_kernel<1, false><<<dim3((M + 7) / 8, (H + 255) / 256), 256, 0, s>>>(d_log_z, a, g, w2, pooled, P, M, H, dW1, db1, dw2, db2);
  return hipGetLastError() == hipSuccess ? RL_OK : RL_ERR_HIP;
}

// ------------------------------------------------------------------ residual-VQ encode
static rl_status rvq_check(int32_t G, int64_t L, int32_t D, int32_t N, int32_t S) {
  if (G < 1 || G > 65535 || L < 1 || L > ((int64_t)1 << 24) || N < 1 || S < 1) return RL_ERR_SHAPE;
  if (D != kRvqD || (S % kRvqChunk) != 0 || S > 65536 || (int64_t)N * S > ((int64_t)1 << 26)) return RL_ERR_SHAPE;
  return RL_OK;
}

// Whether more than 16 vectors of a group are encoded faster by the kernel that takes 32 of them per workgroup (few) than by the one that takes 256 or 512 (many).  Both keep
// one workgroup on a CU (the second kind of `many` at most two, which slow each other down), 32 on an accelerator die, which the workgroups of a group share: what a launch takes is
// its rounds of workgroups times what one takes to start and per stage.  Now and then `many` looks at a whole stage again, some 50 us each time; that depends on the vectors,
// is rarer in the first two stages, for which nothing is added, and is counted by its mean over N(0, 1) vectors: past 20 thousand decisions more than half of the calls have one.
// Fitted to 1800 calls of 1 to 4096 groups of 17 to 4096 vectors, 1 to 64 stages of 64 to 1024 entries, of which it takes 0.9 % more than the faster kernel would; of 1600 others
// 1.1 %, at worst 2.0 times as long where the inputs need a second look, 1.6 times where they need none.  (Without the cost of a start 3.3 % and 6.0 times.)
// us, few and many (without such a stage / mean of eight inputs):
//   2 stages of 64:   512 groups of 256 172, 31 / 32;  264 of 512 179, 53 / 53        1 of 512: 100 groups of 512 86, 33 / 34
//   4 of 1024:  37 of 512 163, 135 / 136      8 of 64:  128 of 256 124, 54 / 55;  8 of 1024 36, 77 / 78      10 of 256:  12 of 17 47, 75 / 86
//   16 of 512:  264 of 64 356, 292 / 342;  40 of 300 231, - / 424;  256 of 96 360, - / 332      40 of 256:  37 of 17 166, 367 / 395      56 of 1024:  160 of 50 1365, - / 1265
static bool rvq_few_is_faster(int64_t G, int64_t L, int N, int S) {
  const int64_t die = (G + 7) / 8, rows = L > 256 ? 512 : 256;
  const double rounds = (double)(((L + 31) / 32 * die + 31) / 32), n = (double)((L + rows - 1) / rows * die);       // few; workgroups of `many` on a die
  const double few = 4.0 + rounds * (4.5 + N * (2.2 + 0.0094 * S));
  const double share = n <= 32 ? 1.0 : rows == 512 ? 1.08 * (double)(((int64_t)n + 31) / 32) : n <= 64 ? 1.5 + 0.5 * (n - 32) / 32 : 0.85 * n / 32;
  const double d = N > 2 ? (double)G * L * (N - 2) : 0.0;
  return few <= 6.0 + share * (13.0 + N * (rows == 512 ? 5.5 + 0.0255 * S : 3.8 + 0.0177 * S)) + 36.0 * d / (d + 2e4);
}

rl_status rl_rvq_codebook_norms(const void* codebooks, int32_t G, int32_t N, int32_t S, int32_t D, float* norms, void* stream) {
  if (!codebooks || !norms) return RL_ERR_NULL;
  rl_status st = rvq_check(G, 1, D, N, S);
  if (st != RL_OK) return st;
  if (reinterpret_cast<uintptr_t>(codebooks) & 15) return RL_ERR_SHAPE;
  (void)hipGetLastError();
  const int64_t entries = (int64_t)G * N * S;
  rvq_norms_kernel<<<(unsigned)((entries + 255) / 256), 256, 0, static_cast<hipStream_t>(stream)>>>(static_cast<const bf16_t*>(codebooks), entries, norms);
  return hipGetLastError() == hipSuccess ? RL_OK : RL_ERR_HIP;
}

rl_status rl_rvq_encode(const void* vectors, const void* codebooks, const float* norms, int32_t G, int64_t L, int32_t D,
                        int32_t N, int32_t S, int32_t* codes, void* residual, void* stream) {
  return rl_rvq_encode_counted(vectors, codebooks, norms, G, L, D, N, S, codes, residual, nullptr, stream);
}

rl_status rl_rvq_encode_counted(const void* vectors, const void* codebooks, const float* norms, int32_t G, int64_t L, int32_t D,
                                int32_t N, int32_t S, int32_t* codes, void* residual, int32_t* n_exact, void* stream) {
  if (!vectors || !codebooks || !norms || !codes) return RL_ERR_NULL;
  rl_status st = rvq_check(G, L, D, N, S);
  if (st != RL_OK) return st;
  if ((reinterpret_cast<uintptr_t>(vectors) | reinterpret_cast<uintptr_t>(codebooks) | reinterpret_cast<uintptr_t>(residual)) & 15) return RL_ERR_SHAPE;
  (void)hipGetLastError();
  hipStream_t s = static_cast<hipStream_t>(stream);
  // Few vectors: a kernel that reads each codebook once for 16 or 32 of them and scores nothing else (norms 16 bytes at a time).  Up to 16 vectors of
  // a group it is the faster one whatever the number of groups; with more its workgroups read the codebook again, and the cheaper one is taken, see rvq_few_is_faster.
  const int nv = L <= 16 ? 1 : 2;
  const bool few = L <= 16 || rvq_few_is_faster(G, L, N, S);
  if (few && S <= rvq_few_max_entries(nv) && reinterpret_cast<uintptr_t>(norms) % 16 == 0) {
    const unsigned n = (unsigned)((L + 16 * nv - 1) / (16 * nv) * (8 * (((int64_t)G + 7) / 8)));
    auto kern = nv == 1 ? rvq_few_kernel<1> : rvq_few_kernel<2>;
    kern<<<n, 320, 0, s>>>(static_cast<const bf16_t*>(vectors), static_cast<const bf16_t*>(codebooks), norms, G, (int)L, N, S, codes,
                           static_cast<bf16_t*>(residual), n_exact);
    return hipGetLastError() == hipSuccess ? RL_OK : RL_ERR_HIP;
  }
  const int kw = L > 256 ? 8 : 4;                                   // wavefronts per workgroup, 64 vectors each
  const int64_t n_wg = (L + 64 * kw - 1) / (64 * kw) * (8 * (((int64_t)G + 7) / 8));
  if (n_wg > 0x7fffffff) return RL_ERR_RANGE;
  if (kw == 8)
    rvq_encode_kernel<8><<<(unsigned)n_wg, 512, 0, s>>>(static_cast<const bf16_t*>(vectors), static_cast<const bf16_t*>(codebooks), norms,
                                                        G, (int)L, N, S, codes, static_cast<bf16_t*>(residual), n_exact);
  else
    rvq_encode_kernel<4><<<(unsigned)n_wg, 256, 0, s>>>(static_cast<const bf16_t*>(vectors), static_cast<const bf16_t*>(codebooks), norms,
                                                        G, (int)L, N, S, codes, static_cast<bf16_t*>(residual), n_exact);
  return hipGetLastError() == hipSuccess ? RL_OK : RL_ERR_HIP;
}

}  // extern "C"
