// Lossless acceptance over the per-node logits of a verified draft tree
// (arXiv 2408.15562, Preliminaries, validation phase: strict comparison of the
// tree with the target's results, a differing token dropped with all its
// descendants; Experiments "Settings": temperature 0 and 1, acceptance not
// relaxed). gfx950 (CDNA4) only.
//
// Two kernels per call. The first streams the [B*N, V] fp32 logits once, 16 bytes
// per lane, one workgroup per (row, chunk of 1024..8192 entries), and leaves per-chunk
// statistics: (max, first index of max) for greedy, (max, fp64 sum of
// exp((l-max)/T)) for sampling. The second, one workgroup per sequence, merges the
// chunk statistics of every row at once, walks the tree with wavefront ballots
// out of LDS and, for sampling, draws the last token by an inverse-CDF search that
// descends chunk -> thread segment -> element. (Large sampling calls: see kInnerFirst; greedy calls of small vocabularies, one
// launch: see accept_greedy_small_kernel.)
#include <hip/hip_runtime.h>
#include <algorithm>
#include <stdint.h>

#include <mutex>

#include "fspad.h"
#include "exp_nonpos.h"
#include "greedy_walk.h"

namespace {

using fspad_detail::exp_nonpos;
using fspad_detail::exp_nonpos_table;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4), aligned(4))) float f32x4_at_4;   // rows of any alignment: the load takes it

constexpr int kThreads = 256;
constexpr int kMinChunk = 1024;           // logits per workgroup of the streaming kernel: 1024 .. 8192,
constexpr int kMaxChunk = 8192;           // chosen per call so that small problems still fill the chip
constexpr int kMaxPerThread = kMaxChunk / kThreads;  // 32
constexpr int kNone = 0x7fffffff;

struct AcceptParams {
  const float* logits;
  int64_t row_stride;
  const int32_t* draft_tokens;
  const int32_t* parent;
  const int32_t* n_nodes;
  const float* uniforms;
  int32_t* path;
  int32_t* path_len;
  int32_t* tokens;
  int32_t* n_tokens;
  float* part_max;     // [rows][chunks]
  int32_t* part_idx;   // greedy  [rows][chunks]
  double* part_sum;    // sampling [rows][chunks]
  double inv_temperature;
  double table_scale;  // of exp_nonpos_table: 256 log2(e) / T
  int32_t B, Nmax, V, n_chunks;
  int32_t chunk;       // logits per (row, chunk) workgroup: 256 * PT
  uint32_t* clear_words;   // words this launch sets to zero for the kernel behind it (may be null)
  int32_t clear_count;
  // a second logit array of the same shape for the same launch (grid.z = 2; sampling statistics only), or null
  const float* logits2;
  float* part_max2;
  double* part_sum2;
  int32_t rows;        // kAllRows, ...: which rows' statistics this launch forms (sampling)
};

constexpr int32_t kAllRows = 0;
constexpr int32_t kInnerRows = 1;   // nodes that have children

// Has a node a child among the n nodes of its tree (n <= Nmax), as the walk would test it? my_parent: of the node that is this
// lane's number. (the same answer in every lane)
__device__ __forceinline__ int lane_parent(const int32_t* parent, int Nmax) { return parent[min((int)(threadIdx.x & 63), Nmax - 1)]; }
__device__ __forceinline__ bool has_child(int my_parent, int n, int node) {
  const int lane = threadIdx.x & 63;
  return __ballot(my_parent == node && lane > 0 && lane < n) != 0ull;
}

// Inclusive running sum over the 64 lanes of a wavefront, lane order, with data-parallel-primitive moves
// (no LDS round trips): four shifts inside each row of 16 lanes (a lane without a source adds 0), then the
// last lane of row 0 / 2 onto rows 1 / 3 and lane 31 onto rows 2 and 3.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_take(double v) {
  const unsigned long long bits = __builtin_bit_cast(unsigned long long, v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)bits, CTRL, ROW_MASK, 0xf, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(bits >> 32), CTRL, ROW_MASK, 0xf, true);
  return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double wave_running_sum(double v) {
  v += dpp_take<0x111, 0xf>(v);   // row_shr:1
  v += dpp_take<0x112, 0xf>(v);   // row_shr:2
  v += dpp_take<0x114, 0xf>(v);   // row_shr:4
  v += dpp_take<0x118, 0xf>(v);   // row_shr:8
  v += dpp_take<0x142, 0xa>(v);   // row_bcast:15 onto rows 1 and 3
  v += dpp_take<0x143, 0xc>(v);   // row_bcast:31 onto rows 2 and 3
  return v;
}

__device__ __forceinline__ float clean(float x) { return (x != x) ? -INFINITY : x; }  // NaN ranks lowest

// The largest of the numbers among x (-infinity where there is none): two at a time, NaNs dropped by the instruction. (With the IEEE bit of the mode
// register, which kernels start with and the compiler counts on, a signalling NaN would come back as a quiet one, and the compiler puts an
// instruction in front of every operand to make sure that there is none. The bit is off for these instructions alone: m ties them, first to last, to the
// statements that clear and set it; what else the compiler moves in between are loads, conversions and integers.)
template <int N>
__device__ __forceinline__ float max_of_numbers(const float (&x)[N]) {
  static_assert(N % 2 == 0, "pairs");
  float m;
  asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 9, 1), 0\n\tv_mov_b32 %0, 0xff800000" : "=v"(m));
#pragma unroll
  for (int k = 0; k < N; k += 2) asm("v_max3_f32 %0, %0, %1, %2" : "+v"(m) : "v"(x[k]), "v"(x[k + 1]));
  asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 9, 1), 1" : "+v"(m));
  return m;
}

// The largest m of a wavefront's lanes, in every lane.
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_larger(float m) {
  const int bits = __builtin_bit_cast(int, m);
  return fmaxf(m, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(bits, bits, CTRL, ROW_MASK, 0xf, false)));
}
__device__ __forceinline__ float wave_max(float m) {
  m = dpp_larger<0x111, 0xf>(m);
  m = dpp_larger<0x112, 0xf>(m);
  m = dpp_larger<0x114, 0xf>(m);
  m = dpp_larger<0x118, 0xf>(m);
  m = dpp_larger<0x142, 0xa>(m);
  m = dpp_larger<0x143, 0xc>(m);
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, m), 63));
}

// (value, index) with "larger value, then lower index" order
__device__ __forceinline__ void take_better(float& v, int& i, float ov, int oi) {
  if (ov > v || (ov == v && oi < i)) { v = ov; i = oi; }
}

// The best of the 64 lanes in that order, in every lane (v is no NaN): the largest value, and nearly always one lane
// that has it. (Values and indices exchanged step by step are twelve trips through LDS, some 800 clocks.)
__device__ __forceinline__ void wave_best(float& v, int& i) {
  const float top = wave_max(v);
  const unsigned long long at = __ballot(v == top);
  int first = __builtin_amdgcn_readlane(i, __builtin_ctzll(at));
  if ((at & (at - 1)) != 0ull) {
    int x = v == top ? i : kNone;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) x = min(x, __shfl_xor(x, off));
    first = x;
  }
  v = top;
  i = first;
}

// ------------------------------------------------------------------------------------------------
// Streaming pass. MODE 0: greedy (max, argmax). MODE 1: sampling (max, sum of exp).
// Sixteen bytes per lane and load whatever the rows' alignment (4 bytes at least): entry by entry, as rows that are not 16-byte aligned were
// read before, the texture path takes four times the requests. us a call, entry by entry -> so: 3 x 60 rows of 151001, sampling 43.6 -> 33.8,
// greedy 31.7 -> 24.9, sampled drafts 68.5 -> 50.9; 8 x 60 rows of 50257 41.7 -> 31.1, 30.6 -> 21.0, 66.4 -> 49.1 (with half the instructions a weight).
template <int MODE, int PT>
__global__ __launch_bounds__(kThreads) void accept_rows_kernel(const AcceptParams p) {
  constexpr int kChunk = kThreads * PT;
  constexpr int kPerThread = PT;
  __shared__ float sh_max[4];
  __shared__ int sh_idx[4];
  __shared__ double sh_sum[4];
  __shared__ double exp2_table[fspad_detail::kExp2Entries];
  static_assert(fspad_detail::kExp2Entries == kThreads, "an entry a thread");
  const int row = blockIdx.y, chunk = blockIdx.x;
  const int b = row / p.Nmax, node = row - b * p.Nmax;
  // (asked for together with the tree's size: behind it the first logits were a trip later)
  const int my_parent = MODE == 1 ? lane_parent(p.parent + (int64_t)b * p.Nmax, p.Nmax) : -1;
  if (row == 0 && chunk == 0)
    for (int i = threadIdx.x; i < p.clear_count; i += kThreads) p.clear_words[i] = 0u;
  const int n = p.n_nodes[b];
  if (node >= n) return;  // rows of unused tree slots are never read
  const bool second = blockIdx.z != 0;
  if (MODE == 1 && p.rows == kInnerRows && !has_child(my_parent, min(n, p.Nmax), node)) return;
  const float* rp = (second ? p.logits2 : p.logits) + (int64_t)row * p.row_stride;
  float* const part_max = second ? p.part_max2 : p.part_max;
  double* const part_sum = second ? p.part_sum2 : p.part_sum;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int base = chunk * kChunk;
  const double root = MODE == 1 ? fspad_detail::kExp2Table[tid] : 0.0;

  float x[kPerThread];
#pragma unroll
  for (int k = 0; k < kPerThread / 4; ++k) {
    const int e0 = base + (k * kThreads + tid) * 4;
    if (e0 + 3 < p.V) {
      const f32x4_at_4 v = *reinterpret_cast<const f32x4_at_4*>(rp + e0);
#pragma unroll
      for (int j = 0; j < 4; ++j) x[4 * k + j] = MODE == 1 ? v[j] : clean(v[j]);   // (sampling: a NaN is dropped where it is used)
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) x[4 * k + j] = (e0 + j < p.V) ? (MODE == 1 ? rp[e0 + j] : clean(rp[e0 + j])) : -INFINITY;
    }
  }

  const int64_t slot = (int64_t)row * p.n_chunks + chunk;
  if (MODE == 1) {
    exp2_table[tid] = root;
    __syncthreads();
    // sampling: each wavefront sums exp((x - its own max)/T) over its entries as soon as they arrive (fp64, no waiting for the rest
    // of the workgroup); the wavefronts' (max, sum) pairs are then merged into the chunk's: sum_c = sum_w sum_w * exp((max_w - max_c)/T).
    // (A maximum and a weight of its own for every thread, with exchanges through LDS, was a sixth of the instructions.)
    const float mw = wave_max(max_of_numbers(x));
    double st = 0.0;
    if (mw > -INFINITY) {
      const double mwd = (double)mw;
#pragma unroll
      for (int k = 0; k < kPerThread; ++k) st += exp_nonpos_table((double)x[k] - mwd, p.table_scale, exp2_table);
    }
    st = wave_running_sum(st);
    if (lane == 63) { sh_max[wave] = mw; sh_sum[wave] = st; }
    __syncthreads();
    if (tid < 4) {
      const float own = sh_max[tid];
      const float mc = fmaxf(fmaxf(sh_max[0], sh_max[1]), fmaxf(sh_max[2], sh_max[3]));
      double sum = own > -INFINITY ? sh_sum[tid] * exp_nonpos(((double)own - (double)mc) * p.inv_temperature) : 0.0;
      sum += __shfl_xor(sum, 1);
      sum += __shfl_xor(sum, 2);
      if (tid == 0) { part_max[slot] = mc; part_sum[slot] = sum; }
    }
    return;
  }

  float best = -INFINITY;
  int idx = kNone;
#pragma unroll
  for (int k = 0; k < kPerThread / 4; ++k)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (x[4 * k + j] > best) { best = x[4 * k + j]; idx = base + (k * kThreads + tid) * 4 + j; }

  // workgroup (max, index): wavefront butterflies, then 4 partials through LDS
  wave_best(best, idx);
  if (lane == 0) { sh_max[wave] = best; sh_idx[wave] = idx; }
  __syncthreads();
  best = sh_max[0]; idx = sh_idx[0];
#pragma unroll
  for (int w = 1; w < 4; ++w) take_better(best, idx, sh_max[w], sh_idx[w]);
  if (tid == 0) { part_max[slot] = best; p.part_idx[slot] = idx; }
}

// ------------------------------------------------------------------------------------------------
// Greedy: merge chunk argmaxes per node, then wavefront 0 descends while a child carries the
// target's token.
__global__ __launch_bounds__(kThreads) void accept_greedy_walk_kernel(const AcceptParams p) {
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n = p.n_nodes[b];
  const int64_t o = (int64_t)b * p.Nmax;
  // the tree itself does not depend on the logits: wavefront 0 asks for it before anything else
  int my_par = -2, my_tok = -1;
  if (wave == 0 && lane < n) {
    my_par = p.parent[o + lane];
    my_tok = p.draft_tokens[o + lane];
  }
  // thread (node = lane, quarter = wave) scans every 4th chunk entry of its node, eight loads in
  // flight at a time; the four quarters of a node meet in LDS (no lane exchange needed)
  __shared__ float q_best[4][FSPAD_MAX_NODES];
  __shared__ int q_idx[4][FSPAD_MAX_NODES];
  {
    float best = -INFINITY;
    int idx = kNone;
    if (lane < n) {
      const int64_t slot0 = (o + lane) * p.n_chunks;
      for (int c0 = wave; c0 < p.n_chunks; c0 += 32) {
        float v[8];
        int ix[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          const int c = c0 + 4 * k;
          v[k] = c < p.n_chunks ? p.part_max[slot0 + c] : -INFINITY;
          ix[k] = c < p.n_chunks ? p.part_idx[slot0 + c] : kNone;
        }
#pragma unroll
        for (int k = 0; k < 8; ++k) take_better(best, idx, v[k], ix[k]);
      }
    }
    q_best[wave][lane] = best;
    q_idx[wave][lane] = idx;
  }
  __syncthreads();
  if (wave != 0) return;
  float best = q_best[0][lane];
  int idx = q_idx[0][lane];
#pragma unroll
  for (int w = 1; w < 4; ++w) take_better(best, idx, q_best[w][lane], q_idx[w][lane]);
  idx = idx == kNone ? 0 : idx;  // a row with nothing above -inf: token 0
  fspad_detail::greedy_descend(idx, n, p.Nmax, lane, o, b, my_par, my_tok, p.path, p.tokens, p.path_len, p.n_tokens);
}

// The same in one launch where a row has up to kSmallVocab logits: sixteen to a lane, a wavefront for up to four rows, whose loads are
// under way together and with the tree's. (Four rows of sixteen are 64 of the 128 registers that a wavefront of sixteen can have: longer
// rows would need a loop. Rows of unused tree slots are not read: waiting for the number of nodes first costs 0.13 us.) Such a call is
// launches and trips to memory, us by two launches / so, rows of 1000, a call's share of a graph of fifty: 1 x 20 5.05 / 3.14, 1 x 26 5.35 / 3.58, 1 x 36
// 5.27 / 4.00, 1 x 48 5.47 / 4.93, 4 x 60 5.63 / 5.46, 16 x 60 6.14 / 5.63, 25 x 48 8.29 / 5.32, 200 x 20 12.9 / 3.7. One workgroup per sequence takes longer the more rows it
// has, two launches the more there are in all: 1 x 64 5.47 / 5.75, 8 x 64 5.69 / 6.00, 20 x 64 8.19 / 6.08, 64 x 64 13.1 / 6.1. Rows that are not aligned are read entry
// by entry here, 16 bytes a lane by two launches, so the line lies lower for few sequences (one launch / two, rows of 997 and of 1000 a stride of 1001 apart): 1 x 48 0.95 and 0.94, 4 x 48
// 0.94 and 0.96, 1 x 56 1.04 and 1.04, 2 x 60 1.04 and 1.03, 4 x 60 1.01 and 1.03, 8 x 60 0.99 and 1.02, 16 x 52 0.93 and 0.95, 16 x 60 0.94 and 0.98.
constexpr int kSmallVocab = 1024;
bool takes_small_greedy(int32_t B, int32_t Nmax, int32_t V, bool aligned) {
  const int64_t rows = (int64_t)B * Nmax;
  return V <= kSmallVocab && (Nmax <= 48 || (Nmax <= 60 && (aligned || rows >= 480)) || rows >= 1200);
}
constexpr int kSmallWaves = 16;
constexpr int kSmallRows = FSPAD_MAX_NODES / kSmallWaves;   // per wavefront
template <bool VEC>
__global__ __launch_bounds__(64 * kSmallWaves) void accept_greedy_small_kernel(const AcceptParams p) {
  constexpr int kPieces = kSmallVocab / 256;   // of four logits a lane
  __shared__ int amax[FSPAD_MAX_NODES];
  const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int64_t o = (int64_t)b * p.Nmax;
  const int V = p.V;
  const int n = p.n_nodes[b];
  int my_par = -2, my_tok = -1;
  if (wave == 0 && lane < min(n, p.Nmax)) {
    my_par = p.parent[o + lane];
    my_tok = p.draft_tokens[o + lane];
  }
  auto entry = [&](int k, int j) { return VEC ? (k * 64 + lane) * 4 + j : (4 * k + j) * 64 + lane; };   // (increasing in every lane)
  float x[kSmallRows][4 * kPieces];
#pragma unroll
  for (int r = 0; r < kSmallRows; ++r) {
    if (wave + r * kSmallWaves >= min(n, p.Nmax)) break;   // rows of unused tree slots are never read
    const float* row = p.logits + (o + wave + r * kSmallWaves) * p.row_stride;
#pragma unroll
    for (int k = 0; k < kPieces; ++k) {
      if constexpr (VEC) {   // (V is a multiple of four; a piece past the end: the row's first)
        const f32x4 v = *reinterpret_cast<const f32x4*>(row + (entry(k, 0) < V ? entry(k, 0) : 0));
        x[r][4 * k] = v[0]; x[r][4 * k + 1] = v[1]; x[r][4 * k + 2] = v[2]; x[r][4 * k + 3] = v[3];
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) x[r][4 * k + j] = row[min(entry(k, j), V - 1)];
      }
    }
  }
#pragma unroll
  for (int r = 0; r < kSmallRows; ++r) {
    const int node = wave + r * kSmallWaves;
    if (node >= n || node >= p.Nmax) break;
    float best = -INFINITY;
    int idx = kNone;
#pragma unroll
    for (int k = 0; k < kPieces; ++k)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int e = entry(k, j);
        if (e < V && x[r][4 * k + j] > best) { best = x[r][4 * k + j]; idx = e; }   // (a NaN is above nothing)
      }
    wave_best(best, idx);
    if (lane == 0) amax[node] = idx == kNone ? 0 : idx;   // a row with nothing above -inf: token 0
  }
  __syncthreads();
  if (wave != 0) return;
  fspad_detail::greedy_descend(amax[lane], n, p.Nmax, lane, o, b, my_par, my_tok, p.path, p.tokens, p.path_len, p.n_tokens);
}

// ------------------------------------------------------------------------------------------------
// The sampling walk runs with 1024 threads: its code runs once per call, so what it costs is the
// longest chain of dependent fp64 instructions in any one thread and the number of instruction lines
// fetched (cold at every launch), and both shrink when the same arithmetic is spread over more lanes.
constexpr int kWalkThreads = 1024;
constexpr int kWalkWaves = kWalkThreads / 64;

// Last step of the sampling pass: the workgroup draws the token at which the running sum of the
// residual weights of one chunk crosses `target`. Thread k owns E consecutive entries; their
// weights are formed once and stay in registers, so the thread that owns the crossing finds it
// without touching memory again. If rounding leaves no crossing, the last entry with mass is taken.
struct DrawArgs {
  const float* rp;          // the row
  int first, V;             // first entry of the chunk, vocabulary size
  double M, target, inv_temperature;
  const int* rej_tok;       // tokens rejected at this node: zero weight
  int nrej;
  double* scan_part;        // LDS scratch: kWalkWaves doubles
  int* sh_wave;             // LDS scratch: 2 * kWalkWaves ints
  int32_t* out;
};

template <int E>
__device__ __forceinline__ void draw_in_chunk(const DrawArgs& a) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int e0 = a.first + tid * E;
  float lx[E];
  if constexpr (E % 4 == 0) {
#pragma unroll
    for (int k = 0; k < E / 4; ++k) {
      const int e = e0 + 4 * k;
      if (e + 3 < a.V) {
        const f32x4_at_4 v = *reinterpret_cast<const f32x4_at_4*>(a.rp + e);
        lx[4 * k] = v[0]; lx[4 * k + 1] = v[1]; lx[4 * k + 2] = v[2]; lx[4 * k + 3] = v[3];
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) lx[4 * k + j] = (e + j < a.V) ? a.rp[e + j] : NAN;
      }
    }
  } else {
#pragma unroll
    for (int j = 0; j < E; ++j) lx[j] = (e0 + j < a.V) ? a.rp[e0 + j] : NAN;
  }
  unsigned gone = 0u;   // bit j: entry e0 + j was rejected at this node and has left the residual
  for (int k = 0; k < a.nrej; ++k) {
    const unsigned r = (unsigned)(a.rej_tok[k] - e0);
    if (r < (unsigned)E) gone |= 1u << r;
  }
  double w[E];
  double local = 0.0;
  int last_here = -1;
#pragma unroll
  for (int j = 0; j < E; ++j) {
    double wj = 0.0;
    if (lx[j] == lx[j] && !((gone >> j) & 1u))   // not NaN (entries past the vocabulary were loaded as NaN)
      wj = exp_nonpos(((double)lx[j] - a.M) * a.inv_temperature);
    w[j] = wj;
    local += wj;
    if (wj > 0.0) last_here = e0 + j;
  }
  const double incl = wave_running_sum(local);
  if (lane == 63) a.scan_part[wave] = incl;
  __syncthreads();
  double wave_base = 0.0;   // the wavefronts before this one, in order (every partial is read: the loads go out together)
#pragma unroll
  for (int v = 0; v < kWalkWaves; ++v) {
    const double part = a.scan_part[v];
    if (v < wave) wave_base += part;
  }
  // the owner is the first thread whose inclusive running sum exceeds the target: first lane of a
  // wavefront by ballot, first wavefront through LDS (one slot each: no two lanes meet on an address)
  const double inclusive = wave_base + incl;
  const unsigned long long hits = __ballot(inclusive > a.target && local > 0.0);
  int last_wave = last_here;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) last_wave = max(last_wave, __shfl_xor(last_wave, off));
  if (lane == 0) {
    a.sh_wave[wave] = hits ? wave * 64 + (__ffsll(hits) - 1) : kNone;
    a.sh_wave[kWalkWaves + wave] = last_wave;
  }
  __syncthreads();
  int owner = kNone, last_any = -1;
#pragma unroll
  for (int v = 0; v < kWalkWaves; ++v) {
    owner = min(owner, a.sh_wave[v]);
    last_any = max(last_any, a.sh_wave[kWalkWaves + v]);
  }
  if (owner == kNone) {  // rounding left no crossing: the last entry with mass
    if (tid == 0) *a.out = last_any < 0 ? 0 : last_any;
    return;
  }
  if (tid == owner) {
    double run = inclusive - local;
    int pick = last_here;  // if rounding hides the crossing inside the segment: its last entry with mass
    bool done = false;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      run += w[j];
      if (!done && run > a.target) { pick = e0 + j; done = true; }
    }
    *a.out = pick;
  }
}

// A chunk's statistics by the walk's workgroup, as the first pass forms them but for the order of the sum. wave_max, wave_sum: LDS,
// one slot a wavefront.
__device__ __forceinline__ void form_chunk(const float* rp, int base, int V, double table_scale, const double* exp2_table,
                                           float* wave_max, double* wave_sum, float* out_max, double* out_sum) {
  constexpr int E = kMaxChunk / kWalkThreads;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  float x[E];
#pragma unroll
  for (int k = 0; k < E / 4; ++k) {
    const int e0 = base + (k * kWalkThreads + tid) * 4;
    if (e0 + 3 < V) {
      const f32x4_at_4 v = *reinterpret_cast<const f32x4_at_4*>(rp + e0);
#pragma unroll
      for (int j = 0; j < 4; ++j) x[4 * k + j] = v[j];
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) x[4 * k + j] = rp[min(e0 + j, V - 1)];
    }
  }
  float mt = -INFINITY;
#pragma unroll
  for (int k = 0; k < E; ++k) {
    x[k] = base + ((k >> 2) * kWalkThreads + tid) * 4 + (k & 3) < V ? clean(x[k]) : -INFINITY;
    mt = fmaxf(mt, x[k]);
  }
  float mc = mt;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mc = fmaxf(mc, __shfl_xor(mc, off));
  if (lane == 0) wave_max[wave] = mc;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kWalkWaves; ++w) mc = fmaxf(mc, wave_max[w]);
  double sum = 0.0;
  if (mc > -INFINITY) {
#pragma unroll
    for (int k = 0; k < E; ++k) sum += exp_nonpos_table((double)x[k] - (double)mc, table_scale, exp2_table);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
  if (lane == 0) wave_sum[wave] = sum;
  __syncthreads();
  if (tid == 0) {
    double total = 0.0;
#pragma unroll
    for (int w = 0; w < kWalkWaves; ++w) total += wave_sum[w];
    *out_max = mc;
    *out_sum = total;
  }
}

// Sampling. Everything the walk can need is fetched up front, in parallel, so that the walk itself
// touches no memory: (1) the chunk statistics of every row are merged into the row's max M and
// normaliser Z (four threads per row); (2) every node fetches the weight of its own draft token
// under its parent's distribution (one gather for the whole tree; a token that an earlier sibling
// already proposed weighs nothing, because it has left the residual by the time it is tested);
// (3) wavefront 0 walks the tree out of LDS, testing the children of the current node in index
// order against the running residual; (4) the workgroup draws the last token.
// LARGE (kInnerFirst): leaves have no statistics, and the walk looks at none of theirs. If it ends at one, that row's are formed
// now: every one of the sequence's gridDim.x workgroups walks the tree, to the same end, and takes its share of the chunks; the
// last to finish (an arrival counter, part_idx[b]) draws. Where the walk ends at an inner node the first one goes on alone.
template <bool LARGE>
__global__ __launch_bounds__(kWalkThreads) void accept_sample_walk_kernel(const AcceptParams p) {
  __shared__ int rej_tok[FSPAD_MAX_NODES];
  __shared__ double rej_w[FSPAD_MAX_NODES];
  __shared__ double sh_d[8];
  __shared__ int sh_i[8];
  __shared__ double scan_part[kWalkWaves];
  __shared__ int sh_wave[2 * kWalkWaves];
  __shared__ double row_M[FSPAD_MAX_NODES], row_Z[FSPAD_MAX_NODES], node_w[FSPAD_MAX_NODES];
  __shared__ int node_par[FSPAD_MAX_NODES], node_tok[FSPAD_MAX_NODES];
  __shared__ float node_u[2][FSPAD_MAX_NODES];
  const int b = LARGE ? blockIdx.y : blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t o = (int64_t)b * p.Nmax;
  const float* u_acc = p.uniforms + (int64_t)b * 2 * p.Nmax;

  // (1) row statistics: thread (row = tid / 16, part = tid % 16) takes every 16th chunk of its row,
  // two chunks in flight at a time, keeping a running (max, sum); the sixteen parts of a row are then
  // merged with lane exchanges. Nothing here waits for the tree size: rows past it hold unused numbers.
  const int n_raw = p.n_nodes[b];
  auto merge_row = [&](int row, int q) {   // sixteen threads, q = 0 .. 15
    const bool in_range = row < p.Nmax;
    const float* pm = p.part_max + (o + (in_range ? row : 0)) * p.n_chunks;
    const double* ps = p.part_sum + (o + (in_range ? row : 0)) * p.n_chunks;
    float m_run = -INFINITY;
    double z_run = 0.0;
    for (int c0 = q; c0 < p.n_chunks; c0 += 32) {
      float m_c[2];
      double s_c[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int c = c0 + 16 * k;
        const bool ok = in_range && c < p.n_chunks;
        m_c[k] = ok ? pm[c] : -INFINITY;
        s_c[k] = ok ? ps[c] : 0.0;
      }
      const float m_new = fmaxf(m_run, fmaxf(m_c[0], m_c[1]));
      if (m_new > -INFINITY) {
        double z = m_run > -INFINITY ? z_run * exp_nonpos(((double)m_run - (double)m_new) * p.inv_temperature) : 0.0;
#pragma unroll
        for (int k = 0; k < 2; ++k)
          if (m_c[k] > -INFINITY) z += s_c[k] * exp_nonpos(((double)m_c[k] - (double)m_new) * p.inv_temperature);
        z_run = z;
        m_run = m_new;
      }
    }
    float mx = m_run;
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    double z = m_run > -INFINITY ? z_run * exp_nonpos(((double)m_run - (double)mx) * p.inv_temperature) : 0.0;
#pragma unroll
    for (int off = 1; off < 16; off <<= 1) z += __shfl_xor(z, off);
    if (in_range && q == 0) { row_M[row] = (double)mx; row_Z[row] = z; }
  };
  merge_row(tid >> 4, tid & 15);
  if (tid < FSPAD_MAX_NODES) {
    const bool ok = tid < p.Nmax;
    node_par[tid] = ok ? p.parent[o + tid] : -2;
    node_tok[tid] = ok ? p.draft_tokens[o + tid] : -1;
    node_u[0][tid] = ok ? u_acc[tid] : 0.f;
    node_u[1][tid] = ok ? u_acc[p.Nmax + tid] : 0.f;
  }
  const int n = n_raw;
  __syncthreads();
  // (2) weight of every node's draft token under its parent's row
  if (tid < FSPAD_MAX_NODES) {
    double w = 0.0;
    const int par = node_par[tid], tok = node_tok[tid];
    if (tid > 0 && tid < n && par >= 0 && par < tid && tok >= 0 && tok < p.V) {
      const double M = row_M[par];
      if (M > -INFINITY) {
        const float lx = p.logits[(o + par) * p.row_stride + tok];
        if (lx == lx) w = exp_nonpos(((double)lx - M) * p.inv_temperature);
      }
    }
    node_w[tid] = w;
  }
  __syncthreads();

  int my_path = lane == 0 ? 0 : -1, my_out = -1;
  int cur = 0, len = 1, nrej = 0;
  int my_rej = -1;       // lane k keeps the k-th token rejected at the current node, and its weight
  double my_rej_w = 0.0;
  double M = 0.0, Z = 0.0;
  auto walk = [&] {      // (3), wavefront 0
    const int my_par = node_par[lane], my_tok = node_tok[lane];
    const double my_w = node_w[lane];
    const float my_u = node_u[0][lane];
    auto lane_value = [](double v, int src) {   // src is the same in every lane: scalar reads, no LDS exchange
      const unsigned long long bits = __builtin_bit_cast(unsigned long long, v);
      const unsigned lo = __builtin_amdgcn_readlane((unsigned)bits, src);
      const unsigned hi = __builtin_amdgcn_readlane((unsigned)(bits >> 32), src);
      return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
    };
    for (int iter = 0; iter < p.Nmax; ++iter) {  // one level per iteration; a leaf ends the walk
      M = row_M[cur];
      Z = row_Z[cur];
      nrej = 0;
      my_rej = -1;
      const bool is_kid = lane > 0 && lane < n && my_par == cur;
      unsigned long long kids = __ballot(is_kid);
      int accepted = -1;
      while (kids != 0ull && len < p.Nmax) {
        const int c = __builtin_amdgcn_readfirstlane(__ffsll(kids) - 1);
        kids &= kids - 1ull;
        const int x = __builtin_amdgcn_readlane(my_tok, c);
        // a token that an earlier sibling proposed has left the residual: it weighs nothing now
        const bool gone = __ballot(lane < nrej && my_rej == x) != 0ull;
        const double w = gone ? 0.0 : lane_value(my_w, c);
        const double lhs = (double)__builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, my_u), c)) * Z;
        if (lhs < w) { accepted = c; break; }
        Z -= w;
        if (lane == nrej) { my_rej = x; my_rej_w = w; }
        ++nrej;
      }
      if (accepted < 0) break;
      if (lane == len) my_path = accepted;
      const int accepted_tok = __builtin_amdgcn_readlane(my_tok, accepted);
      if (lane == len - 1) my_out = accepted_tok;
      cur = accepted;
      ++len;
    }
    if constexpr (LARGE) {
      const bool leaf = __ballot(lane > 0 && lane < n && my_par == cur) == 0ull;
      if (lane == 0) { sh_i[5] = cur; sh_i[6] = leaf; }
    }
  };
  auto settle = [&] {    // the results but for the last token, and the chunk that holds it; wavefront 0
    if (lane < nrej) { rej_tok[lane] = my_rej; rej_w[lane] = my_rej_w; }
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    if (lane < p.Nmax) { p.path[o + lane] = my_path; if (lane != len - 1) p.tokens[o + lane] = my_out; }
    if (lane == 0) {
      p.path_len[b] = len; p.n_tokens[b] = len;
      sh_i[0] = cur; sh_i[1] = len; sh_i[2] = nrej;
      sh_d[0] = M; sh_d[1] = Z;
    }

    // bonus, stage 1: which chunk holds the running-sum crossing of t = u * Z
    const double t = (double)node_u[1][cur] * Z;
    const int64_t row = o + cur;
    const float* pm = p.part_max + row * p.n_chunks;
    const double* ps = p.part_sum + row * p.n_chunks;
    double carry = 0.0, before = 0.0;
    int found = -1, last_pos = -1;
    for (int c0 = 0; c0 < p.n_chunks && found < 0; c0 += 64) {
      const int c = c0 + lane;
      double r = 0.0;
      if (c < p.n_chunks && pm[c] > -INFINITY) {
        r = ps[c] * exp_nonpos(((double)pm[c] - M) * p.inv_temperature);
        for (int k = 0; k < nrej; ++k)
          if (rej_tok[k] >= c * p.chunk && rej_tok[k] < (c + 1) * p.chunk && rej_tok[k] < p.V) r -= rej_w[k];
      }
      const double incl = wave_running_sum(r);
      const unsigned long long pos = __ballot(r > 0.0);
      if (pos) last_pos = c0 + 63 - __clzll(pos);
      const unsigned long long hit = __ballot(c < p.n_chunks && carry + incl > t);
      if (hit) {
        const int first = __ffsll(hit) - 1;
        found = c0 + first;
        before = carry + __shfl(incl - r, first);
      } else {
        carry += __shfl(incl, 63);
      }
    }
    if (lane == 0) {
      // rounding fallback: the last chunk that still has mass, searched to its end
      sh_i[3] = found >= 0 ? found : last_pos;
      sh_i[4] = found >= 0;
      sh_d[2] = found >= 0 ? t - before : INFINITY;
    }
  };
  if constexpr (LARGE) {
    if (wave == 0) walk();
    __syncthreads();
    if (sh_i[6]) {
      __shared__ double exp2_table[fspad_detail::kExp2Entries];
      __shared__ float wave_max[kWalkWaves];
      if (tid < fspad_detail::kExp2Entries) exp2_table[tid] = fspad_detail::kExp2Table[tid];
      __syncthreads();
      const int leaf = sh_i[5];
      const int64_t row = o + leaf;
      for (int c = blockIdx.x; c < p.n_chunks; c += gridDim.x)
        form_chunk(p.logits + row * p.row_stride, c * kMaxChunk, p.V, p.table_scale, exp2_table, wave_max, scan_part,
                        p.part_max + row * p.n_chunks + c, p.part_sum + row * p.n_chunks + c);
      // (one thread wrote them all, and one wavefront reads them: a fence in each of the sixteen took 20 us)
      if (tid == 0) {
        __threadfence();
        sh_i[7] = gridDim.x > 1 ? atomicAdd(p.part_idx + b, 1) : 0;
      }
      __syncthreads();
      if (sh_i[7] != (int)gridDim.x - 1) return;
      if (wave == 0) {
        __threadfence();
        merge_row(tid < 16 ? leaf : FSPAD_MAX_NODES, tid & 15);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        M = row_M[leaf];
        Z = row_Z[leaf];
      }
    } else if (blockIdx.x > 0) {
      return;
    }
    if (wave == 0) settle();
  } else if (wave == 0) {
    walk();
    settle();
  }
  __syncthreads();

  // bonus, stage 2: inside the chunk, thread k owns chunk/1024 consecutive entries
  const int stop = sh_i[0], last = sh_i[1] - 1, chunk = sh_i[3];
  if (chunk < 0) {  // no mass anywhere (cannot happen with finite logits): token 0
    if (tid == 0) p.tokens[o + last] = 0;
    return;
  }
  DrawArgs a;
  a.rp = p.logits + (o + stop) * p.row_stride;
  a.first = chunk * p.chunk;
  a.V = p.V;
  a.M = sh_d[0];
  a.target = sh_d[2];
  a.inv_temperature = p.inv_temperature;
  a.rej_tok = rej_tok;
  a.nrej = sh_i[2];
  a.scan_part = scan_part;
  a.sh_wave = sh_wave;
  a.out = p.tokens + o + last;
  switch (p.chunk / kWalkThreads) {
    case 1: draw_in_chunk<1>(a); break;
    case 2: draw_in_chunk<2>(a); break;
    case 4: draw_in_chunk<4>(a); break;
    default: draw_in_chunk<8>(a); break;
  }
}

// Largest chunk that still gives about a thousand workgroups (rows x chunks), so that a few rows of
// a small vocabulary are spread over the whole chip.
constexpr int kTargetWorkgroups = 1024;
int pick_chunk(int32_t B, int32_t Nmax, int32_t V) {
  int chunk = kMaxChunk;
  while (chunk > kMinChunk && (int64_t)B * Nmax * ((V + chunk - 1) / chunk) < kTargetWorkgroups) chunk >>= 1;
  return chunk;
}

fspad_status check_accept_args(int32_t B, int32_t Nmax, int32_t V, const float* logits, int64_t row_stride,
                               const int32_t* draft_tokens, const int32_t* parent, const int32_t* n_nodes,
                               int32_t* path, int32_t* path_len, int32_t* tokens, int32_t* n_tokens,
                               void* workspace, size_t workspace_bytes) {
  if (!logits || !draft_tokens || !parent || !n_nodes || !path || !path_len || !tokens || !n_tokens) return FSPAD_ERR_NULL;
  if (B < 1 || Nmax < 1 || Nmax > FSPAD_MAX_NODES || V < 1 || V > (1 << 30) || row_stride < V) return FSPAD_ERR_SHAPE;
  if ((int64_t)B * Nmax > 65535) return FSPAD_ERR_SHAPE;  // grid.y
  if (((uintptr_t)logits) & 3) return FSPAD_ERR_SHAPE;
  if (!workspace || ((uintptr_t)workspace & 15) || workspace_bytes < fspad_tree_accept_workspace_bytes(B, Nmax, V))
    return FSPAD_ERR_WORKSPACE;
  return FSPAD_OK;
}

void fill_params(AcceptParams& p, int32_t B, int32_t Nmax, int32_t V, const float* logits, int64_t row_stride,
                 const int32_t* draft_tokens, const int32_t* parent, const int32_t* n_nodes, int32_t* path,
                 int32_t* path_len, int32_t* tokens, int32_t* n_tokens, void* workspace) {
  p.logits = logits; p.row_stride = row_stride; p.draft_tokens = draft_tokens; p.parent = parent;
  p.n_nodes = n_nodes; p.path = path; p.path_len = path_len; p.tokens = tokens; p.n_tokens = n_tokens;
  p.B = B; p.Nmax = Nmax; p.V = V;
  p.chunk = pick_chunk(B, Nmax, V);
  p.n_chunks = (V + p.chunk - 1) / p.chunk;
  const size_t slots = (size_t)B * Nmax * p.n_chunks;
  p.part_sum = reinterpret_cast<double*>(workspace);                 // 8-byte entries first
  p.part_max = reinterpret_cast<float*>(p.part_sum + slots);
  p.part_idx = reinterpret_cast<int32_t*>(p.part_max + slots);
  p.uniforms = nullptr;
  p.inv_temperature = 1.0;
  p.table_scale = fspad_detail::kExp2PerE;
}

bool rows_vectorisable(const float* logits, int64_t row_stride) {
  return (((uintptr_t)logits) & 15) == 0 && (row_stride % 4) == 0;
}

template <int MODE>
void launch_rows(const AcceptParams& p, hipStream_t stream) {
  const dim3 grid((unsigned)p.n_chunks, (unsigned)(p.B * p.Nmax), p.logits2 ? 2u : 1u), block(kThreads);
  switch (p.chunk / kThreads) {
    case 4: hipLaunchKernelGGL((accept_rows_kernel<MODE, 4>), grid, block, 0, stream, p); break;
    case 8: hipLaunchKernelGGL((accept_rows_kernel<MODE, 8>), grid, block, 0, stream, p); break;
    case 16: hipLaunchKernelGGL((accept_rows_kernel<MODE, 16>), grid, block, 0, stream, p); break;
    default: hipLaunchKernelGGL((accept_rows_kernel<MODE, 32>), grid, block, 0, stream, p); break;
  }
}

// ------------------------------------------------------------------------------------------------
// Acceptance for drafts that were sampled from a draft distribution q (Introduction: the
// draft-then-verify scheme of speculative sampling), in its multi-candidate form: at a node with
// target distribution p and draft distribution q the children are tested in sibling order,
//     accept x  <=>  u q(x) < p(x);      reject x:  p <- max(p - q, 0) / sum,  q(x) <- 0, q <- q / sum
// and when none is accepted the step's last token is drawn from what p has become.
//
// The streaming pass above leaves the chunk statistics of both logit arrays; one workgroup of 1024
// threads per sequence then walks the tree. Every decision is taken in fp64; all threads take it
// from the same values, so the control flow stays uniform without an exchange. A rejection or the
// draw needs the node's two whole rows: they are then written out unnormalised (fp64, 2 V entries
// per sequence) with their scale factors in registers, and every further rejection is one pass.
constexpr int kDraftThreads = 1024;
constexpr int kDraftWaves = kDraftThreads / 64;

struct DraftAcceptParams {
  const float* logits;        // [B][Nmax][row_stride]
  const float* draft_logits;  // same layout
  int64_t row_stride;
  const int32_t* draft_tokens;
  const int32_t* parent;
  const int32_t* n_nodes;
  const float* uniforms;      // [B][2][Nmax]
  int32_t* path;
  int32_t* path_len;
  int32_t* tokens;
  int32_t* n_tokens;
  double* work;               // [B][3][V]: unnormalised p, a spare for the next p, and q of the current node
  const float* part_max_p;    // [B*Nmax][n_chunks] chunk statistics of logits (accept_rows_kernel<1>)
  const double* part_sum_p;
  const float* part_max_q;    // the same of draft_logits
  const double* part_sum_q;
  double inv_temperature;
  int32_t B, Nmax, V, n_chunks;
};

__device__ __forceinline__ double wg_sum(double v, double* sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  __syncthreads();                  // sh may still be read from the previous reduction
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  double s = 0.0;
#pragma unroll
  for (int i = 0; i < kDraftWaves; ++i) s += sh[i];   // the same order in every thread
  return s;
}

__device__ __forceinline__ float wg_max(float v, float* sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
  __syncthreads();
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  float m = sh[0];
#pragma unroll
  for (int i = 1; i < kDraftWaves; ++i) m = fmaxf(m, sh[i]);
  return m;
}

__global__ __launch_bounds__(kDraftThreads) void accept_sample_draft_kernel(const DraftAcceptParams p) {
  __shared__ double sh_d[kDraftWaves];
  __shared__ float sh_f[kDraftWaves];
  __shared__ int sh_tok, sh_last;
  const int b = blockIdx.x, tid = threadIdx.x;
  const int64_t o = (int64_t)b * p.Nmax;
  const int n = p.n_nodes[b];
  const float* u_acc = p.uniforms + (int64_t)b * 2 * p.Nmax;
  const float* u_draw = u_acc + p.Nmax;
  double* wp = p.work + (int64_t)b * 3 * p.V;   // unnormalised p of the current node
  double* wp_spare = wp + p.V;                  // where a rejection writes the next p
  double* wq = wp + 2 * p.V;                    // unnormalised q
  const int V = p.V;

  for (int i = tid; i < p.Nmax; i += kDraftThreads) { p.path[o + i] = i == 0 ? 0 : -1; p.tokens[o + i] = -1; }

  int cur = 0, len = 1;
  for (;;) {
    // row statistics of the node from the chunk statistics of the streaming pass: p(v) = exp((l[v] - mp) / T) / zp
    const float* lrow = p.logits + (o + cur) * p.row_stride;
    const float* qrow = p.draft_logits + (o + cur) * p.row_stride;
    float mp = -INFINITY, mq = -INFINITY;
    for (int c = tid; c < p.n_chunks; c += kDraftThreads) {
      mp = fmaxf(mp, p.part_max_p[(o + cur) * p.n_chunks + c]);
      mq = fmaxf(mq, p.part_max_q[(o + cur) * p.n_chunks + c]);
    }
    mp = wg_max(mp, sh_f);
    mq = wg_max(mq, sh_f);
    double zp = 0.0, zq = 0.0;
    for (int c = tid; c < p.n_chunks; c += kDraftThreads) {
      const float cp = p.part_max_p[(o + cur) * p.n_chunks + c], cq = p.part_max_q[(o + cur) * p.n_chunks + c];
      if (cp > -INFINITY) zp += p.part_sum_p[(o + cur) * p.n_chunks + c] * exp_nonpos(((double)cp - (double)mp) * p.inv_temperature);
      if (cq > -INFINITY) zq += p.part_sum_q[(o + cur) * p.n_chunks + c] * exp_nonpos(((double)cq - (double)mq) * p.inv_temperature);
    }
    zp = wg_sum(zp, sh_d);
    zq = wg_sum(zq, sh_d);
    double sp = zp > 0.0 ? 1.0 / zp : 0.0, sq = zq > 0.0 ? 1.0 / zq : 0.0;
    // The unnormalised weights of the whole rows are written out only when a rejection or the draw
    // needs them: a node whose first child is accepted costs two logits.
    bool filled = false;
    auto weight_p = [&](int v) {
      const float a = lrow[v];
      return (a == a && mp > -INFINITY) ? exp_nonpos(((double)a - (double)mp) * p.inv_temperature) : 0.0;
    };
    auto weight_q = [&](int v) {
      const float c = qrow[v];
      return (c == c && mq > -INFINITY) ? exp_nonpos(((double)c - (double)mq) * p.inv_temperature) : 0.0;
    };
    auto fill_p = [&]() {   // p alone, for a draw at a node without a rejection: p(v) = wp[v] * sp
      __syncthreads();
      for (int v = tid; v < V; v += kDraftThreads) wp[v] = weight_p(v);
      __syncthreads();
    };

    int next = -1;
    for (int c = cur + 1; c < n && len < p.Nmax; ++c) {
      if (p.parent[o + c] != cur) continue;
      const int x = p.draft_tokens[o + c];
      const bool valid = x >= 0 && x < V;
      double px = 0.0, qx = 0.0;
      if (valid && filled) {
        px = wp[x] * sp; qx = wq[x] * sq;
      } else if (valid) {
        const float a = lrow[x], d = qrow[x];
        px = (a == a && mp > -INFINITY) ? exp_nonpos(((double)a - (double)mp) * p.inv_temperature) * sp : 0.0;
        qx = (d == d && mq > -INFINITY) ? exp_nonpos(((double)d - (double)mq) * p.inv_temperature) * sq : 0.0;
      }
      if ((double)u_acc[c] * qx < px) { next = c; break; }
      // rejected: p <- max(p - q, 0), renormalised; q loses x and is renormalised
      if (!filled) {
        // the first rejection at this node: the rows are formed and the rejection applied in the same pass
        __syncthreads();
        double z = 0.0, s = 0.0;
        for (int v = tid; v < V; v += kDraftThreads) {
          const double qv = weight_q(v);
          const double r = fmax(weight_p(v) * sp - qv * sq, 0.0);
          const double keep = (valid && v == x) ? 0.0 : qv;
          wp[v] = r;
          wq[v] = keep;
          z += r;
          s += keep;
        }
        z = wg_sum(z, sh_d);
        s = wg_sum(s, sh_d);
        if (z > 0.0) {
          sp = 1.0 / z;
        } else {                               // p = q exactly: p is kept
          for (int v = tid; v < V; v += kDraftThreads) wp[v] = weight_p(v);
        }
        sq = s > 0.0 ? 1.0 / s : sq;
        filled = true;
        __syncthreads();
        continue;
      }
      // One pass (a workgroup streams its rows at the rate of one compute unit, so passes are what a
      // rejection costs): the residual goes to the spare buffer while its sum forms, and what q keeps
      // once x is gone is summed from the entries alongside (a difference of the old sum and wq[x]
      // would cancel when the drafter was nearly certain of x).
      __syncthreads();                       // every thread has read wp[x], wq[x]
      double z = 0.0, s = 0.0;
      for (int v = tid; v < V; v += kDraftThreads) {
        const double qv = wq[v];
        const double r = fmax(wp[v] * sp - qv * sq, 0.0);
        wp_spare[v] = r;
        z += r;
        s += (valid && v == x) ? 0.0 : qv;
      }
      z = wg_sum(z, sh_d);
      s = wg_sum(s, sh_d);                   // (its barriers: every thread is done with the old wq[x])
      if (z > 0.0) {                         // else p = q exactly: p is kept
        double* const tmp = wp; wp = wp_spare; wp_spare = tmp;
        sp = 1.0 / z;
      }
      if (valid && tid == 0) wq[x] = 0.0;
      sq = s > 0.0 ? 1.0 / s : sq;
      __syncthreads();
    }
    if (next >= 0) {
      if (tid == 0) { p.tokens[o + len - 1] = p.draft_tokens[o + next]; p.path[o + len] = next; }
      ++len;
      cur = next;
      __syncthreads();                       // the next node overwrites wp / wq
      continue;
    }

    if (!filled) fill_p();
    // no child accepted: inverse-CDF draw from the current p. Wavefront w owns the contiguous range
    // [w * per_wave, (w + 1) * per_wave) and walks it in chunks of 64 consecutive entries (one per
    // lane: the loads are contiguous), summing chunk totals in chunk order; the same chunk totals, in
    // the same order, locate the crossing afterwards.
    const int lane = tid & 63, wave = tid >> 6;
    const int per_wave = (V + kDraftThreads - 1) / kDraftThreads * 64;
    const int w0 = wave * per_wave, w1 = min(V, w0 + per_wave);
    auto chunk_total = [&](double x) {
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off);
      return x;
    };
    double mine = 0.0;
    for (int c0 = w0; c0 < w1; c0 += 64) mine += chunk_total(c0 + lane < w1 ? wp[c0 + lane] : 0.0);
    __syncthreads();                  // sh_d may still be read from the last reduction
    if (lane == 0) sh_d[wave] = mine;
    if (tid == 0) sh_tok = -1;
    __syncthreads();
    double total = 0.0, before = 0.0;
    for (int w = 0; w < kDraftWaves; ++w) {
      if (w == wave) before = total;
      total += sh_d[w];
    }
    const double t = (double)u_draw[cur] * total;
    // the first wavefront whose range brackets t (the same arithmetic in every thread)
    int owner = -1;
    {
      double run = 0.0;
      for (int w = 0; w < kDraftWaves && owner < 0; ++w) {
        run += sh_d[w];
        if (run > t) owner = w;
      }
    }
    if (wave == owner) {
      double run = before;
      int tok = -1;
      for (int c0 = w0; c0 < w1 && tok < 0; c0 += 64) {
        const double x = c0 + lane < w1 ? wp[c0 + lane] : 0.0;
        const double tot = chunk_total(x);
        if (run + tot > t) {
          double incl = x;            // running sum inside the chunk, lane order
#pragma unroll
          for (int off = 1; off < 64; off <<= 1) {
            const double up = __shfl_up(incl, off);
            if (lane >= off) incl += up;
          }
          const unsigned long long hit = __ballot(run + incl > t && x > 0.0);
          const unsigned long long mass = __ballot(x > 0.0);
          // (the chunk's total and its lane-order running sum are formed in different orders: if the
          // running sum falls short by rounding, the chunk's last entry with mass)
          tok = c0 + (hit ? __ffsll(hit) - 1 : 63 - __clzll(mass));
        }
        run += tot;
      }
      if (tok < 0) {   // the range's total said "here", its chunk-by-chunk sum fell short: its last entry with mass
        int last = -1;
        for (int c0 = w0; c0 < w1; c0 += 64)
          if (c0 + lane < w1 && wp[c0 + lane] > 0.0) last = c0 + lane;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) last = max(last, __shfl_xor(last, off));
        tok = last;
      }
      if (lane == 0) sh_tok = tok;
    }
    __syncthreads();
    if (sh_tok < 0) {   // no mass at all, or rounding left no crossing: the last entry with mass (0 if none)
      int last = -1;
      for (int c0 = w0; c0 < w1; c0 += 64)
        if (c0 + lane < w1 && wp[c0 + lane] > 0.0) last = c0 + lane;
      if (tid == 0) sh_last = -1;
      __syncthreads();
#pragma unroll
      for (int off = 32; off > 0; off >>= 1) last = max(last, __shfl_xor(last, off));
      if (lane == 0 && last >= 0) atomicMax(&sh_last, last);   // the highest such entry over the workgroup (one lane a wavefront)
      __syncthreads();
      if (tid == 0) sh_tok = sh_last < 0 ? 0 : sh_last;
      __syncthreads();
    }
    if (tid == 0) {
      p.tokens[o + len - 1] = sh_tok;
      p.path_len[b] = len;
      p.n_tokens[b] = len;
    }
    return;
  }
}


// ------------------------------------------------------------------------------------------------
// The same acceptance spread over the chip. With one workgroup per sequence every rejection is a
// pass over two rows of V fp64 entries at the rate of one compute unit. Here G workgroups share a
// sequence: each thread keeps E consecutive entries of the unnormalised p and q of the current node
// in registers, a rejection is arithmetic on registers plus one exchange between the G workgroups
// (partial sums and the two entries the next test needs go through memory), and the draw is located
// from the workgroups' totals. Every workgroup takes every decision from the same published numbers,
// summed in the same order, so the control flow is the same in all of them.
//
// An exchange is one trip: a workgroup stores its numbers with device scope, and every workgroup polls all of them
// until none is missing. (A stored number is its complement, so that the zero words that the launch before leaves
// mean "not there": the complement of no sum is zero, that would be a NaN with every bit set.) Three sets of places
// are used in turn; who has read round r knows that all are done with round r - 1, and empties its place of that set.
//
// The launch is an ordinary one, and whether all G workgroups run at the same time is found out on the way. Each counts
// itself in when it starts; a workgroup whose numbers of the first round are there is running and will see the walk through.
// The one that came first waits for the others (the compute units may be held by another stream's kernels) for as long as the walk
// would take those who are there, see wait_ticks, and then, if one has not even started, closes the count. Those who came
// until then are the team: they take the G shares in turn, from the root on, with the same arithmetic in the same order. Who has more
// shares than registers forms a node's entries anew in every round, from the logits and the rejections so far; who comes later leaves at once.
// Nobody ever waits for a workgroup that has not started, so calls on several streams cannot hold each other up. A cooperative
// launch, the form before, cost 14 us a call (the runtime orders it with signals), and its barrier (a fence, an arrival counter, a poll,
// a fence, then the loads) 4 us a rejection. 60 nodes, V = 128256, 61.8 -> 32.9 us a call, both on the same inputs.
//
// Waits for running workgroups are bounded all the same: who sees no progress for kSpinLimit polls raises the failure bit,
// reports path_len = n_tokens = -1 and leaves, and so does every other workgroup at its next wait.
constexpr int kGridThreads = 256;
constexpr int kGridWaves = kGridThreads / 64;
constexpr int kGridMaxWgs = 64;          // workgroups per sequence, at most
constexpr unsigned kSpinLimit = 1u << 20;
constexpr int kGridSets = 3;             // sets of places for the exchanges
// the word that counts a sequence's workgroups in (low byte)
constexpr uint32_t kClosed = 1u << 31;   // the count is closed; those who came until then, in the second byte, go on
constexpr uint32_t kFailed = 1u << 30;
constexpr uint32_t kCount = 0xff;
static_assert(kGridMaxWgs <= (int)kCount, "a byte each");
constexpr int64_t kShortestWait = 2000;  // 100 MHz ticks: what a whole walk takes

struct DraftGridParams {
  const float* logits;
  const float* draft_logits;
  int64_t row_stride;
  const int32_t* draft_tokens;
  const int32_t* parent;
  const int32_t* n_nodes;
  const float* uniforms;
  int32_t* path;
  int32_t* path_len;
  int32_t* tokens;
  int32_t* n_tokens;
  float* part_max_p;   // chunk statistics of every row of logits, then of draft_logits; the merge launch leaves the row's own
  double* part_sum_p;  // (maximum, sum of exponentials) in place of its first chunk's
  float* part_max_q;
  double* part_sum_q;
  uint64_t* slots;     // [B][3][G][4]: per set and workgroup: sum of the new p, of what q keeps, of the old p
  uint64_t* pubs;      // [B][3][4]: the next test's entry of the new p, of the old p, of q
  uint32_t* sync;      // [B]: workgroups that have started, kClosed with the team's size, kFailed
  uint32_t* clear;     // all of these, as words that the merge launch sets to zero
  int32_t clear_count;
  double* tests;       // [2][B*Nmax]: p(x), then q(x), of the node's token x at its parent
  double inv_temperature;
  int64_t wait_ticks;  // what the first workgroup waits for the others, times the shares of a team of those who are there
  int32_t B, Nmax, V, n_chunks, G;
#ifdef FSPAD_TEST_LATE_WORKGROUPS
  int32_t late_from;   // workgroups of a sequence from this one on count themselves in when the count is closed, or late_ticks late
  int64_t late_ticks;
#endif
};

// K sums over the workgroup at once: running sums inside the wavefronts (no LDS), the four totals of each
// through LDS, one barrier. `sh` holds two sets of K x 4 doubles used in turn, so that a wavefront that
// runs ahead into the next call writes the other set.
template <int K>
__device__ __forceinline__ void grid_wg_sums(double (&v)[K], double* sh, int& flip) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  double* const buf = sh + flip * (K * kGridWaves);
  flip ^= 1;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const double run = wave_running_sum(v[k]);
    if (lane == 63) buf[k * kGridWaves + wave] = run;
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < K; ++k)
    v[k] = (buf[k * kGridWaves] + buf[k * kGridWaves + 1]) + (buf[k * kGridWaves + 2] + buf[k * kGridWaves + 3]);
}

__device__ __forceinline__ float grid_wg_max(float v, float* sh) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off));
  __syncthreads();
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  return fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
}

// numbers of an exchange, device scope
__device__ __forceinline__ void publish(uint64_t* at, double v) {
  __hip_atomic_store(at, ~(uint64_t)__double_as_longlong(v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t poll(const uint64_t* at) { return __hip_atomic_load(at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ double published(uint64_t bits) { return __longlong_as_double((long long)~bits); }

// Row statistics of both logit arrays from the chunk statistics of the streaming pass, for every row at once
// (one workgroup per row and array), and with them the two probabilities that the test of each child of the row's node takes:
// the walk then finds a node's (max, sum) and its first test ready instead of forming them, node after node, on its critical path.
__global__ __launch_bounds__(kGridThreads) void accept_row_merge_kernel(const DraftGridParams p) {
  __shared__ double sh_sums[2 * kGridWaves];
  __shared__ float sh_f[kGridWaves];
  const int row = blockIdx.x, arr = blockIdx.y, tid = threadIdx.x;
  const int b = row / p.Nmax, node = row - b * p.Nmax;
  const int64_t o = (int64_t)b * p.Nmax;
  for (int i = (int)((blockIdx.y * gridDim.x + blockIdx.x) * kGridThreads) + tid; i < p.clear_count; i += (int)(2 * gridDim.x * kGridThreads))
    p.clear[i] = 0u;
  // Statistics, tree and tokens are asked for together (places of rows without statistics are looked at too, and not used), the logits
  // of the children's tokens (wavefront 0, a lane each) a trip later: 60 nodes, V = 128256, a call 34.3 -> 33.9 us.
  const int my_parent = lane_parent(p.parent + o, p.Nmax);
  const int my_token = p.draft_tokens[o + min(tid & 63, p.Nmax - 1)];
  float* const pm = (arr ? p.part_max_q : p.part_max_p) + (int64_t)row * p.n_chunks;
  double* const ps = (arr ? p.part_sum_q : p.part_sum_p) + (int64_t)row * p.n_chunks;
  const float own_max = pm[min(tid, p.n_chunks - 1)];
  const double own_sum = ps[min(tid, p.n_chunks - 1)];
  const int n_all = p.n_nodes[b], n = min(n_all, p.Nmax);
  if (node >= n_all) return;   // rows of unused tree slots have no chunk statistics
  if (!has_child(my_parent, n, node)) return;   // (nor those of leaves: no child is tested there, and the draw takes none)
  const bool child = tid < 64 && my_parent == node && tid > node && tid < n;
  float at_child = __builtin_nanf("");
  if (child && my_token >= 0 && my_token < p.V) at_child = (arr ? p.draft_logits : p.logits)[(o + node) * p.row_stride + my_token];
  float m = tid < p.n_chunks ? own_max : -INFINITY;
  for (int c = tid + kGridThreads; c < p.n_chunks; c += kGridThreads) m = fmaxf(m, pm[c]);
  m = grid_wg_max(m, sh_f);
  double z[1] = {0.0};
  for (int c = tid; c < p.n_chunks; c += kGridThreads) {
    const float mc = c == tid ? own_max : pm[c];
    if (mc > -INFINITY) z[0] += (c == tid ? own_sum : ps[c]) * exp_nonpos(((double)mc - (double)m) * p.inv_temperature);
  }
  int flip = 0;
  grid_wg_sums<1>(z, sh_sums, flip);
  if (tid == 0) {   // (every thread's loads are done: they are in the sums)
    pm[0] = m;
    ps[0] = z[0];
  }
  if (child) {
    const double scale = z[0] > 0.0 ? 1.0 / z[0] : 0.0;
    p.tests[(int64_t)arr * p.B * p.Nmax + o + tid] =
        (at_child == at_child && m > -INFINITY) ? exp_nonpos(((double)at_child - (double)m) * p.inv_temperature) * scale : 0.0;
  }
}

template <int E>
__global__ __launch_bounds__(kGridThreads) void accept_sample_draft_grid_kernel(const DraftGridParams p) {
  __shared__ double sh_d[kGridWaves];
  __shared__ double sh_sums[2 * 3 * kGridWaves];
  __shared__ float sh_f[kGridWaves];
  __shared__ int sh_w[2 * kGridWaves];
  __shared__ double sh_tot[2];
  // of an exchange: the sums of the new p and of what q keeps, the next test's entries; how it ended
  __shared__ double sh_round[5];
  __shared__ int sh_how, sh_team;
  __shared__ uint32_t sh_order;
  int flip = 0;
  const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int g = blockIdx.x, G = p.G, V = p.V;
  const int64_t o = (int64_t)b * p.Nmax;
  uint32_t* const sync = p.sync + b;
#ifdef FSPAD_TEST_LATE_WORKGROUPS
  if (g >= p.late_from)
    for (const long long began = wall_clock64(); wall_clock64() - began < p.late_ticks;) {
      if (__hip_atomic_load(sync, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & kClosed) break;
      __builtin_amdgcn_s_sleep(16);
    }
#endif
  if (tid == 0) sh_order = __hip_atomic_fetch_add(sync, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int n = min(p.n_nodes[b], p.Nmax);
  uint64_t* const slots = p.slots + (int64_t)b * kGridSets * G * 4;
  uint64_t* const pubs = p.pubs + (int64_t)b * kGridSets * 4;

  // the tree, the uniforms and what the rows' launch left go to LDS once: the walk reads them in loops
  __shared__ int t_tok[FSPAD_MAX_NODES], t_path[FSPAD_MAX_NODES];
  __shared__ float t_ua[FSPAD_MAX_NODES], t_ud[FSPAD_MAX_NODES];
  __shared__ double t_stats[2][FSPAD_MAX_NODES][2];   // (max, sum) of every row of this sequence: logits, draft logits
  __shared__ double t_test[2][FSPAD_MAX_NODES];
  // rejections at the current node: the scales they were applied with, the rejected token, whether p moved
  __shared__ double h_sp[FSPAD_MAX_NODES], h_sq[FSPAD_MAX_NODES];
  __shared__ int h_x[FSPAD_MAX_NODES], h_moved[FSPAD_MAX_NODES];
  static_assert(FSPAD_MAX_NODES <= 64, "a lane per node");
  for (int i = tid; i < 2 * p.Nmax; i += kGridThreads) {
    const int arr = i >= p.Nmax, node = i - arr * p.Nmax;
    t_stats[arr][node][0] = (double)(arr ? p.part_max_q : p.part_max_p)[(o + node) * p.n_chunks];
    t_stats[arr][node][1] = (arr ? p.part_sum_q : p.part_sum_p)[(o + node) * p.n_chunks];
    t_test[arr][node] = p.tests[(int64_t)arr * p.B * p.Nmax + o + node];
  }
  const int my_parent = lane < p.Nmax ? p.parent[o + lane] : -2;
  if (tid < FSPAD_MAX_NODES) {
    const bool ok = tid < p.Nmax;
    t_tok[tid] = ok ? p.draft_tokens[o + tid] : -1;
    t_ua[tid] = ok ? p.uniforms[(int64_t)b * 2 * p.Nmax + tid] : 0.f;
    t_ud[tid] = ok ? p.uniforms[(int64_t)b * 2 * p.Nmax + p.Nmax + tid] : 0.f;
  }
  __syncthreads();
  const uint32_t order = __builtin_amdgcn_readfirstlane(sh_order);
  if (order & kClosed) return;   // too late: the others have gone on
  // this workgroup's shares of the entries: its own one, or every step-th of a team's
  int first = g, step = G;
  bool team = false;

  double rp[E], rq[E];   // unnormalised p and q of the current node, once a rejection or the draw has formed them
  unsigned round = 0;
  double slot_z = 0.0, slot_t = 0.0;   // wavefront 0, a lane per workgroup: its sums of the new and the old p in the last round
  int cur = 0, len = 1;

  // Path and tokens but for the last one, which is its finder's. (threads of one workgroup, after a barrier behind the last step of the walk)
  auto write_walk = [&]() {
    for (int i = tid; i < p.Nmax; i += kGridThreads) {
      p.path[o + i] = i < len ? t_path[i] : -1;
      if (i != len - 1) p.tokens[o + i] = i < len ? t_tok[t_path[i + 1]] : -1;
    }
  };
  auto write_last = [&](int tok) {   // one thread
    p.tokens[o + len - 1] = tok;
    p.path_len[b] = len;
    p.n_tokens[b] = len;
  };
  // The numbers of this round's `set` from all workgroups (pub: and the next test's entries): 1: they are in sh_round and the
  // lanes' slot_z, slot_t; 0: leave; 2: go on as a team of sh_team, from the root.
  auto exchange = [&](unsigned set, bool pub) -> int {
    if (wave == 0) {
      int how = 1, size = 0;
      double z = 0.0, s = 0.0, t = 0.0, e0 = 0.0, e1 = 0.0, e2 = 0.0;
      const uint64_t* const at = slots + ((int64_t)set * G + min(lane, G - 1)) * 4;
      const uint64_t* const next = pubs + set * 4;
      const long long began = wall_clock64();
      for (unsigned polls = 0;; ++polls) {
        const uint64_t a0 = poll(at), a1 = poll(at + 1), a2 = poll(at + 2);
        uint64_t b0 = 1, b1 = 1, b2 = 1;
        if (pub) { b0 = poll(next); b1 = poll(next + 1); b2 = poll(next + 2); }
        const uint32_t polled = __hip_atomic_load(sync, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // (waited for only if the numbers are not there)
        if (__all(a0 != 0 && a1 != 0 && a2 != 0 && b0 != 0 && b1 != 0 && b2 != 0)) {
          if (lane < G) { z = published(a0); s = published(a1); t = published(a2); }
          e0 = published(b0); e1 = published(b1); e2 = published(b2);
          break;
        }
        const uint32_t word = __builtin_amdgcn_readfirstlane(polled);
        if (word & kFailed) { how = 0; break; }
        if (!team && (word & kClosed)) { how = 2; size = (word >> 8) & kCount; break; }
        if (round == 1 && order == 0 && word < (uint32_t)G && wall_clock64() - began > max(kShortestWait, p.wait_ticks * ((G + (int)word - 1) / (int)word))) {
          int closed = 0;
          if (lane == 0) {
            uint32_t expected = word;
            closed = __hip_atomic_compare_exchange_strong(sync, &expected, word | (word << 8) | kClosed, __ATOMIC_RELAXED, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          }
          if (__any(closed)) { how = 2; size = word; break; }
        }
        if (polls > kSpinLimit) {
          if (lane == 0) __hip_atomic_fetch_or(sync, kFailed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          how = 0;
          break;
        }
        __builtin_amdgcn_s_sleep(1);
      }
      if (how == 0 && lane == 0) {
        for (int i = 0; i < p.Nmax; ++i) { p.path[o + i] = i == 0 ? 0 : -1; p.tokens[o + i] = -1; }
        p.path_len[b] = -1;
        p.n_tokens[b] = -1;
      }
      const double Z = wave_running_sum(z), S = wave_running_sum(s);
      slot_z = z;
      slot_t = t;
      if (lane == 63) {
        sh_round[0] = Z; sh_round[1] = S; sh_round[2] = e0; sh_round[3] = e1; sh_round[4] = e2;
        sh_how = how;
        sh_team = size;
      }
      // Who is here has all numbers of this round, so all are done with the round before: its places are emptied (they are used
      // again in the round after the next, and this workgroup's numbers of the next one leave behind this). In a team's first round
      // these are the places of round 1: what was stored there has arrived, see below, before its writer's numbers of this round left.
      if (how == 1) {
        const unsigned old = set == 0 ? kGridSets - 1 : set - 1;
        if (lane * step < G - first) {   // (lane 0 alone, but in a team)
          uint64_t* const place = slots + (old * (unsigned)G + (unsigned)(first + lane * step)) * 4u;
#pragma unroll
          for (int k = 0; k < 3; ++k) __hip_atomic_store(place + k, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (first == 0 && lane == 0) {
#pragma unroll
          for (int k = 0; k < 3; ++k) __hip_atomic_store(pubs + old * 4 + k, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
    }
    __syncthreads();
    return sh_how;
  };
  // the sums of a share in a round, thread 0
  auto leave_sums = [&](unsigned set, int of, double z, double s, double t) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the emptied places are (this wavefront's lanes have emptied them)
    uint64_t* const mine = slots + ((int64_t)set * G + of) * 4;
    publish(mine, z); publish(mine + 1, s); publish(mine + 2, t);
  };

  for (;;) {
    if (tid == 0) t_path[len - 1] = cur;
    const float* lrow = p.logits + (o + cur) * p.row_stride;
    const float* qrow = p.draft_logits + (o + cur) * p.row_stride;
    // (rows of nodes beyond the tree are never walked; a leaf's hold no statistics either, which are for the tests of children)
    const double mp = t_stats[0][cur][0], zp = t_stats[0][cur][1], mq = t_stats[1][cur][0], zq = t_stats[1][cur][1];
    double sp = zp > 0.0 ? 1.0 / zp : 0.0, sq = zq > 0.0 ? 1.0 / zq : 0.0;
    int rejected = 0;
    // E entries of a row from v on as they are, past its end NaN (which weighs nothing)
    auto row_entries = [&](const float* row, int v, float (&x)[E]) {
      if (v + E <= V) {
#pragma unroll
        for (int k = 0; k < E / 4; ++k) {
          const f32x4_at_4 q = *reinterpret_cast<const f32x4_at_4*>(row + v + 4 * k);
          x[4 * k] = q[0]; x[4 * k + 1] = q[1]; x[4 * k + 2] = q[2]; x[4 * k + 3] = q[3];
        }
      } else {
#pragma unroll
        for (int j = 0; j < E; ++j) x[j] = v + j < V ? row[v + j] : __builtin_nanf("");
      }
    };
    auto weight = [&](float a, double m) { return (a == a && m > -INFINITY) ? exp_nonpos(((double)a - m) * p.inv_temperature) : 0.0; };
    // p and q of a share from the logits, and the rejections so far (which only a team does not have in its registers)
    auto form = [&](int v) {
      float xp[E], xq[E];
      row_entries(lrow, v, xp);
      row_entries(qrow, v, xq);
#pragma unroll
      for (int j = 0; j < E; ++j) { rp[j] = weight(xp[j], mp); rq[j] = weight(xq[j], mq); }
      for (int i = 0; i < rejected; ++i) {
        const double a = h_sp[i], c = h_sq[i];
        const int x = h_x[i], moved = h_moved[i];
#pragma unroll
        for (int j = 0; j < E; ++j) {
          const double r = fmax(rp[j] * a - rq[j] * c, 0.0);
          if (moved) rp[j] = r;
          if (v + j == x) rq[j] = 0.0;
        }
      }
    };
    // p alone, for a draw at a node without a rejection, with the shift that a workgroup's own entries give: the largest of them
    auto form_p = [&](int v) -> float {
      float xp[E];
      row_entries(lrow, v, xp);
      float most = -INFINITY;
#pragma unroll
      for (int j = 0; j < E; ++j) most = fmaxf(most, xp[j]);   // (a NaN is left out)
      most = grid_wg_max(most, sh_f);
#pragma unroll
      for (int j = 0; j < E; ++j) rp[j] = weight(xp[j], (double)most);
      return most;
    };

    bool moved = false;                // the last round's totals of the p in the registers are those of the new p
    double pub_p = 0.0, pub_q = 0.0;   // the entries of p and q for the child under test, behind a rejection
    int next = -1, how = 1;
    unsigned long long children = __ballot(my_parent == cur && lane > cur && lane < n);
    while (children && len < p.Nmax) {
      const int c = __ffsll(children) - 1;
      children &= children - 1;
      const int x = t_tok[c];
      const bool valid = x >= 0 && x < V;
      double px = 0.0, qx = 0.0;
      if (valid) {
        px = rejected ? pub_p * sp : t_test[0][c];
        qx = rejected ? pub_q * sq : t_test[1][c];
      }
      if ((double)t_ua[c] * qx < px) { next = c; break; }
      // rejected: p <- max(p - q, 0), renormalised; q loses x and is renormalised. The sibling tested
      // next (if any) needs its entries of the new p and q: their owner publishes them in the same round.
      const int x2 = children ? t_tok[__ffsll(children) - 1] : -1;
      const unsigned set = ++round % kGridSets;
      double rn[E];
      for (int of = first; of < G; of += step) {
        const int e0 = (of * kGridThreads + tid) * E;   // this thread's E consecutive entries
        if (team || !rejected) form(e0);
        double three[3] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int j = 0; j < E; ++j) {
          const int v = e0 + j;
          const double qv = rq[j], pold = rp[j];
          const double r = fmax(pold * sp - qv * sq, 0.0);
          const double keep = (valid && v == x) ? 0.0 : qv;
          rn[j] = r; rq[j] = keep;
          three[0] += r; three[1] += keep; three[2] += pold;
        }
        // (behind the loop: as a branch for every entry in it, 32 rejections of V = 500 000 took 155 us instead of 131)
        if ((unsigned)x2 - (unsigned)e0 < (unsigned)E && x2 < V) {
          double r = rn[0], pold = rp[0], keep = rq[0];
#pragma unroll
          for (int j = 1; j < E; ++j)
            if (e0 + j == x2) { r = rn[j]; pold = rp[j]; keep = rq[j]; }
          publish(pubs + set * 4, r); publish(pubs + set * 4 + 1, pold); publish(pubs + set * 4 + 2, keep);
        }
        grid_wg_sums<3>(three, sh_sums, flip);
        if (tid == 0) leave_sums(set, of, three[0], three[1], three[2]);
      }
      how = exchange(set, x2 >= 0 && x2 < V);
      if (how != 1) break;
      const double Z = sh_round[0], S = sh_round[1];
      moved = Z > 0.0;                       // else p = q exactly: p is kept
      if (tid == 0) { h_sp[rejected] = sp; h_sq[rejected] = sq; h_x[rejected] = valid ? x : -1; h_moved[rejected] = moved; }
      ++rejected;
      if (moved) {
#pragma unroll
        for (int j = 0; j < E; ++j) rp[j] = rn[j];
        sp = 1.0 / Z;
      }
      sq = S > 0.0 ? 1.0 / S : sq;
      pub_p = moved ? sh_round[2] : sh_round[3];
      pub_q = sh_round[4];
      if (team) __syncthreads();   // (the history goes through LDS)
    }
    if (how == 1 && next >= 0) {
      ++len;
      cur = next;
      continue;
    }

    // no child accepted: inverse-CDF draw from the current p, located from the workgroups' totals
    if (how == 1 && !rejected) {
      const unsigned set = ++round % kGridSets;
      for (int of = first; of < G; of += step) {
        const float most = form_p((of * kGridThreads + tid) * E);
        double told[1] = {0.0};
#pragma unroll
        for (int j = 0; j < E; ++j) told[0] += rp[j];
        grid_wg_sums<1>(told, sh_sums, flip);
        if (tid == 0) leave_sums(set, of, (double)most, 0.0, told[0]);
      }
      how = exchange(set, false);
      moved = false;
    }
    if (how == 0) return;
    if (how == 2) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // what this workgroup has stored in round 1 has arrived
      first = (int)order;
      step = __builtin_amdgcn_readfirstlane(sh_team);
      team = true;
      cur = 0;
      len = 1;
      __syncthreads();   // sh_how and sh_team are read
      continue;
    }
    // wavefront 0, one lane per workgroup (G <= 64): running sum of the totals, first workgroup above t
    static_assert(kGridMaxWgs <= 64, "one lane per workgroup");
    if (wave == 0) {
      double mine = moved ? slot_z : slot_t, scale = 1.0;   // (0 in lanes past the workgroups)
      if (!rejected) {   // the workgroups' weights have shifts of their own: slot_z
        double most = lane < G ? slot_z : -INFINITY;   // (a largest entry of +infinity is the whole row's: no entry has mass then)
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) most = fmax(most, __shfl_xor(most, off));
        if (mine > 0.0) scale = exp_nonpos((slot_z - most) * p.inv_temperature);
        mine *= scale;
      }
      const double incl = wave_running_sum(mine);
      const double total = __shfl(incl, 63);
      const double t = (double)t_ud[cur] * total;
      const unsigned long long mass = __ballot(mine > 0.0), hit = __ballot(mine > 0.0 && incl > t);
      const int first = hit ? __ffsll(hit) - 1 : (mass ? 63 - __clzll(mass) : -1);
      // (no crossing by rounding: the last workgroup with mass, to its last entry with mass)
      const int at = first < 0 ? 0 : first;
      const double left = hit ? (t - (__shfl(incl, at) - __shfl(mine, at))) / __shfl(scale, at) : INFINITY;
      if (lane == 0) { sh_w[0] = first; sh_tot[0] = left; }
    }
    __syncthreads();
    const int owner = sh_w[0];
    const double target = sh_tot[0];
    __syncthreads();   // sh_w is written again below
    if (owner < 0) {                                            // no mass at all: token 0
      if (first == 0) {
        write_walk();
        if (tid == 0) write_last(0);
      }
      return;
    }
    if (owner % step != first) return;
    write_walk();
    const int e0 = (owner * kGridThreads + tid) * E;
    if (team) {
      if (rejected) form(e0);
      else form_p(e0);
    }
    double local = 0.0;
    int last_here = -1;
#pragma unroll
    for (int j = 0; j < E; ++j) {
      local += rp[j];
      if (rp[j] > 0.0) last_here = e0 + j;
    }
    const double incl = wave_running_sum(local);
    if (lane == 63) sh_d[wave] = incl;
    __syncthreads();
    double wave_base = 0.0;
#pragma unroll
    for (int w = 0; w < kGridWaves; ++w) {
      const double part = sh_d[w];
      if (w < wave) wave_base += part;
    }
    const double inclusive = wave_base + incl;
    const unsigned long long hits = __ballot(inclusive > target && local > 0.0);
    int last_wave = last_here;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) last_wave = max(last_wave, __shfl_xor(last_wave, off));
    if (lane == 0) {
      sh_w[wave] = hits ? wave * 64 + (__ffsll(hits) - 1) : kNone;
      sh_w[kGridWaves + wave] = last_wave;
    }
    __syncthreads();
    int first_thread = kNone, last_any = -1;
#pragma unroll
    for (int w = 0; w < kGridWaves; ++w) {
      first_thread = min(first_thread, sh_w[w]);
      last_any = max(last_any, sh_w[kGridWaves + w]);
    }
    if (first_thread == kNone) {
      if (tid == 0) write_last(last_any < 0 ? 0 : last_any);
      return;
    }
    if (tid == first_thread) {
      double run = inclusive - local;
      int pick = last_here;
      bool done = false;
#pragma unroll
      for (int j = 0; j < E; ++j) {
        run += rp[j];
        if (!done && run > target && rp[j] > 0.0) { pick = e0 + j; done = true; }
      }
      write_last(pick);
    }
    return;
  }
}

struct GridPlan { int G, E; size_t pubs_at, sync_at, tests_at; };
// E = 0: the chip-wide form does not apply (too many sequences, a vocabulary beyond 256 x 32 entries for each of the workgroups
// that a sequence can have, or too small to hold the exchange area in the workspace's row buffers).
GridPlan plan_draft_grid(int32_t B, int32_t Nmax, int32_t V) {
  GridPlan pl{};
  if (B > 256) return pl;
  const int max_g = std::min(kGridMaxWgs, 256 / B);
  const int64_t per = ((int64_t)V + (int64_t)max_g * kGridThreads - 1) / ((int64_t)max_g * kGridThreads);
  const int E = per <= 4 ? 4 : per <= 8 ? 8 : per <= 16 ? 16 : per <= 32 ? 32 : 0;
  if (E == 0) return pl;
  const int G = (int)(((int64_t)V + (int64_t)kGridThreads * E - 1) / ((int64_t)kGridThreads * E));
  pl.pubs_at = (size_t)B * kGridSets * G * 4 * sizeof(uint64_t);
  pl.sync_at = pl.pubs_at + (size_t)B * kGridSets * 4 * sizeof(uint64_t);
  pl.tests_at = pl.sync_at + (((size_t)B * sizeof(uint32_t) + 15) & ~(size_t)15);
  const size_t end = pl.tests_at + (size_t)2 * B * Nmax * sizeof(double);
  if (end > (size_t)B * 3 * (size_t)V * 8) return GridPlan{};
  pl.G = G; pl.E = E;
  return pl;
}

}  // namespace

#ifdef FSPAD_TEST_LATE_WORKGROUPS   // (a build for the tests, which set these: see DraftGridParams)
extern "C" {
int32_t fspad_test_late_from = 64;
int64_t fspad_test_late_ticks = 0;
}
#endif

extern "C" size_t fspad_tree_accept_workspace_bytes(int32_t B, int32_t Nmax, int32_t V) {
  if (B < 1 || Nmax < 1 || V < 1) return 0;
  const size_t slots = (size_t)B * Nmax * ((V + kMinChunk - 1) / kMinChunk);  // room for the finest split
  return (slots * 16 + 255) & ~(size_t)255;
}

extern "C" fspad_status fspad_tree_accept_greedy(int32_t B, int32_t Nmax, int32_t V, const float* logits,
                                                 int64_t row_stride, const int32_t* draft_tokens,
                                                 const int32_t* parent, const int32_t* n_nodes, int32_t* path,
                                                 int32_t* path_len, int32_t* tokens, int32_t* n_tokens,
                                                 void* workspace, size_t workspace_bytes, void* hip_stream) {
  const fspad_status st = check_accept_args(B, Nmax, V, logits, row_stride, draft_tokens, parent, n_nodes, path,
                                            path_len, tokens, n_tokens, workspace, workspace_bytes);
  if (st != FSPAD_OK) return st;
  AcceptParams p{};
  fill_params(p, B, Nmax, V, logits, row_stride, draft_tokens, parent, n_nodes, path, path_len, tokens, n_tokens, workspace);
  hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
  const bool aligned = rows_vectorisable(logits, row_stride) && V % 4 == 0;
  if (takes_small_greedy(B, Nmax, V, aligned)) {
    const dim3 grid((unsigned)B), block(64 * kSmallWaves);
    if (aligned) hipLaunchKernelGGL(accept_greedy_small_kernel<true>, grid, block, 0, stream, p);
    else hipLaunchKernelGGL(accept_greedy_small_kernel<false>, grid, block, 0, stream, p);
    return hipGetLastError() == hipSuccess ? FSPAD_OK : FSPAD_ERR_HIP;
  }
  launch_rows<0>(p, stream);
  if (hipGetLastError() != hipSuccess) return FSPAD_ERR_HIP;
  hipLaunchKernelGGL(accept_greedy_walk_kernel, dim3((unsigned)B), dim3(kThreads), 0, stream, p);
  if (hipGetLastError() != hipSuccess) return FSPAD_ERR_HIP;
  return FSPAD_OK;
}

// ------------------------------------------------------------------------------------------------
// The greedy acceptance for callers that cannot allocate: the chunk statistics live in a fixed
// device array of the library image. In host code the array's name is only a handle: its device
// address is looked up once per device (with that device current) and kept; the kernels get that
// address exactly as they get a caller's workspace.
namespace {
constexpr int kMaxDevices = 64;
}  // namespace
static __device__ __align__(256) unsigned char scratch[FSPAD_STATIC_SCRATCH_BYTES];
namespace {
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices];   // device address of `scratch` on each device, nullptr until looked up

// Device address of the static array on the current device, or nullptr.
void* static_scratch() {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) {
      (void)hipGetLastError();
      return nullptr;
    }
    g_scratch_ptr[dev] = ptr;
  }
  return g_scratch_ptr[dev];
}
}  // namespace

extern "C" fspad_status fspad_tree_accept_greedy_static(int32_t B, int32_t Nmax, int32_t V, const float* logits,
                                                        int64_t row_stride, const int32_t* draft_tokens,
                                                        const int32_t* parent, const int32_t* n_nodes, int32_t* path,
                                                        int32_t* path_len, int32_t* tokens, int32_t* n_tokens,
                                                        void* hip_stream) {
  if (!logits || !draft_tokens || !parent || !n_nodes || !path || !path_len || !tokens || !n_tokens) return FSPAD_ERR_NULL;
  if (B < 1 || Nmax < 1 || Nmax > FSPAD_MAX_NODES || V < 1 || V > (1 << 30)) return FSPAD_ERR_SHAPE;
  const size_t need = fspad_tree_accept_workspace_bytes(B, Nmax, V);
  if (need == 0 || need > FSPAD_STATIC_SCRATCH_BYTES) return FSPAD_ERR_WORKSPACE;  // beyond the fixed array
  void* ptr = static_scratch();
  if (!ptr) return FSPAD_ERR_HIP;
  // every slot the walk reads is written by the row pass of the same call: nothing to clear
  return fspad_tree_accept_greedy(B, Nmax, V, logits, row_stride, draft_tokens, parent, n_nodes, path, path_len, tokens,
                                  n_tokens, ptr, FSPAD_STATIC_SCRATCH_BYTES, hip_stream);
}

// Sampling, large calls: the rows of leaves are looked at only where the walk ends, for the last draw, and leaves are more than
// half of a tree. From so many logits on, the first pass leaves them out, and the walk kernel forms the one that it ends at, by
// several workgroups a sequence (accept_sample_walk_kernel). us a call, all rows formed first / with the leaf formed between two
// more launches / now: V = 128256, 16 x 60 nodes 131 / 70 / 62, 16 x 20..60 96 / 59 / 50, 6 x 60 56 / 40 / 34, 16 x 16 nodes in
// 60-node buffers 45 / 38 / 31; 64 x 60 nodes, V = 32000, 134 / 75 / 65. Drafts without branches have one leaf: 16 x 32 nodes
// 69.4 / 76.2 / 69.2, 64 x 24, V = 32000, 57.4 / 62.3 / 57.4. The line counts the buffers' places, not the trees' nodes, which the
// host does not see: of a few nodes each, what is spared is little and the leaf's row stands behind the walk (16 x 5..10
// nodes 32.0 / 35.8 / 29.5, 6 x 5..10 21.7 / 29.2 / 23.3, 64 x 3..8, V = 32000, 30.2 / 37.0 / 31.4). Below the line the two forms
// are level (4 x 60: 44.1 / 43.7 with the launches); the least number of nodes keeps short drafts, mostly without branches, out.
constexpr int64_t kInnerFirst = (int64_t)40 << 20;
constexpr int32_t kInnerFirstNodes = 24;
constexpr int kWalkWorkgroups = 256;   // of the walk at most: one a compute unit

extern "C" fspad_status fspad_tree_accept_sample(int32_t B, int32_t Nmax, int32_t V, const float* logits,
                                                 int64_t row_stride, const int32_t* draft_tokens,
                                                 const int32_t* parent, const int32_t* n_nodes, float temperature,
                                                 const float* uniforms, int32_t* path, int32_t* path_len,
                                                 int32_t* tokens, int32_t* n_tokens, void* workspace,
                                                 size_t workspace_bytes, void* hip_stream) {
  if (!(temperature > 0.0f) || temperature > 3.0e38f) return FSPAD_ERR_TEMPERATURE;
  if (!uniforms) return FSPAD_ERR_NULL;
  const fspad_status st = check_accept_args(B, Nmax, V, logits, row_stride, draft_tokens, parent, n_nodes, path,
                                            path_len, tokens, n_tokens, workspace, workspace_bytes);
  if (st != FSPAD_OK) return st;
  AcceptParams p{};
  fill_params(p, B, Nmax, V, logits, row_stride, draft_tokens, parent, n_nodes, path, path_len, tokens, n_tokens, workspace);
  p.uniforms = uniforms;
  p.inv_temperature = 1.0 / (double)temperature;
  p.table_scale = fspad_detail::kExp2PerE / (double)temperature;
  hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
  const bool large = Nmax >= kInnerFirstNodes && (int64_t)B * Nmax * V >= kInnerFirst && p.chunk == kMaxChunk;
  if (large) {
    p.rows = kInnerRows;
    p.clear_words = reinterpret_cast<uint32_t*>(p.part_idx);   // the walk's arrival counters
    p.clear_count = B;
  }
  launch_rows<1>(p, stream);
  if (hipGetLastError() != hipSuccess) return FSPAD_ERR_HIP;
  if (large) {
    const int shares = B < kWalkWorkgroups ? kWalkWorkgroups / B : 1;
    const dim3 grid((unsigned)(p.n_chunks < shares ? p.n_chunks : shares), (unsigned)B);
    hipLaunchKernelGGL(accept_sample_walk_kernel<true>, grid, dim3(kWalkThreads), 0, stream, p);
  } else {
    hipLaunchKernelGGL(accept_sample_walk_kernel<false>, dim3((unsigned)B), dim3(kWalkThreads), 0, stream, p);
  }
  if (hipGetLastError() != hipSuccess) return FSPAD_ERR_HIP;
  return FSPAD_OK;
}

extern "C" size_t fspad_tree_accept_sample_draft_workspace_bytes(int32_t B, int32_t Nmax, int32_t V) {
  if (B < 1 || Nmax < 1 || V < 1) return 0;
  // chunk statistics of both logit arrays, then 3 V fp64 entries per sequence
  return 2 * fspad_tree_accept_workspace_bytes(B, Nmax, V) + (((size_t)B * 3 * (size_t)V * 8 + 255) & ~(size_t)255);
}

extern "C" fspad_status fspad_tree_accept_sample_draft(int32_t B, int32_t Nmax, int32_t V, const float* logits,
                                                       const float* draft_logits, int64_t row_stride,
                                                       const int32_t* draft_tokens, const int32_t* parent,
                                                       const int32_t* n_nodes, float temperature, const float* uniforms,
                                                       int32_t* path, int32_t* path_len, int32_t* tokens,
                                                       int32_t* n_tokens, void* workspace, size_t workspace_bytes,
                                                       void* hip_stream) {
  if (!draft_logits || !uniforms) return FSPAD_ERR_NULL;
  if (((uintptr_t)draft_logits) & 3) return FSPAD_ERR_SHAPE;
  const size_t need = fspad_tree_accept_sample_draft_workspace_bytes(B, Nmax, V);
  const fspad_status st = check_accept_args(B, Nmax, V, logits, row_stride, draft_tokens, parent, n_nodes, path, path_len,
                                            tokens, n_tokens, workspace, workspace_bytes >= need ? workspace_bytes : 0);
  if (st != FSPAD_OK) return st;
  if (!(temperature > 0.0f) || temperature > 3.0e38f) return FSPAD_ERR_TEMPERATURE;
  hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
  const size_t region = fspad_tree_accept_workspace_bytes(B, Nmax, V);
  char* ws = static_cast<char*>(workspace);
  AcceptParams pa{}, pb{};
  fill_params(pa, B, Nmax, V, logits, row_stride, draft_tokens, parent, n_nodes, path, path_len, tokens, n_tokens, ws);
  fill_params(pb, B, Nmax, V, draft_logits, row_stride, draft_tokens, parent, n_nodes, path, path_len, tokens, n_tokens,
              ws + region);
  pa.inv_temperature = pb.inv_temperature = 1.0 / (double)temperature;
  pa.table_scale = pb.table_scale = fspad_detail::kExp2PerE / (double)temperature;
  // Chip-wide form: G workgroups a sequence, E entries a thread, if the shape allows it; else one workgroup a sequence.
  const GridPlan plan = plan_draft_grid(B, Nmax, V);
  char* const work = ws + 2 * region;
  // one streaming launch over both logit arrays (grid.z picks the array)
  AcceptParams both = pa;
  both.logits2 = draft_logits; both.part_max2 = pb.part_max; both.part_sum2 = pb.part_sum;
  // The chip-wide walk needs nothing of the leaves' rows, which are more than half of a tree's: no child is tested there, and the
  // draw forms its weights itself (60 nodes, V = 128256, two sets of inputs: the maximum of every row formed 37.0 and 34.7 us, now 34.3 and 31.7). The one-workgroup form needs all.
  both.rows = plan.E != 0 ? kInnerRows : kAllRows;
  launch_rows<1>(both, stream);
  if (hipGetLastError() != hipSuccess) return FSPAD_ERR_HIP;
  if (plan.E != 0) {
    DraftGridParams gp{};
    gp.logits = logits; gp.draft_logits = draft_logits; gp.row_stride = row_stride;
    gp.draft_tokens = draft_tokens; gp.parent = parent; gp.n_nodes = n_nodes; gp.uniforms = uniforms;
    gp.path = path; gp.path_len = path_len; gp.tokens = tokens; gp.n_tokens = n_tokens;
    gp.part_max_p = pa.part_max; gp.part_sum_p = pa.part_sum; gp.part_max_q = pb.part_max; gp.part_sum_q = pb.part_sum;
    gp.slots = reinterpret_cast<uint64_t*>(work);
    gp.pubs = reinterpret_cast<uint64_t*>(work + plan.pubs_at);
    gp.sync = reinterpret_cast<uint32_t*>(work + plan.sync_at);
    gp.clear = reinterpret_cast<uint32_t*>(work);
    gp.clear_count = (int32_t)(plan.tests_at / 4);
    gp.tests = reinterpret_cast<double*>(work + plan.tests_at);
    gp.inv_temperature = pa.inv_temperature;
    gp.B = B; gp.Nmax = Nmax; gp.V = V; gp.n_chunks = pa.n_chunks; gp.G = plan.G;
    // About what a share costs a team in the walk of a tree whose tests reject a few times (E entries a thread; a share's round takes 3 us
    // with 8, 9 with 32), so that a call takes at most about twice as long as if it had known. Walks with the given number of workgroups
    // there, wait and all, us: 60 nodes, V = 128256 (63 shares, E = 8): 1 770, 4 226, 16 87, 32 to 62 76, all 37; 32 rejections at the
    // root: 1 10100, 16 744, all 104; V = 500 000 (62 shares, E = 32): 32300, 2210, 131, only a draw there 1490, 119, 17. A form that waited 300 us and
    // then walked alone, however many were there: 790, 10100, 32900 and 580.
    gp.wait_ticks = 60 * plan.E;
#ifdef FSPAD_TEST_LATE_WORKGROUPS
    gp.late_from = fspad_test_late_from;
    gp.late_ticks = fspad_test_late_ticks;
#endif
    hipLaunchKernelGGL(accept_row_merge_kernel, dim3((unsigned)(B * Nmax), 2u), dim3(kGridThreads), 0, stream, gp);
    if (hipGetLastError() != hipSuccess) return FSPAD_ERR_HIP;
    const dim3 grid((unsigned)plan.G, (unsigned)B), block(kGridThreads);
    switch (plan.E) {
      case 4: hipLaunchKernelGGL(accept_sample_draft_grid_kernel<4>, grid, block, 0, stream, gp); break;
      case 8: hipLaunchKernelGGL(accept_sample_draft_grid_kernel<8>, grid, block, 0, stream, gp); break;
      case 16: hipLaunchKernelGGL(accept_sample_draft_grid_kernel<16>, grid, block, 0, stream, gp); break;
      default: hipLaunchKernelGGL(accept_sample_draft_grid_kernel<32>, grid, block, 0, stream, gp); break;
    }
    return hipGetLastError() == hipSuccess ? FSPAD_OK : FSPAD_ERR_HIP;
  }
  DraftAcceptParams p{};
  p.logits = logits; p.draft_logits = draft_logits; p.row_stride = row_stride;
  p.draft_tokens = draft_tokens; p.parent = parent; p.n_nodes = n_nodes; p.uniforms = uniforms;
  p.path = path; p.path_len = path_len; p.tokens = tokens; p.n_tokens = n_tokens;
  p.work = reinterpret_cast<double*>(ws + 2 * region);
  p.part_max_p = pa.part_max; p.part_sum_p = pa.part_sum; p.part_max_q = pb.part_max; p.part_sum_q = pb.part_sum;
  p.inv_temperature = pa.inv_temperature;
  p.B = B; p.Nmax = Nmax; p.V = V; p.n_chunks = pa.n_chunks;
  hipLaunchKernelGGL(accept_sample_draft_kernel, dim3((unsigned)B), dim3(kDraftThreads), 0, stream, p);
  return hipGetLastError() == hipSuccess ? FSPAD_OK : FSPAD_ERR_HIP;
}
