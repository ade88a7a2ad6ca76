// Top-k cut of a draft step's output (arXiv 2408.15562, Preliminaries, last paragraph: the output
// of every draft step is cut to its k most probable tokens; their probabilities feed the joint
// scores from which the tree is chosen). Per row of logits: the k largest entries, best first
// (equal logits: lower token first; NaN counts as -infinity), and their log-softmax values.
// gfx950 (CDNA4) only.
//
// Two kernels. The first, one workgroup per (chunk of 1024..8192 logits, row), reads its chunk once
// (16 bytes per lane), keeps it in registers as order-preserving integer keys, and leaves the
// chunk's maximum, its sum of exponentials and its own k best entries. The second, one workgroup
// per row, picks the k best of the chunks' candidates and turns them into log-probabilities.
// Entries are compared as packed (key, ~token) words.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "fspad.h"

namespace {

constexpr int kThreads = 256;
constexpr int kMinChunk = 1024, kMaxChunk = 8192;
constexpr int kMergePerThread = 8;   // candidates per thread of the merge kernel: 2048 in all

struct TopkParams {
  const float* logits;
  int64_t row_stride;
  int32_t* tokens;        // [rows][k]
  float* logp;            // [rows][k]
  unsigned long long* cand;  // [rows][k][n_chunks] packed (key << 32 | ~token), 0 = none
  float* chunk_max;       // [rows][n_chunks]
  double* chunk_sum;      // [rows][n_chunks]  sum of exp(l - chunk_max)
  int32_t rows, V, k, n_chunks, chunk;
};

// float -> unsigned key with the same order; NaN ranks with -infinity, -0 with +0; key 0 is
// reserved for "no entry" (smaller than the key of -infinity)
__device__ __forceinline__ unsigned key_of(float x) {
  x = (x != x) ? -INFINITY : x + 0.0f;
  const unsigned u = __float_as_uint(x);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float value_of(unsigned key) {
  return __uint_as_float((key & 0x80000000u) ? (key & 0x7fffffffu) : ~key);
}
__device__ __forceinline__ int token_of(unsigned long long w) { return (int)(0xffffffffu - (unsigned)w); }

// The value of the lane that a data-parallel-primitive lane pattern pairs this one with (no LDS round trip)
template <int CTRL>
__device__ __forceinline__ unsigned dpp(unsigned x) {
  return (unsigned)__builtin_amdgcn_update_dpp((int)x, (int)x, CTRL, 0xf, 0xf, false);
}
template <int CTRL>
__device__ __forceinline__ unsigned long long dpp(unsigned long long x) {
  return ((unsigned long long)dpp<CTRL>((unsigned)(x >> 32)) << 32) | dpp<CTRL>((unsigned)x);
}
__device__ __forceinline__ unsigned lane_of(unsigned x, int lane) { return (unsigned)__builtin_amdgcn_readlane((int)x, lane); }
__device__ __forceinline__ unsigned long long lane_of(unsigned long long x, int lane) {
  return ((unsigned long long)lane_of((unsigned)(x >> 32), lane) << 32) | lane_of((unsigned)x, lane);
}

// Reduction over the 64 lanes, the same value in every lane: neighbours, pairs, mirrored halves of
// eight and of sixteen lanes (after which a row of 16 agrees), then the four rows through scalars.
template <typename T, typename Op>
__device__ __forceinline__ T wave_reduce(T x, Op op) {
  x = op(x, dpp<0xB1>(x));    // quad_perm [1,0,3,2]
  x = op(x, dpp<0x4E>(x));    // quad_perm [2,3,0,1]
  x = op(x, dpp<0x141>(x));   // row_half_mirror
  x = op(x, dpp<0x140>(x));   // row_mirror
  return op(op(lane_of(x, 0), lane_of(x, 16)), op(lane_of(x, 32), lane_of(x, 48)));
}
template <typename T>
__device__ __forceinline__ T wave_max(T x) { return wave_reduce(x, [](T a, T b) { return b > a ? b : a; }); }
__device__ __forceinline__ double wave_sum(double x) {
  const auto add = [](unsigned long long a, unsigned long long b) {
    return (unsigned long long)__double_as_longlong(__longlong_as_double((long long)a) + __longlong_as_double((long long)b));
  };
  return __longlong_as_double((long long)wave_reduce((unsigned long long)__double_as_longlong(x), add));
}

// The k best of a workgroup's words (key above, `low(q)` below; key 0: no entry), in two barriers.
// `prepare` finds a bound that at least k entries reach, the k-th largest of the maxima of 32 groups of
// threads (every 32nd: neighbours may hold what one chunk has left), and the largest key; `gather` sets aside the few entries that reach it (of random ones k to 1.4 k);
// `emit` counts for each of them the ones above it, which is its place. Before, k rounds of a
// workgroup-wide maximum with a barrier each, in which the winner's thread looked its registers through
// again, were most of both kernels. Where more than kListed entries reach the bound (many equal logits) it
// is found once more by whole words (`gather_by_word`); where they still do (the best ones in a few groups) those rounds do it.
//
// Bound by latency: two launches of 1.6 us, a trip to memory and some 1000 clocks of dependent instructions each. In a
// graph, before (k rounds, the loads of a chunk one behind the other) and now: 4 rows of 32000, k = 4 10.0 -> 6.9 us,
// 40 rows of 32000, k = 10 19.0 -> 8.4, 30 rows of 151001, k = 10 34.0 -> 11.8, 80 rows of 128256, k = 10 48.1 -> 19.3,
// 16 rows of 32000, k = 16 22.6 -> 7.9. Rounds over the lanes of a wavefront, without barriers, took 10.5 us at 40 x 32000;
// 64 groups 8.9; groups of neighbouring threads 11.7 at 16 x 32000 (k = 16: a chunk's list came to few of them).
// Where more than kListed entries reach the bound (a chunk of a masked vocabulary, nothing but -infinity), k rounds took longer behind it than without, and
// the bound by whole words takes their place. us a call, k rounds for every row / behind the first bound / now: 10 rows of 128256 with five finite entries, k = 16
// 25.8 / 34.3 / 13.2, 40 rows of 128255 with sixty, k = 10 33.1 / 37.0 / 20.4, 40 rows of 32000 with seven distinct values 19.3 / 12.6 / 12.8; with
// k = 4 the rounds are few: 4 constant rows of 32000 10.0 / 10.8 / 10.9, with five finite entries 9.9 / 9.2 / 9.3.
constexpr int kWaves = kThreads / 64, kListed = kThreads, kGroups = 32;
template <int PT>
struct BlockBest {
  struct Shared {
    unsigned long long list[kListed];
    unsigned long long slots[2 * kWaves];
    unsigned group[kWaves][kGroups], best[kWaves], bound[kWaves];
    unsigned long long word_group[kWaves][kGroups];
    int count;
  };
  Shared& s;
  unsigned (&key)[PT];
  const int k, tid = threadIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;

  __device__ __forceinline__ BlockBest(Shared& shared, unsigned (&keys)[PT], int k_) : s(shared), key(keys), k(k_) {}

  // (a barrier; returns the largest key)
  __device__ __forceinline__ unsigned prepare() {
    unsigned mine = 0u;
#pragma unroll
    for (int q = 0; q < PT; ++q) mine = key[q] > mine ? key[q] : mine;
    const auto halves = __builtin_amdgcn_permlane32_swap(mine, mine, false, false);   // (both halves of the wavefront, in every lane)
    mine = max(halves[0], halves[1]);
    if (lane < kGroups) s.group[wave][lane] = mine;
    if (lane == 0) s.bound[wave] = 0xffffffffu;
    if (tid == 0) s.count = 0;
    s.list[tid] = 0ull;
    __syncthreads();
    // every wavefront for itself: lanes i and i + 32 place group i (equal maxima share the best place)
    mine = 0u;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) mine = max(mine, s.group[w][lane % kGroups]);
    int place = 0;
#pragma unroll
    for (int i = 0; i < kGroups; ++i) place += lane_of(mine, i) > mine ? 1 : 0;
    if (place < k) atomicMin(&s.bound[wave], mine);
    if (place == 0) s.best[wave] = mine;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    return s.best[wave];
  }
  template <typename Low>
  __device__ __forceinline__ void gather(Low&& low) {
    const unsigned bound = max(s.bound[wave], 1u);
    set_aside([&](int q) { return key[q] >= bound; }, low);
  }
  // behind a barrier after `gather`: put(place, word) for places 0..k-1, each by one thread; word 0: no entry is left
  template <typename Low, typename Put>
  __device__ __forceinline__ void emit(Low&& low, Put&& put) {
    const int n = s.count;
    if (__builtin_expect(n <= kListed, 1)) return emit_listed(n, put);
    const int by_word = gather_by_word(low);
    if (by_word <= kListed) return emit_listed(by_word, put);
    unsigned long long mine = local_best(low);
    for (int r = 0; r < k; ++r) {
      unsigned long long* slots = s.slots + (r & 1) * kWaves;   // in turn: one barrier a round is enough
      const unsigned long long wave_best = wave_max(mine);
      if (lane == 0) slots[wave] = wave_best;
      __syncthreads();
      unsigned long long win = slots[0];
#pragma unroll
      for (int w = 1; w < kWaves; ++w) win = slots[w] > win ? slots[w] : win;
      if (tid == 0) put(r, win);
      if (win != 0ull && win == mine) {
#pragma unroll
        for (int q = 0; q < PT; ++q)
          if (word(q, low) == win) key[q] = 0u;
        mine = local_best(low);
      }
    }
  }

 private:
  template <typename Put>
  __device__ __forceinline__ void emit_listed(int n, Put& put) {
    const unsigned long long mine = s.list[tid];
    if (mine != 0ull) {
      int place = 0;
      for (int i = 0; i < n; i += 4) {   // (0 behind the last entry)
#pragma unroll
        for (int o = 0; o < 4; ++o) place += s.list[i + o] > mine ? 1 : 0;
      }
      if (place < k) put(place, mine);
    } else if (tid < k) {
      put(tid, 0ull);   // fewer than k entries: thread tid >= n has none
    }
  }
  template <typename Low>
  __device__ __forceinline__ unsigned long long word(int q, Low& low) const { return key[q] ? ((unsigned long long)key[q] << 32) | low(q) : 0ull; }
  template <typename Low>
  __device__ __forceinline__ unsigned long long local_best(Low& low) const {
    unsigned long long best = 0ull;
#pragma unroll
    for (int q = 0; q < PT; ++q) {
      const unsigned long long w = word(q, low);
      best = w > best ? w : best;
    }
    return best;
  }
  template <typename In, typename Low>
  __device__ __forceinline__ void set_aside(In&& in_list, Low& low) {
    int n = 0;
#pragma unroll
    for (int q = 0; q < PT; ++q) n += __builtin_popcountll(__ballot(in_list(q)));
    if (n == 0) return;
    int at = 0;
    if (lane == 0) at = atomicAdd(&s.count, n);
    at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
    for (int q = 0; q < PT; ++q) {
      const bool mine = in_list(q);
      const unsigned long long in = __ballot(mine);
      if (in == 0ull) continue;
      const int to = at + (int)__builtin_amdgcn_mbcnt_hi((unsigned)(in >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)in, 0u));
      if (mine && to < kListed) s.list[to] = ((unsigned long long)key[q] << 32) | low(q);
      at += __builtin_popcountll(in);
    }
  }
  // `prepare` and `gather` once more, by whole words, which are all different: of equal entries (of a masked vocabulary's -infinities) those with
  // the lowest tokens. Called by all threads; three barriers; returns how many reach the bound.
  template <typename Low>
  __device__ __forceinline__ int gather_by_word(Low& low) {
    unsigned long long mine = local_best(low);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(mine >> 32), (unsigned)(mine >> 32), false, false);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)mine, (unsigned)mine, false, false);
    mine = max(((unsigned long long)hi[0] << 32) | lo[0], ((unsigned long long)hi[1] << 32) | lo[1]);
    __syncthreads();   // (all have read the count)
    if (lane < kGroups) s.word_group[wave][lane] = mine;
    if (tid == 0) s.count = 0;
    s.list[tid] = 0ull;
    __syncthreads();
    mine = 0ull;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) mine = max(mine, s.word_group[w][lane % kGroups]);
    int place = 0;
#pragma unroll
    for (int i = 0; i < kGroups; ++i) place += lane_of(mine, i) > mine ? 1 : 0;
    const unsigned long long at = __ballot(place == k - 1);   // (none: fewer than k groups have an entry, and all entries are taken)
    const unsigned long long bound = at != 0ull ? max(lane_of(mine, __builtin_ctzll(at)), 1ull) : 1ull;
    set_aside([&](int q) { return word(q, low) >= bound; }, low);
    __syncthreads();
    return s.count;
  }
};

// PT entries per thread, entry j*4+i of thread t is logit chunk0 + (j*256 + t)*4 + i.
// Loads of 16 bytes take rows of any alignment: 30 rows of 151001, k = 10 3.6 us a call less than entry by entry.
template <int PT>
__global__ __launch_bounds__(kThreads) void topk_chunk_kernel(const TopkParams p) {
  __shared__ typename BlockBest<PT>::Shared shared;
  __shared__ double red_d[kWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int c = blockIdx.x, row = blockIdx.y;
  const int chunk0 = c * p.chunk;
  const float* src = p.logits + (size_t)row * p.row_stride;

  // (a whole chunk's loads are one block of code: behind a check each, one waits for the one before it, 80 rows of
  // 128256 21.4 us instead of 19.3)
  typedef float f32x4_at_4 __attribute__((ext_vector_type(4), aligned(4)));
  unsigned key[PT];
  if (chunk0 + PT * kThreads <= p.V) {
    f32x4_at_4 x[PT / 4];
#pragma unroll
    for (int j = 0; j < PT / 4; ++j) x[j] = *reinterpret_cast<const f32x4_at_4*>(src + chunk0 + (j * kThreads + tid) * 4);
#pragma unroll
    for (int q = 0; q < PT; ++q) key[q] = key_of(x[q / 4][q % 4]);
  } else {
#pragma unroll
    for (int j = 0; j < PT / 4; ++j) {
      const int e = chunk0 + (j * kThreads + tid) * 4;
      if (e + 3 < p.V) {
        const f32x4_at_4 x = *reinterpret_cast<const f32x4_at_4*>(src + e);
#pragma unroll
        for (int i = 0; i < 4; ++i) key[j * 4 + i] = key_of(x[i]);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) key[j * 4 + i] = e + i < p.V ? key_of(src[e + i]) : 0u;
      }
    }
  }
  auto low = [&](int q) { return 0xffffffffu - (unsigned)(chunk0 + ((q >> 2) * kThreads + tid) * 4 + (q & 3)); };
  BlockBest<PT> best(shared, key, p.k);
  const unsigned top = best.prepare();

  // the chunk's sum of exponentials (entries past the row end and -infinity add nothing)
  const float cmax = top ? value_of(top) : -INFINITY;
  float sum = 0.f;
  if (cmax > -INFINITY) {
#pragma unroll
    for (int q = 0; q < PT; ++q)
      if (key[q]) sum += __expf(value_of(key[q]) - cmax);
  }
  const double dsum = wave_sum((double)sum);
  if (lane == 0) red_d[wave] = dsum;
  best.gather(low);
  __syncthreads();
  if (tid == 0) {
    p.chunk_max[(size_t)row * p.n_chunks + c] = cmax;
    p.chunk_sum[(size_t)row * p.n_chunks + c] = red_d[0] + red_d[1] + red_d[2] + red_d[3];
  }
  unsigned long long* out = p.cand + (size_t)row * p.n_chunks * p.k + c;
  best.emit(low, [&](int place, unsigned long long word) { out[(size_t)place * p.n_chunks] = word; });
}

__global__ __launch_bounds__(kThreads) void topk_merge_kernel(const TopkParams p) {
  __shared__ BlockBest<kMergePerThread>::Shared shared;
  __shared__ double red_d[kWaves];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = blockIdx.x;
  const int n_cand = p.n_chunks * p.k;
  const unsigned long long* cand = p.cand + (size_t)row * n_cand;
  const float* chunk_max = p.chunk_max + (size_t)row * p.n_chunks;
  const double* chunk_sum = p.chunk_sum + (size_t)row * p.n_chunks;

  unsigned key[kMergePerThread], below[kMergePerThread];
#pragma unroll
  for (int q = 0; q < kMergePerThread; ++q) {
    const int i = q * kThreads + tid;
    const unsigned long long w = i < n_cand ? cand[i] : 0ull;
    key[q] = (unsigned)(w >> 32);
    below[q] = (unsigned)w;
  }
  // (the thread's first chunk: requested with the candidates, not behind the barrier)
  const bool one = tid < p.n_chunks;
  const float first_max = one ? chunk_max[tid] : -INFINITY;
  const double first_sum = one ? chunk_sum[tid] : 0.0;

  auto low = [&](int q) { return below[q]; };
  BlockBest<kMergePerThread> best(shared, key, p.k);
  const unsigned top = best.prepare();
  // normaliser from the chunk statistics
  const float m = top ? value_of(top) : -INFINITY;
  double z = 0.0;
  if (m > -INFINITY) {
    auto add = [&](float cm, double cs) { if (cm > -INFINITY) z += cs * exp((double)cm - (double)m); };
    add(first_max, first_sum);
    for (int c = tid + kThreads; c < p.n_chunks; c += kThreads) add(chunk_max[c], chunk_sum[c]);
  }
  z = wave_sum(z);
  if (lane == 0) red_d[wave] = z;
  best.gather(low);
  __syncthreads();
  z = red_d[0] + red_d[1] + red_d[2] + red_d[3];
  const double lse = (double)m + log(z);
  best.emit(low, [&](int place, unsigned long long word) {
    // k <= V and every chunk hands in its own k best: no place stays empty
    const float v = word ? value_of((unsigned)(word >> 32)) : -INFINITY;
    p.tokens[(size_t)row * p.k + place] = word ? token_of(word) : 0;
    p.logp[(size_t)row * p.k + place] = (m > -INFINITY && v > -INFINITY) ? (float)((double)v - lse) : -INFINITY;
  });
}

// Largest chunk that still gives a few hundred workgroups, and few enough chunks for the merge kernel
int pick_chunk(int32_t rows, int32_t V, int32_t k) {
  int chunk = kMaxChunk;
  while (chunk > kMinChunk && (int64_t)rows * ((V + chunk - 1) / chunk) < 512) chunk >>= 1;
  while (chunk < kMaxChunk && (int64_t)((V + chunk - 1) / chunk) * k > kMergePerThread * kThreads) chunk <<= 1;
  return chunk;
}

}  // namespace

extern "C" size_t fspad_draft_topk_workspace_bytes(int32_t rows, int32_t V, int32_t k) {
  if (rows < 1 || V < 1 || k < 1 || k > FSPAD_MAX_TOPK) return 0;
  const size_t chunks = (size_t)rows * ((V + kMinChunk - 1) / kMinChunk);   // room for the finest split
  return ((chunks * (8 * (size_t)k + 4 + 8)) + 255 + 16) & ~(size_t)255;
}

extern "C" fspad_status fspad_draft_topk(int32_t rows, int32_t V, int32_t k, const float* logits, int64_t row_stride,
                                         int32_t* tokens, float* logp, void* workspace, size_t workspace_bytes,
                                         void* hip_stream) {
  if (!logits || !tokens || !logp) return FSPAD_ERR_NULL;
  if (rows < 1 || rows > 65535 || V < 1 || V > (1 << 30) || row_stride < V) return FSPAD_ERR_SHAPE;
  if (k < 1 || k > FSPAD_MAX_TOPK || k > V) return FSPAD_ERR_SHAPE;
  if (((uintptr_t)logits) & 3) return FSPAD_ERR_SHAPE;
  if (!workspace || ((uintptr_t)workspace & 15) || workspace_bytes < fspad_draft_topk_workspace_bytes(rows, V, k))
    return FSPAD_ERR_WORKSPACE;
  TopkParams p{};
  p.logits = logits; p.row_stride = row_stride; p.tokens = tokens; p.logp = logp;
  p.rows = rows; p.V = V; p.k = k;
  p.chunk = pick_chunk(rows, V, k);
  p.n_chunks = (V + p.chunk - 1) / p.chunk;
  if ((int64_t)p.n_chunks * k > kMergePerThread * kThreads) return FSPAD_ERR_SHAPE;   // V > 8192 * 2048 / k
  const size_t chunks = (size_t)rows * p.n_chunks;
  p.cand = static_cast<unsigned long long*>(workspace);                       // 8-byte entries first
  p.chunk_sum = reinterpret_cast<double*>(p.cand + chunks * k);
  p.chunk_max = reinterpret_cast<float*>(p.chunk_sum + chunks);
  hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
  const dim3 grid((unsigned)p.n_chunks, (unsigned)rows), block(kThreads);
  switch (p.chunk / kThreads) {
    case 4: hipLaunchKernelGGL(topk_chunk_kernel<4>, grid, block, 0, stream, p); break;
    case 8: hipLaunchKernelGGL(topk_chunk_kernel<8>, grid, block, 0, stream, p); break;
    case 16: hipLaunchKernelGGL(topk_chunk_kernel<16>, grid, block, 0, stream, p); break;
    default: hipLaunchKernelGGL(topk_chunk_kernel<32>, grid, block, 0, stream, p); break;
  }
  if (hipGetLastError() != hipSuccess) return FSPAD_ERR_HIP;
  hipLaunchKernelGGL(topk_merge_kernel, dim3((unsigned)rows), dim3(kThreads), 0, stream, p);
  if (hipGetLastError() != hipSuccess) return FSPAD_ERR_HIP;
  return FSPAD_OK;
}
