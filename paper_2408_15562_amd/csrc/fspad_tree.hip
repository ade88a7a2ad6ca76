// Dynamic draft tree from its candidates (arXiv 2408.15562, Preliminaries, last paragraph:
// per-step top-k, joint probabilities from the dependencies, one more top-k over all tokens;
// then the tokens are organised into a tree and the attention mask derived from it).
// One workgroup per sequence, one thread per candidate (256, 512 or 1024 threads), everything in
// LDS: at most 1024 candidates, a few microseconds.
//   1. joint scores, level by level (a candidate is scored once its parent is)
//   2. rank of every candidate = number of candidates that beat it (score, then index): each
//      candidate becomes one 64-bit word (order-preserving score bits, complemented index), so
//      that "beats" is one unsigned comparison against broadcast LDS reads
//   3. kept = rank < n_keep-1, closed under "parent kept" (level by level again)
//   4. node index = number of kept candidates before it; parents, tokens, ancestor words
#include "fspad.h"

#include <hip/hip_runtime.h>
#include <math.h>

namespace {

struct BuildParams {
  const int32_t* cand_parent;
  const int32_t* cand_token;
  const float* cand_logp;
  const int32_t* n_cand;
  int32_t* parent;
  int32_t* tokens;
  int32_t* n_nodes;
  uint64_t* anc_mask;
  int32_t* node_cand;
  int32_t M, Nmax, n_keep;
};

// float -> unsigned with the same order (-0 ranks with +0)
__device__ __forceinline__ unsigned ordered_bits(float x) {
  const unsigned u = __float_as_uint(x + 0.0f);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// What a candidate waits for its parent to leave: a word of which 0 says "not yet". Every thread repeats its look
// until all of its wavefront have an answer, without a barrier: a parent's index is smaller than its child's, and a
// candidate without a valid one answers at once, so that the answers follow from one another and each loop ends. (In
// rounds between barriers a level took some 500 clocks.) An answer is one 64-bit store, read by one 64-bit load.
template <typename Answer>
__device__ __forceinline__ void follow_parents(unsigned long long* words, int c, int parent, bool pending, Answer&& answer) {
  while (__ballot(pending) != 0ull) {
    if (pending) {
      const unsigned long long of_parent = __hip_atomic_load(&words[parent], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      if (of_parent != 0ull) {
        __hip_atomic_store(&words[c], answer(of_parent), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        pending = false;
      }
    }
  }
}

// Bound by latency: a launch of 1.6 us, a trip to memory (what a thread reads is requested at once: candidates past
// n_cand are read too, and not used), the levels of the tree twice, m comparisons a candidate (of 32 bits, with the index only
// among a wavefront's own, they took longer: 26 nodes 5.4 us), the ancestors' chain. us a call in a graph, with the number of
// candidates, the candidates and the tokens in three trips and barriers between the levels -> now: 26 of 85 candidates 7.6 -> 4.6, 60 of
// 511 14.4 -> 9.3, 8 trees of 48 of 211 7.5 -> 5.4.
template <int THREADS>
__global__ __launch_bounds__(THREADS) void tree_build_kernel(const BuildParams p) {
  constexpr int kWavesPerWg = THREADS / 64;
  typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
  __shared__ __attribute__((aligned(16))) unsigned long long keys[THREADS];   // 0: not a competitor
  __shared__ unsigned long long words[2][THREADS];   // joint scores, decisions (follow_parents)
  __shared__ int16_t node_of[THREADS];   // node index of a kept candidate, else -1
  __shared__ int16_t node_par[FSPAD_MAX_NODES];
  __shared__ int wave_count[kWavesPerWg];
  const int b = blockIdx.x, c = threadIdx.x, lane = c & 63, wave = c >> 6;   // candidate c belongs to thread c
  const size_t at = (size_t)b * p.M + (c < p.M ? c : 0);
  const int read_parent = p.cand_parent[at], my_token = p.cand_token[at];
  const float read_logp = p.cand_logp[at];
  int m = p.n_cand[b];
  m = m < 1 ? 1 : (m > p.M ? p.M : m);
  m = m > THREADS ? THREADS : m;

  // 1. joint scores: bit 33 an answer, bit 32 reached from the root, below it the score
  constexpr unsigned long long kAnswer = 2ull << 32, kReached = 3ull << 32;
  const bool inner = c > 0 && c < m;
  int my_par = inner && read_parent >= 0 && read_parent < c ? read_parent : -2;   // -1 root, -2 unreachable / no candidate
  if (c == 0) my_par = -1;
  const float my_lp = (read_logp != read_logp) ? -INFINITY : read_logp;
  const unsigned long long lowest = kAnswer | __float_as_uint(-INFINITY);   // a candidate that is never reached keeps -infinity
  words[0][c] = c == 0 ? kReached : (my_par >= 0 ? 0ull : lowest);
  words[1][c] = 0ull;
  __syncthreads();
  follow_parents(words[0], c, my_par, my_par >= 0, [&](unsigned long long up) {
    return (up & (1ull << 32)) ? kReached | __float_as_uint(__uint_as_float((unsigned)up) + my_lp) : lowest;
  });
  const unsigned long long scored = words[0][c];   // (this thread's own store)
  if (!(scored & (1ull << 32))) my_par = -2;       // not reached (bad parent index somewhere above): cannot be kept
  const float joint = __uint_as_float((unsigned)scored);

  // 2. rank among the non-root candidates: higher joint first, then lower index
  const unsigned long long mine =
      inner ? (((unsigned long long)ordered_bits(joint) << 32) | (0xffffffffu - (unsigned)c)) : 0ull;
  keys[c] = mine;
  __syncthreads();
  int rank = 0;
  const u32x4* keys2 = reinterpret_cast<const u32x4*>(keys);   // two words per read
  for (int j8 = 0; j8 < (m + 7) / 8; ++j8) {   // entries from m on are 0
    u32x4 o[4];   // same addresses in all lanes: four broadcast reads, issued together
#pragma unroll
    for (int u = 0; u < 4; ++u) o[u] = keys2[4 * j8 + u];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const unsigned long long k0 = ((unsigned long long)o[u][1] << 32) | o[u][0];
      const unsigned long long k1 = ((unsigned long long)o[u][3] << 32) | o[u][2];
      rank += (int)(k0 > mine) + (int)(k1 > mine);
    }
  }

  // 3. closure: a candidate among the best is kept once its parent is, dropped once its parent is (1 dropped, 2 kept)
  const bool top = inner && rank < p.n_keep - 1 && my_par >= 0;
  if (!top)   // (others may be waiting for it already)
    __hip_atomic_store(&words[1][c], c == 0 ? 2ull : 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  follow_parents(words[1], c, my_par, top, [&](unsigned long long up) { return up; });

  // 4. node index = kept candidates before it
  const int kept = words[1][c] == 2ull ? 1 : 0;
  int incl = kept;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int v = __shfl_up(incl, off);
    if (lane >= off) incl += v;
  }
  if (lane == 63) wave_count[wave] = incl;
  __syncthreads();
  int before = incl - kept, total = 0;   // total <= n_keep <= Nmax
#pragma unroll
  for (int w2 = 0; w2 < kWavesPerWg; ++w2) {
    before += w2 < wave ? wave_count[w2] : 0;
    total += wave_count[w2];
  }
  const int my_node = kept ? before : -1;
  if (c < m) node_of[c] = (int16_t)my_node;
  __syncthreads();
  int32_t* out_par = p.parent + (size_t)b * p.Nmax;
  int32_t* out_tok = p.tokens + (size_t)b * p.Nmax;
  int32_t* out_cand = p.node_cand + (size_t)b * p.Nmax;
  if (my_node >= 0) {
    const int pi = c == 0 ? -1 : node_of[my_par];
    node_par[my_node] = (int16_t)pi;
    out_par[my_node] = pi;
    out_tok[my_node] = my_token;
    out_cand[my_node] = c;
  }
  __syncthreads();
  if (c < p.Nmax) {
    uint64_t word = 0;
    if (c < total) {
      for (int a = c; a >= 0; a = node_par[a]) word |= 1ull << a;   // parents have smaller indices: it ends
    } else {
      out_par[c] = -1; out_tok[c] = -1; out_cand[c] = -1;
    }
    p.anc_mask[(size_t)b * p.Nmax + c] = word;
  }
  if (c == 0) p.n_nodes[b] = total;
}

}  // namespace

extern "C" fspad_status fspad_tree_build(int32_t B, int32_t M, int32_t Nmax, const int32_t* cand_parent,
                                         const int32_t* cand_token, const float* cand_logp,
                                         const int32_t* n_cand, int32_t n_keep, int32_t* parent,
                                         int32_t* draft_tokens, int32_t* n_nodes, uint64_t* anc_mask,
                                         int32_t* node_cand, void* hip_stream) {
  if (!cand_parent || !cand_token || !cand_logp || !n_cand || !parent || !draft_tokens || !n_nodes || !anc_mask ||
      !node_cand)
    return FSPAD_ERR_NULL;
  if (B < 1 || M < 1 || M > FSPAD_MAX_CANDIDATES || Nmax < 1 || Nmax > FSPAD_MAX_NODES || n_keep < 1 || n_keep > Nmax)
    return FSPAD_ERR_SHAPE;
  BuildParams prm{cand_parent, cand_token, cand_logp, n_cand, parent, draft_tokens, n_nodes, anc_mask, node_cand,
                  M, Nmax, n_keep};
  hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
  if (M <= 256) hipLaunchKernelGGL(tree_build_kernel<256>, dim3((unsigned)B), dim3(256), 0, stream, prm);
  else if (M <= 512) hipLaunchKernelGGL(tree_build_kernel<512>, dim3((unsigned)B), dim3(512), 0, stream, prm);
  else hipLaunchKernelGGL(tree_build_kernel<1024>, dim3((unsigned)B), dim3(1024), 0, stream, prm);
  return hipGetLastError() == hipSuccess ? FSPAD_OK : FSPAD_ERR_HIP;
}
