// Commit of the accepted path to the KV cache (arXiv 2408.15562, Preliminaries: the
// tokens that survive validation extend the sequence the next draft-verify cycle starts
// from; the paper does not spell the cache update out). The keys and values of the
// accepted tree nodes, computed by the verification forward, are appended to each
// sequence's cache in path order, so the next cycle's prefix already holds them.
//
// Pure data movement: a few hundred KB per call. One workgroup per (path position,
// sequence, K or V); each thread moves 16 bytes at a time.
#include "fspad.h"

#include <hip/hip_runtime.h>

namespace {

constexpr int kMaxBatchPerLaunch = 128;

struct CommitParams {
  const char* tree[2];   // k_tree, v_tree of this slice
  char* cache[2];        // k_cache, v_cache of this slice
  const int32_t* path;   // [B,Nmax]
  const int32_t* path_len;
  int32_t* kv_len_out;   // may be null
  int64_t stride_batch, stride_head, stride_token;  // bytes
  int32_t Nmax, Hkv, row_bytes;                     // row_bytes = D * element size
  int32_t kv_len[kMaxBatchPerLaunch];
};

// One workgroup per (path position, sequence, K or V). What a call of this size costs is the chain of memory round
// trips behind the launch: arguments (one batch, fetched as the kernel starts -- left to the compiler they are loaded
// where they are needed, five round trips), path entry and length (together), the rows (four 16-byte pieces per thread
// in flight). Together with the merge's index
// arithmetic (tree_attn_combine_kernel), a step of 32 layers with 32 kv heads, 2048 keys: 638 -> 608 us.
static_assert(offsetof(CommitParams, path) == 32 && offsetof(CommitParams, stride_batch) == 56 && offsetof(CommitParams, Nmax) == 80 &&
              offsetof(CommitParams, kv_len) == 92, "the kernel reads its arguments by their offsets");
__global__ __launch_bounds__(256) void kv_commit_kernel(const CommitParams) {
  typedef int v16i __attribute__((ext_vector_type(16)));
  typedef int v8i __attribute__((ext_vector_type(8)));
  typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
  typedef const __attribute__((address_space(4))) char* KernargPtr;
  const int j = blockIdx.x, b = blockIdx.y, which = blockIdx.z;
  KernargPtr ka = (KernargPtr)__builtin_amdgcn_kernarg_segment_ptr();
  KernargPtr ka_b = ka + 4 * b;
  v16i u;
  v8i v;
  int kv_len;
  asm volatile("s_load_dwordx16 %0, %3, 0x0\n\ts_load_dwordx8 %1, %3, 0x40\n\ts_load_dword %2, %4, 0x5c\n\ts_waitcnt lgkmcnt(0)"
               : "=&s"(u), "=&s"(v), "=&s"(kv_len) : "s"(ka), "s"(ka_b));
  // (pointers formed from integers: told to be global ones, or their accesses are flat instructions)
  auto u64 = [](int lo, int hi) { return ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo; };
  const char* const tree = (const char*)(__attribute__((address_space(1))) const char*)(which ? u64(u[2], u[3]) : u64(u[0], u[1]));
  char* const cache = (char*)(__attribute__((address_space(1))) char*)(which ? u64(u[6], u[7]) : u64(u[4], u[5]));
  const int32_t* const path = (const int32_t*)(__attribute__((address_space(1))) const int32_t*)(u64(u[8], u[9]));
  const int32_t* const path_len = (const int32_t*)(__attribute__((address_space(1))) const int32_t*)(u64(u[10], u[11]));
  int32_t* const kv_len_out = (int32_t*)(__attribute__((address_space(1))) int32_t*)(u64(u[12], u[13]));
  const int64_t stride_batch = (int64_t)u64(u[14], u[15]), stride_head = (int64_t)u64(v[0], v[1]), stride_token = (int64_t)u64(v[2], v[3]);
  const int Nmax = v[4], Hkv = v[5], row_bytes = v[6];

  // (an entry past the path's end may hold anything: it is not used)
  const int node = path[(size_t)b * Nmax + j];
  int len = path_len[b];
  len = len < 0 ? 0 : (len > Nmax ? Nmax : len);
  if (j == 0 && which == 0 && threadIdx.x == 0 && kv_len_out) kv_len_out[b] = kv_len + len;
  if (j >= len) return;
  if (node < 0 || node >= Nmax) return;  // a malformed path moves nothing rather than reading out of bounds
  const int shift = 31 - __builtin_clz((unsigned)row_bytes >> 4);   // 8, 16 or 32 pieces of 16 bytes per head
  const int chunks = Hkv << shift;
  const char* src = tree + ((size_t)b * Nmax + node) * Hkv * row_bytes;
  char* dst = cache + (size_t)b * stride_batch + (size_t)(kv_len + j) * stride_token;
  for (int c0 = threadIdx.x; c0 < chunks; c0 += 4 * 256) {
    u32x4 x[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) x[i] = *reinterpret_cast<const u32x4*>(src + (size_t)min(c0 + 256 * i, chunks - 1) * 16);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int c = c0 + 256 * i, g = c >> shift, o = c - (g << shift);
      if (c < chunks) *reinterpret_cast<u32x4*>(dst + (size_t)g * stride_head + (size_t)o * 16) = x[i];
    }
  }
}

}  // namespace

extern "C" fspad_status fspad_kv_commit(const fspad_attn_desc* desc, const void* k_tree, const void* v_tree,
                                        void* k_cache, void* v_cache, int32_t cache_capacity,
                                        const int32_t* kv_len, const int32_t* path, const int32_t* path_len,
                                        int32_t* kv_len_out, void* hip_stream) {
  if (!desc) return FSPAD_ERR_NULL;
  const fspad_attn_desc& d = *desc;
  if (d.batch < 1 || d.n_nodes_max < 1 || d.n_nodes_max > FSPAD_MAX_NODES) return FSPAD_ERR_SHAPE;
  if (d.n_kv_heads < 1 || (d.head_dim != 64 && d.head_dim != 128)) return FSPAD_ERR_SHAPE;
  if (d.io_dtype != FSPAD_F32 && d.io_dtype != FSPAD_BF16) return FSPAD_ERR_DTYPE;
  if (!k_tree || !v_tree || !k_cache || !v_cache || !kv_len || !path || !path_len) return FSPAD_ERR_NULL;
  const int esz = d.io_dtype == FSPAD_BF16 ? 2 : 4;
  const int64_t align = 16 / esz;
  if (d.cache_stride_token < d.head_dim || d.cache_stride_token % align || d.cache_stride_head % align ||
      d.cache_stride_batch % align || d.cache_stride_head < 0 || d.cache_stride_batch < 0)
    return FSPAD_ERR_SHAPE;
  if (((uintptr_t)k_tree | (uintptr_t)v_tree | (uintptr_t)k_cache | (uintptr_t)v_cache) & 15) return FSPAD_ERR_SHAPE;
  // the path is only known on the device: room for the longest possible one is required
  for (int b = 0; b < d.batch; ++b)
    if (kv_len[b] < 0 || (int64_t)kv_len[b] + d.n_nodes_max > cache_capacity) return FSPAD_ERR_SHAPE;
  hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);

  CommitParams prm{};
  prm.stride_batch = d.cache_stride_batch * esz;
  prm.stride_head = d.cache_stride_head * esz;
  prm.stride_token = d.cache_stride_token * esz;
  prm.Nmax = d.n_nodes_max; prm.Hkv = d.n_kv_heads; prm.row_bytes = d.head_dim * esz;
  for (int b0 = 0; b0 < d.batch; b0 += kMaxBatchPerLaunch) {
    const int nb = d.batch - b0 < kMaxBatchPerLaunch ? d.batch - b0 : kMaxBatchPerLaunch;
    CommitParams sl = prm;
    const size_t tree_off = (size_t)b0 * d.n_nodes_max * d.n_kv_heads * d.head_dim * esz;
    sl.tree[0] = static_cast<const char*>(k_tree) + tree_off;
    sl.tree[1] = static_cast<const char*>(v_tree) + tree_off;
    sl.cache[0] = static_cast<char*>(k_cache) + (size_t)b0 * prm.stride_batch;
    sl.cache[1] = static_cast<char*>(v_cache) + (size_t)b0 * prm.stride_batch;
    sl.path = path + (size_t)b0 * d.n_nodes_max;
    sl.path_len = path_len + b0;
    sl.kv_len_out = kv_len_out ? kv_len_out + b0 : nullptr;
    for (int i = 0; i < nb; ++i) sl.kv_len[i] = kv_len[b0 + i];
    hipLaunchKernelGGL(kv_commit_kernel, dim3((unsigned)d.n_nodes_max, (unsigned)nb, 2), dim3(256), 0, stream, sl);
    if (hipGetLastError() != hipSuccess) return FSPAD_ERR_HIP;
  }
  return FSPAD_OK;
}
