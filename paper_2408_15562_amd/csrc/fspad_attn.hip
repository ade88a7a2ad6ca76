// Tree-masked attention of the draft-tree tokens against the prefix KV cache and
// each other (arXiv 2408.15562, Preliminaries, validation phase: one forward of
// the target over the flattened tree, the tree mask introducing the
// dependencies). gfx950 (CDNA4) only.
//
// bf16 path: one wavefront owns up to 64 query rows (16-row tiles) of one kv head
// and streams 32-key blocks of K and V straight from HBM into registers, each
// byte read once: K rows arrive in the A-operand layout of
// v_mfma_f32_16x16x32_bf16, S^T = K Q^T lands one query row per lane column, so the
// running max / sum of the softmax and the O^T = V^T P^T accumulators of a row
// all live in the same lanes and P never leaves registers. V rows are loaded
// 16 bytes per lane (a whole 256-byte row per 16 lanes) and transposed in
// registers with byte permutes. Wavefronts of a workgroup either split the keys
// (few rows: MHA) and merge through LDS, or take different row slabs of the same
// keys (GQA). A second, tiny kernel merges the split-KV partials.
//
// fp32 path: plain VALU kernel, used for the small fp32 parity configuration.
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <type_traits>

#include "attn_plan.h"
#include "fspad.h"
#include "stream_gemm.h"

namespace {

using fspad_detail::bf16x8;
using fspad_detail::blocks_of;
using fspad_detail::div_rcp;
using fspad_detail::kBlockKeys;
using fspad_detail::kComputeUnits;
using fspad_detail::key_waves;
using fspad_detail::kMaxWorkgroups;
using fspad_detail::Plan;
using fspad_detail::plan_rows;
using fspad_detail::plan_wgs;
using fspad_detail::reciprocal;
using fspad_detail::f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned u32x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int kMaxBatchPerLaunch = 128;
constexpr int64_t kMaxFlatBlocks = 1ll << 30;  // 32-key blocks of one launch, summed over its units
constexpr int kMaxClasses = 4;          // classes of sequences (shared-stage kernels)

// Sequences whose trees fill equally many slab groups, of the shared-stage kernels. The kv heads of a class form one flat list of
// blocks; a *cluster* takes a contiguous range of it (every cluster of the class the same number of blocks) with one workgroup
// per slab group, all of them on the same keys at the same time and on the same die (workgroups eight apart), so that K and V come
// from memory once for all slab groups. With the slab groups one after another in the list, as units of their own, each fetched
// them for itself wherever the pieces of a unit were not a multiple of eight: 16 sequences of 131 to 6011 keys, 17 to 60 nodes,
// 32 / 8 heads 98.5 -> 95.5 us a call; 4 equal ones of 4096 keys, 60 nodes 36.5 -> 34.5, 40 / 8 heads 23.2 -> 22.0.
struct SeqClass {
  int32_t wg_begin, groups, clusters, quot, rem;   // cluster p starts at block p * quot + p * rem / clusters of the class
  uint32_t clusters_rcp, tile_rcp;                 // reciprocals (div_rcp) of clusters and of 8 * groups
  int32_t first_seq, slot0, units;                 // units: (sequence, kv head) pairs
  int32_t first_block;                             // in the launch's flat list
  double inv_total;                                // 1 / blocks of the class
};
// A sequence's prefix length and node count; from bit 8 of `nodes` on its place in the batch, from bit 16 on its class.
struct SeqInfo { int32_t kv_len, nodes; };
constexpr float kNegBig = -1.0e30f;     // finite stand-in for "no key seen yet"
constexpr float kLog2e = 1.4426950408889634f;

struct AttnParams {
  const void* q;
  const void* k_tree;
  const void* v_tree;
  const void* k_cache;
  const void* v_cache;
  const uint64_t* anc_mask;
  void* out;
  float* part;     // partial slots: [slot][rows_per_unit * D] un-normalised outputs (rows, or partial_index), then [rows_per_unit][2] (shift, sum)
  int64_t stride_batch, stride_head, stride_token;  // cache strides, elements
  int32_t B, Nmax, Hq, Hkv, G;
  int32_t WS;       // row slabs per workgroup: 1, 2 or 4 (4/WS wavefronts share a slab and split its keys)
  int32_t ws_shift; // log2(WS)
  int32_t NS;       // row slabs per kv head
  int32_t GY;       // slab groups per kv head (of the launch's only class)
  int32_t n_wgs;    // workgroups of the flat decomposition (clusters of the only class)
  int32_t total_blocks;  // 32-key blocks summed over all units (T)
  int32_t wg_quot, wg_rem;  // T = wg_quot * n_wgs + wg_rem: workgroup w starts at w*wg_quot + w*wg_rem/n_wgs
  uint32_t g_magic;   // ceil(2^32 / G): division by multiplication (unused when the divisor is 1)
  uint32_t tile_rcp;  // reciprocal of 8 * GY
  int32_t out_bf16;
  float scale;      // softmax scale
  // when every sequence of the launch has the same prefix length and node count: the flat blocks of
  // one sequence (0 otherwise) and those two numbers, so that a workgroup finds its sequence and its
  // lengths by arithmetic instead of dependent loads from the arrays below
  int32_t seq_blocks, same_len, same_nodes;
  int32_t setup;    // blocks that every unit counts for beyond its own in the flat list (ragged batches; setup_blocks)
  uint32_t wgs_rcp, seq_rcp, unit_rcp;  // reciprocals (div_rcp) of n_wgs and, with seq_blocks > 0, of that and of the blocks a unit counts for
  int32_t n_classes;
  // Sequences in the order of their classes. A workgroup that knows its sequence reads both entries at once, in one trip: fetched
  // one number after the other, and the merge kernel's own arguments behind them, a ragged call took over half a microsecond more
  // (2 x 40 heads, 91 to 729 keys, 48 nodes 19.8 -> 18.9 us, 4 x 32 heads, D = 64, 1 to 102 keys, 48 nodes 18.1 -> 17.4).
  int32_t bstart[kMaxBatchPerLaunch + 1];  // first flat block of each sequence; bstart[B] = total_blocks
  SeqInfo seq[kMaxBatchPerLaunch];
};
// The arguments of the shared-stage kernels, which the other ones do without: with 200 bytes more, and a sequence's lengths further
// from the scalars, fp32 calls of 4 to 10 us took 0.15 to 0.2 us longer.
struct SharedParams {
  AttnParams a;
  int32_t class_wg[kMaxClasses];   // first workgroup of each class (of those that the launch does not have: none, INT32_MAX)
  SeqClass classes[kMaxClasses];   // where there is more than one
};

// The scalar part of AttnParams as the kernels use it, fetched from the kernel-argument segment in
// ONE batch of scalar loads at the top of a kernel. Left to the compiler, the arguments are loaded
// where they are first needed: eight dependent round trips stood between a wavefront's start and
// its first K/V request (a kernel that lives for ten to a hundred microseconds notices each of
// them). The per-sequence arrays stay in the argument segment and are read from there.
typedef const __attribute__((address_space(4))) int32_t* KernargI32;
typedef const __attribute__((address_space(4))) char* KernargPtr;
struct AttnArgs {
  const void* q;
  const void* k_tree;
  const void* v_tree;
  const void* k_cache;
  const void* v_cache;
  const uint64_t* anc_mask;
  void* out;
  float* part;
  int64_t stride_batch, stride_head, stride_token;
  int32_t B, Nmax, Hq, Hkv, G, WS, ws_shift, NS, GY, n_wgs, total_blocks, wg_quot, wg_rem;
  uint32_t g_magic, tile_rcp;
  int32_t out_bf16;
  float scale;
  int32_t seq_blocks, same_len, same_nodes, setup;
  uint32_t wgs_rcp, seq_rcp, unit_rcp;
  int32_t n_classes;
};
static_assert(sizeof(AttnParams) <= 1728, "a longer argument block costs every launch");
static_assert(offsetof(AttnParams, stride_batch) == 64 && offsetof(AttnParams, B) == 88 && offsetof(AttnParams, total_blocks) == 128 &&
              offsetof(AttnParams, scale) == 152 && offsetof(AttnParams, same_nodes) == 164 && offsetof(AttnParams, setup) == 168 && offsetof(AttnParams, n_classes) == 184 && sizeof(AttnParams) % 8 == 0 && sizeof(SharedParams) % 8 == 0,
              "fetch_args reads the scalars by their offsets");

// Arguments that are read where they are used: the arrays, and in the shared-stage kernels what only a segment's end needs
// (kept in scalar registers for the length of a stream they displaced what the stream needs).
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(4))) T* arg_at(size_t offset) {
  return (const __attribute__((address_space(4))) T*)((KernargPtr)__builtin_amdgcn_kernarg_segment_ptr() + offset);
}
__device__ __forceinline__ KernargI32 arg_bstart() { return arg_at<int32_t>(offsetof(AttnParams, bstart)); }
__device__ __forceinline__ const __attribute__((address_space(4))) SeqClass* arg_classes() { return arg_at<SeqClass>(offsetof(SharedParams, classes)); }

typedef int i32x16 __attribute__((ext_vector_type(16)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ AttnArgs args_from(const i32x16& a, const i32x16& b, const i32x16& c) {
  auto u64 = [](int lo, int hi) { return ((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo; };
  // (a pointer formed from an integer is a generic one: its accesses become flat instructions, which count as LDS accesses
  // too and may return in any order, so that every wait for one is a wait for all that is in flight)
  AttnArgs r;
  r.q = (const void*)(__attribute__((address_space(1))) const void*)u64(a[0], a[1]);
  r.k_tree = (const void*)(__attribute__((address_space(1))) const void*)u64(a[2], a[3]);
  r.v_tree = (const void*)(__attribute__((address_space(1))) const void*)u64(a[4], a[5]);
  r.k_cache = (const void*)(__attribute__((address_space(1))) const void*)u64(a[6], a[7]);
  r.v_cache = (const void*)(__attribute__((address_space(1))) const void*)u64(a[8], a[9]);
  r.anc_mask = (const uint64_t*)(__attribute__((address_space(1))) const uint64_t*)u64(a[10], a[11]);
  r.out = (void*)(__attribute__((address_space(1))) void*)u64(a[12], a[13]);
  r.part = (float*)(__attribute__((address_space(1))) float*)u64(a[14], a[15]);
  r.stride_batch = (int64_t)u64(b[0], b[1]);
  r.stride_head = (int64_t)u64(b[2], b[3]);
  r.stride_token = (int64_t)u64(b[4], b[5]);
  r.B = b[6]; r.Nmax = b[7]; r.Hq = b[8]; r.Hkv = b[9]; r.G = b[10]; r.WS = b[11]; r.ws_shift = b[12]; r.NS = b[13];
  r.GY = b[14]; r.n_wgs = b[15];
  r.total_blocks = c[0]; r.wg_quot = c[1]; r.wg_rem = c[2]; r.g_magic = (uint32_t)c[3]; r.tile_rcp = (uint32_t)c[4];
  r.out_bf16 = c[5];
  const int scale_bits = c[6];   // (a bit cast straight from the vector element reads element 0)
  r.scale = __builtin_bit_cast(float, scale_bits);
  r.seq_blocks = c[7]; r.same_len = c[8]; r.same_nodes = c[9]; r.setup = c[10];
  r.wgs_rcp = (uint32_t)c[11]; r.seq_rcp = (uint32_t)c[12]; r.unit_rcp = (uint32_t)c[13]; r.n_classes = c[14];
  return r;
}
// Registers of their own for what is read throughout: left in the sixteen of their load they are spilled, and fetched back, all
// sixteen at a time (moves from spilled registers in the code of the 48-row tiles at D = 64: 201, now 43; 4 x 52 heads of it,
// 497 keys, 42 to 48 nodes 11.3 -> 10.9 us). Loads of four or two words instead cost more than they spare: 10 x 8 heads, 70 keys,
// 64 nodes 12.6 us, in loads of four 13.2, of two 13.9.
__device__ __forceinline__ AttnArgs args_apart(const i32x16& a, const i32x16& b, const i32x16& c) {
  AttnArgs r = args_from(a, b, c);
  asm volatile("" : "+s"(r.seq_blocks), "+s"(r.same_len), "+s"(r.same_nodes), "+s"(r.setup), "+s"(r.unit_rcp), "+s"(r.g_magic), "+s"(r.out_bf16),
                    "+s"(r.n_classes), "+s"(r.wgs_rcp), "+s"(r.seq_rcp), "+s"(r.scale));
  return r;
}
__device__ __forceinline__ AttnArgs fetch_args() {
  KernargPtr ka = (KernargPtr)__builtin_amdgcn_kernarg_segment_ptr();   // AttnParams is the first argument
  i32x16 a, b, c;
  asm volatile("s_load_dwordx16 %0, %3, 0x0\n\ts_load_dwordx16 %1, %3, 0x40\n\ts_load_dwordx16 %2, %3, 0x80\n\ts_waitcnt lgkmcnt(0)"
               : "=&s"(a), "=&s"(b), "=&s"(c) : "s"(ka));
  return args_apart(a, b, c);
}
// The same with the first workgroups of the classes, for the shared-stage kernels (a trip of their own: two classes, 2 x 12 / 2
// heads, D = 64, 3 and 26 keys 8.6 -> 8.4 us; with one class the load beside the others costs nothing measurable).
__device__ __forceinline__ AttnArgs fetch_args(i32x4& class_wg) {
  KernargPtr ka = (KernargPtr)__builtin_amdgcn_kernarg_segment_ptr();
  i32x16 a, b, c;
  asm volatile("s_load_dwordx16 %0, %4, 0x0\n\ts_load_dwordx16 %1, %4, 0x40\n\ts_load_dwordx16 %2, %4, 0x80\n\ts_load_dwordx4 %3, %4, %5\n\t"
               "s_waitcnt lgkmcnt(0)"
               : "=&s"(a), "=&s"(b), "=&s"(c), "=&s"(class_wg) : "s"(ka), "n"(offsetof(SharedParams, class_wg)));
  int from_1 = class_wg[1], from_2 = class_wg[2], from_3 = class_wg[3];   // (apart too: 32 / 8 heads, 4096 keys 20.0 -> 19.8 us)
  asm volatile("" : "+s"(from_1), "+s"(from_2), "+s"(from_3));
  class_wg = i32x4{0, from_1, from_2, from_3};
  return args_apart(a, b, c);
}
// The same with what the merge needs of a sequence and the merge kernel's own arguments, which lie `tail` bytes into the segment.
struct MergeArgs {
  AttnArgs p;
  int first_block, kv_len, nodes;   // of the sequence (SeqInfo)
  int rows_per_unit, pieces;
  double inv_total;
};
__device__ __forceinline__ MergeArgs fetch_merge_args(int at_seq, size_t tail) {
  KernargPtr ka = (KernargPtr)__builtin_amdgcn_kernarg_segment_ptr();
  i32x16 a, b, c;
  i32x4 own;
  i32x2 seq;
  int first;
  asm volatile("s_load_dwordx16 %0, %6, 0x0\n\ts_load_dwordx16 %1, %6, 0x40\n\ts_load_dwordx16 %2, %6, 0x80\n\t"
               "s_load_dwordx4 %3, %7, 0x0\n\ts_load_dwordx2 %4, %8, 0x0\n\ts_load_dword %5, %9, 0x0\n\ts_waitcnt lgkmcnt(0)"
               : "=&s"(a), "=&s"(b), "=&s"(c), "=&s"(own), "=&s"(seq), "=&s"(first)
               : "s"(ka), "s"(ka + tail), "s"(ka + offsetof(AttnParams, seq) + (unsigned)at_seq * sizeof(SeqInfo)),
                 "s"(ka + offsetof(AttnParams, bstart) + (unsigned)at_seq * sizeof(int32_t)));
  MergeArgs m;
  m.p = args_from(a, b, c);
  m.first_block = first; m.kv_len = seq[0]; m.nodes = seq[1];
  m.rows_per_unit = own[0]; m.pieces = own[1];
  m.inv_total = __builtin_bit_cast(double, i32x2{own[2], own[3]});
  return m;
}
// sequence that flat block r0 belongs to, and the first flat block / lengths of a sequence
__device__ __forceinline__ int seq_of_block(const AttnArgs& p, unsigned r0, int first = 0) {
  if (p.seq_blocks > 0) return (int)div_rcp(r0, (unsigned)p.seq_blocks, p.seq_rcp);
  int b = first;
  while (b + 1 < p.B && r0 >= (unsigned)arg_bstart()[b + 1]) ++b;
  return b;
}
__device__ __forceinline__ unsigned seq_first_block(const AttnArgs& p, int b) {
  return p.seq_blocks > 0 ? (unsigned)b * (unsigned)p.seq_blocks : (unsigned)arg_bstart()[b];
}
// what a workgroup needs to know of a sequence of the launch's order
struct Seq {
  int n, len, place;   // nodes, prefix keys, place in the batch
  unsigned first;      // first flat block
};
__device__ __forceinline__ Seq seq_at(const AttnArgs& p, int b) {
  Seq s{p.same_nodes, p.same_len, b, (unsigned)b * (unsigned)p.seq_blocks};
  if (p.seq_blocks <= 0) {
    KernargPtr ka = (KernargPtr)__builtin_amdgcn_kernarg_segment_ptr();
    i32x2 info;
    int first;
    asm volatile("s_load_dwordx2 %0, %2, 0x0\n\ts_load_dword %1, %3, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=&s"(info), "=&s"(first)
                 : "s"(ka + offsetof(AttnParams, seq) + (unsigned)b * sizeof(SeqInfo)), "s"(ka + offsetof(AttnParams, bstart) + (unsigned)b * sizeof(int32_t)));
    s = Seq{info[1] & 0xff, info[0], (info[1] >> 8) & 0xff, (unsigned)first};
  }
  return s;
}

// flat blocks [r0, r1) of workgroup w: [floor(w*T/W), floor((w+1)*T/W)) with T = wg_quot*W + wg_rem
__device__ __forceinline__ void workgroup_blocks(const AttnArgs& p, unsigned w, unsigned& r0, unsigned& r1) {
  const unsigned wr = w * (unsigned)p.wg_rem, wq = div_rcp(wr, (unsigned)p.n_wgs, p.wgs_rcp);
  r0 = w * (unsigned)p.wg_quot + wq;
  r1 = r0 + (unsigned)p.wg_quot + ((wr - wq * (unsigned)p.n_wgs) + (unsigned)p.wg_rem >= (unsigned)p.n_wgs ? 1u : 0u);
}
// What a workgroup of a shared-stage kernel does: blocks [r0, r1) of the flat list for slab group y. The partial result of the
// unit-th (sequence, kv head) pair of the class goes to slot `slot` + unit.
struct Share {
  unsigned r0, r1;
  int y, first_seq, slot;
};
__device__ __forceinline__ Share share_of(const AttnArgs& p, const i32x4& class_wg, unsigned w) {
  SeqClass c;
  c.wg_begin = 0; c.groups = p.GY; c.clusters = p.n_wgs; c.quot = p.wg_quot; c.rem = p.wg_rem; c.clusters_rcp = p.wgs_rcp;
  c.tile_rcp = p.tile_rcp; c.first_seq = 0; c.slot0 = 0; c.units = p.B * p.Hkv;
  unsigned flat0 = 0;
  if (p.n_classes > 1) {
    const int k = ((int)w >= class_wg[1] ? 1 : 0) + ((int)w >= class_wg[2] ? 1 : 0) + ((int)w >= class_wg[3] ? 1 : 0);
    const __attribute__((address_space(4))) SeqClass& from = arg_classes()[k];
    c.wg_begin = from.wg_begin; c.groups = from.groups; c.clusters = from.clusters; c.quot = from.quot; c.rem = from.rem;
    c.clusters_rcp = from.clusters_rcp; c.tile_rcp = from.tile_rcp; c.first_seq = from.first_seq; c.slot0 = from.slot0; c.units = from.units;
    flat0 = (unsigned)from.first_block;
  }
  // eight clusters at a time: their workgroups for the first slab group, then those for the second, ...
  const unsigned local = w - (unsigned)c.wg_begin, tile = div_rcp(local, 8u * c.groups, c.tile_rcp);
  unsigned in_tile = local - tile * 8u * c.groups;
  const unsigned width = min(8u, (unsigned)c.clusters - 8u * tile);
  Share s;
  s.y = 0;
  if (width == 8u) {
    s.y = (int)(in_tile >> 3);
    in_tile &= 7u;
  } else {
    for (; in_tile >= width; in_tile -= width) ++s.y;
  }
  const unsigned at = 8u * tile + in_tile, ar = at * (unsigned)c.rem, aq = div_rcp(ar, (unsigned)c.clusters, c.clusters_rcp);
  s.r0 = flat0 + at * (unsigned)c.quot + aq;
  s.r1 = s.r0 + (unsigned)c.quot + ((ar - aq * (unsigned)c.clusters) + (unsigned)c.rem >= (unsigned)c.clusters ? 1u : 0u);
  s.first_seq = c.first_seq;
  s.slot = c.slot0 + s.y * (c.units + c.clusters) + (int)at;
  return s;
}
// unit that flat block `rel` of a sequence belongs to, its units counting for `counted` blocks each
__device__ __forceinline__ int unit_of_block(const AttnArgs& p, unsigned rel, int counted) {
  return (int)(p.seq_blocks > 0 ? div_rcp(rel, (unsigned)counted, p.unit_rcp) : rel / (unsigned)counted);
}

// x / d for x*d < 2^32, with magic = ceil(2^32 / d) (d >= 2) from the host
__device__ __forceinline__ unsigned div_magic(unsigned x, int d, unsigned magic) {
  return d == 1 ? x : __umulhi(x, magic);
}

// Row slabs a sequence's tree fills, and the slab groups that hold them: a tree smaller
// than the batch's largest has no work beyond them. The rows past its last group are zeroed by the workgroup
// that holds the first block of its first group (zero_rows). 16 sequences of 17 to 60 nodes, 32 / 8 heads: 98 -> 86 us.
__device__ __forceinline__ int seq_slabs(const AttnArgs& p, int n, int rows_per_slab) { return (int)((unsigned)(n * p.G + rows_per_slab - 1) / (unsigned)rows_per_slab); }
__device__ __forceinline__ int seq_groups(const AttnArgs& p, int slabs) { return (slabs + p.WS - 1) >> p.ws_shift; }

__device__ __forceinline__ float wave_xor_max_16_32(float v) {
  v = fmaxf(v, __shfl_xor(v, 16));
  v = fmaxf(v, __shfl_xor(v, 32));
  return v;
}

// Zeros for the output rows of (sequence b, kv head g) from row `first` of its Nmax * G rows on.
template <int D, int THREADS>
__device__ __forceinline__ void zero_rows(const AttnArgs& p, int b, int g, int first) {
  const int row_bytes = p.out_bf16 ? 2 * D : 4 * D, chunks = row_bytes >> 4;   // 8, 16 or 32 pieces of 16 bytes
  const int shift = 31 - __builtin_clz((unsigned)chunks), total = (p.Nmax * p.G - first) << shift;
  for (int i = threadIdx.x; i < total; i += THREADS) {
    const int rr = first + (i >> shift);
    const int node = (int)div_magic((unsigned)rr, p.G, p.g_magic), hl = rr - node * p.G;
    const int64_t row = ((int64_t)b * p.Nmax + node) * p.Hq + g * p.G + hl;
    *reinterpret_cast<u32x4*>(reinterpret_cast<char*>(p.out) + row * row_bytes + 16 * (i & (chunks - 1))) = u32x4{0u, 0u, 0u, 0u};
  }
}

// Which key a lane's j-th V row / P element refers to inside a 32-key block:
// the accumulator layout of two 16-key S^T tiles puts keys 4*g4+i (tile 0) and
// 16+4*g4+i (tile 1) in lane group g4.
__device__ __forceinline__ int key_of(int g4, int j) { return (j < 4) ? 4 * g4 + j : 16 + 4 * g4 + (j - 4); }

// Partial results of the shared-stage kernel lie in their slots as its lanes hold them, [row tile][store instruction][lane]
// pieces of four dims: a store instruction writes a kilobyte in a row and a merging workgroup, eight rows by all pieces, reads
// whole lines. They are written through to memory (device scope), where the merge kernel, mostly on another die, finds them
// anyway: left dirty in the L2 caches, 17 MB of them were written back when the kernel ended, with nothing else to do. Row by
// row, in 16-byte pieces, each would cost the write of a part of a line. A call with 32 / 8 heads, 60 nodes, 4096 keys:
// 21.2 us row by row, 20.8 in lane order, 19.9 written through; 1000 keys 16.5, 16.0, 15.1; D = 64, 3000 keys 15.9, 14.3, 13.8.
// (The wavefronts that split keys of few rows gain nothing and keep rows: 32 heads, 4 nodes 13.2 us, in lane order 13.7.)
// Offset in floats of piece `piece` (dims 4 * piece .. + 3) of row lr.
template <int D>
__device__ __forceinline__ int partial_index(int lr, int piece) {
  // D = 128: a lane holds dims 8 * x + 4 * h .. + 3 of its row; D = 64: dims 4 * (4 * g4 + i) .. + 3 are stored i-th
  if constexpr (D == 128) return 4 * (((lr >> 5) * 16 + (piece >> 1)) * 64 + (piece & 1) * 32 + (lr & 31));
  else return 4 * (((lr >> 4) * 4 + (piece & 3)) * 64 + (piece >> 2) * 16 + (lr & 15));
}
// (the store reads its data behind its issue: one slot before anything may write those registers)
__device__ __forceinline__ void store_through(float* p, const f32x4& v) {
  asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 0" : : "v"((__attribute__((address_space(1))) float*)p), "v"(v) : "memory");
}

// Where one 32-key block lives and how it is masked.
struct BlockSrc {
  const char* k;       // first key row of the block
  const char* v;
  unsigned row_bytes;  // bytes between consecutive keys
  int nvalid;          // keys of the block that exist (1..32)
  int kind;            // 0 full prefix block, 1 prefix block with a ragged tail, 2 tree block
  int tree_key0;       // first tree node of a tree block
};

// Per-lane byte offsets of a block's rows from its first row. They depend only on the row pitch
// and on how many rows exist (rows past the end of a ragged block are clamped and masked later),
// so they are recomputed only where a stream changes from full blocks to its tail or to the tree.
// K rows arrive in the A-operand layout of the 16x16x32 MFMA: lane (col, g4) holds key 16*kt+col,
// dims 32*ks + 8*g4 .. +7.
__device__ __forceinline__ void k_offsets(unsigned (&off)[2], unsigned row_bytes, int nvalid, int col, int g4) {
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) off[kt] = (unsigned)min(16 * kt + col, nvalid - 1) * row_bytes + 16u * g4;
}
// V rows: lane (col, g4) holds, for its 8 keys, the D/16 consecutive dims starting at (D/16)*col,
// i.e. 16 lanes read one whole row contiguously.
template <int D>
__device__ __forceinline__ void v_offsets(unsigned (&off)[8], unsigned row_bytes, int nvalid, int col, int g4) {
#pragma unroll
  for (int j = 0; j < 8; ++j) off[j] = (unsigned)min(key_of(g4, j), nvalid - 1) * row_bytes + (unsigned)(D / 8) * col;
}

// Scalar base + per-lane byte offset. STREAMED: with the non-temporal hint (kCacheBytes in stream_gemm.h).
template <bool STREAMED, typename T>
__device__ __forceinline__ T load_once(const char* p) {
  if constexpr (STREAMED) return __builtin_nontemporal_load(reinterpret_cast<const T*>(p));
  else return *reinterpret_cast<const T*>(p);
}
template <int D, bool STREAMED>
__device__ __forceinline__ void load_k(bf16x8 (&k)[2][D / 32], const char* base, const unsigned (&off)[2]) {
#pragma unroll
  for (int kt = 0; kt < 2; ++kt)
#pragma unroll
    for (int ks = 0; ks < D / 32; ++ks) k[kt][ks] = load_once<STREAMED, bf16x8>(base + off[kt] + 64 * ks);
}
template <int D, bool STREAMED>
__device__ __forceinline__ void load_v(unsigned (&v)[8][D / 32], const char* base, const unsigned (&off)[8]) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if constexpr (D == 128) {
      const u32x4 w = load_once<STREAMED, u32x4>(base + off[j]);
      v[j][0] = w[0]; v[j][1] = w[1]; v[j][2] = w[2]; v[j][3] = w[3];
    } else {
      const u32x2 w = load_once<STREAMED, u32x2>(base + off[j]);
      v[j][0] = w[0]; v[j][1] = w[1];
    }
  }
}

template <int QT, int D>
struct RowState {
  static constexpr int DT = D / 16;
  f32x4 o[QT][DT];   // O^T accumulators: lane (col,g4), reg i <-> row 16t+col, dim DT*(4*g4+i)+e
  float m[QT];       // softmax shift in use (log2 units, scaled): within kLazyLog2 of the running max
  f32x4 l[QT];       // running sum of the weights, formed on the matrix cores (all 4 entries equal)
};

// The shift of a row only moves when a score exceeds it by more than this (log2 units): weights
// then stay below 2^kLazyLog2, which fp32 sums and bf16 weights hold without loss, and the
// accumulators are rescaled (and lanes exchanged) almost never after the first blocks.
constexpr float kLazyLog2 = 8.0f;

// One 32-key block against the wavefront's 16*QT query rows, two row tiles at a time so that only
// 16 score and 8 weight registers are live and the matrix work of one tile pair can run under the
// vector work of the other:
//   S^T = K Q^T          s[kt][i] of tile t in lane (col,g4) is key 16*kt+4*g4+i against row 16*t+col
//   mask (ragged / tree blocks), lazy shift update, weights p = 2^(s*c - m) rounded to bf16
//   O^T += V^T P^T       V slice of a lane transposed once per block with byte permutes
//   l   += 1^T P^T       row sums on the matrix cores: sums of the bf16 weights actually used, so
//                        numerator and denominator agree (a dominant key is reproduced exactly),
//                        with no vector-ALU adds and no lane exchange.
// Q fragments come from registers, or (large row tiles) from lane-private LDS slots.
// `after_scores()` runs once the last product that reads k has been issued (the caller requests
// the next block's K there when it keeps a single K buffer). `after_transpose()` runs, for tiles
// done in several passes, once v has been transposed and is dead (the caller requests the next
// block's V into the same registers there: a whole block of lead time at no register cost).
template <int QT, int D, typename QFn, typename MaskFn, typename AfterFn, typename AfterVFn>
__device__ __forceinline__ void process_block(RowState<QT, D>& st, const bf16x8 (&k)[2][D / 32],
                                              const unsigned (&v)[8][D / 32], QFn&& q_frag, const BlockSrc& src,
                                              MaskFn&& mask_of_tile, float c, int g4, AfterFn&& after_scores,
                                              AfterVFn&& after_transpose) {
  constexpr int DT = D / 16;
  constexpr int TP = QT >= 2 ? 2 : 1;  // tiles per pass
  bf16x8 ones;
#pragma unroll
  for (int j = 0; j < 8; ++j) ones[j] = (__bf16)1.0f;
  bf16x8 vt[DT];  // transposed V: A operand of d-tile e holds dims DT*col+e of the lane group's 8 keys
#pragma unroll
  for (int t0 = 0; t0 < QT; t0 += TP) {
    f32x4 s[TP][2];
#pragma unroll
    for (int tt = 0; tt < TP; ++tt) {
      if (t0 + tt >= QT) continue;
      f32x4 acc0 = {0.f, 0.f, 0.f, 0.f}, acc1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < D / 32; ++ks) {
        const bf16x8 q = q_frag(t0 + tt, ks);
        acc0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[0][ks], q, acc0, 0, 0, 0);
        acc1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(k[1][ks], q, acc1, 0, 0, 0);
      }
      s[tt][0] = acc0;
      s[tt][1] = acc1;
    }
    if (t0 + TP >= QT) after_scores();
    if (src.kind != 0) {  // wavefront-uniform: ragged tail and tree blocks only
#pragma unroll
      for (int tt = 0; tt < TP; ++tt) {
        if (t0 + tt >= QT) continue;
        // visibility of the block's 32 keys for this lane's row, then shifted to the lane's own keys
        unsigned vis = src.nvalid >= kBlockKeys ? ~0u : ((1u << src.nvalid) - 1u);
        if (src.kind == 2) vis &= (unsigned)(mask_of_tile(t0 + tt) >> src.tree_key0);
        vis >>= 4 * g4;
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
          for (int i = 0; i < 4; ++i) s[tt][kt][i] = ((vis >> (16 * kt + i)) & 1u) ? s[tt][kt][i] : -INFINITY;
      }
    }
    // exponents of the weights under the shift in use: t = s*c - m. Their maximum decides whether
    // the shift has to move (results of an fma are canonical numbers: the maximum needs no
    // quieting of its inputs, unlike one over the raw outputs of the matrix instructions)
    float tv[TP][8];
    bool grow = false;
#pragma unroll
    for (int tt = 0; tt < TP; ++tt) {
      if (t0 + tt >= QT) continue;
      const float m = st.m[t0 + tt];
#pragma unroll
      for (int j = 0; j < 8; ++j) tv[tt][j] = fmaf(s[tt][j >> 2][j & 3], c, -m);
      const float mt = fmaxf(fmaxf(fmaxf(tv[tt][0], tv[tt][1]), fmaxf(tv[tt][2], tv[tt][3])),
                             fmaxf(fmaxf(tv[tt][4], tv[tt][5]), fmaxf(tv[tt][6], tv[tt][7])));
      grow = grow || (mt > kLazyLog2);
    }
    if (__any(grow)) {  // wavefront-uniform and rare: move these rows' shifts to their running maxima
#pragma unroll
      for (int tt = 0; tt < TP; ++tt) {
        if (t0 + tt >= QT) continue;
        const int t = t0 + tt;
        const float mx = fmaxf(fmaxf(fmaxf(s[tt][0][0], s[tt][0][1]), fmaxf(s[tt][0][2], s[tt][0][3])),
                               fmaxf(fmaxf(s[tt][1][0], s[tt][1][1]), fmaxf(s[tt][1][2], s[tt][1][3])));
        const float mnew = fmaxf(st.m[t], wave_xor_max_16_32(mx) * c);
        const float alpha = __builtin_amdgcn_exp2f(st.m[t] - mnew);
        st.m[t] = mnew;
        st.l[t] *= alpha;
#pragma unroll
        for (int e = 0; e < DT; ++e) st.o[t][e] *= alpha;
#pragma unroll
        for (int j = 0; j < 8; ++j) tv[tt][j] = fmaf(s[tt][j >> 2][j & 3], c, -mnew);
      }
    }
    bf16x8 pf[TP];
#pragma unroll
    for (int tt = 0; tt < TP; ++tt) {
      if (t0 + tt >= QT) continue;
#pragma unroll
      for (int j = 0; j < 8; ++j) pf[tt][j] = (__bf16)__builtin_amdgcn_exp2f(tv[tt][j]);
    }
    auto transposed = [&](int e) {  // A operand of d-tile e from the lane's 8 x DT slice of V
      const unsigned sel = (e & 1) ? 0x07060302u : 0x05040100u;
      u32x4 w;
#pragma unroll
      for (int m2 = 0; m2 < 4; ++m2) w[m2] = __builtin_amdgcn_perm(v[2 * m2 + 1][e >> 1], v[2 * m2][e >> 1], sel);
      return __builtin_bit_cast(bf16x8, w);
    };
    constexpr bool kSinglePass = QT <= TP;  // one pass: transpose on the fly, nothing to keep
    if (!kSinglePass && t0 == 0) {
#pragma unroll
      for (int e = 0; e < DT; ++e) vt[e] = transposed(e);
      after_transpose();
    }
#pragma unroll
    for (int tt = 0; tt < TP; ++tt) {
      if (t0 + tt >= QT) continue;
      st.l[t0 + tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf[tt], st.l[t0 + tt], 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < DT; ++e) {
      const bf16x8 va = kSinglePass ? transposed(e) : vt[e];
#pragma unroll
      for (int tt = 0; tt < TP; ++tt) {
        if (t0 + tt >= QT) continue;
        st.o[t0 + tt][e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, pf[tt], st.o[t0 + tt][e], 0, 0, 0);
      }
    }
  }
}

// The (sequence, kv head, slab group) units and their 32-key blocks form one flat list of
// blocks; workgroup w owns the contiguous range [w*T/W, (w+1)*T/W) of it, so every workgroup
// streams the same number of bytes whatever the head count. A workgroup therefore works on one
// or a few *segments* (a run of blocks of one unit). A segment that is a whole unit is written
// to `out` directly; otherwise its un-normalised (O, max, sum) goes to partial slot unit+w and the
// merge kernel finishes the unit.
// RAGGED: units count for p.setup blocks more than they have (a form of its own: in the other one the bookkeeping
// costs the 64-row tiles registers they do not have, 4 x 52 heads, 4096 keys: 83 -> 98 us).
// Two workgroups fit on a compute unit except of 64-row tiles and of 48-row tiles at D = 128 (and of 32-row tiles at D = 128 in
// ragged batches, where 256 registers made it spill): launches of more whole units than compute units need that, so that one's
// set-up and merge run beside another's stream. 16 x 52 heads, 26 nodes, D = 128: 150 keys 25.0 us, with one workgroup per
// compute unit 37.7, 600 keys 55.9 (68.3), 1400 keys 112 (126); D = 64, 40 nodes: 150 keys 19.4 (30.5), 1200 keys 54.4 (66.9). The limit
// stands where the compiler would pass it: asked for it everywhere, D = 64 with 32-row tiles lost up to 13 % in ragged batches
// (184 registers without) and D = 64 with 48-row tiles 1 % (239 without).
template <int QT, int D, bool STREAMED, bool RAGGED>
__global__ __launch_bounds__(256, (QT == 1 || (QT == 2 && D == 128 && !RAGGED) ? 2 : 1)) void tree_attn_bf16_kernel(const AttnParams) {
  const AttnArgs p = fetch_args();
  constexpr int KS = D / 32;
  constexpr int DT = D / 16;
  constexpr int ROWS = 16 * QT;
  // merge buffers: 4 wavefronts x (QT*DT accumulators + QT stats) x 64 lanes. With large row tiles
  // the Q fragments of the 4 wavefronts live in lane-private LDS slots instead of registers; they are
  // dead once a segment's stream is done, so they share the space of the merge buffers.
  constexpr bool kQInLds = QT >= 3;
  // Tiles done in several passes run one wavefront per SIMD: they hide the memory latency by
  // themselves, keeping K and V of the next block in flight for a whole block
  constexpr bool kDeep = QT >= 3;
  constexpr int kMergeBytes = 4 * QT * DT * 64 * 16;
  constexpr int kQBytes = kQInLds ? 4 * QT * KS * 64 * 16 : 0;
  __shared__ __attribute__((aligned(16))) char lds_raw[kMergeBytes > kQBytes ? kMergeBytes : kQBytes];
  __shared__ float2 merge_ml[4][QT][64];
  typedef f32x4 (*MergeO)[QT * DT][64];
  MergeO merge_o = reinterpret_cast<MergeO>(lds_raw);

  // the wavefront index is the same in all 64 lanes: telling the compiler keeps everything that
  // derives from it (key split, block counters, base addresses) in scalar registers
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col = lane & 15, g4 = lane >> 4;
  bf16x8* q_lds = reinterpret_cast<bf16x8*>(lds_raw) + wave * (QT * KS * 64) + lane;
  const int slab_local = wave & (p.WS - 1);
  const int KW = 4 >> p.ws_shift;  // wavefronts that split the keys of one slab
  const int kp = wave >> p.ws_shift;
  const float c = p.scale * kLog2e;
  const unsigned tree_row_bytes = (unsigned)p.Hkv * D * 2u;
  const unsigned cache_row_bytes = (unsigned)p.stride_token * 2u;
  const int rows_per_unit = p.WS * ROWS;

  // A kernel this short-lived spends much of its time fetching instructions it runs once: all
  // index arithmetic up to the first loads is 32-bit, and divisions by the launch's constants
  // are multiplications.
  const unsigned w = blockIdx.x;
  unsigned r0, r1;
  workgroup_blocks(p, w, r0, r1);
  int b = seq_of_block(p, r0);

  for (unsigned r = r0; r < r1;) {
    const Seq seq = seq_at(p, b);
    const int n = seq.n, L = seq.len;
    const int n_prefix_blocks = (L + kBlockKeys - 1) / kBlockKeys;
    const int n_blocks = n_prefix_blocks + (n + kBlockKeys - 1) / kBlockKeys;
    const unsigned rel = r - seq.first;
    const int counted = RAGGED ? n_blocks + p.setup : n_blocks;  // what the unit counts for: its set-up first, then its blocks
    const int ub = unit_of_block(p, rel, counted);                // unit within the sequence: (g, y)
    int seg_begin = (int)(rel - (unsigned)ub * (unsigned)counted);
    int seg_count = min(counted - seg_begin, (int)(r1 - r));
    const int count = seg_count;
    if constexpr (RAGGED) {
      const int end = seg_begin + count - p.setup;
      seg_begin = max(seg_begin - p.setup, 0);
      seg_count = end - seg_begin;
      if (seg_count <= 0) {   // nothing but set-up
        r += (unsigned)count;
        continue;
      }
    }
    const int g = ub;   // one slab group per kv head in every plan of this kernel
    const int unit = b * p.Hkv + ub;
    const bool whole_unit = seg_count == n_blocks;
    const int slab = slab_local;
    const bool slab_live = slab < p.NS;

    // the key-splitting wavefronts of a slab share the segment's blocks evenly
    // interleaved: wavefront kp takes blocks kp, kp+KW, ... so that the workgroup as a whole walks
    // one contiguous stretch of K and of V (neighbouring DRAM pages stay open)
    const int blk_begin = seg_begin + kp;
    const int blk_end = seg_begin + seg_count;
    const bool active = slab_live && blk_begin < blk_end;

    const char* kc = reinterpret_cast<const char*>(p.k_cache) + (b * p.stride_batch + g * p.stride_head) * 2;
    const char* vc = reinterpret_cast<const char*>(p.v_cache) + (b * p.stride_batch + g * p.stride_head) * 2;
    const char* ktr = reinterpret_cast<const char*>(p.k_tree) + ((int64_t)b * p.Nmax * p.Hkv + g) * (D * 2);
    const char* vtr = reinterpret_cast<const char*>(p.v_tree) + ((int64_t)b * p.Nmax * p.Hkv + g) * (D * 2);

    auto locate = [&](int blk) {
      BlockSrc src;
      if (blk < n_prefix_blocks) {
        const int key0 = blk * kBlockKeys;
        const int64_t byte0 = (int64_t)key0 * cache_row_bytes;
        src.k = kc + byte0;
        src.v = vc + byte0;
        src.row_bytes = cache_row_bytes;
        src.nvalid = min(kBlockKeys, L - key0);
        src.kind = src.nvalid == kBlockKeys ? 0 : 1;
        src.tree_key0 = 0;
      } else {
        const int t0 = (blk - n_prefix_blocks) * kBlockKeys;
        src.k = ktr + t0 * tree_row_bytes;
        src.v = vtr + t0 * tree_row_bytes;
        src.row_bytes = tree_row_bytes;
        src.nvalid = min(kBlockKeys, n - t0);
        src.kind = 2;
        src.tree_key0 = t0;
      }
      return src;
    };

    // The stream's first block is requested before anything else is set up. Small tiles (two
    // wavefronts per SIMD) keep one K and one V block in registers: K of the next block is requested
    // right after the scores of this one, V of the next block once this block's products are issued.
    // Large tiles (one wavefront per SIMD) request K of the next block at the top of this one into a
    // second buffer and V of the next block as soon as this block's V has been transposed, into the
    // registers that frees.
    bf16x8 kf[2][KS], kfn[kDeep ? 2 : 1][KS];
    unsigned vr[8][D / 32];
    unsigned koff[2], voff[8];
    unsigned k_rb = 0, v_rb = 0;   // row pitch and row count the offsets were last computed for
    int k_nv = 0, v_nv = 0;
    auto set_k = [&](const BlockSrc& s) {
      if (s.row_bytes != k_rb || s.nvalid != k_nv) {
        k_offsets(koff, s.row_bytes, s.nvalid, col, g4);
        k_rb = s.row_bytes; k_nv = s.nvalid;
      }
    };
    auto set_v = [&](const BlockSrc& s) {
      if (s.row_bytes != v_rb || s.nvalid != v_nv) {
        v_offsets<D>(voff, s.row_bytes, s.nvalid, col, g4);
        v_rb = s.row_bytes; v_nv = s.nvalid;
      }
    };
    BlockSrc cur{};
    if (active) {
      cur = locate(blk_begin);
      set_k(cur);
      load_k<D, STREAMED>(kf, cur.k, koff);
      set_v(cur);
      load_v<D, STREAMED>(vr, cur.v, voff);
    }

    // row of this lane in tile t: query row rr of the kv head's N*G rows = (node, head within group)
    struct RowInfo { bool exists, valid; int node; int64_t out; };
    auto row_info = [&](int t) {
      RowInfo ri;
      const int rr = slab * ROWS + 16 * t + col;
      ri.node = (int)div_magic((unsigned)rr, p.G, p.g_magic);
      const int hl = rr - ri.node * p.G;
      ri.exists = slab_live && rr < p.Nmax * p.G;
      ri.valid = ri.exists && ri.node < n;
      ri.out = ((int64_t)b * p.Nmax + ri.node) * p.Hq + g * p.G + hl;  // index of (b, node, h)
      return ri;
    };
    // every load of the set-up is issued before the first value of any of them is needed (memory
    // returns in order, so a wait for one is a wait for everything requested before it)
    bf16x8 qf[kQInLds ? 1 : QT][KS];
    uint64_t tree_mask[QT];  // ancestor words of the lane's rows (used by the tree blocks only)
    bf16x8 qtmp[kQInLds ? QT : 1][KS];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      const RowInfo ri = row_info(t);
      const __bf16* qrow = reinterpret_cast<const __bf16*>(p.q) + ri.out * D + 8 * g4;
      tree_mask[t] = ri.valid ? p.anc_mask[b * p.Nmax + ri.node] : 0ull;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        bf16x8 zero;
#pragma unroll
        for (int j = 0; j < 8; ++j) zero[j] = (__bf16)0.f;
        const bf16x8 frag = ri.valid ? *reinterpret_cast<const bf16x8*>(qrow + 32 * ks) : zero;
        if constexpr (kQInLds) qtmp[t][ks] = frag; else qf[t][ks] = frag;
      }
    }
    {
      const uint64_t live_bits = (n >= 64) ? ~0ull : ((1ull << n) - 1ull);
#pragma unroll
      for (int t = 0; t < QT; ++t) {
        tree_mask[t] &= live_bits;
        if constexpr (kQInLds) {
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) q_lds[(t * KS + ks) * 64] = qtmp[t][ks];
        }
      }
    }
    auto q_frag = [&](int t, int ks) -> bf16x8 {
      if constexpr (kQInLds) return q_lds[(t * KS + ks) * 64]; else return qf[t][ks];
    };
    auto mask_of_tile = [&](int t) -> uint64_t { return tree_mask[t]; };

    RowState<QT, D> st;
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      st.m[t] = kNegBig;
      st.l[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int e = 0; e < DT; ++e) st.o[t][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    if (active) {
      int blk = blk_begin;
      if constexpr (kDeep) {
        // long streams of full prefix blocks: a loop of its own with nothing in it but the steady state
        // (the next block is a full block too, so bases advance by a constant and the offsets stay)
        const int full_end = min(blk_end, L / kBlockKeys);
        if (blk + KW < full_end) {
          const int64_t step = (int64_t)kBlockKeys * cache_row_bytes * KW;
          const char* kb = cur.k;
          const char* vb = cur.v;
          BlockSrc full{};  // kind 0
          full.nvalid = kBlockKeys;
          for (; blk + KW < full_end; blk += KW) {
            asm volatile("" ::: "memory");  // keep the Q reads inside the loop (they are the point)
            kb += step;
            vb += step;
            load_k<D, STREAMED>(kfn, kb, koff);
            process_block<QT, D>(st, kf, vr, q_frag, full, mask_of_tile, c, g4, [] {},
                                 [&] { load_v<D, STREAMED>(vr, vb, voff); });
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
              for (int ks = 0; ks < KS; ++ks) kf[kt][ks] = kfn[kt][ks];
          }
          cur = locate(blk);
        }
      }
      for (;; blk += KW) {
        if constexpr (kQInLds) asm volatile("" ::: "memory");  // keep the Q reads inside the loop (they are the point)
        const bool more = blk + KW < blk_end;
        BlockSrc nxt = cur;
        if (more) nxt = locate(blk + KW);
        if constexpr (kDeep) {
          if (more) { set_k(nxt); load_k<D, STREAMED>(kfn, nxt.k, koff); }
          process_block<QT, D>(st, kf, vr, q_frag, cur, mask_of_tile, c, g4, [] {},
                               [&] { if (more) { set_v(nxt); load_v<D, STREAMED>(vr, nxt.v, voff); } });
          if (more) {
#pragma unroll
            for (int kt = 0; kt < 2; ++kt)
#pragma unroll
              for (int ks = 0; ks < KS; ++ks) kf[kt][ks] = kfn[kt][ks];
          }
        } else {
          process_block<QT, D>(st, kf, vr, q_frag, cur, mask_of_tile, c, g4,
                               [&] { if (more) { set_k(nxt); load_k<D, STREAMED>(kf, nxt.k, koff); } }, [] {});
          if (more) { set_v(nxt); load_v<D, STREAMED>(vr, nxt.v, voff); }
        }
        if (!more) break;
        cur = nxt;
      }
    }
    float lsum[QT];  // the matrix-core row sums already cover every key of the wavefront's blocks
#pragma unroll
    for (int t = 0; t < QT; ++t) lsum[t] = st.l[t][0];

    // Writes 4 consecutive d-tiles (e0..e0+3) of row tile t: final rows when the segment is the whole
    // unit, a partial slot otherwise. o4[j][i] belongs to dim DT*(4*g4+i)+e0+j of row 16*t+col.
    auto write_quad = [&](int t, int e0, const f32x4 (&o4)[4], float m_row, float l_row) {
      const RowInfo ri = row_info(t);
      if (!ri.exists) return;
      if (whole_unit) {
        const float inv = ri.valid ? 1.0f / l_row : 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int d0 = DT * (4 * g4 + i) + e0;
          float vals[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) vals[j] = ri.valid ? o4[j][i] * inv : 0.f;
          if (p.out_bf16) {
            typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
            bf16x4 pk;
#pragma unroll
            for (int j = 0; j < 4; ++j) pk[j] = (__bf16)vals[j];
            *reinterpret_cast<bf16x4*>(reinterpret_cast<__bf16*>(p.out) + ri.out * D + d0) = pk;
          } else {
            *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(p.out) + ri.out * D + d0) =
                f32x4{vals[0], vals[1], vals[2], vals[3]};
          }
        }
      } else if (ri.valid) {
        float* slot = p.part + (int64_t)(unit + w) * rows_per_unit * (D + 2);
        const int lr = slab_local * ROWS + 16 * t + col;
        if (g4 == 0 && e0 == 0) *reinterpret_cast<float2*>(slot + (int64_t)rows_per_unit * D + 2 * lr) = make_float2(m_row, l_row);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          *reinterpret_cast<f32x4*>(slot + (int64_t)lr * D + DT * (4 * g4 + i) + e0) =
              f32x4{o4[0][i], o4[1][i], o4[2][i], o4[3][i]};
      }
    };

    // The key-splitting wavefronts of a slab leave their states in lane-private LDS slots; after one
    // barrier each of them reduces and writes its own share of the (row tile, 4 d-tiles) quads, so
    // the tail of a short-lived workgroup is spread over all its wavefronts.
    // (KW is 2 or 4. The test stands for the large tiles, whose merge the compiler otherwise mixes with the end of the
    // stream: 20 layers of 4 x 52 heads, 4096 keys, 60 nodes 1665 us with it, 1703 without; smaller tiles are faster without)
    if (!kQInLds || KW > 1) {
      if (kQInLds) __syncthreads();  // every wavefront is done with its Q slots before they are overwritten
#pragma unroll
      for (int t = 0; t < QT; ++t) {
        merge_ml[wave][t][lane] = make_float2(st.m[t], lsum[t]);
#pragma unroll
        for (int e = 0; e < DT; ++e) merge_o[wave][t * DT + e][lane] = st.o[t][e];
      }
      __syncthreads();
      constexpr int kQuadsPerTile = DT / 4;
      for (int q = kp; q < QT * kQuadsPerTile; q += KW) {
        const int t = q / kQuadsPerTile, e0 = 4 * (q - t * kQuadsPerTile);
        float mm = kNegBig;
        for (int k = 0; k < KW; ++k) mm = fmaxf(mm, merge_ml[slab_local + k * p.WS][t][lane].x);
        float l_row = 0.f;
        f32x4 o4[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) o4[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int k = 0; k < KW; ++k) {  // in wavefront order: deterministic
          const int peer = slab_local + k * p.WS;
          const float2 ml = merge_ml[peer][t][lane];
          const float a = __builtin_amdgcn_exp2f(ml.x - mm);
          l_row += ml.y * a;
#pragma unroll
          for (int j = 0; j < 4; ++j) o4[j] += merge_o[peer][t * DT + e0 + j][lane] * a;
        }
        write_quad(t, e0, o4, mm, l_row);
      }
    }
    r += (unsigned)count;
    if (b + 1 < p.B && r >= seq_first_block(p, b + 1)) ++b;
    if (r < r1) __syncthreads();  // the LDS buffers are reused by the next segment
  }
}

// ---------------------------------------------------------------------------------------------
// GQA with many query rows per kv head (more than 128): wavefronts of 32 rows, four to a set that holds 128 rows of one kv head.
// At 32 rows a wavefront cannot afford to fetch every K/V block for itself (four to eight copies of each block through the
// texture path is what would bound the kernel): the set fetches each block once, every wavefront copying a quarter of it into
// LDS with the global-to-LDS load (row-contiguous requests, no registers), and all of them pick their operands out of there.
// A workgroup is two sets (three for head dim 64), its key groups, on the same rows: they take alternate blocks of the
// workgroup's segment and merge their states through LDS at the segment's end. One workgroup of eight (twelve) wavefronts per
// compute unit holds as many wavefronts as two of four, but a cut unit leaves one partial result per workgroup.
// Head dim 64: three stages of one block per key group: stage i is read while i+1 and i+2 are in flight. K is kept swizzled
// (16-byte chunk c of row r at slot c ^ f(r)) so that a fragment read, 16 rows by one chunk, touches 16 different bank groups.
struct Stage {
  static constexpr int D = 64, WAVES = 4;
  static constexpr int kChunks = D / 8;                      // 16-byte chunks per row
  static constexpr int kRowsPerLoad = 64 / kChunks;          // rows one copy instruction covers
  static constexpr int kLoads = kBlockKeys / kRowsPerLoad;   // copy instructions per tensor and block
  static constexpr int kTensorBytes = kBlockKeys * D * 2;
  static constexpr int kBytes = 2 * kTensorBytes;            // K then V
  static constexpr int kPerWave = 2 * kLoads / WAVES;        // copy instructions per wavefront and block
  __device__ static __forceinline__ int swizzle(int r) { return (r >> 1) & 7; }
};
typedef const __attribute__((address_space(1))) void* GlobalPtr;
typedef __attribute__((address_space(3))) void* LdsPtr;

__global__ __launch_bounds__(768) void tree_attn_gqa64_kernel(const SharedParams) {
  i32x4 class_wg;
  const AttnArgs p = fetch_args(class_wg);
  typedef Stage S;
  constexpr int D = S::D, KG = 3, QT = 2, KS = D / 32, DT = D / 16, ROWS = 32, kWaves = S::WAVES, kStages = 3;
  constexpr int kGroupBytes = kStages * S::kBytes;
  // the merge needs (DT + 1) 16-byte slots per lane, tile and wavefront of every key group but the first
  constexpr int kMergeBytes = (KG - 1) * kWaves * QT * (DT + 1) * 64 * 16;
  constexpr int kLdsBytes = KG * kGroupBytes > kMergeBytes ? KG * kGroupBytes : kMergeBytes;
  __shared__ __attribute__((aligned(16))) char lds_all[kLdsBytes];

  const int lane = threadIdx.x & 63, wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kg = wave_all / kWaves;     // key group of this wavefront
  const int wave = wave_all % kWaves;   // its row slab within the workgroup
  char* const stages = lds_all + kg * kGroupBytes;
  const int col = lane & 15, g4 = lane >> 4;
  const float c = p.scale * kLog2e;
  const unsigned tree_row_bytes = (unsigned)p.Hkv * D * 2u;
  const unsigned cache_row_bytes = (unsigned)p.stride_token * 2u;
  constexpr int rows_per_unit = kWaves * ROWS;

  // this wavefront's copy instructions: index x < kLoads is K rows, the others V rows
  int dma_tensor[S::kPerWave], dma_row[S::kPerWave], dma_chunk[S::kPerWave], dma_dst[S::kPerWave];
#pragma unroll
  for (int i = 0; i < S::kPerWave; ++i) {
    const int x = wave + kWaves * i;
    const int n = x % S::kLoads;
    dma_tensor[i] = x / S::kLoads;
    dma_row[i] = n * S::kRowsPerLoad + lane / S::kChunks;
    const int chunk = lane & (S::kChunks - 1);
    dma_chunk[i] = dma_tensor[i] == 0 ? (chunk ^ S::swizzle(dma_row[i])) : chunk;
    dma_dst[i] = dma_tensor[i] * S::kTensorBytes + n * 1024;
  }
  // this lane's operand reads: K fragments (key tile 0; tile 1 is 16 rows further), V rows
  unsigned kfrag[KS], vrow[8];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) kfrag[ks] = (unsigned)col * (D * 2) + 16u * ((4 * ks + g4) ^ S::swizzle(col));
#pragma unroll
  for (int j = 0; j < 8; ++j) vrow[j] = S::kTensorBytes + (unsigned)key_of(g4, j) * (D * 2) + (unsigned)(D / 8) * col;

  const Share share = share_of(p, class_wg, blockIdx.x);
  const unsigned r1 = share.r1;
  const int y = share.y;
  int at_seq = seq_of_block(p, share.r0, share.first_seq);   // place in the launch's order of sequences

  for (unsigned r = share.r0; r < r1;) {
    const Seq seq = seq_at(p, at_seq);
    const int n = seq.n, L = seq.len, b = seq.place;
    const int n_prefix_blocks = (L + kBlockKeys - 1) / kBlockKeys;
    const int n_blocks = n_prefix_blocks + (n + kBlockKeys - 1) / kBlockKeys;
    const unsigned rel = r - seq.first;
    const int counted = n_blocks + p.setup;
    const int g = unit_of_block(p, rel, counted);
    const int from = (int)(rel - (unsigned)g * (unsigned)counted), count = min(counted - from, (int)(r1 - r));
    const int seg_begin = max(from - p.setup, 0), seg_count = from + count - p.setup - seg_begin;
    const int n_slabs = seq_slabs(p, n, ROWS), n_groups = seq_groups(p, n_slabs);
    if (seg_count <= 0 || y >= n_groups) {   // nothing but set-up, or no rows for this slab group (classes put together)
      r += (unsigned)count;
      if (at_seq + 1 < p.B && r >= seq_first_block(p, at_seq + 1)) ++at_seq;
      continue;
    }
    const int unit = share.slot + (at_seq - share.first_seq) * p.Hkv + g;   // partial slot
    const bool whole_unit = seg_count == n_blocks;
    const int slab = y * kWaves + wave;
    const bool slab_live = slab < p.NS;          // has output rows
    const bool slab_works = slab < n_slabs;      // has rows of the tree
    if (seg_begin == 0 && y == 0) {
      const int covered = n_groups * rows_per_unit;
      if (covered < p.Nmax * p.G) zero_rows<D, 64 * kWaves * KG>(p, b, g, covered);
    }

    const char* kc = reinterpret_cast<const char*>(p.k_cache) + (b * p.stride_batch + g * p.stride_head) * 2;
    const char* vc = reinterpret_cast<const char*>(p.v_cache) + (b * p.stride_batch + g * p.stride_head) * 2;
    const char* ktr = reinterpret_cast<const char*>(p.k_tree) + ((int64_t)b * p.Nmax * p.Hkv + g) * (D * 2);
    const char* vtr = reinterpret_cast<const char*>(p.v_tree) + ((int64_t)b * p.Nmax * p.Hkv + g) * (D * 2);

    auto locate = [&](int blk) {
      BlockSrc src;
      if (blk < n_prefix_blocks) {
        const int key0 = blk * kBlockKeys;
        const int64_t byte0 = (int64_t)key0 * cache_row_bytes;
        src.k = kc + byte0;
        src.v = vc + byte0;
        src.row_bytes = cache_row_bytes;
        src.nvalid = min(kBlockKeys, L - key0);
        src.kind = src.nvalid == kBlockKeys ? 0 : 1;
        src.tree_key0 = 0;
      } else {
        const int t0 = (blk - n_prefix_blocks) * kBlockKeys;
        src.k = ktr + t0 * tree_row_bytes;
        src.v = vtr + t0 * tree_row_bytes;
        src.row_bytes = tree_row_bytes;
        src.nvalid = min(kBlockKeys, n - t0);
        src.kind = 2;
        src.tree_key0 = t0;
      }
      return src;
    };
    // request this wavefront's share of a block into a stage (rows past the end are clamped; masked later)
    auto request_block = [&](const BlockSrc& s, int stage) {
#pragma unroll
      for (int i = 0; i < S::kPerWave; ++i) {
        const unsigned off = (unsigned)min(dma_row[i], s.nvalid - 1) * s.row_bytes + 16u * dma_chunk[i];
        const char* src = (dma_tensor[i] == 0 ? s.k : s.v) + off;
        __builtin_amdgcn_global_load_lds((GlobalPtr)src, (LdsPtr)(stages + stage * S::kBytes + dma_dst[i]), 16, 0, 0);
      }
    };
    // key group kg takes blocks kg, kg + KG, ... of the segment
    const int blk_begin = seg_begin + kg, blk_end = seg_begin + seg_count;
    auto request_group = [&](int first, int stage) {
      if (first < blk_end) request_block(locate(first), stage);
    };

    request_group(blk_begin, 0);
    request_group(blk_begin + KG, 1);

    struct RowInfo { bool exists, valid; int node; int64_t out; };
    auto row_info = [&](int t) {
      RowInfo ri;
      const int rr = slab * ROWS + 16 * t + col;
      ri.node = (int)div_magic((unsigned)rr, p.G, p.g_magic);
      const int hl = rr - ri.node * p.G;
      ri.exists = slab_live && rr < p.Nmax * p.G;
      ri.valid = ri.exists && ri.node < n;
      ri.out = ((int64_t)b * p.Nmax + ri.node) * p.Hq + g * p.G + hl;
      return ri;
    };
    bf16x8 qf[QT][KS];
    uint64_t tree_mask[QT];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      const RowInfo ri = row_info(t);
      const __bf16* qrow = reinterpret_cast<const __bf16*>(p.q) + ri.out * D + 8 * g4;
      tree_mask[t] = ri.valid ? p.anc_mask[b * p.Nmax + ri.node] : 0ull;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        bf16x8 zero;
#pragma unroll
        for (int j = 0; j < 8; ++j) zero[j] = (__bf16)0.f;
        qf[t][ks] = ri.valid ? *reinterpret_cast<const bf16x8*>(qrow + 32 * ks) : zero;
      }
    }
    {
      const uint64_t live_bits = (n >= 64) ? ~0ull : ((1ull << n) - 1ull);
#pragma unroll
      for (int t = 0; t < QT; ++t) tree_mask[t] &= live_bits;
    }
    auto q_frag = [&](int t, int ks) -> bf16x8 { return qf[t][ks]; };
    auto mask_of_tile = [&](int t) -> uint64_t { return tree_mask[t]; };

    RowState<QT, D> st;
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      st.m[t] = kNegBig;
      st.l[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int e = 0; e < DT; ++e) st.o[t][e] = f32x4{0.f, 0.f, 0.f, 0.f};
    }

    int stage = 0;
    // every wavefront of the workgroup takes the same number of turns (the barriers are the whole
    // workgroup's): as many as key group 0 has blocks; a group whose blocks have run out idles
    const int n_turns = (seg_count + KG - 1) / KG;
    for (int turn = 0, first = blk_begin; turn < n_turns; ++turn, first += KG) {
      // this turn's copies have landed (the next turn's, requested after them, may still be in
      // flight); the barrier makes every wavefront's share visible and retires the stage that the
      // turn after the next is about to overwrite
      if (first + KG < blk_end) asm volatile("s_waitcnt vmcnt(%0)" : : "n"(S::kPerWave) : "memory");
      else asm volatile("s_waitcnt vmcnt(0)" : : : "memory");
      __syncthreads();
      request_group(first + 2 * KG, stage == 0 ? 2 : stage - 1);
      if (slab_works && first < blk_end) {
        const BlockSrc cur = locate(first);
        const char* sbase = stages + stage * S::kBytes;
        bf16x8 kf[2][KS];
        unsigned vr[8][D / 32];
#pragma unroll
        for (int kt = 0; kt < 2; ++kt)
#pragma unroll
          for (int ks = 0; ks < KS; ++ks)
            kf[kt][ks] = *reinterpret_cast<const bf16x8*>(sbase + kt * 16 * (D * 2) + kfrag[ks]);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const u32x2 x = *reinterpret_cast<const u32x2*>(sbase + vrow[j]);
          vr[j][0] = x[0]; vr[j][1] = x[1];
        }
        process_block<QT, D>(st, kf, vr, q_frag, cur, mask_of_tile, c, g4, [] {}, [] {});
      }
      stage = stage == 2 ? 0 : stage + 1;
    }

    // the other key groups hand their states over in lane-private LDS slots (the stages are free
    // once every wavefront has left the loop); wavefront w of the first group and wavefront w of the
    // second hold the same rows in the same lanes, so the merge is lane by lane and in a fixed order
    __syncthreads();
    constexpr int kGroupSlots = kWaves * QT * (DT + 1) * 64;   // 16-byte slots one group hands over
    f32x4* const mbuf0 = reinterpret_cast<f32x4*>(lds_all) + (wave * QT * (DT + 1)) * 64 + lane;
    if (kg >= 1 && slab_live) {
      f32x4* mbuf = mbuf0 + (kg - 1) * kGroupSlots;
#pragma unroll
      for (int t = 0; t < QT; ++t) {
#pragma unroll
        for (int e = 0; e < DT; ++e) mbuf[(t * (DT + 1) + e) * 64] = st.o[t][e];
        mbuf[(t * (DT + 1) + DT) * 64] = f32x4{st.m[t], st.l[t][0], 0.f, 0.f};
      }
    }
    __syncthreads();
    if (kg == 0 && slab_live) {
#pragma unroll
      for (int other = 1; other < KG; ++other) {   // in group order: deterministic
        const f32x4* mbuf = mbuf0 + (other - 1) * kGroupSlots;
#pragma unroll
        for (int t = 0; t < QT; ++t) {
          const f32x4 ml = mbuf[(t * (DT + 1) + DT) * 64];
          const float mm = fmaxf(st.m[t], ml[0]);
          const float a0 = __builtin_amdgcn_exp2f(st.m[t] - mm), a1 = __builtin_amdgcn_exp2f(ml[0] - mm);
          st.m[t] = mm;
          st.l[t] = st.l[t] * a0 + ml[1] * a1;
#pragma unroll
          for (int e = 0; e < DT; ++e) st.o[t][e] = st.o[t][e] * a0 + mbuf[(t * (DT + 1) + e) * 64] * a1;
        }
      }
    }

    // every wavefront (of the first key group) owns its rows: final rows or a partial slot, straight from registers
    if (slab_live && kg == 0) {
#pragma unroll
      for (int t = 0; t < QT; ++t) {
        const RowInfo ri = row_info(t);
        if (!ri.exists) continue;
        const float l_row = st.l[t][0];
#pragma unroll
        for (int e0 = 0; e0 < DT; e0 += 4) {
          if (whole_unit) {
            const float inv = ri.valid ? 1.0f / l_row : 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int d0 = DT * (4 * g4 + i) + e0;
              float vals[4];
#pragma unroll
              for (int j = 0; j < 4; ++j) vals[j] = ri.valid ? st.o[t][e0 + j][i] * inv : 0.f;
              if (p.out_bf16) {
                typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
                bf16x4 pk;
#pragma unroll
                for (int j = 0; j < 4; ++j) pk[j] = (__bf16)vals[j];
                *reinterpret_cast<bf16x4*>(reinterpret_cast<__bf16*>(p.out) + ri.out * D + d0) = pk;
              } else {
                *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(p.out) + ri.out * D + d0) =
                    f32x4{vals[0], vals[1], vals[2], vals[3]};
              }
            }
          } else if (ri.valid) {
            float* slot = p.part + (int64_t)unit * rows_per_unit * (D + 2);
            const int lr = wave * ROWS + 16 * t + col;
            if (g4 == 0 && e0 == 0) *reinterpret_cast<float2*>(slot + (int64_t)rows_per_unit * D + 2 * lr) = make_float2(st.m[t], l_row);
#pragma unroll
            for (int i = 0; i < 4; ++i)
              store_through(slot + partial_index<D>(lr, (DT * (4 * g4 + i) + e0) / 4), f32x4{st.o[t][e0][i], st.o[t][e0 + 1][i], st.o[t][e0 + 2][i], st.o[t][e0 + 3][i]});
          }
        }
      }
    }
    r += (unsigned)count;
    if (at_seq + 1 < p.B && r >= seq_first_block(p, at_seq + 1)) ++at_seq;
    __syncthreads();  // every wavefront is done with the stages before the next segment refills them
  }
}

// ---------------------------------------------------------------------------------------------
// The same decomposition for head dim 128 (four wavefronts of 32 rows, two key groups, K/V blocks shared through LDS), with
// the matrix products as 32x32x16 tiles and every operand read issued half a turn ahead of its products.
//
// A turn is one 32-key block per wavefront. Its parts bound it about alike (64 / 8 heads, 60 nodes, us per 16384 keys: the
// products alone 15.0, with weights and operand reads 21.6, the copies alone 20.0, all of it 28), so it is written as three
// parts that hide each other:
//   pv      O^T += V^T P^T of block i           under it the K operands of block i + 1 are read from LDS
//   qk      S^T = K Q^T of block i + 1          under it the V operands of block i + 1
//   weights p = 2^(S c - m), row sums           vector work only, no LDS
// Vector and LDS instructions issue beside a 32x32x16 product at their own rate, of the same wavefront and of the SIMD's other
// one (17 products with 48 vector instructions among them 564 clocks, the products alone 548; beside 16x16x32 products the
// vector instructions take 525 instead of 399). The two key groups stand half a turn apart: the turn's one barrier comes
// after `weights` in group 0 and before it in group 1, so that the vector part of one runs beside the products of the other.
// The copies stand behind the products: issued among them they stalled the wavefront (28 -> 37). Rings of five blocks: as four; of three, as
// they are: as four too (64 / 8 heads, 16384 keys 45.3, with four and the query rows in the fourth slot at first 45.7 us a call).
// What a short segment costs is its start. The products begin when block 0 is there, which takes that nothing of a segment's set-up
// is loaded into registers (see the query rows); a segment copies the blocks that it has and no more. Against rows in registers, for
// which the compiler waited for the whole ring, and a fixed number of copies a turn, us a call: 32 / 8 heads, 60 nodes, 300 keys 13.7 -> 12.6,
// 1000 keys 16.4 -> 15.2, 4096 keys 19.9 -> 18.3, 8192 keys 23.6 -> 22.1; 4 sequences of 4096 keys 32.4 -> 31.2; 28 / 4 heads, 9000 keys 19.9 -> 19.4.
// Against 16x16x32 tiles with the reads in front of their products: 64 / 8 heads, 16384 keys 53.9 -> 52.0 us a call, 32 / 8
// heads, 1000 keys 15.0 -> 14.7, 4096 keys 20.3 -> 20.4.
//
// Blocks lie in LDS row by row as they are copied (whole rows per request: as 64-byte pieces a 32 / 8-head call over 4096 keys
// took a microsecond more), with the 16-byte chunks of a K row exchanged by key (c at c ^ (key & 15)) and the 64-byte pieces of
// a V row (d at d ^ (key & 3)): reads then touch every bank once a pass.
constexpr int kWideRing = 3;                        // K and V blocks that a key group holds
constexpr int kWideTensor = kBlockKeys * 128 * 2;  // bytes of one tensor's block
constexpr int kWideGroup = 2 * kWideRing * kWideTensor;
constexpr int kWideQ = 2 * kWideGroup;              // the unit's 128 query rows, behind the rings
constexpr int kWideMasks = kWideQ + 128 * 128 * 2;  // and the lanes' ancestor words
// Weights stay below 2: a score that would go above moves its row's shift to 2^7 times the largest weight so far (the test is
// the exponent's top bit of the packed weights). As with kLazyLog2, shifts move almost never after the first blocks.
constexpr float kWideHeadroom = 7.0f;

// O^T += V^T P^T of a block (v[s][dt]: 16 keys, 32 dims), and the K operands of the next block out of LDS.
__device__ __forceinline__ void pv_reading_k(f32x16 (&o)[4], const bf16x8 (&v)[2][4], const bf16x8 (&w)[2], bf16x8 (&k)[8], unsigned ka) {
  unsigned a0, a1;
  asm volatile(
      "ds_read_b128 %[k0], %[ka]\n\tv_xor_b32 %[a1], 32, %[ka]\n\tds_read_b128 %[k1], %[a1]\n\ts_nop 1\n\t"
      "v_mfma_f32_32x32x16_bf16 %[o0], %[v00], %[w0], %[o0]\n\tv_xor_b32 %[a0], 64, %[ka]\n\tds_read_b128 %[k2], %[a0]\n\t"
      "v_mfma_f32_32x32x16_bf16 %[o1], %[v01], %[w0], %[o1]\n\tv_xor_b32 %[a1], 0x60, %[ka]\n\tds_read_b128 %[k3], %[a1]\n\t"
      "v_mfma_f32_32x32x16_bf16 %[o2], %[v02], %[w0], %[o2]\n\tv_xor_b32 %[a0], 0x80, %[ka]\n\tds_read_b128 %[k4], %[a0]\n\t"
      "v_mfma_f32_32x32x16_bf16 %[o3], %[v03], %[w0], %[o3]\n\tv_xor_b32 %[a1], 0xa0, %[ka]\n\tds_read_b128 %[k5], %[a1]\n\t"
      "v_mfma_f32_32x32x16_bf16 %[o0], %[v10], %[w1], %[o0]\n\tv_xor_b32 %[a0], 0xc0, %[ka]\n\tds_read_b128 %[k6], %[a0]\n\t"
      "v_mfma_f32_32x32x16_bf16 %[o1], %[v11], %[w1], %[o1]\n\tv_xor_b32 %[a1], 0xe0, %[ka]\n\tds_read_b128 %[k7], %[a1]\n\t"
      "v_mfma_f32_32x32x16_bf16 %[o2], %[v12], %[w1], %[o2]\n\tv_mfma_f32_32x32x16_bf16 %[o3], %[v13], %[w1], %[o3]\n\t"
      "s_waitcnt lgkmcnt(0)"
      : [o0] "+v"(o[0]), [o1] "+v"(o[1]), [o2] "+v"(o[2]), [o3] "+v"(o[3]), [k0] "=&v"(k[0]), [k1] "=&v"(k[1]), [k2] "=&v"(k[2]),
        [k3] "=&v"(k[3]), [k4] "=&v"(k[4]), [k5] "=&v"(k[5]), [k6] "=&v"(k[6]), [k7] "=&v"(k[7]), [a0] "=&v"(a0), [a1] "=&v"(a1)
      : [v00] "v"(v[0][0]), [v01] "v"(v[0][1]), [v02] "v"(v[0][2]), [v03] "v"(v[0][3]), [v10] "v"(v[1][0]), [v11] "v"(v[1][1]),
        [v12] "v"(v[1][2]), [v13] "v"(v[1][3]), [w0] "v"(w[0]), [w1] "v"(w[1]), [ka] "v"(ka)
      : "memory");
}
// K operands alone (a segment's first block), and those of the query rows
__device__ __forceinline__ void read_k(bf16x8 (&k)[8], unsigned ka) {
  unsigned a0, a1;
  asm volatile(
      "ds_read_b128 %[k0], %[ka]\n\tv_xor_b32 %[a0], 32, %[ka]\n\tds_read_b128 %[k1], %[a0]\n\tv_xor_b32 %[a1], 64, %[ka]\n\t"
      "ds_read_b128 %[k2], %[a1]\n\tv_xor_b32 %[a0], 0x60, %[ka]\n\tds_read_b128 %[k3], %[a0]\n\tv_xor_b32 %[a1], 0x80, %[ka]\n\t"
      "ds_read_b128 %[k4], %[a1]\n\tv_xor_b32 %[a0], 0xa0, %[ka]\n\tds_read_b128 %[k5], %[a0]\n\tv_xor_b32 %[a1], 0xc0, %[ka]\n\t"
      "ds_read_b128 %[k6], %[a1]\n\tv_xor_b32 %[a0], 0xe0, %[ka]\n\tds_read_b128 %[k7], %[a0]\n\ts_waitcnt lgkmcnt(0)"
      : [k0] "=&v"(k[0]), [k1] "=&v"(k[1]), [k2] "=&v"(k[2]), [k3] "=&v"(k[3]), [k4] "=&v"(k[4]), [k5] "=&v"(k[5]), [k6] "=&v"(k[6]), [k7] "=&v"(k[7]),
        [a0] "=&v"(a0), [a1] "=&v"(a1)
      : [ka] "v"(ka)
      : "memory");
}
// this lane's ancestor word: its halves lie 256 bytes apart
__device__ __forceinline__ uint64_t read_mask(unsigned at) {
  unsigned lo, hi;
  asm volatile("ds_read_b32 %0, %2\n\tds_read_b32 %1, %2 offset:256\n\ts_waitcnt lgkmcnt(0)" : "=&v"(lo), "=&v"(hi) : "v"(at) : "memory");
  return ((uint64_t)hi << 32) | lo;
}
// S^T = K Q^T of a block, and its V operands out of LDS (r: halves of v[s][dt], four keys each). The wait states at the end are
// those between a matrix instruction and a vector instruction that reads its result.
__device__ __forceinline__ void qk_reading_v(f32x16& s, const bf16x8 (&k)[8], const bf16x8 (&q)[8], u32x2 (&r)[16], unsigned va) {
  unsigned a0, a1;
  asm volatile(
      "v_mfma_f32_32x32x16_bf16 %[s], %[k0], %[q0], 0\n\tds_read_b64_tr_b16 %[r0], %[va]\n\t"
      "ds_read_b64_tr_b16 %[r1], %[va] offset:2048\n\tv_mfma_f32_32x32x16_bf16 %[s], %[k1], %[q1], %[s]\n\t"
      "ds_read_b64_tr_b16 %[r8], %[va] offset:4096\n\tds_read_b64_tr_b16 %[r9], %[va] offset:6144\n\t"
      "v_mfma_f32_32x32x16_bf16 %[s], %[k2], %[q2], %[s]\n\tv_xor_b32 %[a1], 0x40, %[va]\n\tds_read_b64_tr_b16 %[r2], %[a1]\n\t"
      "ds_read_b64_tr_b16 %[r3], %[a1] offset:2048\n\tv_mfma_f32_32x32x16_bf16 %[s], %[k3], %[q3], %[s]\n\t"
      "ds_read_b64_tr_b16 %[r10], %[a1] offset:4096\n\tds_read_b64_tr_b16 %[r11], %[a1] offset:6144\n\t"
      "v_mfma_f32_32x32x16_bf16 %[s], %[k4], %[q4], %[s]\n\tv_xor_b32 %[a0], 0x80, %[va]\n\tds_read_b64_tr_b16 %[r4], %[a0]\n\t"
      "ds_read_b64_tr_b16 %[r5], %[a0] offset:2048\n\tv_mfma_f32_32x32x16_bf16 %[s], %[k5], %[q5], %[s]\n\t"
      "ds_read_b64_tr_b16 %[r12], %[a0] offset:4096\n\tds_read_b64_tr_b16 %[r13], %[a0] offset:6144\n\t"
      "v_mfma_f32_32x32x16_bf16 %[s], %[k6], %[q6], %[s]\n\tv_xor_b32 %[a1], 0xc0, %[va]\n\tds_read_b64_tr_b16 %[r6], %[a1]\n\t"
      "ds_read_b64_tr_b16 %[r7], %[a1] offset:2048\n\tv_mfma_f32_32x32x16_bf16 %[s], %[k7], %[q7], %[s]\n\t"
      "ds_read_b64_tr_b16 %[r14], %[a1] offset:4096\n\tds_read_b64_tr_b16 %[r15], %[a1] offset:6144\n\ts_waitcnt lgkmcnt(0)\n\t"
      "s_nop 13"
      : [s] "=&v"(s), [a0] "=&v"(a0), [a1] "=&v"(a1), [r0] "=&v"(r[0]), [r1] "=&v"(r[1]), [r2] "=&v"(r[2]), [r3] "=&v"(r[3]), [r4] "=&v"(r[4]), [r5] "=&v"(r[5]),
        [r6] "=&v"(r[6]), [r7] "=&v"(r[7]), [r8] "=&v"(r[8]), [r9] "=&v"(r[9]), [r10] "=&v"(r[10]), [r11] "=&v"(r[11]),
        [r12] "=&v"(r[12]), [r13] "=&v"(r[13]), [r14] "=&v"(r[14]), [r15] "=&v"(r[15])
      : [k0] "v"(k[0]), [k1] "v"(k[1]), [k2] "v"(k[2]), [k3] "v"(k[3]), [k4] "v"(k[4]), [k5] "v"(k[5]), [k6] "v"(k[6]),
        [k7] "v"(k[7]), [q0] "v"(q[0]), [q1] "v"(q[1]), [q2] "v"(q[2]), [q3] "v"(q[3]), [q4] "v"(q[4]), [q5] "v"(q[5]),
        [q6] "v"(q[6]), [q7] "v"(q[7]), [va] "v"(va)
      : "memory");
}

// Weights p = 2^(s c - m) of a row's 16 keys in bf16, and their sum added to l. `grow`: lanes with a weight of 2 or more.
__device__ __forceinline__ void weights_of(const f32x16& s, float c, float m, unsigned (&p)[8], float& l, uint64_t& grow) {
  float t[16];
  unsigned x;
  asm volatile(
      "v_fma_f32 %[t0], %[s0], %[c], -%[m]\n\tv_fma_f32 %[t1], %[s1], %[c], -%[m]\n\tv_fma_f32 %[t2], %[s2], %[c], -%[m]\n\t"
      "v_fma_f32 %[t3], %[s3], %[c], -%[m]\n\tv_exp_f32 %[t0], %[t0]\n\tv_fma_f32 %[t4], %[s4], %[c], -%[m]\n\t"
      "v_exp_f32 %[t1], %[t1]\n\tv_fma_f32 %[t5], %[s5], %[c], -%[m]\n\tv_exp_f32 %[t2], %[t2]\n\t"
      "v_fma_f32 %[t6], %[s6], %[c], -%[m]\n\tv_exp_f32 %[t3], %[t3]\n\tv_fma_f32 %[t7], %[s7], %[c], -%[m]\n\t"
      "v_exp_f32 %[t4], %[t4]\n\tv_fma_f32 %[t8], %[s8], %[c], -%[m]\n\tv_exp_f32 %[t5], %[t5]\n\t"
      "v_fma_f32 %[t9], %[s9], %[c], -%[m]\n\tv_exp_f32 %[t6], %[t6]\n\tv_fma_f32 %[t10], %[s10], %[c], -%[m]\n\t"
      "v_exp_f32 %[t7], %[t7]\n\tv_fma_f32 %[t11], %[s11], %[c], -%[m]\n\tv_exp_f32 %[t8], %[t8]\n\t"
      "v_fma_f32 %[t12], %[s12], %[c], -%[m]\n\tv_exp_f32 %[t9], %[t9]\n\tv_fma_f32 %[t13], %[s13], %[c], -%[m]\n\t"
      "v_exp_f32 %[t10], %[t10]\n\tv_fma_f32 %[t14], %[s14], %[c], -%[m]\n\tv_exp_f32 %[t11], %[t11]\n\t"
      "v_fma_f32 %[t15], %[s15], %[c], -%[m]\n\tv_exp_f32 %[t12], %[t12]\n\tv_cvt_pk_bf16_f32 %[p0], %[t0], %[t1]\n\t"
      "v_cvt_pk_bf16_f32 %[p1], %[t2], %[t3]\n\tv_exp_f32 %[t13], %[t13]\n\tv_dot2c_f32_bf16 %[l], 0x3f803f80, %[p0]\n\t"
      "v_cvt_pk_bf16_f32 %[p2], %[t4], %[t5]\n\tv_exp_f32 %[t14], %[t14]\n\tv_dot2c_f32_bf16 %[l], 0x3f803f80, %[p1]\n\t"
      "v_cvt_pk_bf16_f32 %[p3], %[t6], %[t7]\n\tv_exp_f32 %[t15], %[t15]\n\tv_dot2c_f32_bf16 %[l], 0x3f803f80, %[p2]\n\t"
      "v_cvt_pk_bf16_f32 %[p4], %[t8], %[t9]\n\tv_dot2c_f32_bf16 %[l], 0x3f803f80, %[p3]\n\t"
      "v_cvt_pk_bf16_f32 %[p5], %[t10], %[t11]\n\tv_dot2c_f32_bf16 %[l], 0x3f803f80, %[p4]\n\t"
      "v_or3_b32 %[x], %[p0], %[p1], %[p2]\n\tv_cvt_pk_bf16_f32 %[p6], %[t12], %[t13]\n\t"
      "v_dot2c_f32_bf16 %[l], 0x3f803f80, %[p5]\n\tv_or3_b32 %[x], %[x], %[p3], %[p4]\n\t"
      "v_cvt_pk_bf16_f32 %[p7], %[t14], %[t15]\n\tv_dot2c_f32_bf16 %[l], 0x3f803f80, %[p6]\n\t"
      "v_or3_b32 %[x], %[x], %[p5], %[p6]\n\tv_dot2c_f32_bf16 %[l], 0x3f803f80, %[p7]\n\tv_or_b32 %[x], %[x], %[p7]\n\t"
      "v_and_b32 %[x], 0x40004000, %[x]\n\tv_cmp_ne_u32_e64 %[g], 0, %[x]"
      : [p0] "=&v"(p[0]), [p1] "=&v"(p[1]), [p2] "=&v"(p[2]), [p3] "=&v"(p[3]), [p4] "=&v"(p[4]), [p5] "=&v"(p[5]),
        [p6] "=&v"(p[6]), [p7] "=&v"(p[7]), [t0] "=&v"(t[0]), [t1] "=&v"(t[1]), [t2] "=&v"(t[2]), [t3] "=&v"(t[3]),
        [t4] "=&v"(t[4]), [t5] "=&v"(t[5]), [t6] "=&v"(t[6]), [t7] "=&v"(t[7]), [t8] "=&v"(t[8]), [t9] "=&v"(t[9]),
        [t10] "=&v"(t[10]), [t11] "=&v"(t[11]), [t12] "=&v"(t[12]), [t13] "=&v"(t[13]), [t14] "=&v"(t[14]), [t15] "=&v"(t[15]),
        [x] "=&v"(x), [l] "+v"(l), [g] "=&s"(grow)
      : [s0] "v"(s[0]), [s1] "v"(s[1]), [s2] "v"(s[2]), [s3] "v"(s[3]), [s4] "v"(s[4]), [s5] "v"(s[5]), [s6] "v"(s[6]),
        [s7] "v"(s[7]), [s8] "v"(s[8]), [s9] "v"(s[9]), [s10] "v"(s[10]), [s11] "v"(s[11]), [s12] "v"(s[12]), [s13] "v"(s[13]),
        [s14] "v"(s[14]), [s15] "v"(s[15]), [c] "v"(c), [m] "v"(m));
}

__global__ __launch_bounds__(512) void tree_attn_gqa128_kernel(const SharedParams) {
  i32x4 class_wg;
  const AttnArgs p = fetch_args(class_wg);
  constexpr int D = 128, KG = 2, WAVES = 4, ROWS = 32, rows_per_unit = WAVES * ROWS;
  __shared__ __attribute__((aligned(1024))) char lds_all[kWideMasks + KG * WAVES * 512];

  const int lane = threadIdx.x & 63, wave_all = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kg = wave_all >> 2, wave = wave_all & 3;   // key group, row slab within the workgroup
  char* const ring = lds_all + kg * kWideGroup;        // K blocks, then V blocks
  const int row = lane & 31, h = lane >> 5;
  const float c = p.scale * kLog2e;
  const unsigned tree_row_bytes = (unsigned)p.Hkv * D * 2u;
  const unsigned cache_row_bytes = (unsigned)p.stride_token * 2u;

  // this wavefront's copies: eight keys of each tensor, four per instruction (this lane: key copy_key, and copy_key + 4)
  const int copy_key = 8 * wave + (lane >> 4);
  const unsigned chunk = lane & 15;
  const unsigned k_chunk[2] = {16u * (chunk ^ (copy_key & 15)), 16u * (chunk ^ ((copy_key + 4) & 15))}, v_chunk = 16u * (chunk ^ (4 * (copy_key & 3)));
  const unsigned copy_dst = 2048u * wave;
  // this lane's operand reads of a block in slot 0
  const unsigned lds0 = (unsigned)(uintptr_t)(LdsPtr)ring;
  const unsigned k_at = lds0 + 256u * row + 16u * (h ^ (row & 15));
  const unsigned q_at = (unsigned)(uintptr_t)(LdsPtr)lds_all + kWideQ + 8192u * wave + 256u * row + 16u * (h ^ (row & 15));
  const unsigned mask_at = (unsigned)(uintptr_t)(LdsPtr)lds_all + kWideMasks + 512u * wave_all + 4u * lane;
  const unsigned v_at = lds0 + kWideRing * kWideTensor + 256u * (4 * h + ((lane >> 2) & 3)) + 64u * ((lane >> 2) & 3) + 32u * ((lane >> 4) & 1) + 8u * (lane & 3);

  const Share share = share_of(p, class_wg, blockIdx.x);
  const unsigned r1 = share.r1;
  const int y = share.y;
  int at_seq = seq_of_block(p, share.r0, share.first_seq);   // place in the launch's order of sequences

  for (unsigned r = share.r0; r < r1;) {
    const Seq seq = seq_at(p, at_seq);
    const int n = seq.n, L = seq.len, b = seq.place;
    const int n_prefix_blocks = (L + kBlockKeys - 1) / kBlockKeys;
    const int n_blocks = n_prefix_blocks + (n + kBlockKeys - 1) / kBlockKeys;
    const unsigned rel = r - seq.first;
    const int counted = n_blocks + p.setup;
    const int g = unit_of_block(p, rel, counted);
    const int from = (int)(rel - (unsigned)g * (unsigned)counted), count = min(counted - from, (int)(r1 - r));
    const int seg_begin = max(from - p.setup, 0), seg_count = from + count - p.setup - seg_begin;
    const int n_slabs = seq_slabs(p, n, ROWS), n_groups = seq_groups(p, n_slabs);
    if (seg_count <= 0 || y >= n_groups) {   // nothing but set-up, or no rows for this slab group (classes put together)
      r += (unsigned)count;
      if (at_seq + 1 < p.B && r >= seq_first_block(p, at_seq + 1)) ++at_seq;
      continue;
    }
    const int unit = share.slot + (at_seq - share.first_seq) * p.Hkv + g;   // partial slot
    const bool whole_unit = seg_count == n_blocks;
    const int slab = y * WAVES + wave;

    const char* kc = reinterpret_cast<const char*>(p.k_cache) + (b * p.stride_batch + g * p.stride_head) * 2;
    const char* vc = reinterpret_cast<const char*>(p.v_cache) + (b * p.stride_batch + g * p.stride_head) * 2;
    const int64_t tree0 = ((int64_t)b * p.Nmax * p.Hkv + g) * (D * 2);

    // blocks of this key group: kg, kg + 2, ... of the segment; those before n_full are whole prefix blocks
    const int blk_begin = seg_begin + kg;
    const int n_own = (seg_count - kg + KG - 1) / KG;
    const int n_full = (min(seg_begin + seg_count, L / kBlockKeys) - blk_begin + KG - 1) >> 1;   // (not positive: none)
    const int64_t first_byte = (int64_t)blk_begin * kBlockKeys * cache_row_bytes;
    const int64_t step = (int64_t)(KG * kBlockKeys) * cache_row_bytes;

    // Where this wavefront's copies of block i of its key group come from: four pieces a block, so that the count of
    // copies in flight tells what has landed.
    const char *k_src = kc + first_byte, *v_src = vc + first_byte;
    unsigned row_at[2] = {(unsigned)copy_key * cache_row_bytes, (unsigned)(copy_key + 4) * cache_row_bytes};
    auto locate_rest = [&](int i) {   // not a whole prefix block
      const int blk = blk_begin + KG * i;
      const bool tree = blk >= n_prefix_blocks;
      const int key0 = (tree ? blk - n_prefix_blocks : blk) * kBlockKeys, left = (tree ? n : L) - key0;
      const unsigned rb = tree ? tree_row_bytes : cache_row_bytes;
      const int64_t at = (int64_t)key0 * rb;
      k_src = (tree ? reinterpret_cast<const char*>(p.k_tree) + tree0 : kc) + at;
      v_src = (tree ? reinterpret_cast<const char*>(p.v_tree) + tree0 : vc) + at;
      row_at[0] = (unsigned)min(copy_key, left - 1) * rb;   // (rows past the end are masked later)
      row_at[1] = (unsigned)min(copy_key + 4, left - 1) * rb;
    };
    auto locate = [&](int i) {   // blocks in order
      if (i >= n_full) locate_rest(i);
      else if (i > 0) { k_src += step; v_src += step; }
    };
    auto copy_block = [&](unsigned at) {
      char* dst = ring + at + copy_dst;
#pragma unroll
      for (int x = 0; x < 2; ++x) __builtin_amdgcn_global_load_lds((GlobalPtr)(k_src + (row_at[x] + k_chunk[x])), (LdsPtr)(dst + 1024 * x), 16, 0, 0);
#pragma unroll
      for (int x = 0; x < 2; ++x)
        __builtin_amdgcn_global_load_lds((GlobalPtr)(v_src + (row_at[x] + v_chunk)), (LdsPtr)(dst + kWideRing * kWideTensor + 1024 * x), 16, 0, 0);
    };
    locate(0);
    if (n_own > 0) copy_block(0);

    // this lane's row: row rr of the kv head's N*G rows = (node, head within group)
    const int rr = slab * ROWS + row;
    const int node = (int)div_magic((unsigned)rr, p.G, p.g_magic);
    const bool exists = rr < p.Nmax * p.G, valid = exists && node < n;
    const int64_t out_row = ((int64_t)b * p.Nmax + node) * p.Hq + g * p.G + (rr - node * p.G);
    // Query rows and ancestor words come through LDS too, and out of it by instructions that the compiler does not track: in front of
    // the first use of anything loaded into registers it waits for every request in flight, a segment's first blocks among them.
    // Sixteen rows per wavefront, four per instruction, their chunks as those of K rows; rows past the tree are its last one again.
    {
      const int last = n * p.G - 1;
      char* const dst = lds_all + kWideQ + 4096 * wave_all;
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const int at = 16 * wave_all + 4 * x + (lane >> 4), qr = min(y * rows_per_unit + at, last);
        const int qn = (int)div_magic((unsigned)qr, p.G, p.g_magic);
        const char* src = reinterpret_cast<const char*>(p.q) + ((((int64_t)b * p.Nmax + qn) * p.Hq + g * p.G + (qr - qn * p.G)) * (D * 2) + (int)(16u * (chunk ^ (at & 15))));
        __builtin_amdgcn_global_load_lds((GlobalPtr)src, (LdsPtr)(dst + 1024 * x), 16, 0, 0);
      }
      const char* word = reinterpret_cast<const char*>(p.anc_mask) + 8 * ((int64_t)b * p.Nmax + min(node, n - 1));
#pragma unroll
      for (int x = 0; x < 2; ++x)
        __builtin_amdgcn_global_load_lds((GlobalPtr)(word + 4 * x), (LdsPtr)(lds_all + kWideMasks + 512 * wave_all + 256 * x), 4, 0, 0);
    }
#pragma unroll 1
    for (int i = 1; i < min(kWideRing, n_own); ++i) {
      locate(i);
      copy_block(i * kWideTensor);
    }

    if (seg_begin == 0 && y == 0) {   // (counted as copies by the waits below, which then wait for more; behind the stream it cost as much)
      const int covered = n_groups * rows_per_unit;
      if (covered < p.Nmax * p.G) zero_rows<D, 64 * WAVES * KG>(p, b, g, covered);
    }

    f32x16 o[4], s;
    float m = kNegBig, l = 0.f;
#pragma unroll
    for (int dt = 0; dt < 4; ++dt)
#pragma unroll
      for (int e = 0; e < 16; ++e) o[dt][e] = 0.f;
    bf16x8 k[8], v[2][4], wt[2];
    u32x2 vr[16];

    // All copies of this wavefront have landed but those of its last block, if there are blocks (`blocks` > 0) behind the one that
    // is needed. (written out: the compiler's form of the choice has four more scalar instructions and a branch more in every turn)
    auto next_landed = [](int blocks) {
      asm volatile("s_cmp_gt_i32 %0, 0\n\ts_cbranch_scc1 .Lone%=\n\ts_waitcnt vmcnt(0)\n.Lone%=:\n\ts_waitcnt vmcnt(4)" : : "s"(blocks) : "scc", "memory");
    };
    auto barrier = [] {
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_barrier" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    };
    // Block 0, the query rows and the ancestor words have landed; blocks 1 and 2 may be in flight.
    if (n_own > 2) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    else next_landed(n_own - 1);
    barrier();
    bf16x8 q[8];
    read_k(q, q_at);
    const uint64_t tree_mask = valid ? read_mask(mask_at) : 0ull;
    if (!valid) {   // (products of zeros: 16 ragged sequences, 17 to 60 nodes 1 % less than with the copied row)
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) q[ks] = bf16x8{};
    }
    read_k(k, k_at);
    unsigned slot = 0;
    for (int i = 0; i < n_own; ++i) {
      const unsigned slot_next = slot + kWideTensor == kWideRing * kWideTensor ? 0u : slot + kWideTensor;
      qk_reading_v(s, k, q, vr, v_at + slot);
      if (kg == 1) {
        next_landed(n_own - 2 - i);
        barrier();
      }
      if (i >= n_full) {   // ragged tail or tree block
        const int blk = blk_begin + KG * i;
        const bool tree = blk >= n_prefix_blocks;
        const int key0 = (tree ? blk - n_prefix_blocks : blk) * kBlockKeys, left = (tree ? n : L) - key0;
        unsigned vis = left >= kBlockKeys ? ~0u : ((1u << left) - 1u);
        if (tree) vis &= (unsigned)(tree_mask >> key0);
        vis >>= 4 * h;
#pragma unroll
        for (int e = 0; e < 16; ++e) s[e] = ((vis >> (8 * (e >> 2) + (e & 3))) & 1u) ? s[e] : -INFINITY;
      }
      unsigned pk[8];
      uint64_t grow;
      const float l_before = l;
      weights_of(s, c, m, pk, l, grow);
      if (grow != 0) {   // rare: move the rows' shifts
        float mx = s[0];
#pragma unroll
        for (int e = 1; e < 16; ++e) mx = fmaxf(mx, s[e]);
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        const float mnew = fmaxf(m, fmaf(mx, c, kWideHeadroom));
        const float alpha = __builtin_amdgcn_exp2f(m - mnew);
        m = mnew;
        l = l_before * alpha;
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) o[dt] *= alpha;
        weights_of(s, c, m, pk, l, grow);
      }
#pragma unroll
      for (int t = 0; t < 2; ++t) wt[t] = __builtin_bit_cast(bf16x8, u32x4{pk[4 * t], pk[4 * t + 1], pk[4 * t + 2], pk[4 * t + 3]});
      if (kg == 0) {
        next_landed(n_own - 2 - i);
        barrier();
      }
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) {
          const int x = 2 * (4 * t + dt);
          v[t][dt] = __builtin_bit_cast(bf16x8, u32x4{vr[x][0], vr[x][1], vr[x + 1][0], vr[x + 1][1]});
        }
      pv_reading_k(o, v, wt, k, k_at + slot_next);
      // block i is read by all four wavefronts: its place in the ring takes a later one
      if (i + kWideRing < n_own) {
        locate(i + kWideRing);
        copy_block(slot);
      }
      slot = slot_next;
    }
    if (kg == 1 && (seg_count & 1)) barrier();   // group 0 has a block more

    // The two key groups hold the same rows in the same lanes. Group 0 finishes dims 0..63 and group 1 dims 64..127: each hands
    // the other half over in lane-private LDS slots (the rings are free), so that all eight wavefronts merge and write.
    // (the compiler does not know that o comes from matrix instructions: the wait states behind the last of them own it, so that
    // no read of it can be placed in front of them)
    asm volatile("s_waitcnt vmcnt(0)\n\ts_nop 15\n\ts_nop 7" : "+v"(o[0]), "+v"(o[1]), "+v"(o[2]), "+v"(o[3]) : : "memory");
    __syncthreads();
    f32x4* const mbuf = reinterpret_cast<f32x4*>(lds_all) + wave * (2 * 8 * 64) + lane;
    float2* const ml = reinterpret_cast<float2*>(lds_all + 65536) + wave * 128 + lane;
    l += __shfl_xor(l, 32);
    ml[kg * 64] = make_float2(m, l);
#pragma unroll
    for (int x = 0; x < 8; ++x) {
      const int e = 4 * (x & 3);
      const f32x16 give = kg == 0 ? o[2 + (x >> 2)] : o[x >> 2];
      mbuf[(kg * 8 + x) * 64] = f32x4{give[e], give[e + 1], give[e + 2], give[e + 3]};
    }
    __syncthreads();
    if (exists) {
      const float2 a = ml[0], bb = ml[64];
      const float mm = fmaxf(a.x, bb.x);
      const float f0 = __builtin_amdgcn_exp2f(a.x - mm), f1 = __builtin_amdgcn_exp2f(bb.x - mm);
      const float l_row = a.y * f0 + bb.y * f1;
      const float own = kg == 0 ? f0 : f1, other = kg == 0 ? f1 : f0;
      const float inv = whole_unit ? (valid ? 1.0f / l_row : 0.f) : 1.0f;
      float* const slot = (float*)*arg_at<__attribute__((address_space(1))) float*>(offsetof(AttnParams, part)) + (int64_t)unit * rows_per_unit * (D + 2);
      void* const out_ptr = (void*)*arg_at<__attribute__((address_space(1))) void*>(offsetof(AttnParams, out));
      const int lr = wave * ROWS + row;
      if (!whole_unit && valid && lane < 32 && kg == 0) *reinterpret_cast<float2*>(slot + (int64_t)rows_per_unit * D + 2 * lr) = make_float2(mm, l_row);
#pragma unroll
      for (int x = 0; x < 8; ++x) {
        const int e = 4 * (x & 3), d0 = 64 * kg + 32 * (x >> 2) + 8 * (x & 3) + 4 * h;
        const f32x16 keep = kg == 0 ? o[x >> 2] : o[2 + (x >> 2)];
        const f32x4 got = mbuf[((kg ^ 1) * 8 + x) * 64];
        f32x4 val;
#pragma unroll
        for (int j = 0; j < 4; ++j) val[j] = keep[e + j] * own + got[j] * other;
        if (!whole_unit) {
          if (valid) store_through(slot + partial_index<D>(lr, d0 / 4), val);
        } else {
#pragma unroll
          for (int j = 0; j < 4; ++j) val[j] = valid ? val[j] * inv : 0.f;
          if (*arg_at<int32_t>(offsetof(AttnParams, out_bf16))) {
            typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
            bf16x4 o4;
#pragma unroll
            for (int j = 0; j < 4; ++j) o4[j] = (__bf16)val[j];
            *reinterpret_cast<bf16x4*>(reinterpret_cast<__bf16*>(out_ptr) + out_row * D + d0) = o4;
          } else {
            *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(out_ptr) + out_row * D + d0) = val;
          }
        }
      }
    }
    r += (unsigned)count;
    if (at_seq + 1 < p.B && r >= seq_first_block(p, at_seq + 1)) ++at_seq;
    __syncthreads();  // every wavefront is done with the merge buffers before the next segment fills the rings
  }
}

// Workgroup (cluster) of n that owns flat block x under the even split: the last w with floor(w T / n) <= x, i.e.
// floor(((x + 1) n - 1) / T). The numerator is below 2^45 and the quotient below 2^15: half a unit up, the product
// with 1/T in fp64 is further from the next integer than its rounding can carry it.
__device__ __forceinline__ int owner_of(unsigned x, int n, double inv_total) {
  return (int)(((double)(x + 1u) * (double)n - 0.5) * inv_total);
}

// Finishes every unit that was cut into several segments:
// out = sum_s 2^(m_s - M) O_s / sum_s 2^(m_s - M) l_s over the unit's partial slots.
// One thread per 4 output dims; rows of nodes past n_nodes are written as zeros.
// pieces: workgroups per unit where every unit of the launch is cut into that many and no workgroup holds parts of two (0 where
// that is not so).
template <bool SHARED>
using MergeParams = std::conditional_t<SHARED, SharedParams, AttnParams>;
template <int D, bool SHARED>
__global__ __launch_bounds__(256) void tree_attn_combine_kernel(const MergeParams<SHARED>, int, int, double) {
  const int at_seq = blockIdx.z, g = blockIdx.y;
  const MergeArgs m = fetch_merge_args(at_seq, sizeof(MergeParams<SHARED>));
  const AttnArgs& p = m.p;
  const int rows_per_unit = m.rows_per_unit, pieces = m.pieces;
  constexpr int TPR = D / 4;  // threads per row
  constexpr int RPW = 256 / TPR;   // rows of this workgroup: in lane order (partial_index) the faster index of its threads
  const int n = m.nodes & 0xff, b = (m.nodes >> 8) & 0xff;
  const int y = SHARED ? (int)(blockIdx.x * RPW) / 128 : 0;   // (128 rows per slab group)
  if (SHARED && y >= seq_groups(p, seq_slabs(p, n, 32))) return;   // a tree smaller than the largest: no such rows of it
  int clusters = p.n_wgs, units = p.B * p.Hkv, first_seq = 0, slot0 = 0, first_block = 0;
  double inv_total = m.inv_total;
  if (SHARED && p.n_classes > 1) {
    const __attribute__((address_space(4))) SeqClass& from = arg_classes()[m.nodes >> 16];
    clusters = from.clusters; units = from.units; first_seq = from.first_seq; slot0 = from.slot0; first_block = from.first_block;
    inv_total = from.inv_total;
  }
  const int unit = (at_seq - first_seq) * p.Hkv + g;
  int w0, n_seg;
  if (pieces > 0) {
    w0 = unit * pieces;
    n_seg = pieces;
  } else {
    const int n_blocks = (m.kv_len + kBlockKeys - 1) / kBlockKeys + (n + kBlockKeys - 1) / kBlockKeys;
    const unsigned fs = (unsigned)(m.first_block - first_block) + (unsigned)g * (unsigned)(n_blocks + p.setup) + (unsigned)p.setup;
    w0 = owner_of(fs, clusters, inv_total);
    n_seg = owner_of(fs + (unsigned)n_blocks - 1u, clusters, inv_total) - w0 + 1;
    if (n_seg == 1) return;  // written directly by the one workgroup that held the whole unit
  }
  const int slot = slot0 + y * (units + clusters) + unit + w0;
  const int lr = (int)(blockIdx.x * RPW) - y * 128 + (int)(SHARED ? threadIdx.x % RPW : threadIdx.x / TPR);
  if (lr >= rows_per_unit) return;
  const int piece = SHARED ? threadIdx.x / RPW : threadIdx.x % TPR, d0 = 4 * piece;
  const int rr = y * rows_per_unit + lr;
  if (rr >= p.Nmax * p.G) return;
  const int node = (int)div_magic((unsigned)rr, p.G, p.g_magic), hl = rr - node * p.G;
  const int64_t row = ((int64_t)b * p.Nmax + node) * p.Hq + g * p.G + hl;
  f32x4 acc = {0.f, 0.f, 0.f, 0.f};
  if (node < n) {
    const int64_t slot_floats = (int64_t)rows_per_unit * (D + 2);
    const float* o_base = p.part + (int64_t)slot * slot_floats + (SHARED ? partial_index<D>(lr, piece) : lr * D + d0);
    const float* ml_base = p.part + (int64_t)slot * slot_floats + (int64_t)rows_per_unit * D + 2 * lr;
    // slots in index order (deterministic), eight at a time so that their loads are in flight together
    float M = kNegBig, denom = 0.f;
    for (int s0 = 0; s0 < n_seg; s0 += 8) {
      float2 ml[8];
      f32x4 o[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const int sidx = min(s0 + k, n_seg - 1);  // clamped duplicates get zero weight below
        // Grouped heads: two, four or eight, as the unit has them. A ragged batch's units are cut in two or three, and eight loads of
        // which five repeat the last one cost the texture path as much as eight: 16 sequences of 131 to 6011 keys 12.3 -> 8.6 us. (Sixteen
        // changed nothing for units of sixteen pieces; elsewhere units have their eight, and the choice costs 0.1 us.)
        if (!SHARED || k < 2 || n_seg - s0 > (k < 4 ? 2 : 4)) {
          ml[k] = *reinterpret_cast<const float2*>(ml_base + sidx * slot_floats);
          o[k] = *reinterpret_cast<const f32x4*>(o_base + sidx * slot_floats);
        } else {
          ml[k] = make_float2(kNegBig, 0.f);
          o[k] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      }
      float mx = M;
#pragma unroll
      for (int k = 0; k < 8; ++k) mx = fmaxf(mx, ml[k].x);
      const float a = __builtin_amdgcn_exp2f(M - mx);
      acc *= a;
      denom *= a;
      M = mx;
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        const float wgt = (s0 + k < n_seg) ? __builtin_amdgcn_exp2f(ml[k].x - M) : 0.f;
        denom += wgt * ml[k].y;
        acc += wgt * o[k];
      }
    }
    acc *= 1.0f / denom;
  }
  if (p.out_bf16) {
    typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
    bf16x4 pk;
#pragma unroll
    for (int e = 0; e < 4; ++e) pk[e] = (__bf16)acc[e];
    *reinterpret_cast<bf16x4*>(reinterpret_cast<__bf16*>(p.out) + row * D + d0) = pk;
  } else {
    *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(p.out) + row * D + d0) = acc;
  }
}

// ---------------------------------------------------------------------------------------------
// fp32 path: vector arithmetic (fp32 inputs need fp32 products and sums for the 1e-5 tolerance of the
// small parity configuration). What bounds it is latency: a call of this size is one or two trips to
// memory and what hangs behind them. A workgroup of eight wavefronts takes QN nodes of one query head;
// the wavefronts take tiles of 8 * 64 / LPK keys in turn, D/4 = LPK lanes per key with four dims each, so
// that a K or V row is one contiguous request and all requests of a tile are in flight together. The dot
// product of a key is a sum over its LPK lanes, which leaves the score -- and so the weight -- in exactly the
// lanes that hold the key's V entries: no exchange between the two products. The wavefronts' (max, sum,
// output) meet in LDS once, at the end. 8 heads, D = 64, 256 keys, 26 nodes: 6.1 us (one wavefront per node, a
// lane per key, the weights exchanged key by key for the second product: 60.6 us).
// WAVES = 1: short prefixes under many rows (launch_f32), where most of the eight would find no key. One wavefront per
// node, which reads only the tree keys that its node sees.
constexpr int kF32Waves = 8;
constexpr int kF32Loads = 8;   // K (and V) rows a lane has in flight per tile

// sum over the LPK lanes that share a key, in every one of them
template <int LPK>
__device__ __forceinline__ float key_sum(float v) {
  auto rotated = [](float x, auto ctrl) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), decltype(ctrl)::value, 0xf, 0xf, true));
  };
  v += rotated(v, std::integral_constant<int, 0x128>{});   // row_ror 8, 4, 2, 1
  v += rotated(v, std::integral_constant<int, 0x124>{});
  v += rotated(v, std::integral_constant<int, 0x122>{});
  v += rotated(v, std::integral_constant<int, 0x121>{});
  if (LPK == 32) v += __shfl_xor(v, 16);
  return v;
}

template <int D, int QN, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void tree_attn_f32_kernel(const AttnParams p) {
  static_assert(WAVES > 1 || QN == 1, "the list of tree keys is one node's");
  constexpr int LPK = D / 4, KPL = 64 / LPK;       // lanes per key, keys per load instruction
  constexpr int kTile = kF32Loads * KPL;           // keys per wavefront and turn
  __shared__ __attribute__((aligned(16))) float sh_o[WAVES][QN][D];
  __shared__ float sh_m[WAVES][QN], sh_l[WAVES][QN];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = blockIdx.x, b = blockIdx.z, node0 = blockIdx.y * QN;
  const int g = h / p.G;
  const int n = p.seq[b].nodes, L = p.seq[b].kv_len;
  int total = L + n;
  const int64_t row0 = ((int64_t)b * p.Nmax + node0) * p.Hq + h;   // (b, node0, h); the next node is Hq rows further
  float* const out0 = reinterpret_cast<float*>(p.out) + row0 * D;
  const int64_t node_stride = (int64_t)p.Hq * D;
  if (node0 >= n) {
    for (int i = tid; i < QN * D; i += 64 * WAVES)
      if (node0 + i / D < p.Nmax) out0[(i / D) * node_stride + i % D] = 0.f;
    return;
  }
  const int sub = lane & (LPK - 1), grp = lane / LPK;
  const float* kc = reinterpret_cast<const float*>(p.k_cache) + b * p.stride_batch + g * p.stride_head;
  const float* vc = reinterpret_cast<const float*>(p.v_cache) + b * p.stride_batch + g * p.stride_head;
  const int64_t tree_stride = (int64_t)p.Hkv * D;
  const int64_t tree0 = ((int64_t)b * p.Nmax * p.Hkv + g) * D;
  const float* ktr = reinterpret_cast<const float*>(p.k_tree) + tree0;
  const float* vtr = reinterpret_cast<const float*>(p.v_tree) + tree0;

  f32x4 q[QN], o[QN];
  uint64_t word[QN];
  float m[QN], l[QN];
#pragma unroll
  for (int t = 0; t < QN; ++t) {
    const int node = min(node0 + t, n - 1);
    q[t] = *reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(p.q) + row0 * D + (node - node0) * node_stride + 4 * sub);
    word[t] = p.anc_mask[b * p.Nmax + node];
    o[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    m[t] = -INFINITY;
    l[t] = 0.f;
  }
  int nth = 0;   // WAVES = 1: lane r holds the r-th tree node that this one sees
  if constexpr (WAVES == 1) {
    const uint64_t own = word[0] & (~0ull >> (64 - n));
    const int n_seen = __popcll(own), below = __popcll(own & ((1ull << lane) - 1));
    nth = __builtin_amdgcn_ds_permute(4 * ((own >> lane) & 1 ? below : n_seen + lane - below), lane);
    total = L + n_seen;
  }
  for (int base = wave * kTile; base < total; base += WAVES * kTile) {
    f32x4 k[kF32Loads], v[kF32Loads];
#pragma unroll
    for (int i = 0; i < kF32Loads; ++i) {   // (keys past the end re-read the last one; they are masked below)
      const int j = min(base + i * KPL + grp, total - 1);
      const bool prefix = j < L;
      int node = j - L;
      if constexpr (WAVES == 1) node = __shfl(nth, max(node, 0));
      const int64_t at = prefix ? j * p.stride_token : node * tree_stride;
      k[i] = *reinterpret_cast<const f32x4*>((prefix ? kc : ktr) + at + 4 * sub);
      v[i] = *reinterpret_cast<const f32x4*>((prefix ? vc : vtr) + at + 4 * sub);
    }
#pragma unroll
    for (int t = 0; t < QN; ++t) {
      float s[kF32Loads], mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < kF32Loads; ++i) {
        const float dot = key_sum<LPK>(fmaf(q[t][3], k[i][3], fmaf(q[t][2], k[i][2], fmaf(q[t][1], k[i][1], q[t][0] * k[i][0]))));
        const int j = base + i * KPL + grp;
        const bool seen = j < L || (j < total && (WAVES == 1 || ((word[t] >> (j - L)) & 1ull)));
        s[i] = seen ? dot * p.scale : -INFINITY;
        mx = fmaxf(mx, s[i]);
      }
#pragma unroll
      for (int off = LPK; off < 64; off <<= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
      const float mnew = fmaxf(m[t], mx);
      // (no key of this wavefront's visible so far: nothing to add, and no -inf minus -inf)
      const float alpha = m[t] > -INFINITY ? expf(m[t] - mnew) : 0.f;
      l[t] *= alpha;
      o[t] *= alpha;
      m[t] = mnew;
#pragma unroll
      for (int i = 0; i < kF32Loads; ++i) {
        const float w = s[i] == -INFINITY ? 0.f : expf(s[i] - mnew);
        l[t] += w;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[t][e] = w == 0.f ? o[t][e] : fmaf(w, v[i][e], o[t][e]);   // a masked V row may hold anything
      }
    }
  }
#pragma unroll
  for (int t = 0; t < QN; ++t) {
#pragma unroll
    for (int off = LPK; off < 64; off <<= 1) {
      l[t] += __shfl_xor(l[t], off);
#pragma unroll
      for (int e = 0; e < 4; ++e) o[t][e] += __shfl_xor(o[t][e], off);
    }
    if (grp == 0) *reinterpret_cast<f32x4*>(&sh_o[wave][t][4 * sub]) = o[t];
    if (lane == 0) { sh_m[wave][t] = m[t]; sh_l[wave][t] = l[t]; }
  }
  __syncthreads();
  for (int i = tid; i < QN * D; i += 64 * WAVES) {
    const int t = i / D, d = i % D, node = node0 + t;
    if (node >= p.Nmax) break;
    float M = sh_m[0][t], num = 0.f, den = 0.f;
#pragma unroll
    for (int w = 1; w < WAVES; ++w) M = fmaxf(M, sh_m[w][t]);
    // (t is the same in a whole wavefront, whose lane w forms the share of wavefront w)
    const float own = sh_m[lane % WAVES][t];
    const float share = own > -INFINITY ? expf(own - M) : 0.f;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) {   // in wavefront order: deterministic
      const float a = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, share), w));
      den += a * sh_l[w][t];
      num += a * sh_o[w][t][d];
    }
    out0[t * node_stride + d] = node < n ? num / den : 0.f;
  }
}

// ---------------------------------------------------------------------------------------------
int host_owner_of(int64_t x, int64_t T, int W) {
  int w = (int)((x * W) / T);
  if (((int64_t)(w + 1) * T) / W <= x) ++w;
  return w;
}

// Slab groups that hold the rows of a tree of n nodes (GY for a full one).
int groups_of(const fspad_attn_desc& d, const Plan& pl, int n) {
  const int rows = n * (d.n_q_heads / d.n_kv_heads), slabs = (rows + 16 * pl.QT - 1) / (16 * pl.QT);
  return (slabs + pl.WS - 1) / pl.WS;
}

constexpr int kWholeSetup = 4096;   // more than the blocks of a launch's units can differ from an even division by

// The flat list of blocks and its division among workgroups: sequences in the order of their classes (see SeqClass), `wgs`
// workgroups shared among the classes by their blocks. Returns the workgroups of the launch (at most wgs, but one per class and
// slab group at least); `any_cut`: some unit is cut among several.
int plan_classes(const fspad_attn_desc& d, const Plan& pl, const int* groups, int64_t wgs, SharedParams& sp, bool& any_cut) {
  AttnParams& sl = sp.a;
  const int nb = sl.B;
  // the kernels of one slab group per kv head: one class. More different numbers of slab groups than a launch has classes
  // (1024 rows per kv head): rounded up, with workgroups that pass over the sequences without rows for them
  int used[kMaxBatchPerLaunch], n_classes = 0, class_groups[kMaxBatchPerLaunch];
  for (int unit = 1;; unit *= 2) {
    n_classes = 0;
    for (int i = 0; i < nb; ++i) {
      used[i] = (groups[i] + unit - 1) / unit * unit;
      if (used[i] > pl.GY) used[i] = pl.GY;
      bool known = false;
      for (int k = 0; k < n_classes; ++k) known = known || class_groups[k] == used[i];
      if (!known) class_groups[n_classes++] = used[i];
    }
    if (n_classes <= kMaxClasses) break;
  }
  SeqInfo in[kMaxBatchPerLaunch];   // in the batch's order
  int len[kMaxBatchPerLaunch];      // blocks of each
  for (int i = 0; i < nb; ++i) {
    in[i] = sl.seq[i];
    len[i] = blocks_of(in[i].kv_len, in[i].nodes);
  }
  // whole units (kWholeSetup): the shorter ones first, so that a workgroup's range ends behind its own unit, in the next one's set-up
  int by[kMaxBatchPerLaunch];
  for (int i = 0; i < nb; ++i) {
    int at = i;
    if (sl.setup == kWholeSetup)
      for (; at > 0 && len[by[at - 1]] > len[i]; --at) by[at] = by[at - 1];
    by[at] = i;
  }
  SeqClass* cls = sp.classes;
  int64_t blocks[kMaxClasses], work = 0, flat = 0, left = wgs;
  for (int k = 0, at = 0; k < n_classes; ++k) {
    cls[k] = SeqClass{};
    cls[k].groups = class_groups[k];
    cls[k].first_seq = at;
    const int64_t flat0 = flat;
    cls[k].first_block = (int32_t)flat0;
    for (int j = 0; j < nb; ++j) {
      const int i = by[j];
      if (used[i] != class_groups[k]) continue;
      sl.seq[at] = SeqInfo{in[i].kv_len, in[i].nodes | i << 8 | k << 16};
      sl.bstart[at] = (int32_t)flat;
      flat += (int64_t)d.n_kv_heads * (len[i] + sl.setup);
      ++at;
    }
    cls[k].units = (at - cls[k].first_seq) * d.n_kv_heads;
    blocks[k] = flat - flat0;
    work += blocks[k] * class_groups[k];
  }
  sl.bstart[nb] = (int32_t)flat;
  for (int k = 0; k < n_classes; ++k) {
    const int64_t n = wgs * blocks[k] / work;   // (= its share of the workgroups over its slab groups)
    cls[k].clusters = (int32_t)(n < 1 ? 1 : n);
    left -= (int64_t)cls[k].groups * cls[k].clusters;
  }
  for (;;) {   // what the rounding left goes to the class with the longest ranges, where there are classes
    int longest = -1;
    for (int k = 0; n_classes > 1 && k < n_classes; ++k)
      if (cls[k].groups <= left && cls[k].clusters < blocks[k] &&
          (longest < 0 || blocks[k] * cls[longest].clusters > blocks[longest] * cls[k].clusters))
        longest = k;
    if (longest < 0) break;
    cls[longest].clusters += 1;
    left -= cls[longest].groups;
  }
  int grid = 0;
  int64_t slot = 0;
  any_cut = false;
  for (int k = 0; k < n_classes; ++k) {
    SeqClass& c = cls[k];
    c.wg_begin = grid;
    grid += c.groups * c.clusters;
    c.quot = (int32_t)(blocks[k] / c.clusters);
    c.rem = (int32_t)(blocks[k] % c.clusters);
    c.clusters_rcp = reciprocal(c.clusters);
    c.tile_rcp = reciprocal(8 * c.groups);
    c.inv_total = 1.0 / (double)blocks[k];
    c.slot0 = (int32_t)slot;
    bool cut = false;
    for (int i = c.first_seq; i < c.first_seq + c.units / d.n_kv_heads && !cut; ++i) {
      const int64_t nblk = len[sl.seq[i].nodes >> 8 & 0xff] + sl.setup;
      for (int g = 0; g < d.n_kv_heads && !cut; ++g) {
        const int64_t fs = sl.bstart[i] - c.first_block + g * nblk;
        cut = host_owner_of(fs + sl.setup, blocks[k], c.clusters) != host_owner_of(fs + nblk - 1, blocks[k], c.clusters);
      }
    }
    any_cut = any_cut || cut;
    if (cut) slot += (int64_t)c.groups * (c.units + c.clusters);   // (at most units + workgroups altogether)
  }
  for (int k = 0; k < kMaxClasses; ++k) sp.class_wg[k] = k < n_classes ? cls[k].wg_begin : INT32_MAX;
  sl.n_classes = n_classes;
  sl.total_blocks = (int32_t)flat;
  sl.GY = cls[0].groups; sl.n_wgs = cls[0].clusters; sl.wg_quot = cls[0].quot; sl.wg_rem = cls[0].rem;
  sl.wgs_rcp = cls[0].clusters_rcp; sl.tile_rcp = cls[0].tile_rcp;
  return grid;
}

// What a unit costs a workgroup beyond its blocks, in blocks: Q, the ramp of the stream, merge and output. In a ragged batch
// the flat list counts every unit for that much more: an even split of the blocks alone gave the workgroups of the
// short sequences a dozen units each, and the call lasted until they were done. Grouped heads, 16 sequences of 131 to
// 6011 keys, 17 to 60 nodes: 98 us without, 77 / 72 / 78 us with 8 / 20 / 40; 64-row tiles, 2 x 32 heads, 100 to 5000 keys: 43,
// 44 / 41 / 42; 32-row tiles, 8 x 32 heads, 200 to 3000 keys: 51, 44 / 46 / 52; 16-row tiles (two workgroups per
// compute unit, which cover each other's set-up), 16 x 32 heads, 64 to 900 keys: 36, 39 / 40 / 39.
int setup_blocks(const Plan& pl) { return pl.shared_stage || pl.QT >= 3 ? 20 : (pl.QT == 2 ? 8 : 0); }

// Partial slots of a plan: one per (unit, workgroup) boundary at most. 32-row tiles get more than two workgroups per
// compute unit only where each holds a whole unit, which leaves no partial results: not more slots then than a cut
// batch of that size needs. More units than a launch has workgroups (kMaxWorkgroups) do not stay whole.
int64_t slots_of(const Plan& pl, int64_t units, int64_t wgs, int64_t total_blocks, int forced) {
  if (forced == 0 && pl.QT == 2 && !pl.shared_stage && wgs > 2 * kComputeUnits && wgs == units) {
    wgs = 2 * kComputeUnits;
    if (wgs > total_blocks / (2 * key_waves(pl))) wgs = total_blocks / (2 * key_waves(pl));
  }
  return units + wgs;
}

size_t slot_bytes(const fspad_attn_desc& d, const Plan& pl) {
  return (size_t)pl.rows_per_unit * (d.head_dim + 2) * sizeof(float);
}

fspad_status check_desc(const fspad_attn_desc* d) {
  if (!d) return FSPAD_ERR_NULL;
  if (d->batch < 1 || d->n_nodes_max < 1 || d->n_nodes_max > FSPAD_MAX_NODES) return FSPAD_ERR_SHAPE;
  if (d->n_q_heads < 1 || d->n_kv_heads < 1 || d->n_q_heads % d->n_kv_heads != 0) return FSPAD_ERR_SHAPE;
  if (d->head_dim != 64 && d->head_dim != 128) return FSPAD_ERR_SHAPE;
  if ((int64_t)d->n_kv_heads * d->head_dim > (1ll << 26)) return FSPAD_ERR_SHAPE;  // 32-bit byte offsets inside a block
  if (d->io_dtype != FSPAD_F32 && d->io_dtype != FSPAD_BF16) return FSPAD_ERR_DTYPE;
  if (d->out_dtype != FSPAD_F32 && d->out_dtype != d->io_dtype) return FSPAD_ERR_DTYPE;
  if (!(d->softmax_scale >= 0.f) || d->softmax_scale > 3.0e38f) return FSPAD_ERR_SHAPE;
  if (d->workgroups < 0) return FSPAD_ERR_SHAPE;
  return FSPAD_OK;
}

template <int QT, int D, bool STREAMED, bool RAGGED>
void launch_bf16(const AttnParams& prm, hipStream_t stream) {
  hipLaunchKernelGGL((tree_attn_bf16_kernel<QT, D, STREAMED, RAGGED>), dim3((unsigned)prm.n_wgs), dim3(256), 0, stream, prm);
}
template <int D, bool STREAMED>
void launch_bf16(const Plan& pl, const AttnParams& prm, hipStream_t stream) {
  const bool ragged = prm.setup > 0;   // (never with 16-row tiles: setup_blocks)
  switch (pl.QT) {
    case 1: launch_bf16<1, D, STREAMED, false>(prm, stream); break;
    case 2: ragged ? launch_bf16<2, D, STREAMED, true>(prm, stream) : launch_bf16<2, D, STREAMED, false>(prm, stream); break;
    case 3: ragged ? launch_bf16<3, D, STREAMED, true>(prm, stream) : launch_bf16<3, D, STREAMED, false>(prm, stream); break;
    default: ragged ? launch_bf16<4, D, STREAMED, true>(prm, stream) : launch_bf16<4, D, STREAMED, false>(prm, stream); break;
  }
}
template <int D>
void launch_bf16(const Plan& pl, const AttnParams& prm, bool streamed, hipStream_t stream) {
  streamed ? launch_bf16<D, true>(pl, prm, stream) : launch_bf16<D, false>(pl, prm, stream);
}

template <int D>
void launch_combine(const Plan& pl, const SharedParams& sp, int pieces, hipStream_t stream) {
  const AttnParams& prm = sp.a;
  const int rows_per_wg = 1024 / D;
  const dim3 grid((unsigned)((pl.rows_per_unit + rows_per_wg - 1) / rows_per_wg * pl.GY), (unsigned)prm.Hkv, (unsigned)prm.B);
  const double inv_total = 1.0 / (double)prm.total_blocks;
  if (pl.shared_stage) hipLaunchKernelGGL((tree_attn_combine_kernel<D, true>), grid, dim3(256), 0, stream, sp, pl.rows_per_unit, pieces, inv_total);
  else hipLaunchKernelGGL((tree_attn_combine_kernel<D, false>), grid, dim3(256), 0, stream, prm, pl.rows_per_unit, pieces, inv_total);
}


// Nodes per workgroup of the fp32 kernel: a node of its own re-reads all of K and V through L2, which costs
// nothing while the chip has room (one node against two: 6.1 / 8.3 us with 8 heads x 26 nodes, 256 keys, D = 64;
// 8.1 / 8.2 us with 8 x 60; 16.9 / 18.5 us with 16 x 48, 600 keys) and is what bounds the call beyond that
// (13.3 / 11.5 us with 16 x 60, 300 keys; 89 / 73 us with 2 x 16 x 64, 700 keys, D = 128; four nodes: 77 us).
// Beyond that, prefixes of up to two tiles of a wavefront's keys (64 at D = 64, 32 at D = 128) leave most of the eight
// wavefronts without one: a single wavefront per node. 16 x 32 / 8 heads, 26 nodes, D = 64: no prefix 14.4 us (58.0 with eight
// wavefronts), 20 keys 14.6 (60.8), 50 keys 23.9 (59.2); 8 x 32 heads, 60 nodes, D = 128, 20 keys 27.6 us (88). With fewer rows
// the eight cost a launch of many workgroups only where a single one has the keys in half a tile (4 x 16 / 4 heads, 10 nodes,
// no prefix: 4.3 us, 6.5; 20 keys 4.3 against 4.4 with 2 x 16 heads, 100 keys 8.7 against 4.5).
template <int D>
void launch_f32(const AttnParams& prm, hipStream_t stream) {
  constexpr int kTile = kF32Loads * 64 / (D / 4);
  const bool few = (int64_t)prm.B * prm.Hq * prm.Nmax <= 768;
  int longest = 0;
  for (int b = 0; b < prm.B; ++b) longest = prm.seq[b].kv_len > longest ? prm.seq[b].kv_len : longest;
  const bool single = longest <= (few ? kTile / 2 : 2 * kTile);
  const bool one = few || single;
  // Sixteen wavefronts where eight take more than a turn and no compute unit gets a second workgroup. us by eight / sixteen, 8 heads of
  // 64: 26 nodes, 256 keys 5.38 / 5.27, 500 6.93 / 6.67, 700 8.52 / 7.43, 4 nodes, 1000 keys 10.3 / 9.0; 16 heads of 128, 16 nodes, 130
  // keys 5.92 / 5.41; 8 of 128, 30 nodes, 400 keys 9.12 / 8.12. (Twelve keys' loads a lane in one turn instead of eight in two: 5.38 -> 5.32.)
  const bool wide = (int64_t)prm.B * prm.Hq * prm.Nmax <= kComputeUnits && longest + prm.Nmax > kF32Waves * kTile;
  const dim3 grid((unsigned)prm.Hq, (unsigned)(one ? prm.Nmax : (prm.Nmax + 1) / 2), (unsigned)prm.B), block(64 * kF32Waves);
  if (single) hipLaunchKernelGGL((tree_attn_f32_kernel<D, 1, 1>), grid, dim3(64), 0, stream, prm);
  else if (wide) hipLaunchKernelGGL((tree_attn_f32_kernel<D, 1, 2 * kF32Waves>), grid, dim3(2 * 64 * kF32Waves), 0, stream, prm);
  else if (one) hipLaunchKernelGGL((tree_attn_f32_kernel<D, 1, kF32Waves>), grid, block, 0, stream, prm);
  else hipLaunchKernelGGL((tree_attn_f32_kernel<D, 2, kF32Waves>), grid, block, 0, stream, prm);
}

}  // namespace

extern "C" size_t fspad_tree_attn_workspace_bytes(const fspad_attn_desc* desc, int32_t max_kv_len) {
  if (check_desc(desc) != FSPAD_OK || max_kv_len < 0) return 0;
  if (desc->io_dtype == FSPAD_F32) return 16;
  // one partial slot per (unit, workgroup) boundary at most: units + workgroups of the largest slice
  Plan pl{};
  plan_rows(*desc, pl);
  const int nb = desc->batch < kMaxBatchPerLaunch ? desc->batch : kMaxBatchPerLaunch;
  const int64_t units = (int64_t)nb * desc->n_kv_heads * pl.GY;
  const int64_t total = units * blocks_of(max_kv_len, desc->n_nodes_max);
  int64_t wgs = plan_wgs(pl, total, units, true, desc->workgroups);
  const int64_t wgs_cut = plan_wgs(pl, total, units, false, desc->workgroups);  // a ragged batch of the same size
  if (wgs_cut > wgs) wgs = wgs_cut;
  return (size_t)slots_of(pl, units, wgs, total, desc->workgroups) * slot_bytes(*desc, pl);
}

extern "C" fspad_status fspad_tree_attn(const fspad_attn_desc* desc, const void* q, const void* k_tree,
                                        const void* v_tree, const void* k_cache, const void* v_cache,
                                        const int32_t* kv_len, const int32_t* n_nodes,
                                        const uint64_t* anc_mask, void* out, void* workspace,
                                        size_t workspace_bytes, void* hip_stream) {
  const fspad_status st = check_desc(desc);
  if (st != FSPAD_OK) return st;
  if (!q || !k_tree || !v_tree || !kv_len || !n_nodes || !anc_mask || !out) return FSPAD_ERR_NULL;
  const fspad_attn_desc& d = *desc;
  const int esz = d.io_dtype == FSPAD_BF16 ? 2 : 4;
  int max_len = 0;
  for (int b = 0; b < d.batch; ++b) {
    if (kv_len[b] < 0 || n_nodes[b] < 1 || n_nodes[b] > d.n_nodes_max) return FSPAD_ERR_SHAPE;
    if (kv_len[b] > max_len) max_len = kv_len[b];
  }
  if (max_len > 0) {
    if (!k_cache || !v_cache) return FSPAD_ERR_NULL;
    const int64_t align = 16 / esz;
    if (d.cache_stride_token < d.head_dim || d.cache_stride_token > (1ll << 26) || d.cache_stride_token % align || d.cache_stride_head % align ||
        d.cache_stride_batch % align || d.cache_stride_head < 0 || d.cache_stride_batch < 0)
      return FSPAD_ERR_SHAPE;
    if (((uintptr_t)k_cache | (uintptr_t)v_cache) & 15) return FSPAD_ERR_SHAPE;
  }
  if (((uintptr_t)q | (uintptr_t)k_tree | (uintptr_t)v_tree | (uintptr_t)out) & 15) return FSPAD_ERR_SHAPE;
  hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);

  AttnParams prm{};
  prm.anc_mask = anc_mask;
  prm.stride_batch = d.cache_stride_batch; prm.stride_head = d.cache_stride_head; prm.stride_token = d.cache_stride_token;
  prm.Nmax = d.n_nodes_max; prm.Hq = d.n_q_heads; prm.Hkv = d.n_kv_heads;
  prm.G = d.n_q_heads / d.n_kv_heads;
  prm.out_bf16 = d.out_dtype == FSPAD_BF16;
  prm.scale = d.softmax_scale > 0.f ? d.softmax_scale : 1.0f / sqrtf((float)d.head_dim);
  prm.WS = 1; prm.NS = 1; prm.GY = 1;
  prm.g_magic = prm.G > 1 ? (uint32_t)(((1ull << 32) + prm.G - 1) / prm.G) : 0u;

  if (d.io_dtype == FSPAD_BF16) prm.part = reinterpret_cast<float*>(workspace);

  // sequences are independent: slices of at most kMaxBatchPerLaunch sequences per launch (the
  // per-sequence lengths travel as kernel arguments), each slice reusing the workspace in stream order
  for (int b0 = 0; b0 < d.batch; b0 += kMaxBatchPerLaunch) {
    const int nb = d.batch - b0 < kMaxBatchPerLaunch ? d.batch - b0 : kMaxBatchPerLaunch;
    SharedParams sp;   // (its classes: plan_classes, for the kernels that take them)
    AttnParams& sl = sp.a;
    sl = prm;
    sl.B = nb;
    const size_t q_rows = (size_t)b0 * d.n_nodes_max * d.n_q_heads * d.head_dim;
    const size_t kv_rows = (size_t)b0 * d.n_nodes_max * d.n_kv_heads * d.head_dim;
    sl.q = static_cast<const char*>(q) + q_rows * esz;
    sl.k_tree = static_cast<const char*>(k_tree) + kv_rows * esz;
    sl.v_tree = static_cast<const char*>(v_tree) + kv_rows * esz;
    if (k_cache) {
      sl.k_cache = static_cast<const char*>(k_cache) + (size_t)b0 * d.cache_stride_batch * esz;
      sl.v_cache = static_cast<const char*>(v_cache) + (size_t)b0 * d.cache_stride_batch * esz;
    }
    sl.anc_mask = anc_mask + (size_t)b0 * d.n_nodes_max;
    sl.out = static_cast<char*>(out) + q_rows * (d.out_dtype == FSPAD_BF16 ? 2 : 4);
    for (int i = 0; i < nb; ++i) sl.seq[i] = SeqInfo{kv_len[b0 + i], n_nodes[b0 + i]};
    if (d.io_dtype == FSPAD_BF16) {
      bool uniform = true;
      int64_t seq_blocks = 0;
      for (int i = 0; i < nb; ++i) {
        uniform = uniform && blocks_of(sl.seq[i].kv_len, sl.seq[i].nodes) == blocks_of(sl.seq[0].kv_len, sl.seq[0].nodes);
        seq_blocks += blocks_of(sl.seq[i].kv_len, sl.seq[i].nodes);
      }
      Plan pl{};
      plan_rows(d, pl);
      sl.WS = pl.WS; sl.NS = pl.NS; sl.GY = pl.GY;
      sl.ws_shift = pl.WS == 4 ? 2 : (pl.WS == 2 ? 1 : 0);
      // units of a sequence: the slab groups that its own tree fills, times the kv heads
      int groups[kMaxBatchPerLaunch];
      const int64_t full_units = (int64_t)nb * d.n_kv_heads * pl.GY;   // (partial slots: as many as if every tree were full)
      const int64_t full_total = (int64_t)d.n_kv_heads * pl.GY * seq_blocks;
      const int64_t full_wgs = plan_wgs(pl, full_total, full_units, uniform, d.workgroups);
      int64_t total = 0, units = 0;
      int longest = 0;
      for (int i = 0; i < nb; ++i) {
        const int blocks = blocks_of(sl.seq[i].kv_len, sl.seq[i].nodes);
        groups[i] = groups_of(d, pl, sl.seq[i].nodes);
        total += (int64_t)d.n_kv_heads * groups[i] * blocks;
        units += (int64_t)d.n_kv_heads * groups[i];
        if (total > kMaxFlatBlocks) return FSPAD_ERR_SHAPE;  // the kernels index blocks with 32 bits
        if (blocks > longest) longest = blocks;
      }
      bool same = true;
      for (int i = 1; i < nb; ++i) same = same && sl.seq[i].kv_len == sl.seq[0].kv_len && sl.seq[i].nodes == sl.seq[0].nodes;
      // never more workgroups than full trees would have: the workspace a call needs does not depend on the trees
      // (units of equally many blocks stay aligned with the workgroups, however many of them a sequence has: 4 x 64 / 8 heads,
      // 16 to 26 keys, trees of 11 to 26 nodes 10.2 us, planned as a ragged batch 17.4)
      int64_t wgs = plan_wgs(pl, total, units, uniform, d.workgroups);
      if (wgs > full_wgs) wgs = uniform && full_wgs >= units ? full_wgs / units * units : full_wgs;
      sl.setup = uniform || total + units * setup_blocks(pl) > kMaxFlatBlocks ? 0 : setup_blocks(pl);
      // Short units of a ragged batch that fit the chip stay whole, as those of an equal one do (plan_wgs): a workgroup each, and
      // so much set-up that the even division falls into it. Whole units leave no partial results, so the workspace does not bound
      // their number. 12 x 40 / 8 heads, 3 to 8 blocks, 26 nodes: 18.3 -> 13.5 us; few units, which an even split of their blocks
      // puts several to a workgroup: 6 x 12 / 2 heads, D = 64, 2 or 3 blocks 21.7 -> 8.9, 4 x 16 / 1 heads, D = 64, 2 to 8 blocks
      // 16.7 -> 10.0, 2 x 12 / 2 heads, 3 to 5 blocks 19.5 -> 11.2.
      if (!uniform && pl.shared_stage && d.workgroups == 0 && units <= kComputeUnits && longest <= 5 * key_waves(pl)) {
        wgs = units;
        sl.setup = kWholeSetup;
      }
      const int64_t kv_blocks = total;
      bool any_cut = false;
      const int grid = plan_classes(d, pl, groups, wgs, sp, any_cut);
      sl.same_len = kv_len[b0];
      sl.same_nodes = n_nodes[b0];
      const int same_blocks = blocks_of(sl.same_len, sl.same_nodes);
      sl.seq_blocks = same ? d.n_kv_heads * same_blocks : 0;
      sl.seq_rcp = reciprocal(sl.seq_blocks);
      sl.unit_rcp = reciprocal(same_blocks + sl.setup);
      const size_t need = (size_t)slots_of(pl, full_units, full_wgs, full_total, d.workgroups) * slot_bytes(d, pl);
      if (!workspace || workspace_bytes < need || ((uintptr_t)workspace & 15)) return FSPAD_ERR_WORKSPACE;
      if (pl.shared_stage) {
        if (d.head_dim == 128) hipLaunchKernelGGL(tree_attn_gqa128_kernel, dim3((unsigned)grid), dim3(512), 0, stream, sp);
        // (head dim 64 leaves registers for three wavefronts per SIMD: three key groups; 43.1 -> 40.6 us on a
        // 64/8-head, 16384-key, 60-node call, 70.7 -> 64.5 us at 32768 keys)
        else hipLaunchKernelGGL(tree_attn_gqa64_kernel, dim3((unsigned)grid), dim3(768), 0, stream, sp);
      } else {
        // keys and values of the call, read once each (one slab group per kv head). Not the 48- and 64-row tiles of
        // D = 128 where a compute unit takes more than two workgroups in turn: 16 x 40 heads, 60 nodes, 2500 keys 172 us
        // without the hint and 178 with it, 32 x 32 heads, 1200 keys 144 and 148 (one or two in turn: 16 x 32 heads, 76 and
        // 74 us; D = 64: 160 and 156; 16-row tiles 107 and 98)
        const bool in_turn = d.head_dim == 128 && pl.QT >= 3 && sl.n_wgs > 2 * kComputeUnits;
        const bool streamed = !in_turn && (size_t)kv_blocks * (2 * kBlockKeys * 2) * d.head_dim > fspad_detail::kCacheBytes;
        if (d.head_dim == 128) launch_bf16<128>(pl, sl, streamed, stream);
        else launch_bf16<64>(pl, sl, streamed, stream);
      }
      if (hipGetLastError() != hipSuccess) return FSPAD_ERR_HIP;
      // the merge pass runs only if some unit was cut across workgroups
      if (any_cut) {
        // every unit of the launch cut into as many pieces, no workgroup with parts of two (0 where that is not so)
        const int64_t pairs = (int64_t)nb * d.n_kv_heads;
        const int pieces = sl.seq_blocks > 0 && sl.n_wgs % pairs == 0 ? (int)(sl.n_wgs / pairs) : 0;
        if (d.head_dim == 128) launch_combine<128>(pl, sp, pieces, stream);
        else launch_combine<64>(pl, sp, pieces, stream);
        if (hipGetLastError() != hipSuccess) return FSPAD_ERR_HIP;
      }
    } else {
      if (d.head_dim == 128) launch_f32<128>(sl, stream);
      else launch_f32<64>(sl, stream);
      if (hipGetLastError() != hipSuccess) return FSPAD_ERR_HIP;
    }
  }
  return FSPAD_OK;
}
