// Streaming core of the skinny bf16 GEMMs of this library (few rows of X, many rows of W, both
// row-major along k): internal to the library. gfx950 (CDNA4) only.
//
// A workgroup of eight wavefronts works on slices of 128 rows of W, sixteen rows per wavefront, and
// walks k in stages; the products run on `v_mfma_f32_16x16x32_bf16` with A = 16 rows of W, B = 16
// rows of X, both operands "8 consecutive k per lane".
//
// W goes from HBM to LDS with global-to-LDS copies, into a ring of two units (16 rows x 128 k = 4 KB
// each) that belongs to the wavefront alone: no registers hold what is in flight, no barrier is
// involved, and a copy instruction may take the bytes of a row in any order. Of row-major weights one
// instruction reads four rows x 256 contiguous bytes (straight into operand registers it has to be
// sixteen rows x 64 bytes), of tile-order weights one contiguous KB. Measured as a pure stream, row-major,
// 32000 x 4096: 44 us (5.9 TB/s) against 53 us for register loads sixteen k-steps ahead; 32000 x 6656:
// 73 us (5.9 TB/s). Two units per wavefront (64 KB requested per compute unit) are enough: with four the same
// streams take 45 and 73 us, with half the row bytes per instruction 48 us and 75 us.
// X (small, L2-resident) is copied the same way for the whole workgroup, a stage ahead, into two
// buffers used in turn. Both are kept XOR-swizzled by 16-byte chunk, so that a 16-row operand read
// touches 16 different bank groups.
//
// Every LDS access of the loop is written out as an instruction with a wait of its own: through
// plain loads the compiler cannot tell them from the ring that the copies are filling, and would wait
// for every copy in flight (vmcnt(0)) first.
#ifndef FSPAD_STREAM_GEMM_H
#define FSPAD_STREAM_GEMM_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace fspad_detail {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef const __attribute__((address_space(1))) void* StreamGlobalPtr;
typedef __attribute__((address_space(3))) void* StreamLdsPtr;

__device__ __forceinline__ unsigned lds_address(const void* p) { return (unsigned)(uintptr_t)(StreamLdsPtr)(p); }
template <int OFF = 0, typename T>
__device__ __forceinline__ void lds_read16(T& v, unsigned addr) {
  static_assert(sizeof(T) == 16, "16 bytes");
  asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(v) : "v"(addr), "n"(OFF));
}
template <typename T>
__device__ __forceinline__ void lds_write16(unsigned addr, const T& v) {
  static_assert(sizeof(T) == 16, "16 bytes");
  asm volatile("ds_write_b128 %0, %1" ::"v"(addr), "v"(v) : "memory");
}
__device__ __forceinline__ void lds_write8(unsigned addr, unsigned long long v) { asm volatile("ds_write_b64 %0, %1" ::"v"(addr), "v"(v) : "memory"); }
__device__ __forceinline__ void lds_read8(unsigned long long& v, unsigned addr) { asm volatile("ds_read_b64 %0, %1" : "=v"(v) : "v"(addr)); }
__device__ __forceinline__ void lds_read4(float& v, unsigned addr) { asm volatile("ds_read_b32 %0, %1" : "=v"(v) : "v"(addr)); }
template <int N>
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(%0)" ::"n"(N) : "memory"); }
template <int N>
__device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
// values read by lds_read16 are only used behind this (volatile instructions keep their order)
template <typename T>
__device__ __forceinline__ void settled(T& v) { asm volatile("" : "+v"(v)); }
// workgroup barrier that orders LDS traffic only: copies in flight stay in flight
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Stage at which workgroup w begins to walk k, of C stages. An XCD's L2 is interleaved over its 16 channels
// every 256 bytes, so rows a power-of-two pitch apart meet on the same channel: if the 32 workgroups of an
// XCD (every eighth workgroup) walk k in step, its traffic crowds one or two channels. Consecutive
// workgroups of an XCD therefore start three stages apart. Pure stream of a row-major 32768 x 4096
// matrix: 6.0 TB/s; with the phases of an XCD's workgroups 8 stages apart 2.9, all equal 4.6 TB/s.
__device__ __forceinline__ unsigned spread_phase(int w, int C) { return (3u * ((unsigned)w / 8u + ((unsigned)w & 7u))) % (unsigned)C; }

// The memory-side cache. What a call reads of more than that -- weights, keys and values, each byte once -- is gone before
// the next call comes back to it, and is read with the non-temporal hint, which spares the caches the replacement: draft
// step of 4 rows (4096 / 11008) 190 -> 180 us, of 40 rows 530 -> 492 us, 20 attention layers of a 33B model 1705 -> 1679 us
// (an 8B head 202 -> 201). What may stay in the cache from one call to the next is slower with the hint: draft step at
// hidden size 2048 88 -> 100 us, 2048 x 32000 head 28 -> 31 us, an attention call over 134 MB repeated by itself 38.8 -> 40.9 us.
// Just above the line both are true: a sampler of 270 MB (60 rows, 4096 / 11008) repeated by itself 60 -> 68 us, with four
// sets of weights in turn, as between two draft steps, 71 -> 68; from 350 MB on the hint is faster either way (70 -> 64 us).
constexpr size_t kCacheBytes = (size_t)256 << 20;

// x / d with rcp = reciprocal(d) from the host: the product's high half is the quotient or one less. A division whose divisor
// the compiler does not know is some 22 instructions with a trip through the vector unit and back; the workgroups of the
// attention made three of them (a merging one too), those of the projections five, before their first request: 32 / 8 heads,
// 60 nodes, 1000 keys 14.76 -> 14.50 us a call, 32 heads, 26 nodes, 2048 keys 16.08 -> 15.94, draft step of 4 rows 180.0 -> 178.0 (with the rotary angles).
__device__ __forceinline__ unsigned div_rcp(unsigned x, unsigned d, unsigned rcp) {
  const unsigned q = __umulhi(x, rcp);
  return q + (x - q * d >= d ? 1u : 0u);
}
inline uint32_t reciprocal(int64_t d) { return d <= 1 ? 0xffffffffu : (uint32_t)((1ull << 32) / (uint64_t)d); }

constexpr int kStreamWaves = 8;
constexpr int kSliceRows = 16 * kStreamWaves;   // rows of W per slice
constexpr int kUnitK = 128;                     // k per unit of a wavefront's ring
constexpr int kUnitBytes = 16 * kUnitK * 2;

// MT: 16-row tiles of X. PACKED: W is stored tile by tile instead of row by row -- the 16 rows x 32 k
// of one operand are 1 KB in lane order (lane (n, g) at byte 16 * (n + 16 g)), the k-steps of a
// 16-row tile follow one another, then the next 16 rows. The sums run in the same order either way.
// STREAMED: the copies of W carry the non-temporal hint (see kCacheBytes).
template <int MT, bool PACKED, bool STREAMED = false>
struct StreamGemm {
  static constexpr int kUnits = MT <= 4 ? 2 : 1;               // units per stage
  static constexpr int kStageK = kUnits * kUnitK;              // 256 or 128
  static constexpr int kXRowBytes = kStageK * 2;
  static constexpr int kXStageBytes = MT * 16 * kXRowBytes;
  static constexpr int kXCopies = kXStageBytes / 1024 / kStreamWaves;   // 16-byte pieces per thread and stage
  static constexpr int kXChunks = kXRowBytes / 16;
  static constexpr int kRing = 2;                           // units of a wavefront's ring
  static constexpr int kRingBytes = kStreamWaves * kRing * kUnitBytes;
  static constexpr int kLdsBytes = kRingBytes + 2 * kXStageBytes;
  static_assert(kXCopies >= 1 && kXCopies * 1024 * kStreamWaves == kXStageBytes, "stage shape");

  struct Source {
    const char* x[2];      // [n_xrows][K] bf16; slices below `split` multiply x[0] / w[0], the others x[1] / w[1]
    const char* w[2];      // [n_wrows][K] bf16
    int split;             // slices of the first problem (0x7fffffff: there is only one)
    int n_xrows, n_wrows, K;
  };

  // Walks `n_stages` stages. A slice is walked from stage `border` of its C = K / kStageK on, around the
  // end of k, back to `border`; then the next slice follows, whose border lies `rot` stages further. The
  // walk begins at stage `at` of `slice`.
  // At a slice's end `slice_end(slice, acc, spare)` takes the sums: acc[t] of lane (n, g) is row
  // 16 t + n of X against rows 128 slice + 16 wave + 4 g .. + 3 of W. `spare` is the LDS address of
  // kXStageBytes that are free from a barrier inside `slice_end` on (plain LDS accesses there would
  // wait for the copies in flight). The range's last sums are handed over too, whole or not.
  template <typename SliceEnd>
  __device__ static __forceinline__ void run(char* lds, const Source& src, int slice, int at, int border, int rot,
                                             int n_stages, SliceEnd&& slice_end) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    const size_t row_bytes = (size_t)src.K * 2;
    char* const ring = lds + wave * kRing * kUnitBytes;
    const unsigned xs = lds_address(lds + kRingBytes);

    // X pieces of this thread: LDS slot s of row r receives the row's chunk s ^ (r & 15) of the stage
    unsigned xoff[kXCopies];
#pragma unroll
    for (int i = 0; i < kXCopies; ++i) {
      const int piece = (wave * kXCopies + i) * 64 + lane, r = piece / kXChunks, s = piece % kXChunks;
      xoff[i] = (unsigned)min(r, src.n_xrows - 1) * (unsigned)row_bytes + (unsigned)(s ^ (r & 15)) * 16u;
    }
    // operand reads: chunk 4 kk + g of row n, kept at slot (4 kk + g) ^ n = (4 kk) ^ (g ^ n)
    const unsigned xread = xs + (unsigned)n * kXRowBytes + ((unsigned)(g ^ n) << 4);
    const unsigned wread = lds_address(ring) + (PACKED ? (unsigned)lane * 16u : (unsigned)n * 256u + ((unsigned)(g ^ n) << 4));

    // W copies: instruction i takes rows 4i .. 4i+3 of the tile (tile order: its i-th KB)
    unsigned woff[4];
    const char* wtile = nullptr;
    auto set_slice = [&](int s) {
      const bool second = s >= src.split;
      const int v0 = (s - (second ? src.split : 0)) * kSliceRows + wave * 16;
      const char* const wb = second ? src.w[1] : src.w[0];
      if constexpr (PACKED) {
        wtile = wb + (size_t)min(v0, (src.n_wrows - 1) & ~15) * row_bytes;
#pragma unroll
        for (int i = 0; i < 4; ++i) woff[i] = (unsigned)lane * 16u + 1024u * i;
      } else {   // (rows past the end are clamped; their sums are never taken)
        const int first = min(v0, src.n_wrows - 1);
        wtile = wb + (size_t)first * row_bytes;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          const int r = 4 * i + (lane >> 4);
          woff[i] = (unsigned)(min(v0 + r, src.n_wrows - 1) - first) * (unsigned)row_bytes + (unsigned)((lane & 15) ^ r) * 16u;
        }
      }
    };
    // a place in the walk: stages (or units) `at` of a slice's `per`, and how many follow it; the last one
    // repeats, so that every turn issues the same number of requests
    struct Cursor {
      int slice, at, border, left, per, rot;
      __device__ __forceinline__ bool next() {   // true: on to the next slice
        if (left == 0) return false;
        --left;
        at = at + 1 == per ? 0 : at + 1;
        if (at != border) return false;
        ++slice;
        border += rot;
        if (border >= per) border -= per;
        at = border;
        return true;
      }
    };
    auto request_unit = [&](const Cursor& at, int slot) {
      const char* b = wtile + (size_t)at.at * (PACKED ? 4096 : 256);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        __builtin_amdgcn_global_load_lds((StreamGlobalPtr)(b + woff[i]), (StreamLdsPtr)(ring + slot * kUnitBytes + i * 1024), 16, 0, STREAMED ? 2 : 0);
    };
    auto request_x = [&](const Cursor& at, int buf) {
      const char* b = (at.slice >= src.split ? src.x[1] : src.x[0]) + (size_t)at.at * kXRowBytes;
#pragma unroll
      for (int i = 0; i < kXCopies; ++i)
        __builtin_amdgcn_global_load_lds((StreamGlobalPtr)(b + xoff[i]),
                                         (StreamLdsPtr)(lds + kRingBytes + buf * kXStageBytes + (wave * kXCopies + i) * 1024), 16, 0, 0);
    };

    // `now` is the stage being multiplied, `xat` the one whose X was requested last (one stage ahead), `wat`
    // the unit of W that was requested last (kRing units ahead)
    const int stages = src.K / kStageK;
    Cursor now{slice, at, border, n_stages - 1, stages, rot}, xat = now;
    Cursor wat{slice, at * kUnits, border * kUnits, n_stages * kUnits - 1, stages * kUnits, rot * kUnits};
    // A unit: its four operands of W and, a k-step ahead of the products, the operands of X. The slot
    // is requested again as soon as its operands have been read.
    f32x4 acc[MT];
    auto unit = [&](int slot, int step0, int buf) {
      const unsigned wa = wread + slot * kUnitBytes, xa = xread + buf * kXStageBytes;
      bf16x8 wf[4], xf[2][MT];
      auto read_x = [&](int j) {
        const unsigned a = xa ^ ((unsigned)(step0 + j) << 6);
        read_tiles(xf[j & 1], a);
      };
      if constexpr (PACKED) {
        lds_read16<0>(wf[0], wa); lds_read16<1024>(wf[1], wa); lds_read16<2048>(wf[2], wa); lds_read16<3072>(wf[3], wa);
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j) lds_read16(wf[j], wa ^ ((unsigned)j << 6));
      }
      read_x(0);
      wait_lds<MT>();
#pragma unroll
      for (int j = 0; j < 4; ++j) settled(wf[j]);
      if (wat.next()) set_slice(wat.slice);
      request_unit(wat, slot);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (j < 3) { read_x(j + 1); wait_lds<MT>(); } else wait_lds<0>();
#pragma unroll
        for (int t = 0; t < MT; ++t) settled(xf[j & 1][t]);
#pragma unroll
        for (int t = 0; t < MT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[j], xf[j & 1][t], acc[t], 0, 0, 0);
      }
    };

    auto clear = [&] {
#pragma unroll
      for (int t = 0; t < MT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    clear();
    request_x(xat, 0);
    set_slice(slice);
    request_unit(wat, 0);
#pragma unroll
    for (int i = 1; i < kRing; ++i) {
      if (wat.next()) set_slice(wat.slice);
      request_unit(wat, i);
    }
    int slot = 0;
    for (int t = 0; t < n_stages; ++t) {
      // this wavefront's share of the stage's X has landed (the units requested after it stay in
      // flight); behind the barrier everybody's has, and the other buffer is free
      if (t == 0) wait_vmem<4 * kRing>();
      else wait_vmem<4 * kUnits>();
      lds_barrier();
      xat.next();
      request_x(xat, (t + 1) & 1);
#pragma unroll
      for (int u = 0; u < kUnits; ++u) {
        // (behind a unit of W: the other units of the ring and this stage's requests for X)
        wait_vmem<4 * (kRing - 1) + kXCopies>();
        unit(slot, 4 * u, t & 1);
        slot = slot == kRing - 1 ? 0 : slot + 1;
      }
      const int ended = now.slice;
      if (now.next() || t + 1 == n_stages) {
        slice_end(ended, acc, xs + (t & 1) * kXStageBytes);
        clear();
      }
    }
    wait_vmem<0>();   // the repeated requests at the end have landed before the ring is given up
  }

 private:
  // the MT operands of one k-step: 16 rows of X apart
  template <int T = 0>
  __device__ static __forceinline__ void read_tiles(bf16x8 (&x)[MT], unsigned a) {
    if constexpr (T < MT) {
      lds_read16<T * 16 * kXRowBytes>(x[T], a);
      read_tiles<T + 1>(x, a);
    }
  }
};

// The same product for more rows of X than the ring's workgroup can hold sums for: 128 rows of W against
// 64 * XT rows of X (XT = 3 or 4) and all of K, eight wavefronts.
//
// At these sizes neither HBM (426 MB of a 32000 x 6656 head: 65 us) nor the matrix cores (46 us for 256 rows) but
// the operand reads bound the kernel if every wavefront keeps rows of W to itself: 16 rows x 256 take an operand of X
// per product, twice what LDS delivers in the time of a product. So the wavefronts form a 2 x 4 grid of
// 64 x (16 XT) tiles: 4 + XT operands for 4 XT products. Both matrices go through LDS, in stages of 64 k copied by
// the global-to-LDS loads, one barrier per stage. Half of the wavefronts copy W (four or five stages, it comes from
// HBM), the others X (three stages, from L2): waits count a wavefront's own requests in order, so a
// wavefront that copied both could not wait for the near one and leave the far one in flight. 16-byte chunk c of a
// row sits at slot c ^ (r >> 1 & 7): two rows fill the 64 banks, and the sixteen rows of an operand read touch
// sixteen different bank groups.
// 32000 x 6656, 240 rows, greedy acceptance: 155 -> 119 us (16 rows of W per wavefront, in registers, before);
// four wavefronts of 64 x 128 tiles 10 % slower; what is left is split over the copies (95 us without most of
// them) and the products (116 us with a quarter of them).
template <int XT, bool PACKED>
struct WideGemm {
  static constexpr int kStageK = 64;
  static constexpr int kWStages = XT == 4 ? 4 : 5, kXStages = 3;
  static constexpr int kRowBytes = kStageK * 2;
  static constexpr int kWBytes = kSliceRows * kRowBytes, kXBytes = 64 * XT * kRowBytes;
  static constexpr int kXAt = kWStages * kWBytes;     // X behind W
  static constexpr int kLdsBytes = kXAt + kXStages * kXBytes;
  static constexpr int kTileBytes = 16 * kRowBytes;   // a 16-row tile of either matrix
  static constexpr int kWCopies = 4, kXCopies = 2 * XT;   // copy instructions of a copying wavefront and stage

  // Stage at which the workgroup of a slice begins, of C stages. The workgroups of an XCD (every eighth) stay
  // within a window of 32 stages, two stages -- the 256 bytes of one L2 channel -- apart, so that they use all
  // channels for W and find the same megabyte of X in L2; each XCD has a window of its own.
  __device__ static __forceinline__ int phase(int slice, int C) {
    return (int)((2u * (((unsigned)slice >> 3) & 15u) + ((unsigned)slice & 7u) * (unsigned)C / 8u) % (unsigned)C);
  }

  // acc[i][t] of lane (n, g): rows v0 + 64 (wave & 1) + 16 i + 4 g .. + 3 of W against row
  // row0 + 16 (XT (wave >> 1) + t) + n of X. The K / 64 stages are walked from `first` on, around the end.
  // Nothing is in flight when it returns, but other wavefronts may still be reading their last stage.
  __device__ static __forceinline__ void run(char* lds, const char* x, const char* w, int n_xrows, int n_wrows, int row0,
                                             int v0, int K, int first, f32x4 (&acc)[4][XT]) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    const size_t row_bytes = (size_t)K * 2;
    const int piece = lane >> 3, slot = lane & 7;   // a copy instruction takes 8 rows x 128 bytes

    // Wavefronts 0..3 copy W (32 rows each), 4..7 X. (Rows past the end of either matrix are clamped; their
    // sums are never taken.)
    const bool copies_w = wave < 4;
    const char* base;
    unsigned off[kXCopies > kWCopies ? kXCopies : kWCopies];
    if (copies_w) {
      if constexpr (PACKED) {
        const int last = (n_wrows - 1) >> 4, tile = (v0 >> 4) + 2 * wave, t0 = min(tile, last);
        base = w + (size_t)t0 * 16 * row_bytes;
#pragma unroll
        for (int i = 0; i < kWCopies; ++i)
          off[i] = (unsigned)(min(tile + i / 2, last) - t0) * 16u * (unsigned)row_bytes + (unsigned)(i & 1) * 1024u + (unsigned)lane * 16u;
      } else {
        const int r0 = min(v0 + 32 * wave, n_wrows - 1);
        base = w + (size_t)r0 * row_bytes;
#pragma unroll
        for (int i = 0; i < kWCopies; ++i) {
          const int r = 8 * i + piece;
          off[i] = (unsigned)(min(v0 + 32 * wave + r, n_wrows - 1) - r0) * (unsigned)row_bytes + (unsigned)(slot ^ ((r >> 1) & 7)) * 16u;
        }
      }
    } else {
      base = x + (size_t)row0 * row_bytes;
#pragma unroll
      for (int i = 0; i < kXCopies; ++i) {
        const int r = 8 * ((wave - 4) * kXCopies + i) + piece;
        off[i] = (unsigned)min(r, n_xrows - 1 - row0) * (unsigned)row_bytes + (unsigned)(slot ^ ((r >> 1) & 7)) * 16u;
      }
    }
    // the copies of this wavefront's matrix: `ahead` is the stage requested last, `to` the slot of the next
    const int stages = K / kStageK;
    int ahead = first, left = stages, to = 0;
    auto request = [&] {
      const char* const src = base + (size_t)ahead * (PACKED && copies_w ? 2048 : kRowBytes);
      if (copies_w) {
#pragma unroll
        for (int i = 0; i < kWCopies; ++i)
          __builtin_amdgcn_global_load_lds((StreamGlobalPtr)(src + off[i]), (StreamLdsPtr)(lds + to * kWBytes + (wave * kWCopies + i) * 1024), 16, 0, 0);
        to = to == kWStages - 1 ? 0 : to + 1;
      } else {
#pragma unroll
        for (int i = 0; i < kXCopies; ++i)
          __builtin_amdgcn_global_load_lds((StreamGlobalPtr)(src + off[i]),
                                           (StreamLdsPtr)(lds + kXAt + to * kXBytes + ((wave - 4) * kXCopies + i) * 1024), 16, 0, 0);
        to = to == kXStages - 1 ? 0 : to + 1;
      }
      // (the last stage repeats: every turn issues the same number of requests)
      if (--left > 0) ahead = ahead + 1 == stages ? 0 : ahead + 1;
    };

    // operand reads of k-step j (32 k): chunk 4 j + g of row n of a tile
    const unsigned swizzled = (unsigned)n * kRowBytes + ((unsigned)(g ^ ((n >> 1) & 7)) << 4);
    const unsigned wread = lds_address(lds) + (unsigned)(wave & 1) * 4u * kTileBytes + (PACKED ? (unsigned)lane * 16u : swizzled);
    const unsigned xread = lds_address(lds) + kXAt + (unsigned)(wave >> 1) * XT * kTileBytes + swizzled;

    // The operands of a k-step are read while the products of the one before it run, a few reads between
    // them (issued in one go they would hold the wavefront up until LDS has taken them all), across the stage's
    // end too: the barrier stands in the middle of a turn, behind the products of the stage's first half, when
    // every wavefront has the operands of the second half in registers -- so that the stage is free as well.
    bf16x8 wf[2][4], xf[2][XT];
    auto multiply = [&](auto step, unsigned wa, unsigned xa) {   // the products of k-step j, the reads of the other one
      constexpr int j = decltype(step)::value, o = 1 - j;
#pragma unroll
      for (int i = 0; i < 4; ++i) settled(wf[j][i]);
#pragma unroll
      for (int i = 0; i < XT; ++i) settled(xf[j][i]);
      products<PACKED ? 1024 * o : 0>(acc, wf[j], xf[j], wf[o], xf[o], PACKED ? wa : wa ^ (64u * o), xa ^ (64u * o));
    };
    const int lead = copies_w ? kWStages : kXStages;
    for (int i = 0; i < lead; ++i) request();
    if (copies_w) wait_vmem<kWCopies * (kWStages - 1)>();
    else wait_vmem<kXCopies * (kXStages - 1)>();
    lds_barrier();
    unsigned wa = wread, xa = xread;
    const unsigned wend = wread + kWStages * kWBytes, xend = xread + kXStages * kXBytes;
    read_tiles<4, 0>(wf[0], wa);
    read_tiles<XT, 0>(xf[0], xa);
    for (int t = 0; t < stages; ++t) {
      wait_lds<0>();
      multiply(std::integral_constant<int, 0>{}, wa, xa);
      // this wavefront's share of the next stage has landed (the ones after it may be in flight)
      if (copies_w) wait_vmem<kWCopies * (kWStages - 2)>();
      else wait_vmem<kXCopies * (kXStages - 2)>();
      lds_barrier();
      request();
      wa = wa + kWBytes == wend ? wread : wa + kWBytes;
      xa = xa + kXBytes == xend ? xread : xa + kXBytes;
      multiply(std::integral_constant<int, 1>{}, wa, xa);   // (reads behind the last stage: a repeated one)
    }
    wait_lds<0>();
#pragma unroll
    for (int i = 0; i < 4; ++i) settled(wf[0][i]);
#pragma unroll
    for (int i = 0; i < XT; ++i) settled(xf[0][i]);
    wait_vmem<0>();   // the repeated requests have landed too
  }

 private:
  // product M of a k-step (tile M / XT of W, M % XT of X) behind, for the first ones, a read for the next
  template <int OFF, int M = 0>
  __device__ static __forceinline__ void products(f32x4 (&acc)[4][XT], const bf16x8 (&wf)[4], const bf16x8 (&xf)[XT],
                                                  bf16x8 (&wn)[4], bf16x8 (&xn)[XT], unsigned wa, unsigned xa) {
    if constexpr (M < 4 * XT) {
      if constexpr (M < 4 + XT) {
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (M < 4) lds_read16<M * kTileBytes + OFF>(wn[M], wa);
        else lds_read16<(M - 4) * kTileBytes>(xn[M - 4], xa);
        __builtin_amdgcn_sched_barrier(0);
      }
      constexpr int i = M / XT, c = M % XT;
      acc[i][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[i], xf[c], acc[i][c], 0, 0, 0);
      products<OFF, M + 1>(acc, wf, xf, wn, xn, wa, xa);
    }
  }
  template <int N, int OFF, int T = 0>
  __device__ static __forceinline__ void read_tiles(bf16x8 (&v)[N], unsigned a) {
    if constexpr (T < N) {
      lds_read16<T * kTileBytes + OFF>(v[T], a);
      read_tiles<N, OFF, T + 1>(v, a);
    }
  }
};

}  // namespace fspad_detail
#endif
