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

constexpr int kStreamWaves = 8;
constexpr int kSliceRows = 16 * kStreamWaves;   // rows of W per slice
constexpr int kUnitK = 128;                     // k per unit of a wavefront's ring
constexpr int kUnitBytes = 16 * kUnitK * 2;

// MT: 16-row tiles of X. PACKED: W is stored tile by tile instead of row by row -- the 16 rows x 32 k
// of one operand are 1 KB in lane order (lane (n, g) at byte 16 * (n + 16 g)), the k-steps of a
// 16-row tile follow one another, then the next 16 rows. The sums run in the same order either way.
template <int MT, bool PACKED>
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
    int n_xrows, n_wrows, row0, K;
  };

  // Walks `n_stages` stages. A slice is walked from stage `border` of its C = K / kStageK on, around the
  // end of k, back to `border`; then the next slice follows, whose border lies `rot` stages further. The
  // walk begins at stage `at` of `slice`.
  // At a slice's end `slice_end(slice, acc, spare)` takes the sums: acc[t] of lane (n, g) is row
  // row0 + 16 t + n of X against rows 128 slice + 16 wave + 4 g .. + 3 of W. `spare` is the LDS address of
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
      xoff[i] = (unsigned)min(src.row0 + r, src.n_xrows - 1) * (unsigned)row_bytes + (unsigned)(s ^ (r & 15)) * 16u;
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
        __builtin_amdgcn_global_load_lds((StreamGlobalPtr)(b + woff[i]), (StreamLdsPtr)(ring + slot * kUnitBytes + i * 1024), 16, 0, 0);
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

// acc[t][nv] += sum over a k range of
//   X[row0 + 16t + n][k] * W[v0 + 16nv + 4g + i][k]      (lane (n, g), accumulator element i)
// for one wavefront of a workgroup of WAVES wavefronts that share X through LDS.
// MT: 16-row tiles of X per workgroup. SPS: k-steps (of 32) per LDS stage of X (stage = 16*MT rows
// x 32*SPS k). kRing: weight operands per 16-row weight tile that a wavefront keeps requested. VT:
// weight tiles per wavefront. x_base / w_base point at the first k of the range, rows are row_bytes
// apart; the range is n_steps k-steps (a multiple of 8) and is walked from first_step on, wrapping
// around (first_step a multiple of SPS; 0 unless n_steps is a multiple of SPS). xs: 2 stages of LDS.
// PACKED: W is stored tile by tile instead of row by row -- the 16 rows x 32 k of one operand are
// 1 KB in lane order (lane (n, g) at byte 16 * (n + 16 g)), the k-steps of a 16-row tile follow one
// another, then the next 16 rows. A wavefront's request is then one contiguous KB instead of sixteen
// 64-byte pieces a row pitch apart; row_bytes is still 2 K, v0 a multiple of 16, and w_base points at
// the first k-step of the range within tile row 0.
template <int MT, int SPS, int kRing, int WAVES, int VT, bool PACKED = false>
struct StreamGemmRegs {
  static constexpr int kStageK = 32 * SPS;
  static constexpr int kRowBytes = kStageK * 2;                        // 256, 512 or 1024
  static constexpr int kStageBytes = MT * 16 * kRowBytes;
  static constexpr int kChunksPerRow = kRowBytes / 16;                 // 16, 32 or 64
  static constexpr int kRowsPerCopy = 1024 / kRowBytes;                // one copy instruction moves 1 KB
  static constexpr int kCopiesPerWave = kStageBytes / 1024 / WAVES;
  static_assert(kCopiesPerWave >= 1 && kRing % SPS == 0 && kRing % 4 == 0, "stage shape");

  __device__ static __forceinline__ void run(char* xs, const char* x_base, const char* w_base, size_t row_bytes,
                                             int n_xrows, int n_wrows, int row0, int v0, int n_steps, int first_step,
                                             f32x4 (&acc)[MT][VT]) {
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    // weight rows of this lane (rows past the vocabulary are clamped; their columns are never taken)
    const char* wrow[VT];
#pragma unroll
    for (int nv = 0; nv < VT; ++nv)
      wrow[nv] = PACKED ? w_base + (size_t)min(v0 + 16 * nv, n_wrows - 16) * row_bytes + lane * 16
                        : w_base + (size_t)min(v0 + 16 * nv + n, n_wrows - 1) * row_bytes + g * 16;

    // hidden-state copies of this wavefront: LDS slot s of row r receives the row's 16-byte chunk
    // s ^ (r & 15) of the stage's k range (chunks past the end of the row are clamped: never used)
    const char* xsrc[kCopiesPerWave];
    int xcol[kCopiesPerWave];
#pragma unroll
    for (int i = 0; i < kCopiesPerWave; ++i) {
      const int r = kRowsPerCopy * (wave * kCopiesPerWave + i) + lane / kChunksPerRow, s = lane % kChunksPerRow;
      xsrc[i] = x_base + (size_t)min(row0 + r, n_xrows - 1) * row_bytes;
      xcol[i] = s ^ (r & 15);
    }
    const int last_chunk = 4 * n_steps - 1;
    // operand reads: lane (n, g) of tile t, k-step kk of the stage reads chunk 4*kk + g of row 16*t + n,
    // kept at slot (4*kk + g) ^ n = (4*kk) ^ (g ^ n)
    const unsigned xread = (unsigned)n * kRowBytes, xswz = (unsigned)(g ^ n) << 4;

    bf16x8 xr[kCopiesPerWave];
    auto fetch_x = [&](int stage_index) {
#pragma unroll
      for (int i = 0; i < kCopiesPerWave; ++i) {
        int stage = stage_index + first_step / SPS;
        stage -= stage * SPS >= n_steps ? n_steps / SPS : 0;
        const int chunk = min(stage * kChunksPerRow + xcol[i], last_chunk);
        xr[i] = *reinterpret_cast<const bf16x8*>(xsrc[i] + ((size_t)chunk << 4));
      }
    };
    auto store_x = [&](int stage_index) {
      char* dst = xs + (stage_index & 1) * kStageBytes + wave * kCopiesPerWave * 1024 + lane * 16;
#pragma unroll
      for (int i = 0; i < kCopiesPerWave; ++i) *reinterpret_cast<bf16x8*>(dst + i * 1024) = xr[i];
    };
    // workgroup barrier that orders LDS traffic only: the weight requests in flight stay in flight
    auto lds_barrier = [] {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    // k-step ks of the weights: lane (n, g) holds k = 32*ks + 8*g .. +7 of its row (steps past the end
    // re-read the last one, so that every turn of the loop issues the same number of requests)
    auto load_w = [&](int nv, int ks) {
      int step = min(ks, n_steps - 1) + first_step;
      step -= step >= n_steps ? n_steps : 0;
      return *reinterpret_cast<const bf16x8*>(wrow[nv] + (size_t)step * (PACKED ? 1024 : 64));
    };

    // The weights are requested kRing k-steps ahead, every operand register being requested again as
    // soon as its products are issued. The hidden states of stage j+1 are requested into registers at
    // the top of stage j and written to the other LDS stage at its end (by then they have long
    // arrived, and the weight requests issued after them stay in flight); the barrier at the top of a
    // stage publishes every wavefront's share of it and retires the other one.
    bf16x8 w[VT][kRing];
    fetch_x(0);
#pragma unroll
    for (int i = 0; i < kRing; ++i)
#pragma unroll
      for (int nv = 0; nv < VT; ++nv) w[nv][i] = load_w(nv, i);
    store_x(0);
    const int n_stages = (n_steps + SPS - 1) / SPS;
    for (int ks0 = 0; ks0 < n_steps; ks0 += kRing) {
#pragma unroll
      for (int kk = 0; kk < kRing; ++kk) {
        const int ks = ks0 + kk;
        if (kk % 4 == 0 && ks >= n_steps) break;   // K is a multiple of 256 and the ring of 4: the end falls on a multiple of 4 steps
        if (kk % SPS == 0) {
          lds_barrier();
          if (ks / SPS + 1 < n_stages) fetch_x(ks / SPS + 1);
        }
        const char* base = xs + ((ks / SPS) & 1) * kStageBytes + xread + ((((unsigned)kk % SPS) << 6) ^ xswz);
        bf16x8 xf[MT];
#pragma unroll
        for (int t = 0; t < MT; ++t) xf[t] = *reinterpret_cast<const bf16x8*>(base + t * (16 * kRowBytes));
#pragma unroll
        for (int nv = 0; nv < VT; ++nv)
#pragma unroll
          for (int t = 0; t < MT; ++t)
            acc[t][nv] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[nv][kk], xf[t], acc[t][nv], 0, 0, 0);
#pragma unroll
        for (int nv = 0; nv < VT; ++nv) w[nv][kk] = load_w(nv, ks + kRing);
        if (kk % SPS == SPS - 1 && ks / SPS + 1 < n_stages) store_x(ks / SPS + 1);
      }
    }

  }
};

}  // namespace fspad_detail
#endif
