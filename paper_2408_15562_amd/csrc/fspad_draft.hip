// Draft-side forward of the draft model (arXiv 2408.15562, Methodology). gfx950 (CDNA4) only.
//
// 1. The Feature Sampler ("Feature Sampling": an Up Projector for the feature f, a Gate Projector
//    for the token embedding e, SiLU on the lifted embedding, element-wise product with the lifted
//    feature, a Down Projector back to the hidden size, and the feature path's residual connection):
//
//        eta = W_down (SiLU(W_gate e) * (W_up f)) + f
//
// 2. The draft model itself (first paragraph of Methodology: a Transformer Decoder Layer; "Partial
//    Alignment Distillation": the output dimension of its MLP is doubled and both halves share one
//    residual connection, giving the features f~ and f): RMSNorm, fused q / k / v projection with
//    rotary encoding, tree attention over the draft's own cache (the attention entry point of this
//    library), output projection and residual, RMSNorm, gated MLP whose down projection is 2 Hd wide.
//
// Both work on the few rows of one draft step (sequences x tree nodes), so every projection is a
// skinny GEMM bound by streaming its weights once (3 x Hd x I bf16 = 270 MB for the Feature
// Sampler of a 4096 / 11008 model, 494 MB for the decoder layer); they share the streaming core of
// the LM head. A projector has too few 128-row slices of its weight matrix to fill the chip (86 for
// the up / gate projectors, 32 for a 4096-wide output), so every slice is also cut along k:
// workgroup (slice, split) leaves an fp32 partial tile, and a small element-wise kernel sums the
// splits in a fixed order (no atomics: the result is the same from run to run) and applies what
// follows the projector -- SiLU and the product for up / gate, the residual for down and for the
// output projection, the rotary encoding for q / k / v.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "fspad.h"
#include "stream_gemm.h"

namespace {

using fspad_detail::bf16x8;
using fspad_detail::div_rcp;
using fspad_detail::reciprocal;
using fspad_detail::f32x4;
using fspad_detail::StreamGemm;

constexpr int kSliceRows = fspad_detail::kSliceRows;   // weight rows per slice
constexpr int kChunkK = 256;         // every k extent is a multiple of this
constexpr int kMaxRows = 128;        // rows of X per call

// Every slice is walked from a stage of its own on, kRot stages of k further than the slice before: the ranges of an XCD would
// otherwise be at the same stage of k, or at few different ones, wherever the length of a range and a slice's stages have a common
// divisor (4096-wide rows: six stages of 16), and rows a power-of-two pitch apart then crowd a few L2 channels.
constexpr int kRot = 3;

// How a projection is spread: its slices (of all problems that share the launch) and their stages
// along k form one flat list, and workgroup w streams the contiguous range
// [floor(w T / W), floor((w + 1) T / W)) of it, so that every compute unit fetches the same number of
// bytes whatever the shape. What a workgroup sums of a slice goes to partial slot (slice + w).
struct Split {
  int32_t n_slices;   // all problems
  int32_t stages;     // per slice
  int32_t total;      // n_slices * stages
  int32_t n_wgs;
  int32_t rot;        // kRot, of as many stages
  uint32_t wgs_rcp, total_rcp, stages_rcp;   // reciprocals (div_rcp)
};
__device__ __forceinline__ int range_begin(const Split& s, int w) { return (int)div_rcp((unsigned)w * (unsigned)s.total, (unsigned)s.n_wgs, s.wgs_rcp); }
// the workgroup whose range holds stage x (32 bits do: at most 2^21 stages and 256 workgroups)
__device__ __forceinline__ int owner_of(const Split& s, int x) { return (int)div_rcp(((unsigned)x + 1u) * (unsigned)s.n_wgs - 1u, (unsigned)s.total, s.total_rcp); }

// Partial sums of a launch: slot (slice + w) holds [rows][128] fp32 for the stages of the slice that
// workgroup w summed.
struct Partials {
  const float* base;
  Split split;
  int32_t rows;

  // Sums over the slots of 4 consecutive columns each (from the first slice `slice0` of a problem), in workgroup order.
  // The slots of a slice are some two to nine, and the passes that sum them are bound by their trips to memory. `request`
  // sends for up to 2 * kInFlight slots of all N sums at once, and a kernel requests whatever else it reads (residual, gain)
  // beside it, so that one trip is over at `finish` (slots behind those are fetched there). With the slots four at a time,
  // the residual behind the sums, the gains behind the normalisation's barrier and the rotary angles (a trip for the
  // position, sine and cosine in fp64) before the first slot, a draft step of 4 rows took 174.8 us instead of 171.8, one of
  // 40 rows (6656 / 17920) 479.5 instead of 475.0; with the slots one by one some 4 us more.
  static constexpr int kInFlight = 4;
  template <int N>
  struct Sums {
    const float* p[N];
    int n[N], longest;
    f32x4 v[2][N][kInFlight];
  };
  template <int N>
  __device__ __forceinline__ void request(const int (&slice0)[N], int row, const int (&col)[N], Sums<N>& s) const {
    const size_t slot = (size_t)rows * kSliceRows;
    s.longest = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int slice = slice0[i] + col[i] / kSliceRows;
      const int w0 = owner_of(split, slice * split.stages), w1 = owner_of(split, slice * split.stages + split.stages - 1);
      s.p[i] = base + (size_t)(slice + w0) * slot + (size_t)row * kSliceRows + col[i] % kSliceRows;
      s.n[i] = w1 - w0 + 1;
      s.longest = max(s.longest, s.n[i]);
    }
    fetch(s, 0, s.v[0]);
    if (s.longest > kInFlight) fetch(s, kInFlight, s.v[1]);
  }
  template <int N>
  __device__ __forceinline__ void finish(Sums<N>& s, f32x4 (&a)[N]) const {
#pragma unroll
    for (int i = 0; i < N; ++i) a[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    add(s, 0, s.v[0], a);
    if (s.longest > kInFlight) add(s, kInFlight, s.v[1], a);
    for (int s0 = 2 * kInFlight; s0 < s.longest; s0 += kInFlight) {
      fetch(s, s0, s.v[0]);
      add(s, s0, s.v[0], a);
    }
  }

 private:
  template <int N>
  __device__ __forceinline__ void fetch(const Sums<N>& s, int s0, f32x4 (&v)[N][kInFlight]) const {
    const size_t slot = (size_t)rows * kSliceRows;
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int k = 0; k < kInFlight; ++k) v[i][k] = *reinterpret_cast<const f32x4*>(s.p[i] + (size_t)min(s0 + k, s.n[i] - 1) * slot);
  }
  template <int N>
  __device__ __forceinline__ void add(const Sums<N>& s, int s0, const f32x4 (&v)[N][kInFlight], f32x4 (&a)[N]) const {
#pragma unroll
    for (int i = 0; i < N; ++i)
#pragma unroll
      for (int k = 0; k < kInFlight; ++k)
        if (s0 + k < s.n[i]) a[i] += v[i][k];
  }
};

struct PartialGemmParams {
  const char* x[2];        // [rows][K] bf16, one per problem (up / gate share a launch)
  const char* w[2];        // [N][K] bf16, row-major or (PACKED) in the tile order of fspad_pack_weight
  float* part;
  int32_t rows, N, K;
  int32_t split;           // slices of the first problem
  Split plan;
};

template <int MT, bool PACKED, bool STREAMED>
__global__ __launch_bounds__(64 * fspad_detail::kStreamWaves, 2) void partial_gemm_kernel(const PartialGemmParams p) {
  typedef StreamGemm<MT, PACKED, STREAMED> G;
  __shared__ __attribute__((aligned(1024))) char lds[G::kLdsBytes];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, g = lane >> 4;
  // an XCD (every eighth workgroup) takes neighbouring ranges
  const int per_xcd = p.plan.n_wgs >> 3;
  const int w = (p.plan.n_wgs & 7) == 0 ? (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3) : (int)blockIdx.x;
  const int t0 = range_begin(p.plan, w), t1 = range_begin(p.plan, w + 1);
  typename G::Source src;
  src.x[0] = p.x[0]; src.x[1] = p.x[1]; src.w[0] = p.w[0]; src.w[1] = p.w[1];
  src.split = p.split; src.n_xrows = p.rows; src.n_wrows = p.N; src.K = p.K;
  const int slice = (int)div_rcp((unsigned)t0, (unsigned)p.plan.stages, p.plan.stages_rcp);
  const unsigned turned = (unsigned)slice * kRot;
  const int border = (int)(turned - (unsigned)p.plan.stages * div_rcp(turned, (unsigned)p.plan.stages, p.plan.stages_rcp));
  int at = t0 - slice * p.plan.stages + border;
  at -= at >= p.plan.stages ? p.plan.stages : 0;
  G::run(lds, src, slice, at, border, p.plan.rot, t1 - t0, [&](int s, const f32x4 (&acc)[MT], unsigned) {
    // lane (n, g) holds columns 16 wave + 4g .. +3 of row 16t + n
    float* out = p.part + (size_t)(s + w) * p.rows * kSliceRows + wave * 16 + 4 * g;
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const int r = 16 * t + n;
      if (r < p.rows) *reinterpret_cast<f32x4*>(out + (size_t)r * kSliceRows) = acc[t];
    }
  });
}

struct CombineParams {
  Partials part;
  const char* f;           // residual input [rows][N] bf16 (MODE 1)
  char* out;               // [rows][N] bf16 (MODE 2: [rows][N/2], columns below N/2)
  char* out2;              // MODE 2: [rows][N/2], columns from N/2 on
  int32_t rows, N, residual;
};

// MODE 0: out = SiLU(gate sums) * up sums (two problems). MODE 1: out = sums (+ f). MODE 2: the N columns
// are two halves that go to two arrays, each half added to the same residual f [rows][N/2]. Four columns
// per thread.
template <int MODE>
__global__ __launch_bounds__(256) void combine_kernel(const CombineParams p) {
  typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
  const int row = blockIdx.y, col = 4 * (int)(blockIdx.x * 256 + threadIdx.x);
  if (col >= p.N) return;
  const int half_n = p.N / 2;
  const bool second = MODE == 2 && col >= half_n;
  const size_t at = MODE == 2 ? ((size_t)row * half_n + (second ? col - half_n : col)) * 2 : ((size_t)row * p.N + col) * 2;   // bytes
  constexpr int kSums = MODE == 0 ? 2 : 1;
  int slice0[kSums] = {0}, cols[kSums] = {col};
  if constexpr (MODE == 0) { slice0[1] = (p.N + kSliceRows - 1) / kSliceRows; cols[1] = col; }
  Partials::Sums<kSums> sums;
  p.part.request<kSums>(slice0, row, cols, sums);
  bf16x4 r = {0, 0, 0, 0};
  if (MODE == 2 || (MODE == 1 && p.residual)) r = *reinterpret_cast<const bf16x4*>(p.f + at);
  f32x4 a[kSums];
  p.part.finish<kSums>(sums, a);
  bf16x4 o;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if constexpr (MODE == 0) o[i] = (__bf16)(a[1][i] / (1.0f + __expf(-a[1][i])) * a[0][i]);   // 0: up, 1: gate
    else o[i] = (__bf16)(MODE == 2 || p.residual ? a[0][i] + (float)r[i] : a[0][i]);
  }
  *reinterpret_cast<bf16x4*>((second ? p.out2 : p.out) + at) = o;
}

// RMSNorm of one row per workgroup: out = x / sqrt(mean(x^2) + eps) * gain, fp32 arithmetic, one
// rounding to bf16. Hd is a multiple of 8.
struct RmsNormParams {
  const char* x;           // [rows][Hd] bf16
  const char* gain;        // [Hd] bf16
  char* out;               // [rows][Hd] bf16
  int32_t Hd;
  float eps;
};
__global__ __launch_bounds__(256) void rms_norm_kernel(const RmsNormParams p) {
  constexpr int kKept = 4;   // of a thread's pieces, in registers
  __shared__ float wave_sum[4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const char* xr = p.x + (size_t)blockIdx.x * p.Hd * 2;
  const int n_vec = p.Hd / 8;
  const auto vec = [](const char* at, int v) { return *reinterpret_cast<const bf16x8*>(at + 16 * v); };
  bf16x8 x[kKept], gain[kKept];
#pragma unroll
  for (int k = 0; k < kKept; ++k)
    if (const int v = tid + 256 * k; v < n_vec) { x[k] = vec(xr, v); gain[k] = vec(p.gain, v); }
  float ss = 0.f;
  auto square = [&](const bf16x8& xv) {
#pragma unroll
    for (int i = 0; i < 8; ++i) { const float t = (float)xv[i]; ss += t * t; }
  };
#pragma unroll
  for (int k = 0; k < kKept; ++k)
    if (tid + 256 * k < n_vec) square(x[k]);
  for (int v = tid + 256 * kKept; v < n_vec; v += 256) square(vec(xr, v));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
  if (lane == 0) wave_sum[wave] = ss;
  __syncthreads();
  const float total = (wave_sum[0] + wave_sum[1]) + (wave_sum[2] + wave_sum[3]);
  const float inv = 1.0f / sqrtf(total / (float)p.Hd + p.eps);
  char* outr = p.out + (size_t)blockIdx.x * p.Hd * 2;
  auto scale = [&](int v, const bf16x8& xv, const bf16x8& gv) {
    bf16x8 o;
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i] = (__bf16)((float)xv[i] * inv * (float)gv[i]);
    *reinterpret_cast<bf16x8*>(outr + 16 * v) = o;
  };
#pragma unroll
  for (int k = 0; k < kKept; ++k)
    if (const int v = tid + 256 * k; v < n_vec) scale(v, x[k], gain[k]);
  for (int v = tid + 256 * kKept; v < n_vec; v += 256) scale(v, vec(xr, v), vec(p.gain, v));
}

// Output projection's epilogue and the normalisation that follows it, one row per workgroup:
// h = sum of the partials + residual (rounded to bf16, written), then out = rmsnorm(h) of the rounded
// values, as rms_norm_kernel would compute it from h. What a thread wrote of h stays in its registers (of rows of more than
// 1024 * 4 * kKept entries the rest is read back, by the same thread). 1024
// threads: with the few rows of a draft step the row's loads must all be in flight at once. (What is under way takes 88 registers, one workgroup a compute unit
// where 36 had room for two, and the other passes 63 to 100; with up to 128 rows, the most a call takes, there are no more workgroups than compute units: 60 calls
// of 32 to 128 rows, hidden size 1024 to 6656, took 0.95 to 1.00 of the time, 4 x 16 rows of 1024 45.6 -> 43.8 us, 8 x 16 of 6656 404.8 -> 402.2.)
struct CombineNormParams {
  Partials part;
  const char* residual;    // [rows][Hd] bf16
  const char* gain;        // [Hd] bf16
  char* h;                 // [rows][Hd] bf16
  char* out;               // [rows][Hd] bf16
  int32_t Hd;
  float eps;
};
__global__ __launch_bounds__(1024) void combine_norm_kernel(const CombineNormParams p) {
  typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
  constexpr int kKept = 2;   // of a thread's quads, in registers
  __shared__ float wave_sum[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const size_t row_at = (size_t)blockIdx.x * p.Hd;
  const int n_quads = p.Hd / 4;
  const auto quad = [](const char* at, size_t i) { return *reinterpret_cast<const bf16x4*>(at + 2 * i); };
  Partials::Sums<1> sums[kKept];
  bf16x4 kept[kKept], gain[kKept];
#pragma unroll
  for (int k = 0; k < kKept; ++k)
    if (const int q = tid + 1024 * k; q < n_quads) {
      p.part.request<1>({0}, blockIdx.x, {4 * q}, sums[k]);
      kept[k] = quad(p.residual, row_at + 4 * q);
      gain[k] = quad(p.gain, 4 * q);
    }
  float ss = 0.f;
  auto state = [&](int q, Partials::Sums<1>& sum, const bf16x4& r) {   // four entries of h
    f32x4 a[1];
    p.part.finish<1>(sum, a);
    bf16x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o[i] = (__bf16)(a[0][i] + (float)r[i]);
      const float t = (float)o[i];
      ss += t * t;
    }
    *reinterpret_cast<bf16x4*>(p.h + (row_at + 4 * q) * 2) = o;
    return o;
  };
#pragma unroll
  for (int k = 0; k < kKept; ++k)
    if (const int q = tid + 1024 * k; q < n_quads) kept[k] = state(q, sums[k], kept[k]);
  for (int q = tid + 1024 * kKept; q < n_quads; q += 1024) {
    Partials::Sums<1> sum;
    p.part.request<1>({0}, blockIdx.x, {4 * q}, sum);
    state(q, sum, quad(p.residual, row_at + 4 * q));
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
  if (lane == 0) wave_sum[wave] = ss;
  __syncthreads();
  float total = 0.f;
#pragma unroll
  for (int i = 0; i < 16; ++i) total += wave_sum[i];
  const float inv = 1.0f / sqrtf(total / (float)p.Hd + p.eps);
  auto scale = [&](int q, const bf16x4& hv, const bf16x4& gv) {
    bf16x4 o;
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = (__bf16)((float)hv[i] * inv * (float)gv[i]);
    *reinterpret_cast<bf16x4*>(p.out + (row_at + 4 * q) * 2) = o;
  };
#pragma unroll
  for (int k = 0; k < kKept; ++k)
    if (const int q = tid + 1024 * k; q < n_quads) scale(q, kept[k], gain[k]);
  for (int q = tid + 1024 * kKept; q < n_quads; q += 1024) scale(q, quad(p.h, row_at + 4 * q), quad(p.gain, 4 * q));
}

// Sum of the q / k / v projection's partials, rotary encoding of the query and key heads, scatter
// into the attention's layouts. A thread owns four columns of the first half of one head of one
// row and the four partner columns of the second half: entry i of the first half and entry i of
// the second half turn by position * theta^(-2i/D). Angles and their sine / cosine are formed in
// fp64 (a position of some thousands times a frequency rounded to fp32 would already be off by
// more than the result's bf16 rounding), once per workgroup (a row's heads share them): one angle for each of its first D/2
// threads instead of four for every thread.
struct QkvRopeParams {
  Partials part;
  const int32_t* positions;  // [rows]
  char* q;                 // [rows][Hq][D] bf16
  char* k;                 // [rows][Hkv][D] bf16
  char* v;                 // [rows][Hkv][D] bf16
  int32_t rows, Hq, Hkv, D;
  double neg_log2_theta_2_over_d;   // -2 log2(theta) / D
};
__global__ __launch_bounds__(256) void qkv_rope_kernel(const QkvRopeParams p) {
  typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
  __shared__ float2 turn[64];   // cosine and sine of entry i
  const int quad_shift = p.D == 128 ? 4 : 3, heads = p.Hq + 2 * p.Hkv, half = p.D / 2;
  const int row = blockIdx.y, t = (int)(blockIdx.x * 256 + threadIdx.x);
  const int j = t & ((1 << quad_shift) - 1), head = t >> quad_shift;
  Partials::Sums<2> sums;
  if (head < heads) p.part.request<2>({0, 0}, row, {head * p.D + 4 * j, head * p.D + 4 * j + half}, sums);   // (on their way beside the angles)
  if ((int)threadIdx.x < half) {
    const double ang = (double)p.positions[row] * exp2((double)threadIdx.x * p.neg_log2_theta_2_over_d);
    double sn, cs;
    sincos(ang, &sn, &cs);
    turn[threadIdx.x] = make_float2((float)cs, (float)sn);
  }
  __syncthreads();
  if (head >= heads) return;
  f32x4 ab[2];
  p.part.finish<2>(sums, ab);
  const f32x4 a = ab[0], b = ab[1];
  char* dst;
  if (head < p.Hq) dst = p.q + ((size_t)row * p.Hq + head) * p.D * 2;
  else if (head < p.Hq + p.Hkv) dst = p.k + ((size_t)row * p.Hkv + (head - p.Hq)) * p.D * 2;
  else dst = p.v + ((size_t)row * p.Hkv + (head - p.Hq - p.Hkv)) * p.D * 2;
  bf16x4 oa, ob;
  if (head < p.Hq + p.Hkv) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float c = turn[4 * j + i].x, s = turn[4 * j + i].y;
      oa[i] = (__bf16)(a[i] * c - b[i] * s);
      ob[i] = (__bf16)(b[i] * c + a[i] * s);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) { oa[i] = (__bf16)a[i]; ob[i] = (__bf16)b[i]; }
  }
  *reinterpret_cast<bf16x4*>(dst + 8 * j) = oa;
  *reinterpret_cast<bf16x4*>(dst + 8 * j + 2 * half) = ob;
}

constexpr int kComputeUnits = 256;
// The flat split of a projection of N columns (per problem) over K. One workgroup per compute unit, and
// not less than two stages for each.
Split plan_split(int N, int K, int problems, int rows) {
  Split s{};
  s.n_slices = problems * ((N + kSliceRows - 1) / kSliceRows);
  s.stages = K / (rows <= 64 ? 256 : 128);
  s.total = s.n_slices * s.stages;
  s.n_wgs = s.total / 2 < kComputeUnits ? (s.total + 1) / 2 : kComputeUnits;
  s.rot = kRot % s.stages;
  s.wgs_rcp = reciprocal(s.n_wgs); s.total_rcp = reciprocal(s.total); s.stages_rcp = reciprocal(s.stages);
  return s;
}
size_t partial_floats(const Split& s, int rows) { return (size_t)(s.n_slices + s.n_wgs) * rows * kSliceRows; }

template <bool PACKED, bool STREAMED>
void launch_partial(const PartialGemmParams& g, hipStream_t stream) {
  const dim3 grid((unsigned)g.plan.n_wgs), block(64 * fspad_detail::kStreamWaves);
  if (g.rows <= 16) hipLaunchKernelGGL((partial_gemm_kernel<1, PACKED, STREAMED>), grid, block, 0, stream, g);
  else if (g.rows <= 32) hipLaunchKernelGGL((partial_gemm_kernel<2, PACKED, STREAMED>), grid, block, 0, stream, g);
  else if (g.rows <= 48) hipLaunchKernelGGL((partial_gemm_kernel<3, PACKED, STREAMED>), grid, block, 0, stream, g);
  else if (g.rows <= 64) hipLaunchKernelGGL((partial_gemm_kernel<4, PACKED, STREAMED>), grid, block, 0, stream, g);
  else hipLaunchKernelGGL((partial_gemm_kernel<8, PACKED, STREAMED>), grid, block, 0, stream, g);
}

// The partial sums of one projection (or of two that share x's shape and w's), on the stream. `streamed`: the weights of
// the whole call exceed the memory-side cache.
fspad_status linear_partials(const void* x0, const void* x1, const void* w0, const void* w1, int rows, int N, int K,
                             const Split& plan, float* part, bool packed, bool streamed, hipStream_t stream) {
  PartialGemmParams g{};
  g.x[0] = static_cast<const char*>(x0); g.x[1] = static_cast<const char*>(x1);
  g.w[0] = static_cast<const char*>(w0); g.w[1] = static_cast<const char*>(w1);
  g.part = part; g.rows = rows; g.N = N; g.K = K;
  g.split = w1 ? plan.n_slices / 2 : plan.n_slices;
  g.plan = plan;
  if (packed) streamed ? launch_partial<true, true>(g, stream) : launch_partial<true, false>(g, stream);
  else streamed ? launch_partial<false, true>(g, stream) : launch_partial<false, false>(g, stream);
  return hipGetLastError() == hipSuccess ? FSPAD_OK : FSPAD_ERR_HIP;
}

template <int MODE>
fspad_status combine(const float* part, const Split& plan, const void* residual, void* out, void* out2, int rows, int N,
                     hipStream_t stream) {
  CombineParams c{};
  c.part = Partials{part, plan, rows};
  c.f = static_cast<const char*>(residual); c.out = static_cast<char*>(out);
  c.out2 = static_cast<char*>(out2); c.rows = rows; c.N = N; c.residual = residual != nullptr;
  hipLaunchKernelGGL(combine_kernel<MODE>, dim3((unsigned)((N / 4 + 255) / 256), (unsigned)rows), dim3(256), 0, stream, c);
  return hipGetLastError() == hipSuccess ? FSPAD_OK : FSPAD_ERR_HIP;
}

struct Plan {
  Split up, down;
  size_t part_floats, s_bytes;
};
Plan make_plan(int rows, int Hd, int I) {
  Plan pl{};
  pl.up = plan_split(I, Hd, 2, rows);
  pl.down = plan_split(Hd, I, 1, rows);
  const size_t up = partial_floats(pl.up, rows), down = partial_floats(pl.down, rows);
  pl.part_floats = up > down ? up : down;
  pl.s_bytes = ((size_t)rows * I * 2 + 255) & ~(size_t)255;
  return pl;
}

}  // namespace

extern "C" size_t fspad_feature_sampler_workspace_bytes(int32_t rows, int32_t hidden_dim, int32_t intermediate_dim) {
  if (rows < 1 || rows > kMaxRows || hidden_dim < kChunkK || hidden_dim % kChunkK || intermediate_dim < kChunkK ||
      intermediate_dim % kChunkK)
    return 0;
  const Plan pl = make_plan(rows, hidden_dim, intermediate_dim);
  return pl.s_bytes + ((pl.part_floats * 4 + 255) & ~(size_t)255);
}

extern "C" fspad_status fspad_feature_sampler(int32_t rows, int32_t hidden_dim, int32_t intermediate_dim, const void* f,
                                              const void* e, const void* w_up, const void* w_gate, const void* w_down,
                                              int32_t flags, void* eta, void* workspace, size_t workspace_bytes,
                                              void* hip_stream) {
  if (flags & ~(FSPAD_SAMPLER_RESIDUAL | FSPAD_WEIGHTS_PACKED)) return FSPAD_ERR_SHAPE;
  const int residual = flags & FSPAD_SAMPLER_RESIDUAL, packed = (flags & FSPAD_WEIGHTS_PACKED) != 0;
  if (!f || !e || !w_up || !w_gate || !w_down || !eta) return FSPAD_ERR_NULL;
  if (rows < 1 || rows > kMaxRows) return FSPAD_ERR_SHAPE;
  if (hidden_dim < kChunkK || hidden_dim % kChunkK || hidden_dim > (1 << 16)) return FSPAD_ERR_SHAPE;
  if (intermediate_dim < kChunkK || intermediate_dim % kChunkK || intermediate_dim > (1 << 18)) return FSPAD_ERR_SHAPE;
  if ((((uintptr_t)f) | ((uintptr_t)e) | ((uintptr_t)w_up) | ((uintptr_t)w_gate) | ((uintptr_t)w_down) | ((uintptr_t)eta)) & 15)
    return FSPAD_ERR_SHAPE;
  if (!workspace || ((uintptr_t)workspace & 15) ||
      workspace_bytes < fspad_feature_sampler_workspace_bytes(rows, hidden_dim, intermediate_dim))
    return FSPAD_ERR_WORKSPACE;
  hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
  const Plan pl = make_plan(rows, hidden_dim, intermediate_dim);
  char* s_buf = static_cast<char*>(workspace);                       // SiLU(gate) * up, [rows][I] bf16
  float* part = reinterpret_cast<float*>(s_buf + pl.s_bytes);

  const bool streamed = (size_t)3 * hidden_dim * intermediate_dim * 2 > fspad_detail::kCacheBytes;

  // up and gate projectors, one launch
  fspad_status st;
  if ((st = linear_partials(f, e, w_up, w_gate, rows, intermediate_dim, hidden_dim, pl.up, part, packed, streamed, stream)) != FSPAD_OK) return st;
  if ((st = combine<0>(part, pl.up, nullptr, s_buf, nullptr, rows, intermediate_dim, stream)) != FSPAD_OK) return st;
  // down projector and residual
  if ((st = linear_partials(s_buf, nullptr, w_down, nullptr, rows, hidden_dim, intermediate_dim, pl.down, part, packed, streamed, stream)) != FSPAD_OK)
    return st;
  return combine<1>(part, pl.down, residual ? f : nullptr, eta, nullptr, rows, hidden_dim, stream);
}

// ------------------------------------------------------------------------------------------------
// The draft decoder layer.
namespace {

size_t align256(size_t n) { return (n + 255) & ~(size_t)255; }

struct LayerPlan {
  int rows, Hd, I, qkv_n, attn_n;
  Split qkv, o, up, down;
  size_t xn_bytes, q_bytes, a_bytes, h_bytes, s_bytes, part_bytes, attn_ws_bytes;
};

bool layer_shape_ok(const fspad_draft_layer_desc* d) {
  const fspad_attn_desc& a = d->attn;
  if (a.batch < 1 || a.n_nodes_max < 1 || a.n_nodes_max > FSPAD_MAX_NODES) return false;
  if ((int64_t)a.batch * a.n_nodes_max > kMaxRows) return false;
  if (a.n_q_heads < 1 || a.n_kv_heads < 1 || a.n_q_heads % a.n_kv_heads) return false;
  if (a.head_dim != 64 && a.head_dim != 128) return false;
  if (d->hidden_dim < kChunkK || d->hidden_dim % kChunkK || d->hidden_dim > (1 << 16)) return false;
  if (d->intermediate_dim < kChunkK || d->intermediate_dim % kChunkK || d->intermediate_dim > (1 << 18)) return false;
  const int64_t attn_n = (int64_t)a.n_q_heads * a.head_dim;
  if (attn_n % kChunkK || attn_n > (1 << 16)) return false;
  if (!(d->rms_eps >= 0.0f) || !(d->rope_theta > 0.0f)) return false;
  if (d->weights_packed != 0 && d->weights_packed != 1) return false;
  return true;
}

LayerPlan make_layer_plan(const fspad_draft_layer_desc* d, int32_t max_kv_len) {
  LayerPlan pl{};
  const fspad_attn_desc& a = d->attn;
  pl.rows = a.batch * a.n_nodes_max;
  pl.Hd = d->hidden_dim;
  pl.I = d->intermediate_dim;
  pl.attn_n = a.n_q_heads * a.head_dim;
  pl.qkv_n = (a.n_q_heads + 2 * a.n_kv_heads) * a.head_dim;
  pl.qkv = plan_split(pl.qkv_n, pl.Hd, 1, pl.rows);
  pl.o = plan_split(pl.Hd, pl.attn_n, 1, pl.rows);
  pl.up = plan_split(pl.I, pl.Hd, 2, pl.rows);
  pl.down = plan_split(2 * pl.Hd, pl.I, 1, pl.rows);
  pl.xn_bytes = align256((size_t)pl.rows * pl.Hd * 2);
  pl.q_bytes = align256((size_t)pl.rows * pl.attn_n * 2);
  pl.a_bytes = pl.q_bytes;
  pl.h_bytes = pl.xn_bytes;
  pl.s_bytes = align256((size_t)pl.rows * pl.I * 2);
  size_t part = 0;
  for (const Split* sp : {&pl.qkv, &pl.o, &pl.up, &pl.down}) part = partial_floats(*sp, pl.rows) > part ? partial_floats(*sp, pl.rows) : part;
  pl.part_bytes = align256(part * 4);
  pl.attn_ws_bytes = align256(fspad_tree_attn_workspace_bytes(&d->attn, max_kv_len));
  return pl;
}

fspad_status rms_norm(const void* x, const void* gain, void* out, int rows, int Hd, float eps, hipStream_t stream) {
  RmsNormParams r{};
  r.x = static_cast<const char*>(x); r.gain = static_cast<const char*>(gain); r.out = static_cast<char*>(out);
  r.Hd = Hd; r.eps = eps;
  hipLaunchKernelGGL(rms_norm_kernel, dim3((unsigned)rows), dim3(256), 0, stream, r);
  return hipGetLastError() == hipSuccess ? FSPAD_OK : FSPAD_ERR_HIP;
}

}  // namespace

extern "C" size_t fspad_draft_layer_workspace_bytes(const fspad_draft_layer_desc* desc, int32_t max_kv_len) {
  if (!desc || max_kv_len < 0 || !layer_shape_ok(desc)) return 0;
  if (desc->attn.io_dtype != FSPAD_BF16 || desc->attn.out_dtype != FSPAD_BF16) return 0;
  const LayerPlan pl = make_layer_plan(desc, max_kv_len);
  return pl.xn_bytes + pl.q_bytes + pl.a_bytes + pl.h_bytes + pl.s_bytes + pl.part_bytes + pl.attn_ws_bytes;
}

extern "C" fspad_status fspad_draft_layer(const fspad_draft_layer_desc* desc, const fspad_draft_layer_weights* w,
                                          const void* eta, const int32_t* positions, const void* k_cache,
                                          const void* v_cache, const int32_t* kv_len, const int32_t* n_nodes,
                                          const uint64_t* anc_mask, void* k_tree, void* v_tree, void* f_tilde, void* f,
                                          void* workspace, size_t workspace_bytes, void* hip_stream) {
  if (!desc || !w || !eta || !positions || !kv_len || !n_nodes || !anc_mask || !k_tree || !v_tree || !f_tilde || !f)
    return FSPAD_ERR_NULL;
  if (!w->w_qkv || !w->w_o || !w->w_gate || !w->w_up || !w->w_down || !w->gain_attn || !w->gain_mlp) return FSPAD_ERR_NULL;
  if (desc->attn.io_dtype != FSPAD_BF16 || desc->attn.out_dtype != FSPAD_BF16) return FSPAD_ERR_DTYPE;
  if (!layer_shape_ok(desc)) return FSPAD_ERR_SHAPE;
  const uintptr_t all = (uintptr_t)eta | (uintptr_t)k_tree | (uintptr_t)v_tree | (uintptr_t)f_tilde | (uintptr_t)f |
                        (uintptr_t)w->w_qkv | (uintptr_t)w->w_o | (uintptr_t)w->w_gate | (uintptr_t)w->w_up |
                        (uintptr_t)w->w_down | (uintptr_t)w->gain_attn | (uintptr_t)w->gain_mlp;
  if (all & 15) return FSPAD_ERR_SHAPE;
  int32_t max_kv = 0;
  for (int b = 0; b < desc->attn.batch; ++b) {
    if (kv_len[b] < 0 || n_nodes[b] < 1 || n_nodes[b] > desc->attn.n_nodes_max) return FSPAD_ERR_SHAPE;
    if (kv_len[b] > max_kv) max_kv = kv_len[b];
  }
  if (!workspace || ((uintptr_t)workspace & 15) || workspace_bytes < fspad_draft_layer_workspace_bytes(desc, max_kv))
    return FSPAD_ERR_WORKSPACE;
  hipStream_t stream = reinterpret_cast<hipStream_t>(hip_stream);
  const LayerPlan pl = make_layer_plan(desc, max_kv);
  const fspad_attn_desc& a = desc->attn;
  const bool packed = desc->weights_packed != 0;

  char* at = static_cast<char*>(workspace);
  char* xn = at; at += pl.xn_bytes;            // normalised input of a projection, [rows][Hd] bf16
  char* q = at; at += pl.q_bytes;              // [rows][Hq][D] bf16
  char* attn = at; at += pl.a_bytes;           // attention output, [rows][Hq][D] bf16
  char* h = at; at += pl.h_bytes;              // state after attention, [rows][Hd] bf16
  char* s = at; at += pl.s_bytes;              // SiLU(gate) * up, [rows][I] bf16
  float* part = reinterpret_cast<float*>(at); at += pl.part_bytes;
  char* attn_ws = at;

  const bool streamed = (size_t)pl.Hd * (pl.qkv_n + pl.attn_n + 4 * (size_t)pl.I) * 2 > fspad_detail::kCacheBytes;

  fspad_status st;
  // q, k, v = rotary(W_qkv rmsnorm(eta))
  if ((st = rms_norm(eta, w->gain_attn, xn, pl.rows, pl.Hd, desc->rms_eps, stream)) != FSPAD_OK) return st;
  if ((st = linear_partials(xn, nullptr, w->w_qkv, nullptr, pl.rows, pl.qkv_n, pl.Hd, pl.qkv, part, packed, streamed, stream)) != FSPAD_OK)
    return st;
  {
    QkvRopeParams r{};
    r.part = Partials{part, pl.qkv, pl.rows}; r.positions = positions; r.q = q; r.k = static_cast<char*>(k_tree); r.v = static_cast<char*>(v_tree);
    r.rows = pl.rows; r.Hq = a.n_q_heads; r.Hkv = a.n_kv_heads; r.D = a.head_dim;
    r.neg_log2_theta_2_over_d = -2.0 * log2((double)desc->rope_theta) / (double)a.head_dim;
    const int threads = (a.n_q_heads + 2 * a.n_kv_heads) * (a.head_dim / 8);   // per row
    hipLaunchKernelGGL(qkv_rope_kernel, dim3((unsigned)((threads + 255) / 256), (unsigned)pl.rows), dim3(256), 0, stream, r);
    if (hipGetLastError() != hipSuccess) return FSPAD_ERR_HIP;
  }
  // tree attention over the draft's own cache
  st = fspad_tree_attn(&desc->attn, q, k_tree, v_tree, k_cache, v_cache, kv_len, n_nodes, anc_mask, attn, attn_ws,
                       pl.attn_ws_bytes, hip_stream);
  if (st != FSPAD_OK) return st;
  // h = eta + W_o attn
  if ((st = linear_partials(attn, nullptr, w->w_o, nullptr, pl.rows, pl.Hd, pl.attn_n, pl.o, part, packed, streamed, stream)) != FSPAD_OK)
    return st;
  // and its normalised form for the MLP (whose doubled down projection adds both halves to h)
  {
    CombineNormParams c{};
    c.part = Partials{part, pl.o, pl.rows}; c.residual = static_cast<const char*>(eta); c.gain = static_cast<const char*>(w->gain_mlp);
    c.h = h; c.out = xn; c.Hd = pl.Hd; c.eps = desc->rms_eps;
    hipLaunchKernelGGL(combine_norm_kernel, dim3((unsigned)pl.rows), dim3(1024), 0, stream, c);
    if (hipGetLastError() != hipSuccess) return FSPAD_ERR_HIP;
  }
  if ((st = linear_partials(xn, xn, w->w_up, w->w_gate, pl.rows, pl.I, pl.Hd, pl.up, part, packed, streamed, stream)) != FSPAD_OK) return st;
  if ((st = combine<0>(part, pl.up, nullptr, s, nullptr, pl.rows, pl.I, stream)) != FSPAD_OK) return st;
  if ((st = linear_partials(s, nullptr, w->w_down, nullptr, pl.rows, 2 * pl.Hd, pl.I, pl.down, part, packed, streamed, stream)) != FSPAD_OK)
    return st;
  return combine<2>(part, pl.down, h, f_tilde, f, pl.rows, 2 * pl.Hd, stream);
}

// ------------------------------------------------------------------------------------------------
// Weight repacking: row-major [N][K] -> tile order (see stream_gemm.h). One thread per 16 bytes.
namespace {
__global__ __launch_bounds__(256) void pack_weight_kernel(const char* w, char* packed, int32_t n_rows, int32_t K) {
  const int steps = K / 32;
  const size_t total = (size_t)((n_rows + 15) / 16) * steps * 64;
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= total) return;
  const int lane = (int)(i & 63), n = lane & 15, g = lane >> 4;
  const size_t tile_step = i >> 6;
  const int step = (int)(tile_step % steps);
  const size_t row = (tile_step / steps) * 16 + n;
  bf16x8 v = {0, 0, 0, 0, 0, 0, 0, 0};
  if (row < (size_t)n_rows) v = *reinterpret_cast<const bf16x8*>(w + (row * K + 32 * step + 8 * g) * 2);
  *reinterpret_cast<bf16x8*>(packed + i * 16) = v;
}
}  // namespace

extern "C" size_t fspad_packed_weight_bytes(int32_t n_rows, int32_t k) {
  if (n_rows < 1 || k < 32 || k % 32) return 0;
  return (size_t)((n_rows + 15) / 16) * 16 * (size_t)k * 2;
}

extern "C" fspad_status fspad_pack_weight(int32_t n_rows, int32_t k, const void* w, void* packed, void* hip_stream) {
  if (!w || !packed) return FSPAD_ERR_NULL;
  if (n_rows < 1 || k < 32 || k % 32) return FSPAD_ERR_SHAPE;
  if ((((uintptr_t)w) | ((uintptr_t)packed)) & 15) return FSPAD_ERR_SHAPE;
  const size_t threads = fspad_packed_weight_bytes(n_rows, k) / 16;
  if ((threads + 255) / 256 > 0x7fffffffu) return FSPAD_ERR_SHAPE;
  hipLaunchKernelGGL(pack_weight_kernel, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0,
                     reinterpret_cast<hipStream_t>(hip_stream), static_cast<const char*>(w), static_cast<char*>(packed),
                     n_rows, k);
  return hipGetLastError() == hipSuccess ? FSPAD_OK : FSPAD_ERR_HIP;
}
