// The decoder around the hot path: the backbone f_theta whose attention the
// Local and Full branches restrict (§2.1), as a pre-norm decoder stack with
// bf16 weights and fp32 activations, so that a whole ODA decode step (Alg. 1:
// Local forward, recall head, conditional Full forward, commit, output
// projection) can be timed against the additive cost model of App. A.6.
//
//   oda_dense_bf16    y = W . RMSNorm(x) (optional), + residual (optional), or
//                     the SwiGLU pair SiLU(W_g . x') * (W_u . x')
//   oda_qk_norm_rope  per-head RMSNorm of q and k, rotary embedding at each
//                     request's current position, bf16 q / K / V candidates
//   oda_embed_bf16    embedding rows of the step's tokens
//   oda_copy_rows     rows of the selected requests from one buffer to another
//   oda_rms_norm_rows RMSNorm (with gain) of the selected requests' rows: the
//                     final normalised hidden state the recall head reads
//   oda_argmax        greedy token of each request's logits
//
// Every kernel can be restricted to a device-side list of requests (the
// recall gate's compacted list), so the Full retry touches only flagged
// requests.  All of them are bound by HBM (bf16 weight streaming for the
// dense layers at small batch), not by arithmetic.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <climits>
#include <cmath>

#include "oda.h"
#include "oda_device.h"
#include "oda_internal.h"

namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kWaves = 4;

constexpr int kDenseMinWaves = 2048;   // grouping rows stops short of fewer wavefronts than this

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }
__device__ __forceinline__ uint16_t to_bf16(float f) { return oda::bf16_rne(f); }
__device__ __forceinline__ float silu(float x) { return x / (1.f + __expf(-x)); }
__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) x += __shfl_xor(x, s);
  return x;
}
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// Requests a launch covers: the listed ones, else all B.
__device__ __forceinline__ int selected_count(const int32_t* n_work, int B) {
  return n_work ? min(max(n_work[0], 0), B) : B;
}
__device__ __forceinline__ int selected_request(const int32_t* work_list, int slot) {
  return work_list ? work_list[slot] : slot;
}

// ---------------------------------------------------------------------------
// dense layer
// ---------------------------------------------------------------------------

struct DenseArgs {
  const uint16_t* W;       // [N][K] bf16 (SwiGLU: [2N][K], gate rows then up rows)
  const float* gain;       // [K] RMSNorm gain of the input, or NULL (no norm)
  const float* x;          // [B][K]
  const float* residual;   // [B][N] or NULL
  float* y;                // [B][N] (may be the residual buffer)
  const int32_t* work_list;
  const int32_t* n_work;
  int N, K, B;
  float eps;
};

// One request per grid row, one wavefront per group of R output rows.  Lanes take 8
// consecutive weights of each row (one 16-byte load per row), so a wavefront
// reads R KiB per 512-element chunk, several chunks in flight; every input
// load serves all R rows.  The inputs come from cache.  The input's sum of
// squares (for RMSNorm) accumulates in the same pass.  R > 1 makes the
// wavefronts of a layer with many short rows fewer and longer.
template <bool kSwiGLU, int R>
__global__ __launch_bounds__(256) void dense_kernel(DenseArgs p) {
  const int lane = threadIdx.x & 63;
  const int wave = uniform(threadIdx.x >> 6);
  const int item = blockIdx.x * kWaves + wave;
  const int row0 = item * R;                   // the host keeps N a multiple of R
  if (row0 >= p.N || (int)blockIdx.y >= selected_count(p.n_work, p.B)) return;
  const int b = selected_request(p.work_list, blockIdx.y);
  if (b < 0 || b >= p.B) return;               // a listed request outside the batch is skipped
  const bool norm = p.gain != nullptr;

  const float* xr = p.x + (int64_t)b * p.K;
  const uint16_t* wrow = p.W + (int64_t)row0 * p.K;
  const uint16_t* wrow2 = kSwiGLU ? p.W + (int64_t)(p.N + row0) * p.K : nullptr;
  float acc[R], acc2[kSwiGLU ? R : 1], ss = 0.f;
#pragma unroll
  for (int j = 0; j < R; ++j) {
    acc[j] = 0.f;
    if (kSwiGLU) acc2[j] = 0.f;
  }
  // 512-element chunks (8 per lane).  In a ragged last chunk the lanes past K
  // read element 0 again and weigh it by zero, so every load is unconditional
  // and the loads of successive chunks overlap.
  const int nchunks = (p.K + 511) / 512;
  // about eight 16-byte weight loads in flight per lane; sixteen for the
  // SwiGLU pair (few registers per load, and the pair is the decoder's
  // largest layer)
  constexpr int kRowsPerChunk = kSwiGLU ? 2 * R : R;
  constexpr int kInFlight = kSwiGLU ? 16 : 8;
  constexpr int kUnroll = kRowsPerChunk >= kInFlight ? 1 : kInFlight / kRowsPerChunk;
#pragma unroll kUnroll
  for (int c = 0; c < nchunks; ++c) {
    const int k0 = c * 512 + 8 * lane;
    const bool in = k0 < p.K;
    const int k = in ? k0 : 0;
    const float mask = in ? 1.f : 0.f;
    u32x4 w[R], w2[kSwiGLU ? R : 1];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      w[j] = *reinterpret_cast<const u32x4*>(wrow + (int64_t)j * p.K + k);
      if (kSwiGLU) w2[j] = *reinterpret_cast<const u32x4*>(wrow2 + (int64_t)j * p.K + k);
    }
    // (asked for before the gains, or the compiler shares the two loads'
    // registers and waits for the first: 520 -> 65536 13.9 us instead of 12.8;
    // not for the pair, which the registers cost more: an MLP of 1688 and 2784
    // 13.1 us instead of 12.7)
    float4 x0, x1;
    auto load_x = [&] {
      x0 = *reinterpret_cast<const float4*>(xr + k);
      x1 = *reinterpret_cast<const float4*>(xr + k + 4);
    };
    if (!kSwiGLU) load_x();
    float g[8];
    if (norm) {
      const float4 g0 = *reinterpret_cast<const float4*>(p.gain + k);
      const float4 g1 = *reinterpret_cast<const float4*>(p.gain + k + 4);
      g[0] = g0.x; g[1] = g0.y; g[2] = g0.z; g[3] = g0.w;
      g[4] = g1.x; g[5] = g1.y; g[6] = g1.z; g[7] = g1.w;
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) g[e] = 1.f;
    }
    if (kSwiGLU) load_x();
    const float xv[8] = {x0.x * mask, x0.y * mask, x0.z * mask, x0.w * mask,
                         x1.x * mask, x1.y * mask, x1.z * mask, x1.w * mask};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (norm) ss += xv[e] * xv[e];
      const float xg = xv[e] * g[e];
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const uint32_t we = w[j][e >> 1];
        acc[j] += ((e & 1) ? bf16_hi(we) : bf16_lo(we)) * xg;
        if (kSwiGLU) {
          const uint32_t we2 = w2[j][e >> 1];
          acc2[j] += ((e & 1) ? bf16_hi(we2) : bf16_lo(we2)) * xg;
        }
      }
    }
  }

  // reduce over the wavefront; lane j keeps row row0 + j
  const float sum_sq = norm ? wave_sum(ss) : 0.f;
  float v = 0.f, v2 = 0.f;
#pragma unroll
  for (int j = 0; j < R; ++j) {
    const float a = wave_sum(acc[j]);
    const float a2 = kSwiGLU ? wave_sum(acc2[j]) : 0.f;
    if (lane == j) {
      v = a;
      v2 = a2;
    }
  }
  if (lane >= R) return;
  const int row = row0 + lane;
  const float inv = norm ? rsqrtf(sum_sq / (float)p.K + p.eps) : 1.f;
  float out;
  if (kSwiGLU) {
    out = silu(v * inv) * (v2 * inv);
  } else {
    out = v * inv;
    if (p.residual) out += p.residual[(int64_t)b * p.N + row];
  }
  p.y[(int64_t)b * p.N + row] = out;
}

// ---------------------------------------------------------------------------
// dense layer for several requests, on the matrix cores
// ---------------------------------------------------------------------------

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kMfmaWaves = 8;      // wavefronts per workgroup; they split K
constexpr int kMfmaRows = 16;      // rows and requests of one MFMA tile
constexpr int kChunk = 64;         // elements of K a wavefront stages at a time
constexpr int kMfmaMaxK = 1 << 28; // a tile's sixteen rows stay within 32-bit element offsets
constexpr int kTargetGroups = 256; // workgroups a launch aims for (one per CU)

// x = p[0] + p[1] + p[2] with bf16 pieces, exactly where the last piece is no
// subnormal (|x| from 2^-110): each piece is the leading eight significant bits
// of what the ones before it leave (truncation, so no piece overflows).  An
// infinity is its own first piece; a NaN stays one.
__device__ __forceinline__ void split_bf16x3(const float (&x)[8], bf16x8 (&p)[3]) {
  float r[8];
  float mx = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    r[e] = x[e];
    mx = __builtin_elementwise_maximum(mx, fabsf(x[e]));   // (a NaN if there is one)
  }
  const bool odd = __any(!(mx < INFINITY));
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    u32x4 w;
#pragma unroll
    for (int e = 0; e < 4; ++e)   // the high halves of two floats
      w[e] = __builtin_amdgcn_perm(__float_as_uint(r[2 * e + 1]), __float_as_uint(r[2 * e]), 0x07060302u);
    if (q < 2) {
#pragma unroll
      for (int e = 0; e < 8; ++e) r[e] -= __uint_as_float(__float_as_uint(r[e]) & 0xffff0000u);
      if (q == 0 && odd) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          if (x[e] != x[e]) w[e / 2] |= 0x40u << (16 * (e & 1));   // quiet: a NaN whose payload is cut stays one
          r[e] = fabsf(x[e]) == INFINITY ? 0.f : r[e];
        }
      }
    }
    p[q] = __builtin_bit_cast(bf16x8, w);
  }
}

// y = W x' for up to 16 selected requests per workgroup on
// v_mfma_f32_16x16x32_bf16, W's rows as the A operand (lane h, j: row h,
// elements 8j..8j+7 of a 32-element step) and the requests as columns.  The
// fp32 inputs enter as three bf16 pieces each (split_bf16x3), so every product
// is exact and the sums are fp32, as in the one-request kernel; the leading
// pieces' products and the others' are summed apart, so fewer roundings happen
// at the size of the result.
//
// The eight wavefronts split K into contiguous stretches and add their tiles
// through LDS in wavefront order.  A wavefront walks its stretch in chunks of
// kChunk elements, the next chunk's inputs and weights in flight while this
// one is multiplied.  Both are read as long contiguous runs (inputs: four
// request rows of 256 bytes per load, weights: eight rows of 128 bytes) and
// turned into operands through the wavefront's own part of LDS: with each lane
// reading its operand straight from memory (16 rows of 64 bytes per load,
// neighbouring lanes on different rows) the loads, not HBM, set the time
// (2048 -> 151936, 4 requests: 142 us against 106; 6144 -> 2048, 32 requests:
// 18.5 against 11.7).  The bound is HBM for large layers (2048 -> 151936: 5.8
// TB/s up to eight requests) and start-up, one wait for the first chunk, and
// the reduction for small ones.  Two chunks of weights in flight, 16
// wavefronts, and chunks of 128 were all slower.
//   P       row tiles of the workgroup (SwiGLU: gate and up tiles each)
//   kHalf   tiles of eight rows, for at most eight requests at a time: tile
//           rows and columns 8..15 hold the same rows and requests over the
//           second half of K (the two off-diagonal quadrants are not used), so
//           that a layer of few rows still fills the chip
template <bool kSwiGLU, bool kNorm, int P, bool kHalf>
__global__ __launch_bounds__(kMfmaWaves * 64) __attribute__((amdgpu_waves_per_eu(2)))
void dense_mfma_kernel(DenseArgs p) {
  constexpr int S = kSwiGLU ? 2 * P : P;              // weight streams: stream P + i is tile i's up projection
  constexpr int kEdge = kHalf ? 8 : kMfmaRows;        // rows and requests per tile
  constexpr int U = kChunk / 32;                      // steps per chunk
  constexpr int kLanes = kChunk / 4;                  // lanes that read one input row of a chunk
  constexpr int kRowsAt = 64 / kLanes;                // input rows per load
  constexpr int kPairs = kMfmaRows / kRowsAt;         // loads that read a chunk of the sixteen input rows
  constexpr int kPitch = kChunk + 4;                  // floats per staged input row: rows on different banks
  constexpr int kWLanes = kChunk / 8;                 // lanes that read one weight row of a chunk
  constexpr int kWLoads = kMfmaRows * kWLanes / 64;   // loads that read a chunk of one tile
  constexpr int kWPitch = kChunk + 8;
  __shared__ union {
    struct {
      float x[kMfmaWaves][kMfmaRows][kPitch];
      uint16_t w[kMfmaWaves][S][kMfmaRows][kWPitch];
    };
    f32x4 acc[kMfmaWaves][S][64];
  } sm;
  __shared__ float sm_ss[kMfmaWaves][kMfmaRows];
  const int lane = threadIdx.x & 63;
  const int wave = uniform(threadIdx.x >> 6);
  const int h = lane & 15, j = lane >> 4;
  const int count = selected_count(p.n_work, p.B);
  // the batch tiles of a row group run next to each other on one XCD
  // (workgroup i runs on XCD i mod 8), so its weights come from HBM once
  const int groups = (p.N + P * kEdge - 1) / (P * kEdge);
  const int span = 8 * ((p.B + kEdge - 1) / kEdge);
  const int rg = (int)(blockIdx.x / span) * 8 + (int)(blockIdx.x % 8);
  const int s0 = (int)(blockIdx.x % span) / 8 * kEdge;
  if (rg >= groups || s0 >= count) return;
  const int nb = min(kEdge, count - s0);
  const int row0 = rg * P * kEdge;

  // K in 32-element steps, a contiguous stretch per wavefront; kHalf: tile
  // rows and columns 8..15 start at the second half
  const int khalf = kHalf ? ((p.K / 8 + 1) / 2) * 8 : p.K;
  const int steps = (khalf + 31) / 32;
  const int per = (steps + kMfmaWaves - 1) / kMfmaWaves;
  const int step0 = min(steps, wave * per);
  const int n = min(steps, step0 + per) - step0;
  const int chunks = (n + U - 1) / U;
  // end of this wavefront's stretch within either half (kHalf: loads of tile
  // rows and columns 8..15 take the second)
  static_assert(!kHalf || (kMfmaRows / kRowsAt == 4 && kWLoads == 2), "a load stays within one half");
  const int stop0 = min(khalf, (step0 + n) * 32), stop1 = min(p.K - khalf, (step0 + n) * 32);

  // input row 4m + lane / 16 of load m: its request's row (columns past the
  // last request repeat it and are not stored; a listed request outside
  // [0, B) is computed as request 0 and not stored) and half of K
  const float* xrow[kPairs];
#pragma unroll
  for (int m = 0; m < kPairs; ++m) {
    const int v = kRowsAt * m + lane / kLanes;
    const int b = selected_request(p.work_list, s0 + min(v & (kEdge - 1), nb - 1));
    xrow[m] = p.x + (int64_t)(b >= 0 && b < p.B ? b : 0) * p.K + (kHalf && m >= kPairs / 2 ? khalf : 0);
  }
  // tile row kMfmaRows / kWLoads * i + lane / kWLanes of weight load i, as an
  // offset from the stream's first row; rows past the last repeat it
  const uint16_t* wbase[S];
  uint32_t woff[P][kWLoads];                          // (the host keeps K below kMfmaMaxK)
#pragma unroll
  for (int s = 0; s < S; ++s) wbase[s] = p.W + (int64_t)((s < P ? 0 : p.N) + min(row0 + (s % P) * kEdge, p.N - 1)) * p.K;
#pragma unroll
  for (int i = 0; i < kWLoads; ++i) {
    const int v = kMfmaRows / kWLoads * i + lane / kWLanes;
#pragma unroll
    for (int s = 0; s < P; ++s)
      woff[s][i] = (uint32_t)max(0, min(v & (kEdge - 1), p.N - 1 - (row0 + s * kEdge))) * (uint32_t)p.K;
  }
  // the epilogue's outputs of this thread; their residuals are read now
  constexpr int kOut = P * kEdge * kEdge;
  constexpr int kThreads = kMfmaWaves * 64;
  constexpr int kPer = (kOut + kThreads - 1) / kThreads;
  int out_b[kPer];
  float res[kPer];
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const int e = threadIdx.x + q * kThreads;
    const int row = row0 + (e / (kEdge * kEdge)) * kEdge + e % kEdge;
    const int slot = e / kEdge % kEdge;
    out_b[q] = -1;
    res[q] = 0.f;
    if (e < kOut && row < p.N && slot < nb) {
      const int b = selected_request(p.work_list, s0 + slot);
      if (b >= 0 && b < p.B) {
        out_b[q] = b;
        if (!kSwiGLU && p.residual) res[q] = p.residual[(int64_t)b * p.N + row];
      }
    }
  }

  f32x4 acc[S], low[S];
  float ss[kPairs];
#pragma unroll
  for (int s = 0; s < S; ++s) acc[s] = low[s] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int m = 0; m < kPairs; ++m) ss[m] = 0.f;
  u32x4 w[S][kWLoads];
  f32x4 x[kPairs], g[kHalf ? 2 : 1] = {};
  const int kx = step0 * 32 + 4 * (lane % kLanes);                                // of chunk 0, within a half
  const int kw = step0 * 32 + 8 * (lane % kWLanes);
  // an element past the end reads the row's start and counts as zero
  auto back_x = [&](int m) { return kHalf && m >= kPairs / 2 ? -khalf : 0; };
  auto load_x = [&](int c) {
#pragma unroll
    for (int m = 0; m < kPairs; ++m) {
      const int k = kx + c * kChunk;
      x[m] = *reinterpret_cast<const f32x4*>(xrow[m] + (k < (kHalf && m >= kPairs / 2 ? stop1 : stop0) ? k : back_x(m)));
    }
    if (kNorm) {
#pragma unroll
      for (int q = 0; q < (kHalf ? 2 : 1); ++q) {
        const int k = kx + c * kChunk + q * khalf;
        g[q] = *reinterpret_cast<const f32x4*>(p.gain + (k < p.K ? k : 0));
      }
    }
  };
  auto load_w = [&](int c) {
#pragma unroll
    for (int i = 0; i < kWLoads; ++i) {
      const int k = kw + c * kChunk;
      const bool second = kHalf && i == 1;
      const uint32_t at = k < (second ? stop1 : stop0) ? (uint32_t)(k + (second ? khalf : 0)) : 0u;
#pragma unroll
      for (int s = 0; s < S; ++s) w[s][i] = *reinterpret_cast<const u32x4*>(wbase[s] + (woff[s % P][i] + at));
    }
  };
  float (&stage)[kMfmaRows][kPitch] = sm.x[wave];
  // Only a stretch's last chunk can reach past its end (kHalf: the second
  // half's, which is no longer than the first): there inputs, gains and weights
  // are zeroed, all of them, since 0 times an infinity would be NaN.
  const bool ragged = n % U != 0 || (step0 + n) * 32 > (kHalf ? p.K - khalf : p.K);
  auto put_x = [&](int c, bool last) {
#pragma unroll
    for (int m = 0; m < kPairs; ++m) {
      f32x4 v = x[m], gk = g[kHalf && m >= kPairs / 2 ? 1 : 0];
      if (last) {
        if (kx + c * kChunk >= (kHalf && m >= kPairs / 2 ? stop1 : stop0)) v = gk = f32x4{0.f, 0.f, 0.f, 0.f};
      }
      if (kNorm) {
        ss[m] += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
        v = f32x4{v[0] * gk[0], v[1] * gk[1], v[2] * gk[2], v[3] * gk[3]};
      }
      *reinterpret_cast<f32x4*>(&stage[kRowsAt * m + lane / kLanes][4 * (lane % kLanes)]) = v;
    }
  };
  auto put_w = [&](int c, bool last) {
#pragma unroll
    for (int i = 0; i < kWLoads; ++i) {
      if (last) {
        if (kw + c * kChunk >= (kHalf && i == 1 ? stop1 : stop0)) {
#pragma unroll
          for (int s = 0; s < S; ++s) w[s][i] = u32x4{0u, 0u, 0u, 0u};
        }
      }
#pragma unroll
      for (int s = 0; s < S; ++s)
        *reinterpret_cast<u32x4*>(&sm.w[wave][s][kMfmaRows / kWLoads * i + lane / kWLanes][8 * (lane % kWLanes)]) = w[s][i];
    }
  };
  auto step = [&](int u) {
    float xv[8];
    const f32x4 lo = *reinterpret_cast<const f32x4*>(&stage[h][32 * u + 8 * j]);
    const f32x4 hi = *reinterpret_cast<const f32x4*>(&stage[h][32 * u + 8 * j + 4]);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      xv[e] = lo[e];
      xv[4 + e] = hi[e];
    }
    bf16x8 px[3];
    split_bf16x3(xv, px);
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const bf16x8 ws = *reinterpret_cast<const bf16x8*>(&sm.w[wave][s][h][32 * u + 8 * j]);
      acc[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ws, px[0], acc[s], 0, 0, 0);
      low[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ws, px[2], low[s], 0, 0, 0);
      low[s] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ws, px[1], low[s], 0, 0, 0);
    }
  };
  if (chunks > 0) {
    load_x(0);
    load_w(0);
    for (int c = 0; c + 1 < chunks; ++c) {
      put_x(c, false);
      load_x(c + 1);
      put_w(c, false);
      load_w(c + 1);
      oda::wave_lds_fence();
#pragma unroll
      for (int u = 0; u < U; ++u) step(u);
      oda::wave_lds_fence();
    }
    put_x(chunks - 1, ragged);
    put_w(chunks - 1, ragged);
    oda::wave_lds_fence();
#pragma unroll
    for (int u = 0; u < U; ++u) step(u);
  }

  // add the wavefronts' tiles in order
  if (kNorm) {
#pragma unroll
    for (int m = 0; m < kPairs; ++m) {
#pragma unroll
      for (int s = kLanes / 2; s >= 1; s >>= 1) ss[m] += __shfl_xor(ss[m], s);
      if ((lane % kLanes) == 0) sm_ss[wave][kRowsAt * m + lane / kLanes] = ss[m];
    }
  }
  __syncthreads();   // the staged chunks are no longer read
#pragma unroll
  for (int s = 0; s < S; ++s) {
    // an infinite weight makes `low` NaN where an input's lower pieces are
    // zero: a sum of the leading pieces that is not finite is the result
    f32x4 t;
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = fabsf(acc[s][i]) < INFINITY ? acc[s][i] + low[s][i] : acc[s][i];
    sm.acc[wave][s][lane] = t;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    if (out_b[q] < 0) continue;
    const int e = threadIdx.x + q * kThreads;
    const int tile = e / (kEdge * kEdge), row = e % kEdge, col = e / kEdge % kEdge;
    float v = 0.f, v2 = 0.f, sq = 0.f;
#pragma unroll
    for (int half = 0; half < (kHalf ? 2 : 1); ++half) {
      const int hr = row + 8 * half, hcol = col + 8 * half;
      const int at = (hr / 4) * 16 + hcol;              // the lane that holds rows 4j..4j+3 of the column
#pragma unroll
      for (int wv = 0; wv < kMfmaWaves; ++wv) {
        v += sm.acc[wv][tile][at][hr % 4];
        if (kSwiGLU) v2 += sm.acc[wv][P + tile][at][hr % 4];
        if (kNorm) sq += sm_ss[wv][hcol];
      }
    }
    const float inv = kNorm ? rsqrtf(sq / (float)p.K + p.eps) : 1.f;
    const float out = kSwiGLU ? silu(v * inv) * (v2 * inv) : v * inv + res[q];
    p.y[(int64_t)out_b[q] * p.N + row0 + tile * kEdge + row] = out;
  }
}

template <bool kSwiGLU, int P, bool kHalf>
oda_status launch_dense_mfma(const DenseArgs& a, hipStream_t stream) {
  constexpr int kEdge = kHalf ? 8 : kMfmaRows;
  const int64_t groups = oda::ceil_div(oda::ceil_div(a.N, P * kEdge), 8) * 8 * oda::ceil_div(a.B, kEdge);
  if (groups > INT_MAX) return oda::fail(ODA_ERR_SHAPE, "layer too large");
  const dim3 grid((unsigned)groups), block(kMfmaWaves * 64);
  if (a.gain)
    hipLaunchKernelGGL((dense_mfma_kernel<kSwiGLU, true, P, kHalf>), grid, block, 0, stream, a);
  else
    hipLaunchKernelGGL((dense_mfma_kernel<kSwiGLU, false, P, kHalf>), grid, block, 0, stream, a);
  return ODA_OK;
}

// ---------------------------------------------------------------------------
// per-head RMSNorm + rotary embedding, bf16 candidates
// ---------------------------------------------------------------------------

struct RopeArgs {
  const float* qkv;        // [B][(Hq + 2 Hkv) D]: q heads, then k heads, then v heads
  const float* q_gain;     // [D] or NULL
  const float* k_gain;     // [D] or NULL
  const int32_t* seq_lens; // position of the current token = seq_lens[b] - 1
  uint16_t* q_out;         // [B][Hq][D]
  uint16_t* k_out;         // [B][Hkv][D]
  uint16_t* v_out;         // [B][Hkv][D]
  const int32_t* work_list;
  const int32_t* n_work;
  double log2_theta;
  float eps;
  int B, Hq, Hkv, D, heads_per_group;
};

// One wavefront per (selected request, head); q and k heads go through
// oda::head_norm and rotate_pair (the same code the fused attention calls run), v heads
// are only rounded.
__global__ __launch_bounds__(256) void qk_norm_rope_kernel(RopeArgs p) {
  const int lane = threadIdx.x & 63;
  const int wave = uniform(threadIdx.x >> 6);
  const int heads = p.Hq + 2 * p.Hkv;
  const int slot = blockIdx.x / p.heads_per_group;
  const int h = (blockIdx.x % p.heads_per_group) * kWaves + wave;
  if (slot >= selected_count(p.n_work, p.B) || h >= heads) return;
  const int b = selected_request(p.work_list, slot);
  if (b < 0 || b >= p.B) return;   // a listed request outside the batch is skipped
  const int half = p.D / 2;
  const bool active = lane < half;   // lane i holds the pair (i, i + D/2)
  const float* src = p.qkv + ((int64_t)b * heads + h) * p.D;
  float x1 = active ? src[lane] : 0.f, x2 = active ? src[lane + half] : 0.f;
  uint16_t* dst;
  if (h < p.Hq + p.Hkv) {
    const bool is_q = h < p.Hq;
    const int n = p.seq_lens[b];
    oda::head_norm(x1, x2, active, lane, p.D, is_q ? p.q_gain : p.k_gain, p.eps);
    if (!active) return;
    oda::rotate_pair(x1, x2, (double)(n - 1), oda::rope_frequency(lane, p.D, p.log2_theta));
    dst = is_q ? p.q_out + ((int64_t)b * p.Hq + h) * p.D : p.k_out + ((int64_t)b * p.Hkv + (h - p.Hq)) * p.D;
  } else {
    if (!active) return;
    dst = p.v_out + ((int64_t)b * p.Hkv + (h - p.Hq - p.Hkv)) * p.D;
  }
  dst[lane] = to_bf16(x1);
  dst[lane + half] = to_bf16(x2);
}

// ---------------------------------------------------------------------------
// embedding, row copy, argmax
// ---------------------------------------------------------------------------

// One workgroup per request; a token outside [0, vocab) gives a NaN row.
__global__ __launch_bounds__(256) void embed_kernel(const uint16_t* table, int vocab, int d, const int32_t* tokens,
                                                   float* x) {
  const int b = blockIdx.x;
  const int t = tokens[b];
  float* dst = x + (int64_t)b * d;
  const bool ok = t >= 0 && t < vocab;
  for (int k = threadIdx.x * 8; k < d; k += 256 * 8) {
    if (ok) {
      const u32x4 w = *reinterpret_cast<const u32x4*>(table + (int64_t)t * d + k);
      *reinterpret_cast<float4*>(dst + k) = make_float4(bf16_lo(w[0]), bf16_hi(w[0]), bf16_lo(w[1]), bf16_hi(w[1]));
      *reinterpret_cast<float4*>(dst + k + 4) =
          make_float4(bf16_lo(w[2]), bf16_hi(w[2]), bf16_lo(w[3]), bf16_hi(w[3]));
    } else {
      const float nan = __builtin_nanf("");
      *reinterpret_cast<float4*>(dst + k) = make_float4(nan, nan, nan, nan);
      *reinterpret_cast<float4*>(dst + k + 4) = make_float4(nan, nan, nan, nan);
    }
  }
}

// One workgroup per selected request slot.
__global__ __launch_bounds__(256) void copy_rows_kernel(const float* src, float* dst, int row_len, int B,
                                                       const int32_t* work_list, const int32_t* n_work) {
  const int slot = blockIdx.x;
  if (slot >= selected_count(n_work, B)) return;
  const int b = selected_request(work_list, slot);
  if (b < 0 || b >= B) return;   // a listed request outside the batch is skipped
  const int64_t base = (int64_t)b * row_len;
  for (int k = threadIdx.x * 4; k < row_len; k += 256 * 4)
    *reinterpret_cast<float4*>(dst + base + k) = *reinterpret_cast<const float4*>(src + base + k);
}

// One workgroup per selected request slot: y = x / sqrt(mean(x^2) + eps) * gain.
// The sum of squares is reduced in a fixed order (lanes, then wavefronts), so
// the result is the same on every run.
__global__ __launch_bounds__(256) void rms_norm_rows_kernel(const float* x, const float* gain, float eps, float* y,
                                                           int row_len, int B, const int32_t* work_list,
                                                           const int32_t* n_work) {
  __shared__ float sred[4];
  const int slot = blockIdx.x;
  if (slot >= selected_count(n_work, B)) return;
  const int b = selected_request(work_list, slot);
  if (b < 0 || b >= B) return;   // a listed request outside the batch is skipped
  const int64_t base = (int64_t)b * row_len;
  float ss = 0.f;
  for (int k = threadIdx.x * 4; k < row_len; k += 256 * 4) {
    const float4 v = *reinterpret_cast<const float4*>(x + base + k);
    ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
  }
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) ss += __shfl_xor(ss, s);
  if ((threadIdx.x & 63) == 0) sred[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float inv = rsqrtf((sred[0] + sred[1] + sred[2] + sred[3]) / (float)row_len + eps);
  for (int k = threadIdx.x * 4; k < row_len; k += 256 * 4) {
    const float4 v = *reinterpret_cast<const float4*>(x + base + k);
    const float4 g = *reinterpret_cast<const float4*>(gain + k);
    *reinterpret_cast<float4*>(y + base + k) = make_float4(v.x * inv * g.x, v.y * inv * g.y, v.z * inv * g.z,
                                                           v.w * inv * g.w);
  }
}

constexpr int kArgThreads = 1024;

// Greedy choice: the first index of the largest non-NaN value (-1 if every
// value is NaN).  One workgroup per request, bound by what one CU reads: the
// values pass in groups of four, of which a thread keeps the best group's
// maximum and number (five operations a group; tracking each value's index
// took four times as many and, at 151,936 values, 16.7 us instead of 8.8).
// The winning group is read again for the position.  kInFlight: 16-byte loads
// in flight per thread (4 or 8 where one round of them covers the row: loads
// past the end read its last group again, and 16 of them took 5.0 us at 16,400
// values instead of 4.0).
template <int kInFlight>
__global__ __launch_bounds__(kArgThreads) void argmax_kernel(const float* x, int n, int32_t* index) {
  __shared__ float sv[kArgThreads / 64];
  __shared__ int si[kArgThreads / 64];
  const int b = blockIdx.x;
  const float* row = x + (int64_t)b * n;
  const int n4 = n / 4;                        // the host keeps n a multiple of 4
  float best = -INFINITY;
  int group = INT_MAX;
  for (int j0 = threadIdx.x; j0 < n4; j0 += kArgThreads * kInFlight) {
    float4 v[kInFlight];
#pragma unroll
    for (int u = 0; u < kInFlight; ++u)     // past the end: the last group again (not a new maximum)
      v[u] = *reinterpret_cast<const float4*>(row + 4 * (int64_t)min(j0 + u * kArgThreads, n4 - 1));
#pragma unroll
    for (int u = 0; u < kInFlight; ++u) {
      const float m = fmaxf(fmaxf(v[u].x, v[u].y), fmaxf(v[u].z, v[u].w));   // ignores NaNs
      if (m > best) {                          // a thread's groups ascend: the first of equals stays
        best = m;
        group = min(j0 + u * kArgThreads, n4 - 1);
      }
    }
  }
  // wavefront, then workgroup: the largest value, of equals the first group
  auto take = [&](float ov, int og) {
    if (ov > best || (ov == best && og < group)) {
      best = ov;
      group = og;
    }
  };
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) {
    const float ov = __shfl_xor(best, s);
    const int og = __shfl_xor(group, s);
    take(ov, og);
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
    sv[wave] = best;
    si[wave] = group;
  }
  __syncthreads();
  best = sv[0];
  group = si[0];
  for (int w = 1; w < kArgThreads / 64; ++w) take(sv[w], si[w]);
  if (group != INT_MAX) {
    if (threadIdx.x == 0) {
      const float4 v = *reinterpret_cast<const float4*>(row + 4 * (int64_t)group);
      index[b] = 4 * group + (v.x == best ? 0 : v.y == best ? 1 : v.z == best ? 2 : 3);
    }
    return;
  }
  // nothing above -infinity: the first value that is not NaN, if any
  int first = INT_MAX;
  for (int i = threadIdx.x; i < n && first == INT_MAX; i += kArgThreads)
    if (row[i] == row[i]) first = i;
#pragma unroll
  for (int s = 32; s >= 1; s >>= 1) first = min(first, __shfl_xor(first, s));
  __syncthreads();
  if (lane == 0) si[wave] = first;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < kArgThreads / 64; ++w) first = min(first, si[w]);
    index[b] = first == INT_MAX ? -1 : first;
  }
}

oda_status launch_status() {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return oda::fail(ODA_ERR_HIP, "kernel launch failed: %s", hipGetErrorString(e));
  return oda::ok();
}

}  // namespace

extern "C" oda_status oda_dense_bf16(const oda_dense_desc* desc, int32_t batch, const float* x,
                                    const float* residual, float* y, const int32_t* work_list,
                                    const int32_t* n_work, hipStream_t stream) {
  if (desc == nullptr) return oda::fail(ODA_ERR_NULL, "desc is NULL");
  if (!desc->weight || !x || !y) return oda::fail(ODA_ERR_NULL, "weight, x and y are required");
  if ((work_list == nullptr) != (n_work == nullptr))
    return oda::fail(ODA_ERR_NULL, "work_list and n_work must both be NULL or both be set");
  if (desc->mode != ODA_DENSE_PLAIN && desc->mode != ODA_DENSE_SWIGLU)
    return oda::fail(ODA_ERR_UNSUPPORTED, "unknown dense mode %d", desc->mode);
  if (batch < 1 || desc->in_features < 8 || desc->in_features % 8 || desc->out_features < 1)
    return oda::fail(ODA_ERR_SHAPE, "batch >= 1, in_features a positive multiple of 8, out_features >= 1 required "
                     "(got %d, %d, %d)", batch, desc->in_features, desc->out_features);
  if (desc->mode == ODA_DENSE_SWIGLU && residual != nullptr)
    return oda::fail(ODA_ERR_UNSUPPORTED, "the SwiGLU mode takes no residual");
  if (!(desc->rms_eps >= 0.f) || !std::isfinite(desc->rms_eps)) return oda::fail(ODA_ERR_SHAPE, "rms_eps must be >= 0");
  if (!oda::aligned(desc->weight, 16) || !oda::aligned(x, 16) || (desc->norm_gain && !oda::aligned(desc->norm_gain, 16)))
    return oda::fail(ODA_ERR_SHAPE, "weight, x and norm_gain must be 16-byte aligned");
  const int N = desc->out_features;
  const bool swiglu = desc->mode == ODA_DENSE_SWIGLU;
  DenseArgs a{desc->weight, desc->norm_gain, x, residual, y, work_list, n_work, N, desc->in_features, batch,
              desc->rms_eps};
  (void)hipGetLastError();
  // Several requests: the narrowest workgroup (row tiles and tile edge) that
  // still needs no more than one per CU, so that the launch is one even round;
  // layers too large for that take the widest.  Narrower ones re-split and
  // re-read the inputs more often, wider ones leave CUs idle: 6144 -> 2048, 8
  // requests 7.4 us with 8-row workgroups against 10.6 with 16, 32 requests
  // 11.7 with 16 against 19.9 with 8; gate and up 2048 -> 6144, 32 requests
  // 16.6 with 48 rows, 21.6 with 32, 19.9 with 16.  A layer of many rounds
  // takes this path for one request too, where the wavefronts' stretches are
  // whole chunks of lines: 2048 -> 151936 99 us against 105, 4096 -> 151936 205
  // against 240, 1536 -> 65536 35.1 against 35.8, but 1624 -> 151936 97 against
  // 83 and 2112 -> 151936 112 against 106.
  const auto groups_of = [&](int tiles, int edge) {
    return oda::ceil_div(N, tiles * edge) * oda::ceil_div(batch, edge);
  };
  const bool one = !swiglu && groups_of(2, kMfmaRows) >= 8 * kTargetGroups && a.K >= 3 * kMfmaWaves * kChunk &&
                   a.K % (kMfmaWaves * kChunk) == 0;
  if ((batch > 1 || one) && a.K < kMfmaMaxK) {
    oda_status st;
    const auto fits = [&](int tiles, int edge) { return groups_of(tiles, edge) <= kTargetGroups; };
    if (swiglu) {
      if (fits(1, 8)) st = launch_dense_mfma<true, 1, true>(a, stream);
      else if (fits(2, 8)) st = launch_dense_mfma<true, 2, true>(a, stream);
      else if (fits(3, 8)) st = launch_dense_mfma<true, 3, true>(a, stream);
      else if (fits(1, kMfmaRows)) st = launch_dense_mfma<true, 1, false>(a, stream);
      else if (fits(2, kMfmaRows)) st = launch_dense_mfma<true, 2, false>(a, stream);
      else st = launch_dense_mfma<true, 3, false>(a, stream);
    } else {
      if (fits(1, 8)) st = launch_dense_mfma<false, 1, true>(a, stream);
      else if (fits(2, 8)) st = launch_dense_mfma<false, 2, true>(a, stream);
      else if (fits(1, kMfmaRows)) st = launch_dense_mfma<false, 1, false>(a, stream);
      else st = launch_dense_mfma<false, 2, false>(a, stream);
    }
    return st == ODA_OK ? launch_status() : st;
  }
  // one request (or rows too long for the tiles): the most rows per wavefront
  // that still leave >= kDenseMinWaves wavefronts
  int rows = 1;
  for (int r = swiglu ? 4 : 8; r > 1; r /= 2)
    if (N % r == 0 && N / r >= kDenseMinWaves) {
      rows = r;
      break;
    }
  const int64_t groups = oda::ceil_div(N / rows, kWaves);
  const dim3 grid((unsigned)groups, (unsigned)batch), block(256);
#define ODA_DENSE_LAUNCH(SW, R) hipLaunchKernelGGL((dense_kernel<SW, R>), grid, block, 0, stream, a)
  if (swiglu) {
    if (rows == 4) ODA_DENSE_LAUNCH(true, 4);
    else if (rows == 2) ODA_DENSE_LAUNCH(true, 2);
    else ODA_DENSE_LAUNCH(true, 1);
  } else {
    if (rows == 8) ODA_DENSE_LAUNCH(false, 8);
    else if (rows == 4) ODA_DENSE_LAUNCH(false, 4);
    else if (rows == 2) ODA_DENSE_LAUNCH(false, 2);
    else ODA_DENSE_LAUNCH(false, 1);
  }
#undef ODA_DENSE_LAUNCH
  return launch_status();
}

extern "C" oda_status oda_qk_norm_rope(int32_t batch, int32_t num_q_heads, int32_t num_kv_heads, int32_t head_dim,
                                      const float* qkv, const float* q_gain, const float* k_gain, float rms_eps,
                                      double rope_theta, const int32_t* seq_lens, uint16_t* q_out,
                                      uint16_t* k_out, uint16_t* v_out, const int32_t* work_list,
                                      const int32_t* n_work, hipStream_t stream) {
  if (!qkv || !seq_lens || !q_out || !k_out || !v_out)
    return oda::fail(ODA_ERR_NULL, "qkv, seq_lens, q_out, k_out and v_out are required");
  if ((work_list == nullptr) != (n_work == nullptr))
    return oda::fail(ODA_ERR_NULL, "work_list and n_work must both be NULL or both be set");
  if (batch < 1 || num_kv_heads < 1 || num_q_heads < 1 || num_q_heads % num_kv_heads)
    return oda::fail(ODA_ERR_SHAPE, "batch >= 1 and num_q_heads a positive multiple of num_kv_heads required");
  if (head_dim < 2 || head_dim > 128 || head_dim % 2)
    return oda::fail(ODA_ERR_UNSUPPORTED, "head_dim must be even and at most 128 (got %d)", head_dim);
  if (!(rope_theta > 1.0) || !std::isfinite(rope_theta)) return oda::fail(ODA_ERR_SHAPE, "rope_theta must be > 1");
  if (!(rms_eps >= 0.f) || !std::isfinite(rms_eps)) return oda::fail(ODA_ERR_SHAPE, "rms_eps must be >= 0");
  RopeArgs a{};
  a.qkv = qkv;
  a.q_gain = q_gain;
  a.k_gain = k_gain;
  a.seq_lens = seq_lens;
  a.q_out = q_out;
  a.k_out = k_out;
  a.v_out = v_out;
  a.work_list = work_list;
  a.n_work = n_work;
  a.log2_theta = std::log2(rope_theta);
  a.eps = rms_eps;
  a.B = batch;
  a.Hq = num_q_heads;
  a.Hkv = num_kv_heads;
  a.D = head_dim;
  a.heads_per_group = (int)oda::ceil_div(num_q_heads + 2 * num_kv_heads, kWaves);
  (void)hipGetLastError();
  hipLaunchKernelGGL(qk_norm_rope_kernel, dim3((unsigned)(batch * a.heads_per_group)), dim3(256), 0, stream, a);
  return launch_status();
}

extern "C" oda_status oda_embed_bf16(const uint16_t* table, int32_t vocab, int32_t d_model, int32_t batch,
                                    const int32_t* tokens, float* x, hipStream_t stream) {
  if (!table || !tokens || !x) return oda::fail(ODA_ERR_NULL, "table, tokens and x are required");
  if (vocab < 1 || batch < 1 || d_model < 8 || d_model % 8)
    return oda::fail(ODA_ERR_SHAPE, "vocab, batch >= 1 and d_model a positive multiple of 8 required");
  if (!oda::aligned(table, 16) || !oda::aligned(x, 16))
    return oda::fail(ODA_ERR_SHAPE, "table and x must be 16-byte aligned");
  (void)hipGetLastError();
  hipLaunchKernelGGL(embed_kernel, dim3((unsigned)batch), dim3(256), 0, stream, table, vocab, d_model, tokens, x);
  return launch_status();
}

extern "C" oda_status oda_copy_rows(int32_t batch, int32_t row_len, const float* src, float* dst,
                                   const int32_t* work_list, const int32_t* n_work, hipStream_t stream) {
  if (!src || !dst) return oda::fail(ODA_ERR_NULL, "src and dst are required");
  if ((work_list == nullptr) != (n_work == nullptr))
    return oda::fail(ODA_ERR_NULL, "work_list and n_work must both be NULL or both be set");
  if (batch < 1 || row_len < 4 || row_len % 4)
    return oda::fail(ODA_ERR_SHAPE, "batch >= 1 and row_len a positive multiple of 4 required");
  if (!oda::aligned(src, 16) || !oda::aligned(dst, 16))
    return oda::fail(ODA_ERR_SHAPE, "src and dst must be 16-byte aligned");
  (void)hipGetLastError();
  hipLaunchKernelGGL(copy_rows_kernel, dim3((unsigned)batch), dim3(256), 0, stream, src, dst, row_len, batch,
                     work_list, n_work);
  return launch_status();
}

extern "C" oda_status oda_rms_norm_rows(int32_t batch, int32_t row_len, const float* x, const float* gain,
                                       float rms_eps, float* y, const int32_t* work_list, const int32_t* n_work,
                                       hipStream_t stream) {
  if (!x || !gain || !y) return oda::fail(ODA_ERR_NULL, "x, gain and y are required");
  if ((work_list == nullptr) != (n_work == nullptr))
    return oda::fail(ODA_ERR_NULL, "work_list and n_work must both be NULL or both be set");
  if (batch < 1 || row_len < 4 || row_len % 4)
    return oda::fail(ODA_ERR_SHAPE, "batch >= 1 and row_len a positive multiple of 4 required");
  if (!(rms_eps >= 0.f) || !std::isfinite(rms_eps)) return oda::fail(ODA_ERR_SHAPE, "rms_eps must be >= 0");
  if (!oda::aligned(x, 16) || !oda::aligned(gain, 16) || !oda::aligned(y, 16))
    return oda::fail(ODA_ERR_SHAPE, "x, gain and y must be 16-byte aligned");
  (void)hipGetLastError();
  hipLaunchKernelGGL(rms_norm_rows_kernel, dim3((unsigned)batch), dim3(256), 0, stream, x, gain, rms_eps, y, row_len,
                     batch, work_list, n_work);
  return launch_status();
}

extern "C" oda_status oda_argmax(int32_t batch, int32_t n, const float* x, int32_t* index, hipStream_t stream) {
  if (!x || !index) return oda::fail(ODA_ERR_NULL, "x and index are required");
  if (batch < 1 || n < 1) return oda::fail(ODA_ERR_SHAPE, "batch and n must be >= 1");
  if (!oda::aligned(x, 16) || n % 4) return oda::fail(ODA_ERR_SHAPE, "x must be 16-byte aligned and n a multiple of 4");
  (void)hipGetLastError();
  if (n / 4 <= 4 * kArgThreads)
    hipLaunchKernelGGL(argmax_kernel<4>, dim3((unsigned)batch), dim3(kArgThreads), 0, stream, x, n, index);
  else if (n / 4 <= 8 * kArgThreads)
    hipLaunchKernelGGL(argmax_kernel<8>, dim3((unsigned)batch), dim3(kArgThreads), 0, stream, x, n, index);
  else
    hipLaunchKernelGGL(argmax_kernel<16>, dim3((unsigned)batch), dim3(kArgThreads), 0, stream, x, n, index);
  return launch_status();
}
