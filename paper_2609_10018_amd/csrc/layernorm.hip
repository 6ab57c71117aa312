// LayerNorm over the feature axis: u = (x - mean) / sqrt(var + eps) * g + b,
// biased variance, statistics in fp32.  Memory-bound: each lane holds its
// share of a row in registers (two passes over registers, one read of the row
// from HBM, one write).
//
// The bf16 path gives each row half a wave and reads and writes 16-byte
// (8-element) bf16 vectors; the class-token rows of the residual stream are
// fp32 and come from their own buffer.  Row stride is free.
#include "common.h"
#include "kernels.h"

namespace elasto {
namespace {

constexpr int kMaxChunks = 8;  // 8-element chunks per lane: d <= 2048
constexpr int kLnGroups = 1280;  // workgroups that walk rows: five on each of 256 CUs

__device__ __forceinline__ float half_sum(float v) {
#pragma unroll
  for (int off = 16; off >= 1; off >>= 1) v += __shfl_xor(v, off, 32);
  return v;
}

// Two rows per wave (32 lanes each), so a load instruction moves 16 bytes per
// lane; NC = ceil(d / 256) chunks per lane.
//
// Bound by HBM and the last-level cache.  A chunk's load was behind the test
// for a class-token row, so the row's loads waited for one another: 50432 x 768
// with class rows 37.5 us from HBM and 28.8 with its rows in the last-level
// cache, now 31.7 and 24.6.  (The rest with rows in the cache:) the loads ahead
// of the test gave most of it, 25.6.  Rows that fill the chip more than once
// (WALK): a half-wave walks rows `step` apart, the next row's load in flight
// under the current row's sums, with g and b, four times a row's bytes, staged
// in LDS once: 25.1 us, 25000 x 768 15.0 -> 13.1, 50432 x 384 15.0 -> 13.4 (768
// to 2048 workgroups: 24.9 to 27.6; 1280 is best or within 2%).  Not for
// d > 1024, where the registers of a row ahead cost wavefronts (50432 x 2048:
// 84.4 against 81.4).
// step = step_q * tokens + step_r, so a row's image needs no division.
struct LnRows {
  int64_t step, step_q;
  int step_r;
};

template <int NC, bool WALK>
__global__ __launch_bounds__(256) void layernorm_bf16_kernel(const uint16_t* __restrict__ x,
                                                             int64_t x_stride,
                                                             const float* __restrict__ xcls,
                                                             int tokens, LnRows walk,
                                                             uint16_t* __restrict__ out,
                                                             int64_t rows, int d,
                                                             const float* __restrict__ g,
                                                             const float* __restrict__ b,
                                                             float eps) {
  // Half h of chunk ci of g (then of b) at [h][ci]: a wave's reads are contiguous.
  __shared__ f32x4 gb[WALK ? 4 * NC * 32 : 1];
  const int nch = d >> 3, hl = threadIdx.x & 31;
  if constexpr (WALK) {
    for (int q = threadIdx.x; q < 2 * nch; q += 256) {
      gb[(q & 1) * NC * 32 + (q >> 1)] = *reinterpret_cast<const f32x4*>(g + 4 * q);
      gb[(2 + (q & 1)) * NC * 32 + (q >> 1)] = *reinterpret_cast<const f32x4*>(b + 4 * q);
    }
  }
  int64_t row = (int64_t)blockIdx.x * 8 + (threadIdx.x >> 5);
  bool live = row < rows;  // the same for a half-wave: the sums below stay inside one
  int64_t bi = 0;
  int tok = 1;  // row = bi * tokens + tok; without class rows never 0
  if (xcls != nullptr) {
    bi = row / tokens;
    tok = (int)(row - bi * tokens);
  }
  u32x4 raw[NC];
  auto load_row = [&]() {
    const uint16_t* xr = x + row * x_stride;
#pragma unroll
    for (int i = 0; i < NC; ++i)
      if (hl + 32 * i < nch) raw[i] = *reinterpret_cast<const u32x4*>(xr + 8 * (hl + 32 * i));
  };
  if (live && tok != 0) load_row();
  if constexpr (WALK) __syncthreads();
  const float inv_d = 1.0f / (float)d;
  while (live) {
    float v[NC][8];
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int ci = hl + 32 * i;
      if (ci < nch) {
        if (tok == 0) {
          const float* xc = xcls + bi * (int64_t)d;
          const f32x4 w0 = *reinterpret_cast<const f32x4*>(xc + 8 * ci);
          const f32x4 w1 = *reinterpret_cast<const f32x4*>(xc + 8 * ci + 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v[i][e] = w0[e];
            v[i][4 + e] = w1[e];
          }
        } else {
          const u32x4 w = raw[i];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v[i][2 * e] = __uint_as_float(w[e] << 16);
            v[i][2 * e + 1] = __uint_as_float(w[e] & 0xffff0000u);
          }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) s += v[i][e];
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[i][e] = 0.0f;
      }
    }
    uint16_t* orow = out + row * (int64_t)d;
    if constexpr (WALK) {
      row += walk.step;
      live = row < rows;
      if (xcls != nullptr) {
        bi += walk.step_q;
        tok += walk.step_r;
        if (tok >= tokens) {
          tok -= tokens;
          ++bi;
        }
      }
      if (live && tok != 0) load_row();
    } else {
      live = false;
    }

    const float mean = half_sum(s) * inv_d;
    float ss = 0.0f;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      if (hl + 32 * i < nch) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float c = v[i][e] - mean;
          ss += c * c;
        }
      }
    }
    const float rstd = rsqrtf(half_sum(ss) * inv_d + eps);
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      const int ci = hl + 32 * i;
      if (ci < nch) {
        u32x4 w;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          f32x4 gv, bv;
          if constexpr (WALK) {
            gv = gb[h * NC * 32 + ci];
            bv = gb[(2 + h) * NC * 32 + ci];
          } else {
            gv = *reinterpret_cast<const f32x4*>(g + 8 * ci + 4 * h);
            bv = *reinterpret_cast<const f32x4*>(b + 8 * ci + 4 * h);
          }
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            const int j = 2 * e;
            w[2 * h + e] = pack_bf16x2((v[i][4 * h + j] - mean) * rstd * gv[j] + bv[j],
                                       (v[i][4 * h + j + 1] - mean) * rstd * gv[j + 1] + bv[j + 1]);
          }
        }
        *reinterpret_cast<u32x4*>(orow + 8 * ci) = w;
      }
    }
  }
}

// fp32 rows, any d <= 2048 (element-wise access).
__global__ __launch_bounds__(256) void layernorm_f32_kernel(const float* __restrict__ x,
                                                            int64_t x_stride,
                                                            float* __restrict__ out, int64_t rows,
                                                            int d, const float* __restrict__ g,
                                                            const float* __restrict__ b,
                                                            float eps) {
  constexpr int kMax = 32;
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const float* xr = x + row * x_stride;
  float v[kMax];
  float s = 0.0f;
#pragma unroll
  for (int i = 0; i < kMax; ++i) {
    const int c = lane + 64 * i;
    v[i] = c < d ? xr[c] : 0.0f;
    s += v[i];
  }
  const float mean = wave_sum(s) / (float)d;
  float ss = 0.0f;
#pragma unroll
  for (int i = 0; i < kMax; ++i) {
    const int c = lane + 64 * i;
    if (c < d) ss += (v[i] - mean) * (v[i] - mean);
  }
  const float rstd = 1.0f / sqrtf(wave_sum(ss) / (float)d + eps);
  float* orow = out + row * (int64_t)d;
#pragma unroll
  for (int i = 0; i < kMax; ++i) {
    const int c = lane + 64 * i;
    if (c < d) orow[c] = (v[i] - mean) * rstd * g[c] + b[c];
  }
}

template <int NC>
hipError_t launch_ln(const uint16_t* x, int64_t x_stride, const float* xcls, int tokens,
                     uint16_t* out, int64_t rows, int d, const float* g, const float* b, float eps,
                     hipStream_t s) {
  const int64_t groups = (rows + 7) / 8;
  LnRows walk{0, 0, 0};
  if (groups <= kLnGroups || NC > 4) {
    hipLaunchKernelGGL((layernorm_bf16_kernel<NC, false>), dim3((unsigned)groups), dim3(256), 0, s,
                       x, x_stride, xcls, tokens, walk, out, rows, d, g, b, eps);
    return hipGetLastError();
  }
  // As many workgroups as stay resident together, each with the same count of
  // rows give or take one.
  const int64_t each = (groups + kLnGroups - 1) / kLnGroups, grid = (groups + each - 1) / each;
  walk.step = grid * 8;
  if (xcls != nullptr) {
    walk.step_q = walk.step / tokens;
    walk.step_r = (int)(walk.step - walk.step_q * tokens);
  }
  constexpr bool kWalk = NC <= 4;  // (past that not reached)
  hipLaunchKernelGGL((layernorm_bf16_kernel<NC, kWalk>), dim3((unsigned)grid), dim3(256), 0, s, x,
                     x_stride, xcls, tokens, walk, out, rows, d, g, b, eps);
  return hipGetLastError();
}

// Weights of a LayerNorm folded into the following linear layer: one wave
// per output row n.  Sums over the row accumulate in fp64 (the folded column
// sum is of the bf16-rounded products the GEMM multiplies).  NW: most widths
// this launch sums for; with one width (no elastic embedding) the sums for the
// other 15 were most of its time (3072 x 768: 26 us, now 10 us).
constexpr int kFoldMaxWidths = 16;
struct FoldWidths {
  int n;
  int e[kFoldMaxWidths];
};

template <int NW>
__global__ __launch_bounds__(256) void ln_fold_kernel(const uint16_t* __restrict__ W, int N, int D,
                                                      const float* __restrict__ gamma,
                                                      const float* __restrict__ beta,
                                                      const float* __restrict__ bias,
                                                      FoldWidths wd, uint16_t* __restrict__ Wf,
                                                      float* __restrict__ colsum,
                                                      float* __restrict__ cbias, int64_t ldv) {
  const int lane = threadIdx.x & 63;
  const int n = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (n >= N) return;
  const uint16_t* w = W + (int64_t)n * D;
  uint16_t* wf = Wf + (int64_t)n * D;
  double sw[NW], sb[NW];
#pragma unroll
  for (int i = 0; i < NW; ++i) sw[i] = sb[i] = 0.0;
  for (int k = lane; k < D; k += 64) {
    const float wv = bf16_to_f32(w[k]);
    const uint16_t f = f32_to_bf16(gamma[k] * wv);
    wf[k] = f;
    const double fv = (double)bf16_to_f32(f), bv = (double)beta[k] * (double)wv;
#pragma unroll
    for (int i = 0; i < NW; ++i)
      if (i < wd.n && k < wd.e[i]) {
        sw[i] += fv;
        sb[i] += bv;
      }
  }
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    if (i >= wd.n) break;
    double a = sw[i], c = sb[i];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
      a += __shfl_xor(a, off, 64);
      c += __shfl_xor(c, off, 64);
    }
    if (lane == 0) {
      colsum[i * ldv + n] = (float)a;
      cbias[i * ldv + n] = (float)((double)bias[n] + c);
    }
  }
}

}  // namespace

hipError_t launch_layernorm_bf16(const void* x, int64_t x_stride, const float* xcls, int tokens,
                                 void* out, int64_t rows, int d, const float* g, const float* b,
                                 float eps, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  if (xcls != nullptr && tokens < 1) return hipErrorInvalidValue;
  if ((d & 7) != 0 || d > 8 * 32 * kMaxChunks) return hipErrorInvalidValue;
  const uint16_t* xp = static_cast<const uint16_t*>(x);
  uint16_t* op = static_cast<uint16_t*>(out);
  switch ((d + 255) / 256) {
    case 1: return launch_ln<1>(xp, x_stride, xcls, tokens, op, rows, d, g, b, eps, s);
    case 2: return launch_ln<2>(xp, x_stride, xcls, tokens, op, rows, d, g, b, eps, s);
    case 3: return launch_ln<3>(xp, x_stride, xcls, tokens, op, rows, d, g, b, eps, s);
    case 4: return launch_ln<4>(xp, x_stride, xcls, tokens, op, rows, d, g, b, eps, s);
    default: return launch_ln<kMaxChunks>(xp, x_stride, xcls, tokens, op, rows, d, g, b, eps, s);
  }
}

hipError_t launch_layernorm_f32(const void* x, int64_t x_stride, void* out, int64_t rows, int d,
                                const float* g, const float* b, float eps, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  const int64_t blocks = (rows + 3) / 4;
  hipLaunchKernelGGL(layernorm_f32_kernel, dim3((unsigned)blocks), dim3(256), 0, s,
                     static_cast<const float*>(x), x_stride, static_cast<float*>(out), rows, d,
                     g, b, eps);
  return hipGetLastError();
}

hipError_t launch_ln_fold(const void* W, int N, int D, const float* gamma, const float* beta,
                          const float* bias, const int32_t* widths, int nw, void* Wf,
                          float* colsum, float* cbias, int64_t ldv, hipStream_t s) {
  if (N <= 0) return hipSuccess;
  if (nw < 1 || nw > kFoldMaxWidths || D < 1 || ldv < N) return hipErrorInvalidValue;
  FoldWidths wd{};
  wd.n = nw;
  for (int i = 0; i < nw; ++i) {
    if (widths[i] < 1 || widths[i] > D) return hipErrorInvalidValue;
    wd.e[i] = widths[i];
  }
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3((unsigned)((N + 3) / 4)), dim3(256), 0, s,
                       static_cast<const uint16_t*>(W), N, D, gamma, beta, bias, wd,
                       static_cast<uint16_t*>(Wf), colsum, cbias, ldv);
    return hipGetLastError();
  };
  if (nw == 1) return go(ln_fold_kernel<1>);
  return nw <= 4 ? go(ln_fold_kernel<4>) : go(ln_fold_kernel<kFoldMaxWidths>);
}

}  // namespace elasto
