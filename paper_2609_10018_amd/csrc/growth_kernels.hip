// Kernels of the growth step (Section 4.2): the weights' transposes for the
// backward, the weight and bias gradients, LayerNorm backward, the
// cross-entropy loss, the selective clipping norm (Eq. 9's G is applied by computing gradients only for the
// re-introduced slices), and the masked update with fp32 master weights.
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace elasto {
namespace {

inline unsigned grid_for(int64_t n, int block) { return (unsigned)((n + block - 1) / block); }

// ------------------------------------------------------------ transposes
// out[c][r] = in[r][c] of every job (blockIdx.y), 64x64 tiles through LDS: the
// weights that the backward multiplies transposed, all in one launch.
constexpr int kTT = 64;
__global__ __launch_bounds__(256) void transpose_kernel(const TransposeJob* __restrict__ jobs,
                                                        const uint16_t* __restrict__ in_base,
                                                        uint16_t* __restrict__ out_base) {
  __shared__ __attribute__((aligned(16))) uint16_t tile[kTT][kTT + 8];
  const TransposeJob jb = jobs[blockIdx.y];
  const int tiles_c = (jb.cols + kTT - 1) / kTT;
  const int tr = blockIdx.x / tiles_c, r0 = tr * kTT, c0 = (blockIdx.x - tr * tiles_c) * kTT;
  if (r0 >= jb.rows) return;
  const uint16_t* in = in_base + jb.in_off;
  const int t = threadIdx.x;
  // 16-byte chunks: rows of ldi elements (a multiple of 8) reach past cols.
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = (t >> 3) + 32 * i, c = min(c0 + (t & 7) * 8, jb.ldi - 8);
    *reinterpret_cast<u32x4*>(&tile[r][(t & 7) * 8]) =
        *reinterpret_cast<const u32x4*>(in + (int64_t)min(r0 + r, jb.rows - 1) * jb.ldi + c);
  }
  __syncthreads();
  const int oc = t >> 2, seg = (t & 3) * 16;  // output row c0 + oc, input rows r0 + seg + [0, 16)
  if (c0 + oc >= jb.cols) return;
  uint16_t* op = out_base + jb.out_off + (int64_t)(c0 + oc) * jb.ldo + r0 + seg;
  if (r0 + seg + 16 <= jb.rows) {
    u32x4 w0, w1;
#pragma unroll
    for (int h = 0; h < 4; ++h) {
      w0[h] = (uint32_t)tile[seg + 2 * h][oc] | ((uint32_t)tile[seg + 2 * h + 1][oc] << 16);
      w1[h] = (uint32_t)tile[seg + 8 + 2 * h][oc] | ((uint32_t)tile[seg + 9 + 2 * h][oc] << 16);
    }
    *reinterpret_cast<u32x4*>(op) = w0;
    *reinterpret_cast<u32x4*>(op + 8) = w1;
  } else {
    for (int e = 0; e < 16 && r0 + seg + e < jb.rows; ++e) op[e] = tile[seg + e][oc];
  }
}

// -------------------------------------------------------- weight gradients
// out[r][c] = sum_m P[m][pc + r] Q[m][qc + c] for the problems of one layer in
// one launch (and the bias gradient sum_m P[m][pc + r], by one more MFMA with a
// matrix of ones).  Both operands are read as they lie, rows of m: the MFMA
// operands, eight m of one column a lane, come from LDS through the transpose
// read (ds_read_b64_tr_b16: in a group of 16 lanes, lane i receives element
// i%4 of the 8-byte pieces that lanes i/4, 4 + i/4, 8 + i/4 and 12 + i/4
// address), so no transposed copy of an activation is written.
// 128x128 output tiles, 4 waves of 64x64, steps of 64 rows in two LDS stages
// (two workgroups per CU), rows of 256 bytes whose 16-byte chunk c sits at
// c ^ 4 (row % 4): the four rows x 32 bytes that 32 lanes read at once lie in
// different banks.  M is split until the launch has about two workgroups per
// CU; split tiles are summed in split order by wgrad_reduce_kernel.
// ViT-B, 12608 rows, one layer of mode 0 grown from mode 1 (44.6 GFLOP): 84 us
// and 9 for the sums; with transposed copies, four split-K GEMMs, their sums and
// row sums of the transposes for the biases it took 430 us.
constexpr int kWT = 128, kWStage = 64 * 256 * 2;
struct WgradTile {
  const uint16_t *P, *Q;
  int ldp, ldq, pa, qa;  // first column of the tile grid (a multiple of 8)
  int sp, sq, ra, rb;    // wanted columns: [sp, sp + ra) x [sq, sq + rb) of the grid
  int tile0, tc;         // first tile, tiles across
  float *out, *bias;
  int ldo;
};
struct WgradP {
  WgradTile t[kWgradMax];
  int n, tiles, split, M, kchunk;
  float *part, *bpart;
  int bstride;
};
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) void global_void;
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

__device__ __forceinline__ int wgrad_problem(const WgradP& a, int tile) {
  int q = 0;
#pragma unroll
  for (int i = 1; i < kWgradMax; ++i)
    if (i < a.n && tile >= a.t[i].tile0) q = i;
  return q;
}

__global__ __launch_bounds__(256, 2) void wgrad_kernel(WgradP a) {
  __shared__ __attribute__((aligned(1024))) char smem[2 * kWStage];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Workgroups of one XCD (workgroup i runs on XCD i % 8) take neighbouring
  // tiles of the same rows, which their L2 then holds.
  const int nblk = gridDim.x, b = blockIdx.x;
  const int q8 = nblk >> 3, r8 = nblk & 7, xcd = b & 7, idx = b >> 3;
  const int logical = (xcd < r8) ? xcd * (q8 + 1) + idx : r8 * (q8 + 1) + (xcd - r8) * q8 + idx;
  const int sl = logical / a.tiles, tile = logical - sl * a.tiles;
  const WgradTile& w = a.t[wgrad_problem(a, tile)];
  const int ti = (tile - w.tile0) / w.tc, tj = tile - w.tile0 - ti * w.tc;
  const int r0 = ti * kWT, c0 = tj * kWT;
  const int k0 = sl * a.kchunk, rows = min(a.M - k0, a.kchunk), nk = (rows + 63) >> 6;

  // Loads: waves 0-1 bring P, waves 2-3 Q; a 1-KB block is 4 rows, lane l
  // landing at row l/16, physical chunk l%16.
  const bool is_q = wave >= 2;
  const uint16_t* const src = is_q ? w.Q : w.P;
  const int ld = is_q ? w.ldq : w.ldp, lrow = lane >> 4;
  const int col = min((is_q ? w.qa + c0 : w.pa + r0) + ((lane & 15) ^ (4 * lrow)) * 8, ld - 8);
  auto issue = [&](int stage, int kt) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int blk = (wave & 1) * 8 + i;
      const int m = min(k0 + kt * 64 + blk * 4 + lrow, a.M - 1);
      __builtin_amdgcn_global_load_lds(
          (global_void*)(src + (int64_t)m * ld + col),
          (lds_void*)(smem + stage * kWStage + (is_q ? kWStage / 2 : 0) + blk * 1024), 16, 0, 0);
    }
  };
  const int wm = wave >> 1, wn = wave & 1, g = lane >> 4, lq = lane & 15;
  const int trow = 8 * (g >> 1) + (lq >> 2), tcol = 16 * (g & 1) + 4 * (lq & 3);
  // Eight rows (16 kk + 8 (lane/32) ..) of column cb + lane%32.
  auto frag = [&](const char* st, int cb, int kk) {
    const int c = cb + tcol, off = (((c >> 3) ^ (4 * (lq >> 2))) << 4) + (c & 7) * 2;
    const char* p0 = st + (kk * 16 + trow) * 256 + off;
    const u32x2 lo = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)p0));
    const u32x2 hi =
        __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4*)(p0 + 4 * 256)));
    return u32x4{lo[0], lo[1], hi[0], hi[1]};
  };
  f32x16 acc[2][2], accb[2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[i][0][e] = acc[i][1][e] = accb[i][e] = 0.0f;
  const bool bias = w.bias != nullptr && tj == 0 && wn == 0;
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = static_cast<__bf16>(1.0f);
  issue(0, 0);
  for (int kt = 0; kt < nk; ++kt) {
    __builtin_amdgcn_s_waitcnt((0x7 << 4) | (0xF << 8));  // this wave's loads of step kt
    __syncthreads();
    if (kt + 1 < nk) issue((kt + 1) & 1, kt + 1);
    const char* st = smem + (kt & 1) * kWStage;
    const int left = rows - kt * 64;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
      u32x4 fp[2], fq[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        fp[i] = frag(st, wm * 64 + 32 * i, kk);
        fq[i] = frag(st + kWStage / 2, wn * 64 + 32 * i, kk);
      }
      if (left < 64) {  // rows past the last: zero in both operands
        const int kb = kk * 16 + 8 * (lane >> 5);
#pragma unroll
        for (int d = 0; d < 4; ++d) {
          const uint32_t m = (kb + 2 * d < left ? 0x0000ffffu : 0u) |
                             (kb + 2 * d + 1 < left ? 0xffff0000u : 0u);
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            fp[i][d] &= m;
            fq[i][d] &= m;
          }
        }
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const bf16x8 x = __builtin_bit_cast(bf16x8, fp[i]);
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, __builtin_bit_cast(bf16x8, fq[j]),
                                                              acc[i][j], 0, 0, 0);
        if (bias) accb[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, ones, accb[i], 0, 0, 0);
      }
    }
  }
  // Element e: row 8*(e/4) + 4*(lane/32) + e%4 of a 32-row block, column lane%32.
  const int lr = lane & 31, lg = lane >> 5;
  float* const part = a.part + (int64_t)logical * (kWT * kWT);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const int r = wm * 64 + 32 * i + 8 * (e >> 2) + 4 * lg + (e & 3);
      const int rr = r0 + r - w.sp;
      const bool row_in = rr >= 0 && rr < w.ra;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const int c = wn * 64 + 32 * j + lr, cc = c0 + c - w.sq;
        if (a.split > 1)
          part[r * kWT + c] = acc[i][j][e];
        else if (row_in && cc >= 0 && cc < w.rb)
          w.out[(int64_t)rr * w.ldo + cc] = acc[i][j][e];
      }
      if (bias && lr == 0 && row_in) {
        if (a.split > 1)
          a.bpart[(int64_t)(sl * kWgradMax + wgrad_problem(a, tile)) * a.bstride + rr] = accb[i][e];
        else
          w.bias[rr] = accb[i][e];
      }
    }
}

// Sums the split tiles (16 workgroups a tile, four values a thread), and in the
// workgroups past the last tile the split bias gradients.
__global__ __launch_bounds__(256) void wgrad_reduce_kernel(WgradP a) {
  const int tile = blockIdx.x >> 4;
  if (tile >= a.tiles) {
    const int i = (blockIdx.x - a.tiles * 16) * 256 + threadIdx.x;
    const int q = i / a.bstride, r = i - q * a.bstride;
    if (q >= a.n || a.t[q].bias == nullptr || r >= a.t[q].ra) return;
    float v = 0.0f;
    for (int s = 0; s < a.split; ++s) v += a.bpart[(int64_t)(s * kWgradMax + q) * a.bstride + r];
    a.t[q].bias[r] = v;
    return;
  }
  const WgradTile& w = a.t[wgrad_problem(a, tile)];
  const int ti = (tile - w.tile0) / w.tc, tj = tile - w.tile0 - ti * w.tc;
  const int o = ((blockIdx.x & 15) * 256 + threadIdx.x) * 4, r = o / kWT, c = o - r * kWT;
  const int rr = ti * kWT + r - w.sp, cc = tj * kWT + c - w.sq;
  if (rr < 0 || rr >= w.ra || cc + 3 < 0 || cc >= w.rb) return;
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < a.split; ++s)
    v += *reinterpret_cast<const f32x4*>(a.part + ((int64_t)s * a.tiles + tile) * (kWT * kWT) + o);
  float* out = w.out + (int64_t)rr * w.ldo + cc;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (cc + e >= 0 && cc + e < w.rb) out[e] = v[e];
}

// --------------------------------------------------------- LayerNorm bwd
// xhat = (x - mean) * rstd recomputed from x (bf16), g = dy * gamma,
// dx = rstd * (g - mean(g) - xhat * mean(g * xhat)); dX[row] += dx (fp32) and
// dXb[row] = bf16(dX[row]).  Half a wave a row, 8-element chunks, every load of
// a row issued before its first sum; NC = ceil(d / 256) chunks a lane.  Bound:
// memory (14 bytes an element); 12608 x 768 rows: 79 us with one element a
// load, now 27 us (5.1 TB/s).
constexpr int kLnMaxChunks = 8;  // d <= 2048
__device__ __forceinline__ float half_sum(float v) {
#pragma unroll
  for (int off = 16; off >= 1; off >>= 1) v += __shfl_xor(v, off, 32);
  return v;
}
__device__ __forceinline__ void unpack8(u32x4 w, float (&v)[8]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    v[2 * e] = __uint_as_float(w[e] << 16);
    v[2 * e + 1] = __uint_as_float(w[e] & 0xffff0000u);
  }
}
template <int NC>
__global__ __launch_bounds__(256) void layernorm_bwd_kernel(
    const uint16_t* __restrict__ x, int64_t ldx, const uint16_t* __restrict__ dy, int64_t ldy,
    const float* __restrict__ gamma, float eps, int rows, int d, float* __restrict__ dX,
    int64_t lddx, uint16_t* __restrict__ dXb, int64_t lddxb) {
  const int hl = threadIdx.x & 31, nch = d >> 3;
  const int row_raw = blockIdx.x * 8 + (threadIdx.x >> 5);
  const bool live = row_raw < rows;
  const int row = live ? row_raw : rows - 1;
  const uint16_t* xr = x + (int64_t)row * ldx;
  const uint16_t* gr = dy + (int64_t)row * ldy;
  float* dxr = dX + (int64_t)row * lddx;
  u32x4 xw[NC], yw[NC];
  f32x4 dw[NC][2];
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = min(hl + 32 * i, nch - 1) * 8;
    xw[i] = *reinterpret_cast<const u32x4*>(xr + c);
    yw[i] = *reinterpret_cast<const u32x4*>(gr + c);
    dw[i][0] = *reinterpret_cast<const f32x4*>(dxr + c);
    dw[i][1] = *reinterpret_cast<const f32x4*>(dxr + c + 4);
  }
  float xv[NC][8], gv[NC][8];
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    unpack8(xw[i], xv[i]);
    unpack8(yw[i], gv[i]);
    const bool in = hl + 32 * i < nch;
    const int c = min(hl + 32 * i, nch - 1) * 8;
    const f32x4 g0 = *reinterpret_cast<const f32x4*>(gamma + c);
    const f32x4 g1 = *reinterpret_cast<const f32x4*>(gamma + c + 4);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      gv[i][e] = in ? gv[i][e] * (e < 4 ? g0[e & 3] : g1[e & 3]) : 0.f;
      xv[i][e] = in ? xv[i][e] : 0.f;
      s += xv[i][e];
    }
  }
  const float mean = half_sum(s) / (float)d;
  float v = 0.f;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const bool in = hl + 32 * i < nch;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      xv[i][e] = in ? xv[i][e] - mean : 0.f;
      v = fmaf(xv[i][e], xv[i][e], v);
    }
  }
  const float rstd = 1.0f / sqrtf(half_sum(v) / (float)d + eps);
  float sg = 0.f, sgx = 0.f;
#pragma unroll
  for (int i = 0; i < NC; ++i)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      xv[i][e] *= rstd;
      sg += gv[i][e];
      sgx = fmaf(gv[i][e], xv[i][e], sgx);
    }
  sg = half_sum(sg) / (float)d;
  sgx = half_sum(sgx) / (float)d;
  if (!live) return;
  uint16_t* dbr = dXb + (int64_t)row * lddxb;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int ci = hl + 32 * i;
    if (ci >= nch) continue;
    float o[8];
#pragma unroll
    for (int e = 0; e < 8; ++e)
      o[e] = dw[i][e >> 2][e & 3] + rstd * (gv[i][e] - sg - xv[i][e] * sgx);
    *reinterpret_cast<f32x4*>(dxr + 8 * ci) = f32x4{o[0], o[1], o[2], o[3]};
    *reinterpret_cast<f32x4*>(dxr + 8 * ci + 4) = f32x4{o[4], o[5], o[6], o[7]};
    u32x4 w;
#pragma unroll
    for (int e = 0; e < 4; ++e) w[e] = pack_bf16x2(o[2 * e], o[2 * e + 1]);
    *reinterpret_cast<u32x4*>(dbr + 8 * ci) = w;
  }
}

// ---------------------------------------------------------- cross-entropy
// One workgroup per image: loss_b = log sum exp(z) - z[label];
// dlogits = (softmax(z) - onehot(label)) / batch, bf16.  A label outside
// [0, C) gives a NaN loss and no one-hot term.
__global__ __launch_bounds__(256) void cross_entropy_kernel(const float* __restrict__ logits,
                                                            int64_t ldl,
                                                            const int32_t* __restrict__ labels,
                                                            int C, int batch,
                                                            uint16_t* __restrict__ dlogits,
                                                            int64_t ldd,
                                                            float* __restrict__ rowloss) {
  __shared__ float red[8];
  const int b = blockIdx.x, t = threadIdx.x;
  const float* z = logits + (int64_t)b * ldl;
  float mx = -INFINITY;
  for (int c = t; c < C; c += 256) mx = fmaxf(mx, z[c]);
  for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, 64));
  if ((t & 63) == 0) red[t >> 6] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  __syncthreads();
  float s = 0.f;
  for (int c = t; c < C; c += 256) s += expf(z[c] - mx);
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((t & 63) == 0) red[4 + (t >> 6)] = s;
  __syncthreads();
  s = (red[4] + red[5]) + (red[6] + red[7]);
  const int y = labels[b];
  const bool ok = y >= 0 && y < C;
  const float inv = 1.0f / s, ib = 1.0f / (float)batch;
  for (int c = t; c < C; c += 256) {
    const float pr = expf(z[c] - mx) * inv;
    dlogits[(int64_t)b * ldd + c] = f32_to_bf16((pr - (ok && c == y ? 1.0f : 0.0f)) * ib);
  }
  if (t == 0) rowloss[b] = ok ? logf(s) + mx - z[y] : NAN;
}

// --------------------------------------------------------- small reductions
// Sum of squares of a fp32 array: one partial per workgroup.
constexpr int kSqBlocks = 1024;
__global__ __launch_bounds__(256) void sumsq_kernel(const float* __restrict__ g, int64_t n,
                                                    float* __restrict__ part) {
  __shared__ float red[4];
  float s = 0.f;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256)
    s = fmaf(g[i], g[i], s);
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o, 64);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = (red[0] + red[1]) + (red[2] + red[3]);
}

// stats = {mean loss, |G . grad|, clip factor}; the factor is also what the
// update kernel reads.
__global__ __launch_bounds__(256) void growth_finish_kernel(const float* __restrict__ part,
                                                            int nparts,
                                                            const float* __restrict__ rowloss,
                                                            int batch, float clip,
                                                            float* __restrict__ stats) {
  __shared__ float red[8];
  float s = 0.f, l = 0.f;
  for (int i = threadIdx.x; i < nparts; i += 256) s += part[i];
  for (int i = threadIdx.x; i < batch; i += 256) l += rowloss[i];
  for (int o = 32; o > 0; o >>= 1) {
    s += __shfl_xor(s, o, 64);
    l += __shfl_xor(l, o, 64);
  }
  if ((threadIdx.x & 63) == 0) {
    red[threadIdx.x >> 6] = s;
    red[4 + (threadIdx.x >> 6)] = l;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    const float norm = sqrtf((red[0] + red[1]) + (red[2] + red[3]));
    stats[0] = ((red[4] + red[5]) + (red[6] + red[7])) / (float)batch;
    stats[1] = norm;
    stats[2] = norm > clip ? clip / norm : 1.0f;
  }
}

// ----------------------------------------------------------------- update
// One workgroup row per slice (blockIdx.y), elements strided over blockIdx.x.
__global__ __launch_bounds__(256) void growth_update_kernel(const GrowthSlice* __restrict__ sl,
                                                            const float* __restrict__ grad,
                                                            float* __restrict__ master,
                                                            uint8_t* __restrict__ packed,
                                                            const float* __restrict__ stats,
                                                            float lr) {
  const GrowthSlice d = sl[blockIdx.y];
  const int64_t n = (int64_t)d.rows * d.cols;
  const float step = lr * stats[2];
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    const int r = (int)(i / d.cols), c = (int)(i - (int64_t)r * d.cols);
    const float g = grad[d.grad_off + (int64_t)r * d.grad_ld + c];
    const int64_t e = (int64_t)r * d.ld + c;
    if (d.is_bf16) {
      const int64_t idx = d.packed_off / 2 + e;  // master element of this bf16 weight
      const float w = master[idx] - step * g;
      master[idx] = w;
      reinterpret_cast<uint16_t*>(packed)[idx] = f32_to_bf16(w);
    } else {
      float* w = reinterpret_cast<float*>(packed + d.packed_off) + e;
      *w = *w - step * g;
    }
  }
}

// master[i] = packed bf16 element i, for i in [off, off + n) (elements).
__global__ __launch_bounds__(256) void master_init_kernel(const uint16_t* __restrict__ packed,
                                                          int64_t off, int64_t n,
                                                          float* __restrict__ master) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) master[off + i] = bf16_to_f32(packed[off + i]);
}

}  // namespace

hipError_t launch_transposes_bf16(const TransposeJob* jobs, int njobs, int max_tiles, const void* in,
                                  void* out, hipStream_t s) {
  if (njobs <= 0 || max_tiles <= 0) return hipSuccess;
  hipLaunchKernelGGL(transpose_kernel, dim3((unsigned)max_tiles, (unsigned)njobs), dim3(256), 0, s,
                     jobs, static_cast<const uint16_t*>(in), static_cast<uint16_t*>(out));
  return hipGetLastError();
}

hipError_t launch_wgrad_bf16(const WgradArgs* probs, int n, int64_t M, float* part,
                             int64_t part_floats, float* bpart, int bstride, hipStream_t s) {
  if (n < 0 || n > kWgradMax || M >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
  WgradP a{};
  a.M = (int)M;
  a.part = part;
  a.bpart = bpart;
  a.bstride = bstride;
  for (int i = 0; i < n; ++i) {
    const WgradArgs& g = probs[i];
    if (g.ra <= 0 || g.rb <= 0) continue;
    // Whole 16-byte chunks of rows of ldp / ldq elements.
    if (g.ldp % 8 || g.ldq % 8 || g.pc < 0 || g.qc < 0 || g.pc + g.ra > g.ldp ||
        g.qc + g.rb > g.ldq || g.ra > bstride)
      return hipErrorInvalidValue;
    WgradTile& t = a.t[a.n++];
    t.P = static_cast<const uint16_t*>(g.P);
    t.Q = static_cast<const uint16_t*>(g.Q);
    t.ldp = g.ldp; t.ldq = g.ldq;
    t.sp = g.pc & 7; t.sq = g.qc & 7;
    t.pa = g.pc - t.sp; t.qa = g.qc - t.sq;
    t.ra = g.ra; t.rb = g.rb;
    t.out = g.out; t.bias = g.bias; t.ldo = g.rb;
    t.tile0 = a.tiles;
    t.tc = (g.rb + t.sq + kWT - 1) / kWT;
    a.tiles += (g.ra + t.sp + kWT - 1) / kWT * t.tc;
  }
  if (a.n == 0 || M <= 0) return hipSuccess;
  // About two workgroups per CU, of at least four steps of 64 rows.
  const int64_t steps = (M + 63) / 64;
  int64_t split = std::max<int64_t>(1, std::min<int64_t>({kWgradSlots / a.tiles, steps / 4, kWgradMaxSplit}));
  a.kchunk = (int)((steps + split - 1) / split) * 64;
  a.split = (int)((M + a.kchunk - 1) / a.kchunk);
  if (a.split > 1 && (int64_t)a.split * a.tiles * kWT * kWT > part_floats) return hipErrorInvalidValue;
  hipLaunchKernelGGL(wgrad_kernel, dim3((unsigned)(a.tiles * a.split)), dim3(256), 0, s, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.split == 1) return e;
  const int bias_blocks = (kWgradMax * bstride + 255) / 256;
  hipLaunchKernelGGL(wgrad_reduce_kernel, dim3((unsigned)(a.tiles * 16 + bias_blocks)), dim3(256), 0,
                     s, a);
  return hipGetLastError();
}

hipError_t launch_layernorm_bwd_bf16(const void* x, int64_t ldx, const void* dy, int64_t ldy,
                                     const float* gamma, float eps, int rows, int d, float* dX,
                                     int64_t lddx, void* dXb, int64_t lddxb, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  // 16-byte chunks of every row (the growth step's rows are d elements, d % 8 == 0).
  if (d < 8 || d > 256 * kLnMaxChunks || d % 8 || ldx % 8 || ldy % 8 || lddx % 4 || lddxb % 8)
    return hipErrorInvalidValue;
  auto go = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(grid_for(rows, 8)), dim3(256), 0, s,
                       static_cast<const uint16_t*>(x), ldx, static_cast<const uint16_t*>(dy), ldy,
                       gamma, eps, rows, d, dX, lddx, static_cast<uint16_t*>(dXb), lddxb);
    return hipGetLastError();
  };
  switch ((d + 255) / 256) {
    case 1: return go(layernorm_bwd_kernel<1>);
    case 2: return go(layernorm_bwd_kernel<2>);
    case 3: return go(layernorm_bwd_kernel<3>);
    case 4: return go(layernorm_bwd_kernel<4>);
    default: return go(layernorm_bwd_kernel<kLnMaxChunks>);
  }
}

hipError_t launch_cross_entropy(const float* logits, int64_t ldl, const int32_t* labels, int C,
                                int batch, void* dlogits, int64_t ldd, float* rowloss,
                                hipStream_t s) {
  if (batch <= 0) return hipSuccess;
  hipLaunchKernelGGL(cross_entropy_kernel, dim3((unsigned)batch), dim3(256), 0, s, logits, ldl,
                     labels, C, batch, static_cast<uint16_t*>(dlogits), ldd, rowloss);
  return hipGetLastError();
}

int growth_sumsq_parts() { return kSqBlocks; }

hipError_t launch_growth_norm(const float* grad, int64_t n, float* part, const float* rowloss,
                              int batch, float clip, float* stats, hipStream_t s) {
  hipLaunchKernelGGL(sumsq_kernel, dim3(kSqBlocks), dim3(256), 0, s, grad, n, part);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(growth_finish_kernel, dim3(1), dim3(256), 0, s, part, kSqBlocks, rowloss,
                     batch, clip, stats);
  return hipGetLastError();
}

hipError_t launch_growth_update(const GrowthSlice* slices, int nslices, const float* grad,
                                float* master, void* packed, const float* stats, float lr,
                                hipStream_t s) {
  if (nslices <= 0) return hipSuccess;
  hipLaunchKernelGGL(growth_update_kernel, dim3(256, (unsigned)nslices), dim3(256), 0, s, slices,
                     grad, master, static_cast<uint8_t*>(packed), stats, lr);
  return hipGetLastError();
}

hipError_t launch_master_init(const void* packed, int64_t off, int64_t n, float* master,
                              hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(master_init_kernel, dim3(grid_for(n, 256)), dim3(256), 0, s,
                     static_cast<const uint16_t*>(packed), off, n, master);
  return hipGetLastError();
}

}  // namespace elasto
