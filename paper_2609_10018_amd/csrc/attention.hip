// Multi-head self-attention over the active heads (Eq. 3):
// o = softmax(q k^T * scale) v per (sequence, head slot).
//
// bf16 path (head_dim 64): one workgroup of 8 waves per (sequence, head
// slot), so no wave takes more than two of the (up to 15) query blocks (two
// workgroups, each with a share of the blocks, when the pairs are too few to
// fill the CUs: small batches).  K and
// V are staged whole in LDS by direct global->LDS loads, both in token-row
// layout (rows of 128 B, 16-byte chunks XOR-swizzled); padding keys past the
// last token repeat that token and are masked (zero probability).  Each wave
// takes 16-query blocks in turn and computes the score block transposed,
// S^T = K Q^T, with v_mfma_f32_16x16x32_bf16: lane l then holds the scores of
// query l%16 against keys 16j + 4*(l/16) + {0..3}.  The softmax of a query is
// reduced over its 4 lanes with two xor-shuffles and is exact (single pass:
// the whole key row fits in registers).  The probabilities are rounded to
// bf16 and are reused unchanged as the k-slots of the second product, which
// is also taken transposed, O^T = V^T P^T: the MFMA's k-slots are only
// labels, so the 8 keys a lane holds for two adjacent key tiles form its
// k-slots, and the V^T operand is read from the row-major V with the LDS
// transpose read (ds_read_b64_tr_b16: in each group of 16 lanes, lane i
// receives element i%4 of the 8-byte pieces that lanes i/4, 4 + i/4, 8 + i/4
// and 12 + i/4 address, so four key rows x 16 feature columns come back as
// four keys per lane, one column per lane).  Lane l then holds features
// 16n + 4*(l/16) + {0..3} of query l%16: the 1/rowsum normalisation is
// applied in fp32 and each lane writes 8-byte pieces of its query's row.
//
// fp32 path: the same transposed products on the fp32 matrix instruction
// (attention_f32_kernel).
#include <algorithm>

#include "common.h"
#include "kernels.h"

namespace elasto {
namespace {

typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(1))) void global_void;
typedef short i16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4 lds_i16x4;

constexpr int kHd = 64;
constexpr int kWaves = 8;
constexpr int kThreads = 64 * kWaves;
constexpr int kRsrcWord3 = 0x00020000;  // buffer resource: raw (unswizzled) 32-bit records

// Byte offset of logical 16-byte chunk c of token row r in a staged K or V.
__device__ __forceinline__ int kv_off(int r, int c) { return r * 128 + ((c ^ (r & 7)) << 4); }

struct AttnP {
  const uint16_t* qkv;
  int64_t qs;
  uint16_t* o;
  int64_t os;
  int T, heads;
  int parts;  // workgroups per (sequence, head slot), each a share of the query blocks
  float scale_log2;
};

// NT = ceil(T / 16) key tiles, fixed at compile time so that every loop over
// keys is fully unrolled and only the last tile carries the key < T mask.
template <int NT>
__global__ __launch_bounds__(kThreads, 2) void attention_bf16_kernel(AttnP p) {
  constexpr int KV = NT * 16 * 128;  // bytes of the staged K (and of V)
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int T = p.T;
  const char* kl = smem;
  const char* vl = smem + KV;

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int bs = blockIdx.x / p.parts, part = blockIdx.x - bs * p.parts;
  const int b = bs / p.heads, s = bs - b * p.heads;
  // Query blocks of this workgroup: part * 8 + wave, then every 8 * parts.
  const int qb0 = part * kWaves + wave, qstep = kWaves * p.parts;
  const uint16_t* base = p.qkv + (int64_t)b * T * p.qs + (int64_t)s * 3 * kHd;

  const int lq = lane & 15, lg = lane >> 4;
  // Q fragments of a 16-query block (B operand of S^T = K Q^T); rows past the
  // last token re-read token T-1 and their outputs are dropped.
  auto load_q = [&](int qb, bf16x8* qf) {
    const int q = min(qb * 16 + lq, T - 1);
    const uint16_t* qp = base + (int64_t)q * p.qs + lg * 8;
    qf[0] = *reinterpret_cast<const bf16x8*>(qp);
    qf[1] = *reinterpret_cast<const bf16x8*>(qp + 32);
  };
  bf16x8 qf[2];
  if (qb0 < NT) load_q(qb0, qf);

  // K and V: direct global->LDS loads in 1-KB blocks of 8 token rows (blocks
  // 0 .. 2NT-1 are K, the next 2NT are V).  Lane l lands at block + 16 l,
  // i.e. row 8*blk + l/8, physical chunk l%8, so it fetches the logical chunk
  // that kv_off() places there.  Rows past the last token re-read token T-1:
  // their scores are masked out and their probabilities are 0.  Each wave
  // issues its K blocks first, then as many V blocks (wave + 8i < 2NT for
  // both), so the first scores are computed while V is still arriving.
  constexpr int kLoadIters = (2 * NT + kWaves - 1) / kWaves;
#pragma unroll
  for (int isv = 0; isv < 2; ++isv)
#pragma unroll
    for (int i = 0; i < kLoadIters; ++i) {
      const int rb = wave + kWaves * i;  // block of 8 rows within K or V
      if (rb < 2 * NT) {
        const int r = rb * 8 + (lane >> 3);
        const int c = (lane & 7) ^ (r & 7);
        const uint16_t* src = base + (int64_t)min(r, T - 1) * p.qs + (1 + isv) * kHd + c * 8;
        __builtin_amdgcn_global_load_lds((global_void*)src,
                                         (lds_void*)(smem + (isv * 2 * NT + rb) * 1024), 16, 0, 0);
      }
    }
  // Nothing reads the staged rows by register dependence.  K: wait until at
  // most this wave's V loads are in flight (loads complete in issue order for
  // the counter; the Q loads came first), then for every wave.
  const int nkv = wave < 2 * NT ? (2 * NT - 1 - wave) / kWaves + 1 : 0;
  static_assert(kLoadIters <= 4, "K/V loads per wave exceed the wait cases");
  switch (nkv) {
    case 0: __builtin_amdgcn_s_waitcnt(0 | (0x7 << 4) | (0xF << 8)); break;
    case 1: __builtin_amdgcn_s_waitcnt(1 | (0x7 << 4) | (0xF << 8)); break;
    case 2: __builtin_amdgcn_s_waitcnt(2 | (0x7 << 4) | (0xF << 8)); break;
    case 3: __builtin_amdgcn_s_waitcnt(3 | (0x7 << 4) | (0xF << 8)); break;
    default: __builtin_amdgcn_s_waitcnt(4 | (0x7 << 4) | (0xF << 8)); break;
  }
  __syncthreads();

  // Output rows of this (sequence, head slot): T rows of p.os elements from
  // column s*64; an offset of nrec drops the store (rows past the last token).
  const int nrec = T * (int)p.os * 2;
  const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
      p.o + (int64_t)b * T * p.os + (int64_t)s * kHd, (short)0, nrec, kRsrcWord3);
  const float c2 = p.scale_log2;
  for (int qb = qb0; qb < NT; qb += qstep) {
    const int q0 = qb * 16;
    f32x4 st[NT];
#pragma unroll
    for (int j = 0; j < NT; ++j) {
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(kl + kv_off(j * 16 + lq, kk * 4 + lg));
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qf[kk], acc, 0, 0, 0);
      }
      st[j] = acc;
      // Bound how far the scheduler hoists LDS reads (register pressure).
      if ((j & 3) == 3) __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_sched_barrier(0);
    bf16x8 qn[2];
    if (qb + qstep < NT) load_q(qb + qstep, qn);
    // Keys of the last tile at or past T do not exist.
    bool valid[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) valid[r] = (NT - 1) * 16 + 4 * lg + r < T;
    float mx = -INFINITY;
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        mx = fmaxf(mx, (j < NT - 1 || valid[r]) ? st[j][r] : -INFINITY);
    mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
    mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
    const float off = -mx * c2;
    float sum = 0.f;
#pragma unroll
    for (int j = 0; j < NT; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float e = __builtin_amdgcn_exp2f(fmaf(st[j][r], c2, off));
        if (j == NT - 1) e = valid[r] ? e : 0.f;
        st[j][r] = e;
        sum += e;
      }
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    __builtin_amdgcn_sched_barrier(0);
    // V: before the first product with it, every V load of every wave.  Each
    // wave passes this barrier once (here on its first block, or after the
    // loop when it has none).
    if (qb == qb0) {
      __builtin_amdgcn_s_waitcnt((0x7 << 4) | (0xF << 8));
      __syncthreads();
    }

    // O^T = V^T P^T over key pairs of tiles (2kb, 2kb+1): k-slot 8*lg + r is
    // key 32kb + 4lg + r, k-slot 8*lg + 4 + r is key 32kb + 16 + 4lg + r.
    f32x4 o[4];
#pragma unroll
    for (int n = 0; n < 4; ++n) o[n] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int vr = 4 * lg + (lq >> 2);  // key row this lane addresses, within a 32-key pair
#pragma unroll
    for (int kb = 0; kb < (NT + 1) / 2; ++kb) {
      const bool has_hi = 2 * kb + 1 < NT;
      bf16x8 pa;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        pa[r] = static_cast<__bf16>(st[2 * kb][r]);
        pa[4 + r] = has_hi ? static_cast<__bf16>(st[has_hi ? 2 * kb + 1 : 2 * kb][r])
                           : static_cast<__bf16>(0.f);
      }
#pragma unroll
      for (int n = 0; n < 4; ++n) {
        // This lane addresses columns 16n + 4(lq%4) .. +3 of key row 32kb + vr
        // (and of the row 16 keys further for the upper k-slots).
        const int col = n * 16 + 4 * (lq & 3), half = (col & 4) * 2;
        const int r0 = kb * 32 + vr;
        const u32x2 lo = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
            (lds_i16x4*)(vl + kv_off(r0, col >> 3) + half)));
        u32x2 hi = {0u, 0u};
        if (has_hi)
          hi = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
              (lds_i16x4*)(vl + kv_off(r0 + 16, col >> 3) + half)));
        const u32x4 w = {lo[0], lo[1], hi[0], hi[1]};
        o[n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w), pa, o[n],
                                                       0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    // Lane (lg, lq) holds O[q0 + lq][16n + 4lg + r], r = 0..3.
    const float inv = 1.0f / sum;  // for query lq
    const int q = q0 + lq;
#pragma unroll
    for (int n = 0; n < 4; ++n) {
      const u32x2 w = {pack_bf16x2(o[n][0] * inv, o[n][1] * inv),
                       pack_bf16x2(o[n][2] * inv, o[n][3] * inv)};
      __builtin_amdgcn_raw_buffer_store_b64(w, ro, q < T ? (q * (int)p.os + 16 * n + 4 * lg) * 2 : nrec,
                                            0, 0);
    }
    qf[0] = qn[0];
    qf[1] = qn[1];
  }
  if (qb0 >= NT) {
    __builtin_amdgcn_s_waitcnt((0x7 << 4) | (0xF << 8));
    __syncthreads();
  }
}

template <int NT>
hipError_t launch_attn_nt(AttnP p, int batch, int heads, hipStream_t s) {
  const size_t lds = 2 * (size_t)NT * 16 * 128;
  // Few (sequence, head slot) pairs (small batches, narrow modes): split each
  // one's query blocks over more workgroups (each stages K and V itself), so
  // that more CUs work and a wave takes one block instead of two.
  constexpr int kCUs = 256;
  const int pairs = batch * heads;
  p.parts = std::max(1, std::min((NT + kWaves - 1) / kWaves, kCUs / std::max(pairs, 1)));
  hipLaunchKernelGGL(attention_bf16_kernel<NT>, dim3((unsigned)(pairs * p.parts)), dim3(kThreads),
                     lds, s, p);
  return hipGetLastError();
}

struct AttnF {
  const float* qkv;
  int64_t qs;
  float* o;
  int64_t os;
  int T, heads, hd, qblocks;
  float scale;
};

constexpr int kHdMaxF32 = 128;
constexpr int kWavesF32 = 4;

// N consecutive floats, as wide as N allows (p aligned to that width).
template <int N>
__device__ __forceinline__ void load_run(const float* p, float* v) {
  if constexpr (N % 4 == 0) {
#pragma unroll
    for (int i = 0; i < N / 4; ++i) {
      const f32x4 w = *reinterpret_cast<const f32x4*>(p + 4 * i);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[4 * i + e] = w[e];
    }
  } else if constexpr (N == 2) {
    const f32x2 w = *reinterpret_cast<const f32x2*>(p);
    v[0] = w[0];
    v[1] = w[1];
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = p[i];
  }
}

// fp32 attention on the fp32 matrix instruction (v_mfma_f32_16x16x4_f32, full
// fp32 products and sums).  A workgroup takes 16 queries of one
// (sequence, head slot); its four waves share out the 16-key tiles (wave w:
// tiles w, w + 4, ...) and merge their running maxima, sums and outputs in LDS
// at the end, so a short sequence still gives four waves work per query block.
// K, V and Q go from memory straight to registers: the MFMA's k-slots are only
// labels, so a lane loads four consecutive features of its K row for four
// MFMAs, and the S^T layout (lane l: query l%16, keys 4*(l/16) + r) is the B
// operand of O^T = V^T P^T as it stands, with feature NB*i + n as row i of
// block n, so a V row is loaded NB floats a lane.
// NB = ceil(hd / 16); VEC: hd = 16 NB and every row 16-byte aligned (else
// element loads with a bound on the feature).  KT key tiles are loaded at a
// time per wave (all of a 256-token sequence for hd <= 64: no rescaling).
// Bound: the MFMAs (64 FLOP a cycle and SIMD) and one memory latency per wave.
// 16 sequences x 6 heads, 197 tokens, hd 64: 24 us, 40 TFLOP/s (4115 us with
// one thread per query and its vectors in scratch); 32 queries a workgroup,
// for half the reads of K and V, measured the same (24.8 us) and slower for
// one sequence (9.7 against 6.6 us).
template <int NB, bool VEC>
__global__ __launch_bounds__(64 * kWavesF32) void attention_f32_kernel(AttnF p) {
  constexpr int KT = NB <= 4 ? 4 : 2;
  constexpr int OS = 16 * NB + 4;
  __shared__ __attribute__((aligned(16))) float so[kWavesF32][16][OS];
  __shared__ float sm[kWavesF32][16], ss[kWavesF32][16];
  const int lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int b = blockIdx.x / p.heads, s = blockIdx.x - b * p.heads;
  const int T = p.T, hd = p.hd, tiles = (T + 15) / 16;
  const float* base = p.qkv + (int64_t)b * T * p.qs + (int64_t)s * 3 * hd;
  // Features c*16 + 4lg .. +3 of a row (Q and K).
  auto load4 = [&](const float* row, int c) {
    const int f = c * 16 + 4 * lg;
    f32x4 v;
    if constexpr (VEC) {
      v = *reinterpret_cast<const f32x4*>(row + f);
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = f + e < hd ? row[f + e] : 0.0f;
    }
    return v;
  };
  for (int qb = blockIdx.y; qb < p.qblocks; qb += gridDim.y) {
    f32x4 qf[NB], o[NB];
    float m = -INFINITY, sum = 0.0f;
    const float* qrow = base + (int64_t)min(qb * 16 + li, T - 1) * p.qs;
#pragma unroll
    for (int c = 0; c < NB; ++c) {
      qf[c] = load4(qrow, c);
      o[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    for (int t0 = wave; t0 < tiles; t0 += kWavesF32 * KT) {
      f32x4 kf[KT][NB];
      float vf[KT][4][NB];
#pragma unroll
      for (int i = 0; i < KT; ++i) {
        const int k0 = (t0 + kWavesF32 * i) * 16;
        const float* row = base + (int64_t)min(k0 + li, T - 1) * p.qs + hd;
#pragma unroll
        for (int c = 0; c < NB; ++c) kf[i][c] = load4(row, c);
      }
#pragma unroll
      for (int i = 0; i < KT; ++i) {
        const int k0 = (t0 + kWavesF32 * i) * 16;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float* row = base + (int64_t)min(k0 + 4 * lg + r, T - 1) * p.qs + 2 * hd;
          if constexpr (VEC) {
            load_run<NB>(row + NB * li, vf[i][r]);
          } else {
#pragma unroll
            for (int n = 0; n < NB; ++n) vf[i][r][n] = NB * li + n < hd ? row[NB * li + n] : 0.0f;
          }
        }
      }
      f32x4 st[KT];
      float mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < KT; ++i) {
        const int k0 = (t0 + kWavesF32 * i) * 16;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NB; ++c)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            acc = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[i][c][r], qf[c][r], acc, 0, 0, 0);
        // Keys past the last do not exist.
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          st[i][r] = k0 + 4 * lg + r < T ? acc[r] * p.scale : -INFINITY;
          mx = fmaxf(mx, st[i][r]);
        }
      }
      mx = fmaxf(mx, __shfl_xor(mx, 16, 64));
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      mx = fmaxf(m, mx);
      // Nothing above -inf so far: any reference will do (all terms are 0).
      const float ref = mx == -INFINITY ? 0.0f : mx;
      if (t0 >= kWavesF32 * KT) {
        const float f = expf(m - ref);
        sum *= f;
#pragma unroll
        for (int n = 0; n < NB; ++n) o[n] *= f;
      }
      m = mx;
#pragma unroll
      for (int i = 0; i < KT; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          st[i][r] = expf(st[i][r] - ref);
          sum += st[i][r];
        }
#pragma unroll
      for (int i = 0; i < KT; ++i) {
        const int k0 = (t0 + kWavesF32 * i) * 16;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const bool in = k0 + 4 * lg + r < T;  // a missing key's 0 must not meet an inf or NaN
#pragma unroll
          for (int n = 0; n < NB; ++n)
            o[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? vf[i][r][n] : 0.0f, st[i][r], o[n], 0,
                                                        0, 0);
        }
      }
    }
    // Merge the waves: lane (lg, li) holds features NB*(4lg + r) + n of query li.
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int n = 0; n < NB; ++n) so[wave][li][NB * (4 * lg + r) + n] = o[n][r];
    if (lg == 0) {
      sm[wave][li] = m;
      ss[wave][li] = sum;
    }
    __syncthreads();
    const int ql = threadIdx.x >> 4, row = qb * 16 + ql;
    float top = sm[0][ql];
#pragma unroll
    for (int w = 1; w < kWavesF32; ++w) top = fmaxf(top, sm[w][ql]);
    float den = 0.0f, v[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n) v[n] = 0.0f;
#pragma unroll
    for (int w = 0; w < kWavesF32; ++w) {
      const float f = expf(sm[w][ql] - top);  // 0 for a wave without keys (all -inf: NaN, as 0/0)
      den = fmaf(f, ss[w][ql], den);
#pragma unroll
      for (int n = 0; n < NB; ++n) v[n] = fmaf(f, so[w][ql][NB * li + n], v[n]);
    }
    if (row < T) {
      const float inv = 1.0f / den;
      float* op = p.o + ((int64_t)b * T + row) * p.os + (int64_t)s * hd + NB * li;
      if constexpr (VEC && NB % 4 == 0) {
#pragma unroll
        for (int n = 0; n < NB; n += 4)
          *reinterpret_cast<f32x4*>(op + n) =
              f32x4{v[n] * inv, v[n + 1] * inv, v[n + 2] * inv, v[n + 3] * inv};
      } else {
#pragma unroll
        for (int n = 0; n < NB; ++n)
          if (NB * li + n < hd) op[n] = v[n] * inv;
      }
    }
    __syncthreads();
  }
}

template <int NB, bool VEC>
hipError_t launch_attn_f32(AttnF p, int batch, hipStream_t s) {
  p.qblocks = (p.T + 15) / 16;
  hipLaunchKernelGGL((attention_f32_kernel<NB, VEC>),
                     dim3((unsigned)(batch * p.heads), (unsigned)std::min(p.qblocks, 65535)),
                     dim3(64 * kWavesF32), 0, s, p);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attention_bf16(const AttnArgs& a, hipStream_t s) {
  if (a.batch <= 0 || a.heads <= 0 || a.tokens <= 0) return hipSuccess;
  if (a.head_dim != kHd || a.tokens > kAttnMaxTokens) return hipErrorInvalidValue;
  // The output of a (sequence, head slot) is addressed as one buffer range of
  // T rows: the rows must hold every head slot and the range must fit 31 bits.
  if (a.o_stride < (int64_t)a.heads * kHd || a.qkv_stride < (int64_t)a.heads * 3 * kHd ||
      (int64_t)a.tokens * a.o_stride * 2 > INT32_MAX)
    return hipErrorInvalidValue;
  AttnP p;
  p.qkv = static_cast<const uint16_t*>(a.qkv);
  p.qs = a.qkv_stride;
  p.o = static_cast<uint16_t*>(a.o);
  p.os = a.o_stride;
  p.T = a.tokens;
  p.heads = a.heads;
  p.scale_log2 = a.scale * 1.4426950408889634f;
  switch ((a.tokens + 15) / 16) {
    case 1: return launch_attn_nt<1>(p, a.batch, a.heads, s);
    case 2: return launch_attn_nt<2>(p, a.batch, a.heads, s);
    case 3: return launch_attn_nt<3>(p, a.batch, a.heads, s);
    case 4: return launch_attn_nt<4>(p, a.batch, a.heads, s);
    case 5: return launch_attn_nt<5>(p, a.batch, a.heads, s);
    case 6: return launch_attn_nt<6>(p, a.batch, a.heads, s);
    case 7: return launch_attn_nt<7>(p, a.batch, a.heads, s);
    case 8: return launch_attn_nt<8>(p, a.batch, a.heads, s);
    case 9: return launch_attn_nt<9>(p, a.batch, a.heads, s);
    case 10: return launch_attn_nt<10>(p, a.batch, a.heads, s);
    case 11: return launch_attn_nt<11>(p, a.batch, a.heads, s);
    case 12: return launch_attn_nt<12>(p, a.batch, a.heads, s);
    case 13: return launch_attn_nt<13>(p, a.batch, a.heads, s);
    case 14: return launch_attn_nt<14>(p, a.batch, a.heads, s);
    case 15: return launch_attn_nt<15>(p, a.batch, a.heads, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_attention_f32(const AttnArgs& a, hipStream_t s) {
  if (a.batch <= 0 || a.heads <= 0 || a.tokens <= 0) return hipSuccess;
  if (a.head_dim > kHdMaxF32 || a.head_dim <= 0) return hipErrorInvalidValue;
  AttnF p;
  p.qkv = static_cast<const float*>(a.qkv);
  p.qs = a.qkv_stride;
  p.o = static_cast<float*>(a.o);
  p.os = a.o_stride;
  p.T = a.tokens;
  p.heads = a.heads;
  p.hd = a.head_dim;
  p.scale = a.scale;
  // Vector loads: whole 16-feature groups and 16-byte aligned rows.
  const bool vec = a.head_dim % 16 == 0 && a.qkv_stride % 4 == 0 && a.o_stride % 4 == 0 &&
                   reinterpret_cast<uintptr_t>(a.qkv) % 16 == 0 &&
                   reinterpret_cast<uintptr_t>(a.o) % 16 == 0;
  switch ((a.head_dim + 15) / 16) {
    case 1: return launch_attn_f32<1, false>(p, a.batch, s);
    case 2: return vec ? launch_attn_f32<2, true>(p, a.batch, s) : launch_attn_f32<2, false>(p, a.batch, s);
    case 3: return launch_attn_f32<3, false>(p, a.batch, s);
    case 4: return vec ? launch_attn_f32<4, true>(p, a.batch, s) : launch_attn_f32<4, false>(p, a.batch, s);
    case 5: return launch_attn_f32<5, false>(p, a.batch, s);
    case 6: return launch_attn_f32<6, false>(p, a.batch, s);
    case 7: return launch_attn_f32<7, false>(p, a.batch, s);
    default: return vec ? launch_attn_f32<8, true>(p, a.batch, s) : launch_attn_f32<8, false>(p, a.batch, s);
  }
}

}  // namespace elasto
