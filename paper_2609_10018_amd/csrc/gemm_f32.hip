// fp32 width-sliced GEMM, C[m][n] = epi(sum_k A[m][k] W[n][k] + bias[n]),
// on the fp32 matrix instruction v_mfma_f32_32x32x2_f32: full fp32 products
// and sums, at twice the rate of the unpacked vector FMA (64 FLOP a cycle and
// SIMD).  Any shape and stride: nothing outside the active K prefix / N rows
// is read.
//
// A workgroup of 4 waves owns a BM x BN output tile and walks K 32 at a time.
// The next step's A and W values are loaded into registers while the present
// step is multiplied from LDS (two LDS stages, one barrier a step).  The
// MFMA's two k-slots are only labels: lane l reads the four consecutive
// values 4*(l/32) .. +3 of an 8-value chunk of its row with one 16-byte LDS
// read, and value r of both halves is one MFMA.  LDS rows are 36 floats long,
// so that 16 consecutive rows start on distinct groups of four banks.
//
// Bound: the matrix units (80% busy in the long K loop of 128x128 tiles, 66% in
// 64x64 ones at K 1536), and for short K the loads before and the stores after a
// tile's loop (53% at K 384).  6304 x 1152 x 384, 1782 64x64 tiles, at most four
// on a CU: 59 us, 94 TFLOP/s (97 us on the vector ALU); 8000 x 3072 x 3072,
// 128x128 tiles: 1190 us, 127 TFLOP/s (2270 us).
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "gemm_small.h"
#include "kernels.h"

namespace elasto {
namespace {

struct P32 {
  const float* A;
  int64_t lda;
  const float* W;
  int64_t ldw;
  void* C;
  int64_t ldc;
  const float* bias;
  int64_t M;
  int N, K;
  const float* img;
  int img_size, patch, chans, grid, tokens;
  const float* cls;
  const float* pos;
  int64_t ldpos;
  int tiles_n;
};

constexpr int kBK32 = 32;            // K per step
constexpr int kLds32 = kBK32 + 4;    // floats per LDS row

// Values k .. k+3 of a row that starts at `row`.  VEC: the row and every k are
// 16-byte aligned.  WHOLE: all four lie below K (else those at and past K read
// as zeros, nothing past them is touched).
template <bool VEC, bool WHOLE>
__device__ __forceinline__ f32x4 load_k4(const float* row, int k, int K) {
  if constexpr (VEC && WHOLE) return *reinterpret_cast<const f32x4*>(row + k);
  f32x4 v;
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = WHOLE || k + e < K ? row[k + e] : 0.0f;
  return v;
}

// The same for the image patch of token row gm (zeros for a class row): value
// k is channel k / P^2, patch row (k / P) % P, patch column k % P.  VEC: P and
// the image rows are multiples of 4 values, so four values share a patch row.
template <bool VEC>
__device__ __forceinline__ f32x4 load_patch4(const P32& p, int64_t gm, int k) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  const int64_t bi = gm / p.tokens;
  const int t = (int)(gm - bi * p.tokens);
  if (t == 0) return v;
  const int n = t - 1, py = n / p.grid, px = n - py * p.grid, pp = p.patch * p.patch;
  auto at = [&](int kk) {
    const int c = kk / pp, rem = kk - c * pp, ii = rem / p.patch, jj = rem - ii * p.patch;
    return p.img + ((bi * p.chans + c) * p.img_size + py * p.patch + ii) * (int64_t)p.img_size +
           px * p.patch + jj;
  };
  if (VEC) {
    if (k < p.K) v = *reinterpret_cast<const f32x4*>(at(k));
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (k + e < p.K) v[e] = *at(k + e);
  }
  return v;
}

// The 16 outputs of a lane in one column (rows `row0` + 8*(e/4) + e%4) from
// their product sums.  Everything the epilogue reads is loaded before the
// first store (C may not alias the inputs, but the compiler cannot know).
template <Epi E>
__device__ __forceinline__ void store_column(const P32& p, int64_t row0, int col, float bias,
                                             const f32x16& acc) {
  if (col >= p.N) return;
  float* const c = static_cast<float*>(p.C) + col;
  const float cls = E == Epi::Patch ? p.cls[col] : 0.0f;
  float add[16], base[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    base[e] = bias;
    const int64_t row = std::min(row0 + 8 * (e >> 2) + (e & 3), p.M - 1);
    if constexpr (E == Epi::BiasResid) {
      add[e] = c[row * p.ldc];
    } else if constexpr (E == Epi::Patch) {
      const int t = (int)(row % p.tokens);
      add[e] = p.pos[(int64_t)t * p.ldpos + col];
      base[e] = t == 0 ? cls : bias;
    } else {
      add[e] = 0.0f;
    }
  }
#pragma unroll
  for (int e = 0; e < 16; ++e) {
    const int64_t row = row0 + 8 * (e >> 2) + (e & 3);
    if (row >= p.M) continue;
    const float v = acc[e];
    float r;
    if constexpr (E == Epi::Bias || E == Epi::BiasF32)
      r = v + base[e];
    else if constexpr (E == Epi::BiasGelu)
      r = gelu_erf(v + base[e]);
    else if constexpr (E == Epi::BiasResid)
      r = add[e] + (v + base[e]);
    else
      r = v + base[e] + add[e];
    c[row * p.ldc] = r;
  }
}

template <Epi E, int BM, int BN, bool VEC>
__global__ __launch_bounds__(256, 2) void gemm_f32_kernel(P32 p) {
  constexpr int TM = BM / 64, TN = BN / 64;            // 32x32 blocks per wave
  constexpr int LA = BM * kBK32 / 4 / 256, LW = BN * kBK32 / 4 / 256;
  constexpr int STAGE = (BM + BN) * kLds32;
  __shared__ __attribute__((aligned(16))) float smem[2 * STAGE];
  const int tid = threadIdx.x, lane = tid & 63, lr = lane & 31, lg = lane >> 5;
  const int wave = tid >> 6, wm = (wave >> 1) * (BM / 2), wn = (wave & 1) * (BN / 2);
  // Tiles, N innermost: workgroup i runs on XCD i % 8, so each XCD takes a
  // contiguous run of tiles and its L2 holds the A rows that they share.
  const unsigned q = gridDim.x >> 3, r8 = gridDim.x & 7, xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
  const unsigned tile = xcd < r8 ? xcd * (q + 1) + idx : r8 * (q + 1) + (xcd - r8) * q + idx;
  const int64_t m0 = (int64_t)(tile / (unsigned)p.tiles_n) * BM;
  const int n0 = (int)(tile % (unsigned)p.tiles_n) * BN;
  const int kc = (tid & 7) * 4, r0 = tid >> 3;  // this thread's chunk; rows r0 + 32 i
  const float* wrow[LW];
  const float* arow[LA];
#pragma unroll
  for (int i = 0; i < LA; ++i) arow[i] = p.A + std::min(m0 + r0 + 32 * i, p.M - 1) * p.lda;
#pragma unroll
  for (int i = 0; i < LW; ++i) wrow[i] = p.W + (int64_t)std::min(n0 + r0 + 32 * i, p.N - 1) * p.ldw;
  f32x4 ra[LA], rw[LW];
  // Step kt's values of this thread; only the last step can be ragged.
  auto load_step = [&](auto whole, int k) {
#pragma unroll
    for (int i = 0; i < LA; ++i) {
      if constexpr (E == Epi::Patch)
        ra[i] = load_patch4<VEC>(p, std::min(m0 + r0 + 32 * i, p.M - 1), k);
      else
        ra[i] = load_k4<VEC, decltype(whole)::value>(arow[i], k, p.K);
    }
#pragma unroll
    for (int i = 0; i < LW; ++i) rw[i] = load_k4<VEC, decltype(whole)::value>(wrow[i], k, p.K);
  };
  auto stash = [&](float* st) {
#pragma unroll
    for (int i = 0; i < LA; ++i) *reinterpret_cast<f32x4*>(st + (r0 + 32 * i) * kLds32 + kc) = ra[i];
#pragma unroll
    for (int i = 0; i < LW; ++i)
      *reinterpret_cast<f32x4*>(st + (BM + r0 + 32 * i) * kLds32 + kc) = rw[i];
  };
  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
  // Fragments of 8-value chunk kk of a stage, and their 4 * TM * TN MFMAs.
  auto frags = [&](const float* st, int kk, f32x4 (&fa)[TM], f32x4 (&fw)[TN]) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
      fa[i] = *reinterpret_cast<const f32x4*>(st + (wm + 32 * i + lr) * kLds32 + 8 * kk + 4 * lg);
#pragma unroll
    for (int j = 0; j < TN; ++j)
      fw[j] = *reinterpret_cast<const f32x4*>(st + (BM + wn + 32 * j + lr) * kLds32 + 8 * kk + 4 * lg);
  };
  auto product = [&](const f32x4 (&fa)[TM], const f32x4 (&fw)[TN]) {
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fa[i][r], fw[j][r], acc[i][j], 0, 0, 0);
  };
  // Step in stage st: each chunk's fragments are read while the chunk before
  // it is multiplied; `mid` (the next step's way to LDS) runs before the last
  // chunk's MFMAs, which then cover it.
  auto step = [&](const float* st, auto mid) {
    f32x4 fa[2][TM], fw[2][TN];
    frags(st, 0, fa[0], fw[0]);
#pragma unroll
    for (int kk = 0; kk < kBK32 / 8; ++kk) {
      __builtin_amdgcn_sched_barrier(0);
      if (kk + 1 < kBK32 / 8)
        frags(st, kk + 1, fa[(kk + 1) & 1], fw[(kk + 1) & 1]);
      else
        mid();
      __builtin_amdgcn_sched_barrier(0);
      product(fa[kk & 1], fw[kk & 1]);
    }
  };
  const int nwhole = p.K / kBK32;
  if (nwhole > 0) {
    load_step(std::true_type{}, kc);
    stash(smem);
  }
  for (int kt = 0; kt < nwhole; ++kt) {
    __syncthreads();
    const bool more = kt + 1 < nwhole;
    if (more) load_step(std::true_type{}, (kt + 1) * kBK32 + kc);
    step(smem + (kt & 1) * STAGE, [&] {
      if (more) stash(smem + ((kt + 1) & 1) * STAGE);
    });
  }
  if (p.K % kBK32 != 0) {  // ragged last step (the other stage: read two steps ago at the latest)
    load_step(std::false_type{}, nwhole * kBK32 + kc);
    float* st = smem + (nwhole & 1) * STAGE;
    stash(st);
    __syncthreads();
    step(st, [] {});
  }
  // acc[i][j][e]: row 8*(e/4) + 4*(lane/32) + e%4 of block i, column lane%32
  // of block j.
  float bias[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) bias[j] = p.bias[std::min(n0 + wn + 32 * j + lr, p.N - 1)];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
      store_column<E>(p, m0 + wm + 32 * i + 4 * lg, n0 + wn + 32 * j + lr, bias[j], acc[i][j]);
}

// GEMM for launches of few tiles (gemm_small.h): 16-byte aligned rows.
template <Epi E, int TMB, int TNB>
__global__ __launch_bounds__(256) void gemm_f32_small(P32 p) {
  using T = SmallTile<float, TMB, TNB, 4, 3>;
  __shared__ __attribute__((aligned(1024))) char smem[T::SMEM];
  int tm, tn;
  small_tile_of((p.M + T::R - 1) / T::R, &tm, &tn);
  const int64_t m0 = (int64_t)tm * T::R;
  const int n0 = tn * T::CN;
  T::run(
      smem, p.K,
      [&](int i, int r) {
        return i < T::ABLK ? p.A + std::min(m0 + r, p.M - 1) * p.lda
                           : p.W + (int64_t)std::min(n0 + r, p.N - 1) * p.ldw;
      },
      [](int, int k) { return k; },
      [&](int, const float* q, int k) {
        return __builtin_bit_cast(u32x4, k + 4 <= p.K ? load_k4<true, true>(q, 0, 4)
                                                      : load_k4<false, false>(q, 0, p.K - k));
      },
      [] {});
  constexpr int CPR = T::CN / 8;
  for (int c = threadIdx.x; c < T::R * CPR; c += 256) {
    const int rl = c / CPR, cl = (c - rl * CPR) * 8;
    const int64_t row = m0 + rl;
    if (row >= p.M) continue;
    float v[8], add[8], bias[8];
    T::sum8(smem, rl, cl, v);
    float* const out = static_cast<float*>(p.C) + row * p.ldc + n0 + cl;
    const int left = p.N - (n0 + cl);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      bias[e] = e < left ? p.bias[n0 + cl + e] : 0.0f;
      add[e] = E == Epi::BiasResid && e < left ? out[e] : 0.0f;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (e >= left) break;
      const float z = v[e] + bias[e];
      out[e] = E == Epi::BiasGelu ? gelu_erf(z) : E == Epi::BiasResid ? add[e] + z : z;
    }
  }
}

template <Epi E, int TMB, int TNB>
hipError_t launch_small(const P32& p, hipStream_t s) {
  const int64_t blocks = (p.M + 16 * TMB - 1) / (16 * TMB) * ((p.N + 16 * TNB - 1) / (16 * TNB));
  hipLaunchKernelGGL((gemm_f32_small<E, TMB, TNB>), dim3((unsigned)blocks), dim3(256), 0, s, p);
  return hipGetLastError();
}

template <Epi E, int BM, int BN, bool VEC>
hipError_t launch_tile(P32 p, hipStream_t s) {
  p.tiles_n = (p.N + BN - 1) / BN;
  const int64_t tiles = (p.M + BM - 1) / BM * p.tiles_n;
  if (tiles > INT32_MAX) return hipErrorInvalidValue;
  hipLaunchKernelGGL((gemm_f32_kernel<E, BM, BN, VEC>), dim3((unsigned)tiles), dim3(256), 0, s, p);
  return hipGetLastError();
}

template <Epi E, bool VEC>
hipError_t launch(const P32& p, hipStream_t s) {
  // Tile shape by the work of the busiest CU (its tiles x a tile's area), the
  // larger where they are equal: 8000 x 3072 x 3072 takes 1180 us with 128x128
  // tiles and 1224 with 64x64, 6304 x 1536 x 384 107 and 79 us, 6304 x 384 x
  // 384 34 and 25 us.
  if constexpr (VEC && E != Epi::Patch) {
    constexpr SmallShape kSmall[] = {{1, 1}, {1, 2}, {2, 2}};
    switch (small_pick(kSmall, p.M, p.N)) {
      case 0: return launch_small<E, 1, 1>(p, s);
      case 1: return launch_small<E, 1, 2>(p, s);
      case 2: return launch_small<E, 2, 2>(p, s);
    }
  }
  constexpr int64_t kCUs = 256;
  auto load = [&](int bm, int bn) {
    const int64_t t = (p.M + bm - 1) / bm * ((p.N + bn - 1) / bn);
    return (t + kCUs - 1) / kCUs * (int64_t)(bm * bn);
  };
  if (load(128, 128) <= load(64, 64)) return launch_tile<E, 128, 128, VEC>(p, s);
  return launch_tile<E, 64, 64, VEC>(p, s);
}

}  // namespace

hipError_t launch_gemm_f32(Epi epi, const GemmArgs& a, hipStream_t s) {
  if (a.M <= 0 || a.N <= 0) return hipSuccess;
  P32 p{};
  p.A = static_cast<const float*>(a.A);
  p.lda = a.lda;
  p.W = static_cast<const float*>(a.W);
  p.ldw = a.ldw;
  p.C = a.C;
  p.ldc = a.ldc;
  p.bias = a.bias;
  p.M = a.M;
  p.N = a.N;
  p.K = a.K;
  p.img = static_cast<const float*>(a.img);
  p.img_size = a.img_size;
  p.patch = a.patch;
  p.chans = a.chans;
  p.grid = a.grid;
  p.tokens = a.tokens;
  p.cls = a.cls;
  p.pos = a.pos;
  p.ldpos = a.ldpos > 0 ? a.ldpos : a.N;
  // 16-byte loads: aligned rows of both operands (patches: of the images).
  auto al = [](const void* q) { return reinterpret_cast<uintptr_t>(q) % 16 == 0; };
  const bool vec = al(p.W) && p.ldw % 4 == 0 &&
                   (epi == Epi::Patch ? al(p.img) && p.patch % 4 == 0 && p.img_size % 4 == 0
                                      : al(p.A) && p.lda % 4 == 0);
#define ELASTO_F32(E) return vec ? launch<E, true>(p, s) : launch<E, false>(p, s)
  switch (epi) {
    case Epi::Bias: ELASTO_F32(Epi::Bias);
    case Epi::BiasGelu: ELASTO_F32(Epi::BiasGelu);
    case Epi::BiasResid: ELASTO_F32(Epi::BiasResid);
    case Epi::BiasF32: ELASTO_F32(Epi::BiasF32);
    case Epi::Patch: ELASTO_F32(Epi::Patch);
    case Epi::GeluBwd: break;
  }
#undef ELASTO_F32
  return hipErrorInvalidValue;
}

}  // namespace elasto
