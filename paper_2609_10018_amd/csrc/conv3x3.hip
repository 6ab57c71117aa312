// 3x3 convolution, stride 1, padding 1 (a bottleneck's middle layer), NHWC
// bf16, with bias and ReLU: MFMA over K = (32 channels, kernel row, kernel
// column), the input patch resident in LDS.
//
// In flat pixel order (image, row, column) tap (ti, tj) of output pixel m reads
// input pixel m + (ti - 1) W + (tj - 1), so the patch of BM consecutive output
// pixels is the BM + 2 W + 2 pixels around them, whatever rows or images the
// tile crosses: a workgroup loads it once per 32 channels and the nine taps read
// it at nine row offsets.  A tap outside the image reads a row of zeros
// instead (resolved to an LDS offset per tap and pixel before the K loop, which
// holds no address arithmetic beyond the buffer's).
//
// As an implicit GEMM with 64 channels a step, each tap brought the pixels
// again from L2, with a test and a select per load, K was padded to 64
// channels a tap (88: 72 MFMA steps instead of 54) and N to 128.  Bound now by
// MFMA and LDS reads together (MFMA busy 57% of the cycles at 256 x 14x14 x
// 256).  In us, before and after: 64 x 28x28 x 88: 31.7 and 15.2; 256 x 56x56 x
// 64: 125 and 82; 256 x 28x28 x 128: 124 and 66.5; 256 x 7x7 x 512: 91 and
// 62.5; 8 x 14x14 x 256: 27.9 and 11.1.
//
// K runs in the same order in every tile, so a result's bits do not depend on
// the tile chosen.
#include "common.h"
#include "kernels.h"
#include "lds_load.h"

#include <algorithm>

namespace elasto {
namespace {

constexpr int kThreads = 256;
constexpr int kCB = 32;          // channels per block of K
constexpr int kRow = kCB * 2;    // bytes of an LDS row: one pixel or one filter tap
constexpr int kLoadRows = kThreads * 16 / kRow;  // rows one load instruction of all waves brings

struct C3Params {
  const uint16_t* x;
  const uint16_t* w;
  uint16_t* out;
  const float* bias;
  int64_t ldc;
  int M, N, H, W, Cs, Ca, ldw, wseg;
  int x_bytes, w_bytes, tiles_n, relu;
};

// 16-byte chunk c of row r lies at slot c ^ ((r >> 2) & 3), so that the rows
// 0-3, 12-15, 20-23, 24-27 (from any first row) that a 16-byte read takes in one
// pass cover all banks (with r >> 1 the layers above took up to 6% longer).
__device__ __forceinline__ int slot_of(int r, int c) { return (c ^ (r >> 2)) & 3; }

// WM x WN = 4 waves.  AP: patch loads per thread, BM / 64 + 1 for W <= 31,
// BM / 64 + 2 for W <= 63.
template <int BM, int BN, int WM, int WN, int AP>
__global__ __launch_bounds__(kThreads, 2) void conv3x3_kernel(C3Params p) {
  static_assert(WM * WN == 4, "four waves");
  constexpr int WTM = BM / WM, WTN = BN / WN, TM = WTM / 32, TN = WTN / 32;
  constexpr int ABUF = AP * kThreads * 16 + kRow;  // a patch and a row of zeros
  constexpr int WSLOTS = 3 * BN * 4, WBUF = WSLOTS * 16, WP = (WSLOTS + kThreads - 1) / kThreads;
  constexpr int ES = WTN * 2 + 16;  // bytes of a staged output row
  constexpr int MAIN = 2 * ABUF + 2 * WBUF, EPI = 4 * WTM * ES;
  __shared__ __attribute__((aligned(1024))) char smem[MAIN > EPI ? MAIN : EPI];
  char* const wbuf = smem + 2 * ABUF;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN, lr = lane & 31, lg = lane >> 5;

  // Workgroup i runs on XCD i % 8: each XCD takes a run of tiles, the N tiles
  // of a row panel next to each other, so they share the panel in its L2.
  const int nblk = gridDim.x, b = blockIdx.x;
  const int q = nblk >> 3, r8 = nblk & 7, xcd = b & 7, idx = b >> 3;
  const int logical = (xcd < r8) ? xcd * (q + 1) + idx : r8 * (q + 1) + (xcd - r8) * q + idx;
  const int tile_m = logical / p.tiles_n, tile_n = logical - tile_m * p.tiles_n;
  const int m0 = tile_m * BM, n0 = tile_n * BN;

  const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(p.x), (short)0, p.x_bytes, kRsrcWord3);
  const __amdgpu_buffer_rsrc_t rs_w = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint16_t*>(p.w), (short)0, p.w_bytes, kRsrcWord3);

  // Load i brings patch row (or filter row) i * kLoadRows + tid / 4; the
  // thread's chunk of it is the same for every i.
  const int chunk = slot_of(tid >> 2, tid & 3);
  unsigned aoff[AP], woff[WP];
#pragma unroll
  for (int i = 0; i < AP; ++i) {
    const int r = i * kLoadRows + (tid >> 2), px = m0 - p.W - 1 + r;
    const bool ok = r < BM + 2 * p.W + 2 && (unsigned)px < (unsigned)p.M;
    aoff[i] = ok ? (unsigned)px * (unsigned)(p.Cs * 2) + chunk * 16 : kOutOfRange;
  }
#pragma unroll
  for (int i = 0; i < WP; ++i) {
    const int r = i * kLoadRows + (tid >> 2), tj = r / BN, n = n0 + r - tj * BN;
    woff[i] = n < p.N ? ((unsigned)n * (unsigned)p.ldw + (unsigned)(tj * p.wseg)) * 2u + chunk * 16
                      : kOutOfRange;
  }
  auto issue_a = [&](int cb) {
    const bool ok = cb * kCB + chunk * 8 < p.Ca;
    char* base = smem + (cb & 1) * ABUF + wave * 1024;
#pragma unroll
    for (int i = 0; i < AP; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_x, (lds_void*)(base + i * kThreads * 16), 16,
                                               ok ? (unsigned)(aoff[i] + cb * kRow) : kOutOfRange, 0, 0, 0);
  };
  auto issue_w = [&](int cb, int ti) {
    const bool ok = cb * kCB + chunk * 8 < p.Ca;
    const unsigned step = (unsigned)(ti * 3 * p.wseg) * 2u + cb * kRow;
    char* base = wbuf + ((cb + ti) & 1) * WBUF + wave * 1024;
#pragma unroll
    for (int i = 0; i < WP; ++i)
      if ((i + 1) * kThreads <= WSLOTS || i * kThreads + wave * 64 < WSLOTS)  // whole waves
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs_w, (lds_void*)(base + i * kThreads * 16), 16,
                                                 ok ? (unsigned)(woff[i] + step) : kOutOfRange, 0, 0, 0);
  };
  issue_a(0);
  issue_w(0, 0);
  if (tid < 8)
    *reinterpret_cast<u32x4*>(smem + (tid >> 2) * ABUF + AP * kThreads * 16 + (tid & 3) * 16) =
        u32x4{0u, 0u, 0u, 0u};

  // LDS offset of this lane's fragment of tap t, row block i (first half of
  // the 32 channels; the second half is at the offset ^ 32).
  int ar[TM][9];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int rl = wm * WTM + i * 32 + lr, m = m0 + rl;
    const int hw = p.H * p.W, rem = m - m / hw * hw, oh = rem / p.W, ow = rem - oh * p.W;
#pragma unroll
    for (int t = 0; t < 9; ++t) {
      const int ti = t / 3, tj = t - ti * 3, r = rl + ti * p.W + tj;
      const bool in = (unsigned)(oh + ti - 1) < (unsigned)p.H &&
                      (unsigned)(ow + tj - 1) < (unsigned)p.W;
      ar[i][t] = in ? r * kRow + slot_of(r, lg) * 16 : AP * kThreads * 16 + lg * 16;
    }
  }
  int wr[2];
  wr[0] = (wn * WTN + lr) * kRow + slot_of(lr, lg) * 16;
  wr[1] = wr[0] ^ 32;

  f32x16 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;

  const int ncb = (p.Ca + kCB - 1) / kCB;
  for (int cb = 0; cb < ncb; ++cb) {
    const bool half = p.Ca - cb * kCB <= 16;  // the last block's second half is empty
    const char* abuf = smem + (cb & 1) * ABUF;
#pragma unroll
    for (int ti = 0; ti < 3; ++ti) {
      // The step's filters have landed, and before a block's first step its
      // patch; the next patch, issued after the second step's filters, may
      // stay in flight over that step.
      if (ti == 1 && cb + 1 < ncb) wait_vm_lds<AP>();
      else wait_vm_lds<0>();
      __builtin_amdgcn_s_barrier();
      if (ti < 2) issue_w(cb, ti + 1);
      else if (cb + 1 < ncb) issue_w(cb + 1, 0);
      if (ti == 0 && cb + 1 < ncb) issue_a(cb + 1);
      const char* wb = wbuf + ((cb + ti) & 1) * WBUF;
#pragma unroll
      for (int tj = 0; tj < 3; ++tj) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          if (k == 1 && half) continue;
          bf16x8 af[TM], wf[TN];
#pragma unroll
          for (int i = 0; i < TM; ++i)
            af[i] = *reinterpret_cast<const bf16x8*>(abuf + (ar[i][ti * 3 + tj] ^ (k * 32)));
#pragma unroll
          for (int j = 0; j < TN; ++j)
            wf[j] = *reinterpret_cast<const bf16x8*>(wb + wr[k] + (tj * BN + j * 32) * kRow);
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[j], af[i], acc[i][j], 0, 0, 0);
        }
      }
    }
  }

  // Epilogue: D = W A^T, so lane l holds pixel l % 32 and channels
  // 8 (e / 4) + 4 (l / 32) + e % 4; each wave turns its block in LDS into rows
  // of 16-byte chunks.
  wait_lds();  // every wave has read the last step's fragments
  __builtin_amdgcn_s_barrier();
  char* const stg = smem + wave * (WTM * ES);
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int nl = j * 32 + 8 * g + 4 * lg, col = n0 + wn * WTN + nl;
      f32x4 bz = {0.f, 0.f, 0.f, 0.f};
      if (p.bias != nullptr && col < p.N) bz = *reinterpret_cast<const f32x4*>(p.bias + col);
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[e] = acc[i][j][4 * g + e] + bz[e];
          if (p.relu) v[e] = fmaxf(v[e], 0.0f);
        }
        *reinterpret_cast<u32x2*>(stg + (i * 32 + lr) * ES + nl * 2) =
            u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
      }
    }
  __syncthreads();
  constexpr int CH = WTN / 8;
#pragma unroll
  for (int it = 0; it < WTM * CH / 64; ++it) {
    const int id = it * 64 + lane, row = id / CH, c = id - row * CH;
    const int m = m0 + wm * WTM + row, col = n0 + wn * WTN + c * 8;
    if (m < p.M && col < p.N)
      *reinterpret_cast<u32x4*>(p.out + (int64_t)m * p.ldc + col) =
          *reinterpret_cast<const u32x4*>(stg + row * ES + c * 16);
  }
}

// Tiles for W > 31 too: not 256x96, which would be alone on its CU (162 against
// 82 us for 256 x 56x56 x 64).
template <int BM, int BN>
constexpr bool kWideTile = !(BM == 256 && BN == 96);

template <int BM, int BN, int WM, int WN>
hipError_t launch_tile(C3Params p, hipStream_t s) {
  p.tiles_n = (p.N + BN - 1) / BN;
  const int64_t tiles = (int64_t)((p.M + BM - 1) / BM) * p.tiles_n;
  if (tiles > INT32_MAX) return hipErrorInvalidValue;
  if (p.W <= 31) {
    hipLaunchKernelGGL((conv3x3_kernel<BM, BN, WM, WN, BM / 64 + 1>), dim3((unsigned)tiles),
                       dim3(kThreads), 0, s, p);
  } else {
    if constexpr (kWideTile<BM, BN>)
      hipLaunchKernelGGL((conv3x3_kernel<BM, BN, WM, WN, BM / 64 + 2>), dim3((unsigned)tiles),
                         dim3(kThreads), 0, s, p);
    else
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

bool conv3x3_applies(const ConvArgs& a) {
  return a.KH == 3 && a.KW == 3 && a.stride == 1 && a.pad == 1 && a.row_window == 0 &&
         a.W <= 63 && a.N % 8 == 0;
}

hipError_t launch_conv3x3(const ConvArgs& a, const void* x, int images, int64_t w_bytes, void* out,
                          hipStream_t s) {
  C3Params p{};
  p.x = static_cast<const uint16_t*>(x);
  p.w = static_cast<const uint16_t*>(a.weight);
  p.out = static_cast<uint16_t*>(out);
  p.bias = a.bias;
  p.ldc = a.ldc;
  p.M = images * a.H * a.W;
  p.N = a.N;
  p.H = a.H;
  p.W = a.W;
  p.Cs = a.Cs;
  p.Ca = a.Ca;
  p.ldw = (int)a.ldw;
  p.wseg = (int)a.wseg;
  p.x_bytes = (int)((int64_t)p.M * a.Cs * 2);
  p.w_bytes = (int)w_bytes;
  p.relu = a.relu ? 1 : 0;
  // Estimated time of each tile: what a CU's share of the tiles takes, with the
  // steps (32 channels x a kernel row) of one tile alone on its CU, or of a tile
  // among two or more that share it, and the tile's patch load and epilogue,
  // in microseconds, fitted to 22 layers of 1 to 256 images (7x7 to 56x56, 16
  // to 512 channels); the choice is within 9% of the best tile on all of them.
  // 96 outputs a wave spend a quarter less time on 88 than two tiles of 64 do
  // (64 x 28x28, 88 channels: 15.2 and 17.1 us), and lose where N fills 64s.
  constexpr struct { int bm, bn; double alone, shared, edge; } kTiles[] = {
      {256, 64, 0.84, 0.63, 2.6}, {256, 96, 1.15, 1.02, 2.8}, {128, 64, 0.54, 0.37, 1.4},
      {128, 96, 0.65, 0.55, 2.0}, {64, 64, 0.36, 0.26, 0.7}};
  constexpr int kCUs = 256;
  const int steps = 3 * ((p.Ca + kCB - 1) / kCB);
  int best = 0;
  double best_t = 1e300;
  for (int i = 0; i < 5; ++i) {
    const auto& c = kTiles[i];
    if (p.W > 31 && i == 1) continue;  // kWideTile
    const int64_t tiles = (int64_t)((p.M + c.bm - 1) / c.bm) * ((p.N + c.bn - 1) / c.bn);
    const double each = (double)((tiles + kCUs - 1) / kCUs);
    const double t = steps * (each < 2 ? c.alone : each * c.shared) + each * c.edge;
    if (t < best_t) { best_t = t; best = i; }
  }
  switch (best) {
    case 0: return launch_tile<256, 64, 4, 1>(p, s);
    case 1: return launch_tile<256, 96, 4, 1>(p, s);
    case 2: return launch_tile<128, 64, 2, 2>(p, s);
    case 3: return launch_tile<128, 96, 4, 1>(p, s);
    default: return launch_tile<64, 64, 2, 2>(p, s);
  }
}

}  // namespace elasto
