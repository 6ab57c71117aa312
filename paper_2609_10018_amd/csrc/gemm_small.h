// Product core of the GEMM kernels for launches of few tiles (small M: one
// image is 197 rows), where a workgroup's K chain is the critical path: in the
// tiled kernels every step costs about a memory latency (~0.7-1 us) of a chip
// that is mostly idle.  A workgroup takes a (16 TMB) x (16 TNB) output tile
// and its WK waves share out the K steps (one 128-byte line of a row: 64 bf16
// or 32 fp32 values).  Each wave brings its own steps to its own LDS ring, D
// steps in flight, and multiplies them with no barrier before the end, where
// the caller sums the waves' fp32 partial tiles in wave order: a row's result
// depends on K and WK alone, not on the tile shape.
//
// The direct loads move 8 rows x 128 bytes per wave instruction with a row's
// lanes adjacent.  What matters is that neighbouring lanes read neighbouring
// addresses: with the MFMA's own lane order (16 rows in 16 neighbouring lanes,
// straight to registers) a CU got 40 GB/s from L2, with this one 115, and a
// step costs a wave no register.
#pragma once

#include "common.h"

namespace elasto {

typedef __attribute__((address_space(3))) void small_lds_void;
typedef __attribute__((address_space(1))) void small_global_void;

template <typename S, int TMB, int TNB, int WK, int D>
struct SmallTile {
  static constexpr bool BF = sizeof(S) == 2;
  static constexpr int R = 16 * TMB, CN = 16 * TNB;  // output tile
  static constexpr int EPC = 16 / sizeof(S);         // elements per 16-byte chunk
  static constexpr int STEP = 128 / sizeof(S);       // K per step
  static constexpr int ABLK = 2 * TMB, PL = 2 * (TMB + TNB);  // 1-KB blocks (8 rows) of a step
  static constexpr int RING = D * PL * 1024, SS = CN + 4;
  static constexpr int SMEM = WK * RING;
  static_assert(R * SS * 4 <= RING && D <= 3 && D * PL < 64, "ring");

  // Chunk c of row r sits at c ^ swz(r) in its row.
  static __device__ __forceinline__ int swz(int r) { return (r ^ (r >> 3)) & 7; }

  // Wait until at most N vector-memory operations of this wave are in flight
  // and every LDS operation has completed.
  template <int N>
  static __device__ __forceinline__ void wait_vm() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4));
    asm volatile("" ::: "memory");
  }
  static __device__ __forceinline__ void wait_lds() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xF | (0x7 << 4) | (0x3 << 14));
    asm volatile("" ::: "memory");
  }

  // Elements [k, kend) of the chunk that starts at k (at and past kend: 0).
  static __device__ __forceinline__ u32x4 masked(u32x4 v, int k, int kend) {
    u32x4 o;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      if constexpr (BF) {
        const uint32_t lo = k + 2 * w < kend ? 0x0000ffffu : 0u;
        const uint32_t hi = k + 2 * w + 1 < kend ? 0xffff0000u : 0u;
        o[w] = v[w] & (lo | hi);
      } else {
        o[w] = k + w < kend ? v[w] : 0u;
      }
    }
    return o;
  }

  // Leaves wave w's partial tile at part(smem, w) ([R][SS] floats), all waves
  // past the barrier.  row(i, r): source row of tile row r (loads i < ABLK: A,
  // else W); koff(i, k): element offset of k there.  A ragged last step goes
  // through registers, masked in both operands; tail(i, ptr, k) reads its chunk
  // at k < K (K - k elements may exist past ptr).  mid() runs once the first
  // loads are in flight.
  template <class Row, class Koff, class Tail, class Mid>
  static __device__ __forceinline__ void run(char* smem, int K, Row row, Koff koff, Tail tail,
                                             Mid mid) {
    const int lane = threadIdx.x & 63, li = lane & 15, lg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    char* const ring = smem + wave * RING;
    const int prow = lane >> 3, pc = lane & 7;
    const S* src[PL];
    int chunk[PL];
#pragma unroll
    for (int i = 0; i < PL; ++i) {
      const int r = (i < ABLK ? i : i - ABLK) * 8 + prow;
      chunk[i] = (pc ^ swz(r)) * EPC;
      src[i] = row(i, r);
    }
    // This wave's steps [s0, s1); a ragged last step is kept apart.
    const int ns = (K + STEP - 1) / STEP, per = (ns + WK - 1) / WK;
    const int s0 = min(wave * per, ns), s1 = min(s0 + per, ns);
    const bool ragged = K % STEP != 0 && s0 < s1 && s1 == ns;
    const int cnt = s1 - s0 - (ragged ? 1 : 0);
    auto issue = [&](int slot, int s) {
#pragma unroll
      for (int i = 0; i < PL; ++i)
        __builtin_amdgcn_global_load_lds(
            (small_global_void*)(src[i] + koff(i, s * STEP + chunk[i])),
            (small_lds_void*)(ring + (slot * PL + i) * 1024), 16, 0, 0);
    };
#pragma unroll
    for (int u = 0; u < D; ++u)
      if (u < cnt) issue(u, s0 + u);
    mid();
    f32x4 acc[TMB][TNB];
#pragma unroll
    for (int i = 0; i < TMB; ++i)
#pragma unroll
      for (int j = 0; j < TNB; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // The step in `slot`: lane l holds chunks lg and lg + 4 of row l%16 of a
    // 16-row block (k-slots are labels, the same for both operands).  D = W
    // A^T, so that a lane ends up with 4 consecutive columns of row l%16.
    auto step = [&](int slot, auto release) {
      const char* st = ring + slot * PL * 1024;
      u32x4 fa[TMB][2], fw[TNB][2];
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int i = 0; i < TMB; ++i) {
          const int r = 16 * i + li;
          fa[i][h] = *reinterpret_cast<const u32x4*>(st + r * 128 + (((lg + 4 * h) ^ swz(r)) << 4));
        }
#pragma unroll
        for (int j = 0; j < TNB; ++j) {
          const int r = 16 * j + li;
          fw[j][h] = *reinterpret_cast<const u32x4*>(st + (R + r) * 128 +
                                                     (((lg + 4 * h) ^ swz(r)) << 4));
        }
      }
      release();
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        if constexpr (BF) {
#pragma unroll
          for (int i = 0; i < TMB; ++i)
#pragma unroll
            for (int j = 0; j < TNB; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                  __builtin_bit_cast(bf16x8, fw[j][h]), __builtin_bit_cast(bf16x8, fa[i][h]),
                  acc[i][j], 0, 0, 0);
        } else {
#pragma unroll
          for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int i = 0; i < TMB; ++i)
#pragma unroll
              for (int j = 0; j < TNB; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(
                    __uint_as_float(fw[j][h][r]), __uint_as_float(fa[i][h][r]), acc[i][j], 0, 0, 0);
        }
      }
    };
    int slot = 0;
    for (int c = 0; c < cnt; ++c) {
      // This step's loads have landed when no more than the later steps' are in flight.
      const int ahead = min(D - 1, cnt - 1 - c);
      if (ahead >= 2) wait_vm<2 * PL>();
      else if (ahead == 1) wait_vm<PL>();
      else wait_vm<0>();
      step(slot, [&] {
        if (c + D < cnt) {  // the slot's values are in registers: refill it
          wait_lds();
          issue(slot, s0 + c + D);
        }
      });
      slot = slot + 1 == D ? 0 : slot + 1;
    }
    if (ragged) {  // slot 0 (every load of this wave has been waited for and read)
      u32x4 v[PL];
#pragma unroll
      for (int i = 0; i < PL; ++i) {
        const int k = (ns - 1) * STEP + chunk[i], kk = k < K ? k : 0;
        v[i] = masked(tail(i, src[i] + koff(i, kk), kk), k, K);
      }
      wait_lds();
#pragma unroll
      for (int i = 0; i < PL; ++i) *reinterpret_cast<u32x4*>(ring + i * 1024 + lane * 16) = v[i];
      wait_lds();
      step(0, [] {});
    }
    wait_lds();  // the partial tile goes over the wave's own ring
    float* const out = part(smem, wave);
#pragma unroll
    for (int i = 0; i < TMB; ++i)
#pragma unroll
      for (int j = 0; j < TNB; ++j)
        *reinterpret_cast<f32x4*>(out + (16 * i + li) * SS + 16 * j + 4 * lg) = acc[i][j];
    __syncthreads();
  }
  static __device__ __forceinline__ float* part(char* smem, int wave) {
    return reinterpret_cast<float*>(smem + wave * RING);
  }
  // Sum over the waves of columns cl .. cl + 7 of tile row rl.
  static __device__ __forceinline__ void sum8(char* smem, int rl, int cl, float (&v)[8]) {
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = 0.0f;
#pragma unroll
    for (int w = 0; w < WK; ++w) {
      const float* pw = part(smem, w) + rl * SS + cl;
      const f32x4 lo = *reinterpret_cast<const f32x4*>(pw);
      const f32x4 hi = *reinterpret_cast<const f32x4*>(pw + 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        v[e] += lo[e];
        v[4 + e] += hi[e];
      }
    }
  }
};

// Tile of workgroup blockIdx.x: row tiles innermost, a contiguous run of tiles
// per XCD (workgroup i runs on XCD i % 8), so that the tiles that share W
// columns share an L2.
__device__ __forceinline__ void small_tile_of(int64_t tiles_m, int* tm, int* tn) {
  const unsigned nblk = gridDim.x, b = blockIdx.x;
  const unsigned q = nblk >> 3, r8 = nblk & 7, xcd = b & 7, idx = b >> 3;
  const unsigned logical = (xcd < r8) ? xcd * (q + 1) + idx : r8 * (q + 1) + (xcd - r8) * q + idx;
  *tn = (int)(logical / (unsigned)tiles_m);
  *tm = (int)(logical - (unsigned)*tn * (unsigned)tiles_m);
}

// The smallest tile of the given list whose workgroups all run at once, one
// per CU (index into the list, -1: none).  With one round a workgroup's stream
// of operands sets the time, and the smallest tile has the shortest; a second
// round loses to the tiled kernels' better reuse (197 x 1152 x 768: 16x32 tiles
// 4.2, 32x32 3.85, 32x64 4.8, 64x64 6.5 us, tiled 11.6; 788 x 1152 x 768: 32x64
// in two rounds 8.4, 64x64 in one 6.9, tiled 12.0; 1576 x 1536 x 768: 64x64 in
// three 17.3, tiled 12.8).
struct SmallShape {
  int tmb, tnb;
};
template <int N>
inline int small_pick(const SmallShape (&list)[N], int64_t M, int64_t Ncols) {
  for (int i = 0; i < N; ++i) {
    const int64_t r = 16 * list[i].tmb, c = 16 * list[i].tnb;
    if ((M + r - 1) / r * ((Ncols + c - 1) / c) <= 256) return i;
  }
  return -1;
}

}  // namespace elasto
