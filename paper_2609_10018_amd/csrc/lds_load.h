// Direct loads to LDS and the waits that go with them.
#pragma once

#include "common.h"

namespace elasto {

typedef __attribute__((address_space(3))) void lds_void;

// Buffer descriptor word 3 for raw (unswizzled, stride 0) buffers on CDNA.
constexpr int kRsrcWord3 = 0x00020000;
constexpr unsigned kOutOfRange = 0x80000000u;  // at or past every buffer's size

// Wait until at most N vector-memory operations of this wave are in flight
// and every LDS operation has completed.
template <int N>
__device__ __forceinline__ void wait_vm_lds() {
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4));
}

// Wait until every LDS operation of this wave has completed (vector memory
// operations may still be in flight).
__device__ __forceinline__ void wait_lds() {
  __builtin_amdgcn_s_waitcnt(0xF | (0x7 << 4) | (0x0 << 8) | (0x3 << 14));
}

}  // namespace elasto
