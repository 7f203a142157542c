// A span of F (a run of whole blocks, starting at any element) between memory and a wave's own LDS region, in aligned
// 16-byte pieces.  The region holds the span at the phase (address modulo 16) it has in memory.
#pragma once

#include "pbz_device.h"

namespace pbz {

__device__ __forceinline__ int phase_of(const void* p) { return int(reinterpret_cast<uintptr_t>(p) & 15u); }

typedef uint32_t raw16 __attribute__((ext_vector_type(4)));   // not uint4: an array of that struct in flight stayed in
                                                              // scratch memory (five operations on 512^3 values, 4x4x4, three
                                                              // tenths kept: 295 us, 281 so)

// [p, p + len) -> LDS, at the phase of p.  Only 16-byte pieces that lie inside the operand [lo, hi) are read as such
// (they may hold bytes of neighbouring blocks, which nobody uses); the bytes of the others are read one by one.
// kBatch: 16-byte loads in flight per lane.
template <int kBatch>
__device__ __forceinline__ void stage_span(const uint8_t* lo, const uint8_t* hi, const uint8_t* p, int len, uint8_t* lds) {
  const int lane = threadIdx.x & 63;
  const int a = phase_of(p);
  const uint8_t* base = p - a;
  const int pieces = (a + len + 15) >> 4;
  const int first = base < lo ? 1 : 0;
  const int last = base + 16 * int64_t(pieces) > hi ? pieces - 1 : pieces;
  for (int i0 = first; i0 < last; i0 += 64 * kBatch) {
    raw16 v[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = i0 + u * 64 + lane;
      v[u] = reinterpret_cast<const raw16*>(base)[i < last ? i : last - 1];
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int i = i0 + u * 64 + lane;
      if (i < last) reinterpret_cast<raw16*>(lds)[i] = v[u];
    }
  }
  if (first != 0 && lane < 16 - a && lane < len) lds[a + lane] = p[lane];
  if (last < pieces) {
    const int i = 16 * last + lane;
    if (lane < 16 && i >= a && i < a + len) lds[i] = base[i];
  }
}

// The same copy, requested only: the pieces go from memory to LDS past the registers (64 lanes' pieces are consecutive there, too).
// span_arrived() waits for them.  `lds`: the same in every lane.
__device__ __forceinline__ void request_span(const uint8_t* lo, const uint8_t* hi, const uint8_t* p, int len, uint8_t* lds) {
  const int lane = threadIdx.x & 63;
  const int a = phase_of(p);
  const uint8_t* base = p - a;
  const int pieces = (a + len + 15) >> 4;
  const int first = base < lo ? 1 : 0;
  const int last = base + 16 * int64_t(pieces) > hi ? pieces - 1 : pieces;
  // what the wave still has to read or write in the region comes first: these writes do not queue with its LDS operations
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  for (int i0 = 0; i0 < last; i0 += 64) {
    const int i = i0 + lane;
    if (i >= first && i < last)
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(base + 16 * i),
                                       (__attribute__((address_space(3))) void*)(lds + 16 * i0), 16, 0, 0);
  }
  if (first != 0 && lane < 16 - a && lane < len) lds[a + lane] = p[lane];
  if (last < pieces) {
    const int i = 16 * last + lane;
    if (lane < 16 && i >= a && i < a + len) lds[i] = base[i];
  }
}
__device__ __forceinline__ void span_arrived() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  wave_lds_sync();
}

// LDS -> [p, p + len), from the phase of p; nothing outside is written
__device__ __forceinline__ void unstage_span(const uint8_t* lds, uint8_t* p, int len) {
  const int lane = threadIdx.x & 63;
  const int a = phase_of(p);
  uint8_t* base = p - a;
  const int first = a != 0 ? 1 : 0, last = (a + len) >> 4;
  for (int i = first + lane; i < last; i += 64) reinterpret_cast<uint4*>(base)[i] = reinterpret_cast<const uint4*>(lds)[i];
  if (a != 0) {
    const int i = a + lane;
    if (i < 16 && i < a + len) base[i] = lds[i];
  }
  const int i = 16 * last + lane;
  if (i >= a && i < a + len) base[i] = lds[i];
}

}  // namespace pbz
