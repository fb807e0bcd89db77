// Device code shared by the bf16 attention kernels.
#pragma once
#include "qcf_device.h"

namespace qcf {

constexpr uint32_t kOob = 0x80000000u;  // a buffer offset past every descriptor's range

__device__ __forceinline__ bf16x8 as_bf16x8(const uint4& v) { return __builtin_bit_cast(bf16x8, v); }

typedef int i32x4 __attribute__((ext_vector_type(4)));

// Raw buffer descriptor (stride 0): base address, byte range, gfx9 data format word.
__device__ __forceinline__ i32x4 make_rsrc(const void* base, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  return i32x4{(int)(uint32_t)a, (int)(uint32_t)(a >> 32) & 0xffff, (int)bytes, 0x00020000};
}

// LDS byte address of a __shared__ object (32 bits, as the LDS instructions take it)
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
  return (uint32_t)reinterpret_cast<uintptr_t>((const __attribute__((address_space(3))) void*)p);
}

// 16 bytes per lane from the buffer at byte offset voff into LDS at byte
// address lds + 16 * lane (zeros when voff is past the descriptor's range).
// Issued as inline assembly so that the compiler adds no waits of its own for
// it: the caller orders the LDS traffic with explicit counter waits and barriers.
__device__ __forceinline__ void dma16(const i32x4& rsrc, uint32_t voff, uint32_t lds) {
  // the LDS address is wave-uniform; readfirstlane keeps it in a scalar register
  const uint32_t la = __builtin_amdgcn_readfirstlane(lds);
  asm volatile("s_mov_b32 m0, %0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
               :
               : "s"(la), "v"(voff), "s"(rsrc)
               : "memory");
}

// s_waitcnt with vmcnt <= n and lgkmcnt == 0 (expcnt unconstrained); gfx9 encoding
template <int N>
__device__ __forceinline__ void wait_vm_lgkm0() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
}

// Turns a lane's query fragments by the rotation of its row's position (Section
// 2.1.3: a recomputed row's fresh query is rotated at its request position).  The
// lane holds pieces 16 st + 8 hi + e (e < 8) of slots st < D/16; rotate-half pairs
// (j, j + D/2) sit in slots st and st + D/32 of the same lane.  tr is the row's
// D/2 (cos, sin) pairs of qcf_rope_table, and the arithmetic is rope_pair's, so
// the result is bit for bit the scatter's rotated query.
template <int D>
__device__ __forceinline__ void rotate_query(bf16x8 (&qr)[D / 16], const float2* __restrict__ tr,
                                             int hi) {
  constexpr int H = D / 32;
#pragma unroll
  for (int st = 0; st < H; ++st) {
    const float4* t4 = reinterpret_cast<const float4*>(tr + 16 * st + 8 * hi);
    float4 c4[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) c4[i] = t4[i];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float4 c = c4[e >> 1];
      const float2 cs = (e & 1) ? make_float2(c.z, c.w) : make_float2(c.x, c.y);
      float y1, y2;
      rope_pair((float)qr[st][e], (float)qr[st + H][e], cs, y1, y2);
      qr[st][e] = (__bf16)y1;
      qr[st + H][e] = (__bf16)y2;
    }
  }
}

}  // namespace qcf
