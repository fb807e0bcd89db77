// Device code shared by the bf16 attention kernels.
#pragma once
#include "qcf_device.h"

namespace qcf {

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
