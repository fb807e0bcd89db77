// float32 attention of the recomputed rows and of the query probe (the same
// definitions as the bf16 kernels of attention.hip), on the float32 matrix
// instruction v_mfma_f32_16x16x4_f32.
//
// Bound: at small sizes (a test-sized layer of a few hundred rows and keys)
// latency, at larger ones the float32 matrix rate (256 FLOP per clock and CU,
// the vector rate, but without the per-key cross-lane sums a vector dot needs).
// One block holds 16 query vectors of one KV head (consecutive rows times the
// heads that share it) and its 8 waves take the 16-key tiles in turn, each
// with its own online softmax, so a few hundred query vectors already occupy
// every CU and no wave walks the whole key range; the waves' (max, sum, O)
// are combined once at the end through LDS, in wave order.  No K/V staging in
// LDS: a lane's fragment is 16 contiguous bytes, 64 bytes per row and four
// lanes, and the waves of a block never read the same key.
//  * S^T = K Q^T: a lane holds 4 keys' logits of one query vector (register r
//    of lane l: key 4 (l / 16) + r, query vector l % 16).  Product (sb, e)
//    takes the d-columns 16 sb + 4 (l / 16) + e of both operands, so both are
//    float4 loads; the blocks sb sum into four accumulators (sb mod 4).
//  * O^T += V^T P^T with P^T straight from those registers: product (r, mb)
//    contracts over the keys 4 (l / 16) + r and fills the d-columns
//    NB (l % 16) + mb, so a lane's V operands are NB contiguous floats.
//  * K(t+1) is requested before the softmax of tile t and V(t+1) after its
//    products, into the registers those just freed.
// 8 x 64 heads over 4 x 128 + 32 keys: 184 rows 224.9 -> 11.5 us, the 32-row
// probe 33.3 -> 5.1 us (before: one wave per (row, head), one key at a time).
//  * At head size 128 the fragments, O and the next tiles fill the 256 registers of two waves
//    per SIMD; 14 (explicit positions) and 8 spill to scratch.
//  * exp2f, not the bare instruction: weights below 2^-126 stay subnormal numbers (0 to 7%
//    of a call's time, 2000-key probe of 8/2 heads of 64 63.1 -> 67.5 us).
// Error against float64, mean of 14 small layers: 2.2e-7 -> 1.5e-7 (rows), 3.3e-7
// -> 2.7e-7 (probe); two logit accumulators instead of four gave 5e-7.
#include <limits.h>
#include <math.h>

#include <algorithm>

#include "qcf_device.h"
#include "qcf_launch.h"

namespace qcf {
namespace {

constexpr int kW = 8;              // waves per block
constexpr int kQv = 16;            // query vectors per block
constexpr int kKeys = 16;          // keys per tile
constexpr int kMaxTilesX = 1 << 20;  // blocks along x; more query tiles are strided over

// a running maximum as the reference of exponentials: 0 while nothing has been seen
__device__ __forceinline__ float finite(float m) { return m == -INFINITY ? 0.f : m; }

template <int D, bool kPos>
__global__ __launch_bounds__(kW * 64) void attn_f32_kernel(
    float* __restrict__ out, float* __restrict__ lse, const float* __restrict__ q,
    const int32_t* __restrict__ row_pos, int64_t n_rows, const int32_t* __restrict__ cu_rows,
    const float* __restrict__ kc, const float* __restrict__ vc, int64_t n_kv_rows,
    int64_t kv_stride, const int32_t* __restrict__ cu_kv, const int32_t* __restrict__ kv_pos,
    int hq, int lg, float scale2) {
  constexpr int SB = D / 16;       // 16-column blocks of a row
  constexpr int NB = D / 16;       // output columns per lane
  constexpr int OSTR = D + 4;      // padded LDS row
  __shared__ __attribute__((aligned(16))) float o_l[kW * kQv * OSTR];
  __shared__ float2 ml_l[kW][kQv];
  const int g = blockIdx.y, b = blockIdx.z;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l = threadIdx.x & 63, li = l & 15, lk = l >> 4;
  const int64_t r0 = cu_rows[b];
  const int nr = cu_rows[b + 1] - (int)r0;
  const int64_t kv0 = cu_kv[b];
  int nkv = cu_kv[b + 1] - (int)kv0;
  if (kv0 + nkv > n_kv_rows) nkv = (int)(n_kv_rows - kv0);
  const int64_t nqv = (int64_t)max(nr, 0) << lg;
  for (int64_t tile = blockIdx.x; tile * kQv < nqv; tile += gridDim.x) {
    const int64_t qv = tile * kQv + li;
    const int64_t grow = r0 + (qv >> lg);
    const int head = (g << lg) + (int)(qv & ((1 << lg) - 1));
    const bool valid = qv < nqv && grow >= 0 && grow < n_rows;
    const int64_t crow = min(max(grow, (int64_t)0), n_rows - 1);
    const int pos_raw = row_pos[crow];
    float4 qf[SB];
#pragma unroll
    for (int sb = 0; sb < SB; ++sb)
      qf[sb] = *reinterpret_cast<const float4*>(q + (crow * hq + head) * D + 16 * sb + 4 * lk);
    const int qpos = valid ? pos_raw : INT_MIN;
    const int wmin = wave_min_i(valid ? qpos : INT_MAX);
    const int jend = kPos ? nkv : min(nkv, max(wave_max_i(valid ? qpos : -1), -1) + 1);
    const float* kb = kc + kv0 * kv_stride + (int64_t)g * D;
    const float* vb = vc + kv0 * kv_stride + (int64_t)g * D;
    float4 kf[SB], vf[4][NB / 4];
    int kp[4];
    auto load_k = [&](int kt0) {
      const float* p = kb + (int64_t)min(kt0 + li, nkv - 1) * kv_stride + 4 * lk;
#pragma unroll
      for (int sb = 0; sb < SB; ++sb) kf[sb] = *reinterpret_cast<const float4*>(p + 16 * sb);
      if (kPos) {
#pragma unroll
        for (int r = 0; r < 4; ++r) kp[r] = kv_pos[kv0 + min(kt0 + 4 * lk + r, nkv - 1)];
      }
    };
    auto load_v = [&](int kt0) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float* p = vb + (int64_t)min(kt0 + 4 * lk + r, nkv - 1) * kv_stride + NB * li;
#pragma unroll
        for (int c = 0; c < NB / 4; ++c) vf[r][c] = *reinterpret_cast<const float4*>(p + 4 * c);
      }
    };
    f32x4 o[NB];
#pragma unroll
    for (int mb = 0; mb < NB; ++mb) o[mb] = f32x4{};
    // m in log2 units, shared by the four lanes of a query vector; -inf until a key is seen
    // (finite() keeps a masked logit's p at 0 then; any finite logit is a valid maximum).  ls is
    // the lane's own keys' sum.
    float m = -INFINITY, ls = 0.f;
    int kt0 = w * kKeys;
    if (kt0 < jend) {
      load_k(kt0);
      load_v(kt0);
    }
    // Q has to be there before the loop (a wait for it inside would count the next tile's loads)
#pragma unroll
    for (int sb = 0; sb < SB; ++sb)
      asm volatile("" : "+v"(qf[sb].x), "+v"(qf[sb].y), "+v"(qf[sb].z), "+v"(qf[sb].w));
    for (; kt0 < jend; kt0 += kW * kKeys) {
      f32x4 s[4] = {};  // summed pairwise: shorter chains round less
      bool vis[4];  // key visible to this lane's query vector
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int j = kt0 + 4 * lk + r;
        vis[r] = j < nkv && (kPos ? kp[r] : j) <= qpos;
      }
#pragma unroll
      for (int sb = 0; sb < SB; sb += 4) {
#pragma unroll
        for (int c = 0; c < 4; ++c)
          s[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[sb + c].x, qf[sb + c].x, s[c], 0, 0, 0);
#pragma unroll
        for (int c = 0; c < 4; ++c)
          s[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[sb + c].y, qf[sb + c].y, s[c], 0, 0, 0);
#pragma unroll
        for (int c = 0; c < 4; ++c)
          s[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[sb + c].z, qf[sb + c].z, s[c], 0, 0, 0);
#pragma unroll
        for (int c = 0; c < 4; ++c)
          s[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[sb + c].w, qf[sb + c].w, s[c], 0, 0, 0);
      }
      const f32x4 dot = (s[0] + s[1]) + (s[2] + s[3]);
      const int kn = kt0 + kW * kKeys;
      if (kn < jend) load_k(kn);
      float x[4], mt = -INFINITY;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        x[r] = vis[r] ? dot[r] * scale2 : -INFINITY;
        mt = fmaxf(mt, x[r]);
      }
      // lazy rescale: a stale max stays unless some vector's max grew by more than 2^8
      if (__ballot(mt > m + 8.f)) {
        mt = fmaxf(mt, __shfl_xor(mt, 16, 64));
        mt = fmaxf(mt, __shfl_xor(mt, 32, 64));
        const float mn = fmaxf(m, mt);
        const float alpha = exp2f(m - finite(mn));
        ls *= alpha;
#pragma unroll
        for (int mb = 0; mb < NB; ++mb) o[mb] *= alpha;
        m = mn;
      }
      float p[4];
      const float mr = finite(m);
#pragma unroll
      for (int r = 0; r < 4; ++r) p[r] = exp2f(x[r] - mr);
      ls += (p[0] + p[1]) + (p[2] + p[3]);
      const bool edge = kPos || kt0 + kKeys > wmin + 1 || kt0 + kKeys > nkv;
      bool fin = true;
      if (edge) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int c = 0; c < NB / 4; ++c)
            fin = fin && isfinite(vf[r][c].x) && isfinite(vf[r][c].y) && isfinite(vf[r][c].z) &&
                  isfinite(vf[r][c].w);
      }
      if (__ballot(!fin) == 0) {
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
          for (int mb = 0; mb < NB; ++mb) {
            const float4 c = vf[r][mb / 4];
            const float ve = mb % 4 == 0 ? c.x : mb % 4 == 1 ? c.y : mb % 4 == 2 ? c.z : c.w;
            o[mb] = __builtin_amdgcn_mfma_f32_16x16x4f32(ve, p[r], o[mb], 0, 0, 0);
          }
      } else {
        // a tile with masked keys and a value that is not finite (an unwritten row, say): a
        // masked key must not reach its query vectors, where 0 * inf would be NaN, so the
        // visible keys' products are added one by one
        for (int k = 0; k < kKeys; ++k) {
          const int src = (k >> 2) * 16 + li;
          const float pk = __shfl(k & 2 ? (k & 1 ? p[3] : p[2]) : (k & 1 ? p[1] : p[0]), src, 64);
          const int vk = __shfl((int)(k & 2 ? (k & 1 ? vis[3] : vis[2]) : (k & 1 ? vis[1] : vis[0])), src, 64);
          const float* vr = vb + (int64_t)min(kt0 + k, nkv - 1) * kv_stride;
          if (vk) {
#pragma unroll
            for (int mb = 0; mb < NB; ++mb)
#pragma unroll
              for (int r = 0; r < 4; ++r) o[mb][r] += pk * vr[NB * (4 * lk + r) + mb];
          }
        }
      }
      if (kn < jend) load_v(kn);
    }
    // the waves' partials: lane l holds columns NB (4 lk + r) + mb of query vector li
    ls += __shfl_xor(ls, 16, 64);
    ls += __shfl_xor(ls, 32, 64);
    if (lk == 0) ml_l[w][li] = make_float2(m, ls);
    float* op = o_l + (w * kQv + li) * OSTR;
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int c = 0; c < NB / 4; ++c)
        *reinterpret_cast<float4*>(op + NB * (4 * lk + r) + 4 * c) =
            make_float4(o[4 * c][r], o[4 * c + 1][r], o[4 * c + 2][r], o[4 * c + 3][r]);
    __syncthreads();
    const int t = threadIdx.x;
    if (t < kQv * D / 4) {
      const int i = t / (D / 4), c = 4 * (t % (D / 4));
      float mx = -INFINITY;
#pragma unroll
      for (int ww = 0; ww < kW; ++ww) mx = fmaxf(mx, ml_l[ww][i].x);
      float lt = 0.f;
      float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int ww = 0; ww < kW; ++ww) {
        const float2 ml = ml_l[ww][i];
        const float f = exp2f(ml.x - finite(mx));
        const float4 x = *reinterpret_cast<const float4*>(o_l + (ww * kQv + i) * OSTR + c);
        lt += f * ml.y;
        acc.x += f * x.x;
        acc.y += f * x.y;
        acc.z += f * x.z;
        acc.w += f * x.w;
      }
      const int64_t ov = tile * kQv + i, orow = r0 + (ov >> lg);
      const int oh = (g << lg) + (int)(ov & ((1 << lg) - 1));
      if (ov < nqv && orow >= 0 && orow < n_rows) {
        const float inv = lt > 0.f ? 1.f / lt : 0.f;
        *reinterpret_cast<float4*>(out + (orow * hq + oh) * D + c) =
            make_float4(acc.x * inv, acc.y * inv, acc.z * inv, acc.w * inv);
        if (lse && c == 0) lse[orow * hq + oh] = lt > 0.f ? (mx + log2f(lt)) * kLn2 : -INFINITY;
      }
    }
    __syncthreads();  // the LDS is rewritten by the next tile
  }
}

}  // namespace

hipError_t launch_attn_f32(float* out, float* lse, const float* q, const int32_t* row_pos,
                           int64_t n_rows, const int32_t* cu_rows, const float* k_cache,
                           const float* v_cache, int64_t n_kv_rows, int64_t kv_row_stride,
                           const int32_t* cu_kv, const int32_t* kv_pos, const AttnShape& s,
                           float scale, hipStream_t stream) {
  int lg = 0;
  while ((1 << lg) < s.hq / s.hkv) ++lg;
  // no request has more rows than there are (max_rows is only a bound)
  const int64_t qv = std::min<int64_t>(s.max_rows, n_rows) << lg;
  const dim3 grid((unsigned)std::min<int64_t>((qv + kQv - 1) / kQv, kMaxTilesX), s.hkv, s.batch);
#define QCF_A32(D, P)                                                                              \
  attn_f32_kernel<D, P><<<grid, kW * 64, 0, stream>>>(out, lse, q, row_pos, n_rows, cu_rows,       \
                                                      k_cache, v_cache, n_kv_rows, kv_row_stride, \
                                                      cu_kv, kv_pos, s.hq, lg, scale * kLog2e)
  if (s.d == 64) {
    if (kv_pos) QCF_A32(64, true); else QCF_A32(64, false);
  } else {
    if (kv_pos) QCF_A32(128, true); else QCF_A32(128, false);
  }
#undef QCF_A32
  return hipGetLastError();
}

}  // namespace qcf
