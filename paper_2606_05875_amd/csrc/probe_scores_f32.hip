// float32 importance scores (eq. single_layer_importance) on the float32 matrix
// instruction v_mfma_f32_16x16x4_f32, in two launches:
//   stats   : one block per 16 query vectors of a KV head (query rows times the
//             heads that share it); its 8 waves take the 16-key tiles in turn and
//             every lane keeps an online (max, sum) of its own keys, combined once
//             at the end -> (max, 1 / sum) per query vector.
//   columns : one block per 16 keys; its 8 waves take the (KV head, 16 query
//             vectors) units in turn, recompute the logits and add 2^(logit - max)
//             / sum over the vectors; one sum over lanes and waves per key.
// Bound: latency at the sizes float32 is used at (a test-sized layer), the float32
// matrix rate beyond.  Both passes spread one dimension over the grid and the
// other over the waves, so a 512-key, 256-vector layer runs on 16 and 32 blocks of
// 8 waves with 4 and 2 tiles each; before, a thread owned a key and walked every
// query vector (2 blocks: 224.7 us), and a wave owned a query row and head (15.5
// us).  Now 7.0 and 8.9 us on that layer; error against float64 over 14 small
// layers 1.6e-7 -> 0.7e-7.
//
// Fragments come straight from memory (a lane's piece is 16 contiguous bytes): in
// both passes lane l holds row l % 16 of its operand tile and the d-columns 16 sb
// + 4 (l / 16) + e, the contraction order of product (sb, e).  Every reduction has
// a fixed order.  With kRot the keys are turned in registers by their rotation
// table row (rope_pair, the arithmetic of the stored re-positioned keys).  exp2f, not the
// bare instruction: weights below 2^-126 stay subnormal numbers and rank their keys.
#include <math.h>

#include <algorithm>

#include "qcf_device.h"
#include "qcf_launch.h"

namespace qcf {
namespace {

constexpr int kW = 8;               // waves per block
constexpr int kTile = 16;           // query vectors and keys per tile
constexpr int kMaxTilesX = 1 << 20;  // blocks along x; more tiles are strided over

// a running maximum as the reference of exponentials: 0 while nothing has been seen
__device__ __forceinline__ float finite(float m) { return m == -INFINITY ? 0.f : m; }

__device__ __forceinline__ float2 combine_ml(float2 a, float2 b) {
  const float m = fmaxf(a.x, b.x), r = finite(m);
  return make_float2(m, a.y * exp2f(a.x - r) + b.y * exp2f(b.x - r));
}

template <int D>
struct Frag {  // one row's columns 16 sb + 4 (lane / 16) + {0..3}
  static constexpr int SB = D / 16;
  float4 f[SB];
  __device__ __forceinline__ void load(const float* row, int lk) {
#pragma unroll
    for (int sb = 0; sb < SB; ++sb) f[sb] = *reinterpret_cast<const float4*>(row + 16 * sb + 4 * lk);
  }
  // rotate-half pairs (j, j + D/2) sit in blocks sb and sb + SB/2 of the same lane
  __device__ __forceinline__ void rotate(const float2* cs, int lk) {
#pragma unroll
    for (int sb = 0; sb < SB / 2; ++sb) {
      const float2* c = cs + 16 * sb + 4 * lk;
      float4 a = f[sb], b = f[sb + SB / 2];
      rope_pair(f[sb].x, f[sb + SB / 2].x, c[0], a.x, b.x);
      rope_pair(f[sb].y, f[sb + SB / 2].y, c[1], a.y, b.y);
      rope_pair(f[sb].z, f[sb + SB / 2].z, c[2], a.z, b.z);
      rope_pair(f[sb].w, f[sb + SB / 2].w, c[3], a.w, b.w);
      f[sb] = a;
      f[sb + SB / 2] = b;
    }
  }
};

// rows of `a` times columns of `b`: register r of lane l is row 4 (l / 16) + r, column l % 16
template <int D>
__device__ __forceinline__ f32x4 product(const Frag<D>& a, const Frag<D>& b) {
  f32x4 s[4] = {};  // summed pairwise: shorter chains round less
#pragma unroll
  for (int sb = 0; sb < D / 16; sb += 4) {
#pragma unroll
    for (int c = 0; c < 4; ++c)
      s[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.f[sb + c].x, b.f[sb + c].x, s[c], 0, 0, 0);
#pragma unroll
    for (int c = 0; c < 4; ++c)
      s[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.f[sb + c].y, b.f[sb + c].y, s[c], 0, 0, 0);
#pragma unroll
    for (int c = 0; c < 4; ++c)
      s[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.f[sb + c].z, b.f[sb + c].z, s[c], 0, 0, 0);
#pragma unroll
    for (int c = 0; c < 4; ++c)
      s[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(a.f[sb + c].w, b.f[sb + c].w, s[c], 0, 0, 0);
  }
  return (s[0] + s[1]) + (s[2] + s[3]);
}

template <int D, bool kRot>
__global__ __launch_bounds__(kW * 64) void scores_stats_f32(
    float2* __restrict__ stats, const float* __restrict__ q, int64_t n_q_rows,
    const float* __restrict__ k, int64_t n_kv_rows, int64_t k_stride,
    const int32_t* __restrict__ key_rot, const float2* __restrict__ rot_tab, int n_rot,
    const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_kv,
    const int32_t* __restrict__ ctx_len, int hq, int lg, int max_q_len, float scale2) {
  __shared__ float2 ml_l[kW][kTile];
  const int g = blockIdx.y, b = blockIdx.z;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l = threadIdx.x & 63, li = l & 15, lk = l >> 4;
  const int64_t q0 = cu_q[b];
  const int nq = min(cu_q[b + 1] - (int)q0, max_q_len);
  const int64_t nqv = (int64_t)max(nq, 0) << lg;
  const int64_t k0 = cu_kv[b];
  const int N = (int)min((int64_t)ctx_len[b], n_kv_rows - k0);
  const float* kb = k + (int64_t)g * D;
  for (int64_t tile = blockIdx.x; tile * kTile < nqv; tile += gridDim.x) {
    const int64_t qv = tile * kTile + li;
    const int i = (int)(qv >> lg), head = (g << lg) + (int)(qv & ((1 << lg) - 1));
    Frag<D> qf, kf, kn;
    qf.load(q + (min(q0 + i, n_q_rows - 1) * hq + head) * D, lk);
    auto load_k = [&](Frag<D>& f, int kt0) {
      const int64_t row = k0 + min(kt0 + li, N - 1);
      f.load(kb + row * k_stride, lk);
      if constexpr (kRot) f.rotate(rot_tab + (int64_t)min(max(key_rot[row], 0), n_rot - 1) * (D / 2), lk);
    };
    // a masked key's logit is -inf and its term 0; any finite logit is a valid maximum
    float m = -INFINITY, ls = 0.f;
    int kt0 = w * kTile;
    if (kt0 < N) load_k(kf, kt0);
    // Q has to be there before the loop (a wait for it inside would count the next tile's loads)
#pragma unroll
    for (int sb = 0; sb < D / 16; ++sb)
      asm volatile("" : "+v"(qf.f[sb].x), "+v"(qf.f[sb].y), "+v"(qf.f[sb].z), "+v"(qf.f[sb].w));
    for (; kt0 < N; kt0 += kW * kTile) {
      if (kt0 + kW * kTile < N) load_k(kn, kt0 + kW * kTile);
      const f32x4 s = product<D>(kf, qf);
      float x[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) x[r] = kt0 + 4 * lk + r < N ? s[r] * scale2 : -INFINITY;
      const float mn = fmaxf(m, fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])));
      const float mr = finite(mn);
      float p = 0.f;
#pragma unroll
      for (int r = 0; r < 4; ++r) p += exp2f(x[r] - mr);
      ls = ls * exp2f(m - mr) + p;
      m = mn;
      kf = kn;
    }
    float2 ml = make_float2(m, ls);
    ml = combine_ml(ml, make_float2(__shfl_xor(ml.x, 16, 64), __shfl_xor(ml.y, 16, 64)));
    ml = combine_ml(ml, make_float2(__shfl_xor(ml.x, 32, 64), __shfl_xor(ml.y, 32, 64)));
    if (lk == 0) ml_l[w][li] = ml;
    __syncthreads();
    if (threadIdx.x < kTile) {
      ml = ml_l[0][li];
#pragma unroll
      for (int ww = 1; ww < kW; ++ww) ml = combine_ml(ml, ml_l[ww][li]);
      if (qv < nqv && q0 + i < n_q_rows)
        stats[((int64_t)b * hq + head) * max_q_len + i] =
            make_float2(finite(ml.x), ml.y > 0.f ? 1.f / ml.y : 0.f);
    }
    __syncthreads();  // ml_l is rewritten by the next tile
  }
}

template <int D, bool kRot>
__global__ __launch_bounds__(kW * 64) void scores_cols_f32(
    float* __restrict__ scores, int accumulate, const float2* __restrict__ stats,
    const float* __restrict__ q, int64_t n_q_rows, const float* __restrict__ k, int64_t n_kv_rows,
    int64_t k_stride, const int32_t* __restrict__ key_rot, const float2* __restrict__ rot_tab,
    int n_rot, const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_kv,
    const int32_t* __restrict__ ctx_len, int hq, int hkv, int lg, int max_q_len, float scale2) {
  __shared__ float col_l[kW][kTile];
  const int b = blockIdx.y;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l = threadIdx.x & 63, li = l & 15, lk = l >> 4;
  const int64_t k0 = cu_kv[b];
  const int N = (int)min((int64_t)ctx_len[b], n_kv_rows - k0);
  const int64_t q0 = cu_q[b];
  const int nq = (int)min((int64_t)min(cu_q[b + 1] - (int)q0, max_q_len), n_q_rows - q0);
  const int64_t nqv = (int64_t)max(nq, 0) << lg;
  const int n_qt = (int)((nqv + kTile - 1) / kTile);
  const int units = n_qt * hkv;
  for (int64_t kt = blockIdx.x; kt * kTile < N; kt += gridDim.x) {
    const int t = (int)kt * kTile + li;
    const int64_t row = k0 + min(t, N - 1);
    const float2* cs = nullptr;
    if constexpr (kRot) cs = rot_tab + (int64_t)min(max(key_rot[row], 0), n_rot - 1) * (D / 2);
    Frag<D> qf, kf;
    float2 st[4];  // (max, 1 / sum) of the unit's vectors 4 lk + r
    auto load = [&](int u) {
      const int g = u / n_qt;
      const int64_t v0 = (int64_t)(u - g * n_qt) * kTile;
      const int64_t qv = min(v0 + li, nqv - 1);
      qf.load(q + ((q0 + (qv >> lg)) * hq + (g << lg) + (int)(qv & ((1 << lg) - 1))) * D, lk);
      kf.load(k + row * k_stride + (int64_t)g * D, lk);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t rv = min(v0 + 4 * lk + r, nqv - 1);
        st[r] = stats[((int64_t)b * hq + (g << lg) + (int)(rv & ((1 << lg) - 1))) * max_q_len + (rv >> lg)];
        if (v0 + 4 * lk + r >= nqv) st[r].y = 0.f;  // a padding vector adds nothing
      }
      if constexpr (kRot) kf.rotate(cs, lk);
    };
    float acc = 0.f;
    if (w < units) load(w);
    for (int u = w; u < units; u += kW) {
      const f32x4 s = product<D>(qf, kf);
      float2 sv[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) sv[r] = st[r];
      if (u + kW < units) load(u + kW);  // in flight during this unit's exponentials
#pragma unroll
      for (int r = 0; r < 4; ++r) acc += exp2f(s[r] * scale2 - sv[r].x) * sv[r].y;
    }
    acc += __shfl_xor(acc, 16, 64);
    acc += __shfl_xor(acc, 32, 64);
    if (lk == 0) col_l[w][li] = acc;
    __syncthreads();
    if (threadIdx.x < kTile && t < N) {
      float sum = 0.f;
#pragma unroll
      for (int ww = 0; ww < kW; ++ww) sum += col_l[ww][li];
      scores[row] = accumulate ? scores[row] + sum : sum;
    }
    __syncthreads();  // col_l is rewritten by the next tile
  }
}

}  // namespace

hipError_t launch_scores_f32(float* scores, int accumulate, const float* q, int64_t n_q_rows,
                             const float* k, int64_t n_kv_rows, int64_t k_row_stride,
                             const KeyRot& rot, const int32_t* cu_q, const int32_t* cu_kv,
                             const int32_t* ctx_len, const ProbeShape& s, float scale, void* ws,
                             hipStream_t stream) {
  if (n_kv_rows <= 0) return hipSuccess;
  const float scale2 = scale * kLog2e;
  int lg = 0;
  while ((1 << lg) < s.hq / s.hkv) ++lg;
  float2* stats = static_cast<float2*>(ws);
  const float2* tab = reinterpret_cast<const float2*>(rot.table);
  // no request has more query rows or keys than there are (the maxima are only bounds)
  const int64_t qv = std::min<int64_t>(s.max_q_len, n_q_rows) << lg;
  const int64_t keys = std::min<int64_t>(s.max_ctx_len, n_kv_rows);
  const dim3 g1((unsigned)std::min<int64_t>((qv + kTile - 1) / kTile, kMaxTilesX), s.hkv, s.batch);
  const dim3 g2((unsigned)std::min<int64_t>((keys + kTile - 1) / kTile, kMaxTilesX), s.batch);
#define QCF_F32(D, R)                                                                              \
  do {                                                                                             \
    if (qv > 0)                                                                                    \
      scores_stats_f32<D, R><<<g1, kW * 64, 0, stream>>>(stats, q, n_q_rows, k, n_kv_rows,         \
                                                         k_row_stride, rot.row, tab, (int)rot.n,   \
                                                         cu_q, cu_kv, ctx_len, s.hq, lg,           \
                                                         s.max_q_len, scale2);                     \
    scores_cols_f32<D, R><<<g2, kW * 64, 0, stream>>>(scores, accumulate, stats, q, n_q_rows, k,   \
                                                      n_kv_rows, k_row_stride, rot.row, tab,       \
                                                      (int)rot.n, cu_q, cu_kv, ctx_len, s.hq,      \
                                                      s.hkv, lg, s.max_q_len, scale2);             \
  } while (0)
  if (s.d == 64) {
    if (rot.row) QCF_F32(64, true); else QCF_F32(64, false);
  } else {
    if (rot.row) QCF_F32(128, true); else QCF_F32(128, false);
  }
#undef QCF_F32
  return hipGetLastError();
}

}  // namespace qcf
