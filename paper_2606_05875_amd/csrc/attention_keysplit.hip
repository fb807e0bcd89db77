// bf16 attention for calls that are short of query vectors: the query probe over
// [anchor cache ; query] (Section 3.3.2, eq. anchor_query_state: a few dozen rows,
// explicit key positions) and the recomputed rows of a small layer.
//
// Bound: latency.  A probe of 64 rows has 256 query vectors per KV head; blocks of
// 128 vectors that walk all the keys put it on 16 of the 256 CUs, one 64-key tile
// after another.  Here a block holds 32 query vectors and its KW waves split the
// KEYS: wave w takes every KW-th 32-key tile, with an online softmax of its own and
// no barrier in the loop; the waves' O are summed once at the end through LDS.
// Long key ranges are also cut over n_split blocks, whose float32 partials
// attn_keysplit_merge_kernel sums in order.
//  * Products as in attention.hip: S^T = K Q^T and O^T += V^T P^T on
//    v_mfma_f32_32x32x16_bf16, fragments from wave-private LDS tiles.  (K fragments
//    straight from memory, 32 bytes of a row per two lanes, were slower: 16.5
//    against 14.5 us for the 1104-key probe, 99 against 69 us uncut for 10304 keys.)
//  * The next tile's K and V are in flight in registers during this tile's work.
//  * Every wave moves its own tiles (16 KB per 32 keys at head size 128), which
//    bounds the loop at about a third of the matrix rate, so calls with enough
//    query vectors to fill the chip take the kernels that share tiles.
// Probe of 64 rows, 32/8 heads of 128: 224 keys 18.6 -> 8.1 us, 1104 keys 65.7 ->
// 14.5 us, 10304 keys 549 -> 30 us; 128 rows, 64/8 heads, 1152 keys 66.6 -> 16.1 us.
#include <limits.h>
#include <math.h>

#include <algorithm>

#include "qcf_attn.h"
#include "qcf_device.h"
#include "qcf_launch.h"

namespace qcf {
namespace {

constexpr int kKeys = 32;  // keys per tile
constexpr int kQv = 32;    // query vectors per block (every wave holds all of them)

// 16 bytes at byte offset off of the buffer (zeros past its range)
__device__ __forceinline__ uint4 bld16(const __amdgpu_buffer_rsrc_t& r, uint32_t off) {
  return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
}

template <int D, int KW, bool kPos, bool kRot>
__global__ __launch_bounds__(KW * 64) void attn_keysplit_kernel(
    uint16_t* __restrict__ out, float* __restrict__ lse, const uint16_t* __restrict__ q,
    const int32_t* __restrict__ row_pos, int64_t n_rows, const int32_t* __restrict__ cu_rows,
    const uint16_t* __restrict__ kc, const uint16_t* __restrict__ vc, int64_t n_kv_rows,
    int64_t kv_stride, const int32_t* __restrict__ cu_kv, const int32_t* __restrict__ kv_pos,
    int max_units, int hkv, int hq, int lg, float scale2, int n_split, float4* __restrict__ part_o,
    float2* __restrict__ part_ml, const int32_t* __restrict__ q_src, int64_t n_q_src,
    const float2* __restrict__ rtab, int n_tab) {
  constexpr int CPR = D / 8;                   // 16-byte chunks per row
  // padded LDS rows: conflict-free fragment (K) and transposing (V) reads
  constexpr int KSTR = (CPR + 1) * 8, VSTR = (CPR + 4) * 8;
  constexpr int KST = kKeys * KSTR, VST = kKeys * VSTR;  // elements of a wave's tiles
  constexpr int TL = kKeys * CPR / 64;         // chunks of a tile per lane
  constexpr int NG = D / 8;                    // groups of 4 output columns per lane
  constexpr int LDS_T = KW * (KST + VST) * 2, LDS_R = KW * 8 * 64 * 16;
  __shared__ __attribute__((aligned(16))) uint8_t lds[LDS_T > LDS_R ? LDS_T : LDS_R];
  __shared__ float2 ml_l[KW][kQv];
  __shared__ __attribute__((aligned(16))) int kp_l[kPos ? KW : 1][kKeys];

  // the KV head fastest: with 8 heads a head's blocks share one XCD's L2
  const int g = blockIdx.x % hkv;
  int rest = blockIdx.x / hkv;
  const int split = rest % n_split;
  rest /= n_split;
  const int unit = rest % max_units, b = rest / max_units;  // 32-vector unit of request b
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l = threadIdx.x & 63, lq = l & 31, hi = l >> 5;
  const int64_t r0 = cu_rows[b];
  const int nr = cu_rows[b + 1] - (int)r0;
  const int64_t nqv = (int64_t)max(nr, 0) << lg;
  if ((int64_t)unit * kQv >= nqv) return;
  const int64_t kv0 = cu_kv[b];
  int nkv = cu_kv[b + 1] - (int)kv0;
  if (kv0 + nkv > n_kv_rows) nkv = (int)(n_kv_rows - kv0);
  const int64_t qv = (int64_t)unit * kQv + lq;
  const int64_t grow = r0 + (qv >> lg);
  const int head = (g << lg) + (int)(qv & ((1 << lg) - 1));
  const bool valid = qv < nqv && grow < n_rows;
  const int64_t crow = min(grow, n_rows - 1);
  const int pos_raw = row_pos[crow];
  bf16x8 qreg[D / 16];
  {
    int64_t qrow = crow;
    if (kRot && q_src) qrow = min(max((int64_t)q_src[crow], (int64_t)0), n_q_src - 1);
    const uint16_t* qp = q + (qrow * hq + head) * D + 8 * hi;
#pragma unroll
    for (int st = 0; st < D / 16; ++st) qreg[st] = __builtin_bit_cast(bf16x8, ld16(qp + 16 * st));
  }
  const int qpos = valid ? pos_raw : INT_MIN;
  const int wmin = wave_min_i(valid ? qpos : INT_MAX);
  const int jend = kPos ? nkv : min(nkv, wave_max_i(valid ? max(qpos, -1) : -1) + 1);
  if (kRot) rotate_query<D>(qreg, rtab + (int64_t)min(max(pos_raw, 0), n_tab - 1) * (D / 2), hi);
  // this block's share of the tiles, then this wave's
  const int nt = max(jend + kKeys - 1, 0) / kKeys;
  const int t_hi = (int)((int64_t)nt * (split + 1) / n_split);
  int t = (int)((int64_t)nt * split / n_split) + w;

  const uint16_t* kb = kc + kv0 * kv_stride + (int64_t)g * D;
  const uint16_t* vb = vc + kv0 * kv_stride + (int64_t)g * D;
  uint16_t* kl = reinterpret_cast<uint16_t*>(lds) + w * (KST + VST);
  uint16_t* vl = kl + KST;
  const int tg = l >> 4, te = (l >> 2) & 3, tq = l & 3;
  const uint16_t* vrd = vl + (4 * (tg >> 1) + te) * VSTR + 16 * (tg & 1) + 4 * tq;
  const uint16_t* krd = kl + lq * KSTR + 8 * hi;
  const uint32_t row_b = (uint32_t)(kv_stride * 2);
  const int range = nkv > 0 ? (int)((uint32_t)(nkv - 1) * row_b + D * 2) : 0;
  const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc((void*)kb, 0, range, 0x00020000);
  const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc((void*)vb, 0, range, 0x00020000);
  uint4 kt[TL], vt[TL];
  int kp = 0;
  // Causal calls read through descriptors that end at the request's last key (their row offsets are
  // below 2^31): rows past it are zeros, so that their weight 0 meets no value that is not finite
  // (the last key repeated there, its value zeroed in LDS: 32.7 us against 31.8 for 390 rows over
  // 2438 keys with 8 heads of 128).  Probes, as in the shared-tile kernel, repeat the last key.
  auto load = [&](int kt0) {
    if (kPos) kp = kv_pos[kv0 + min(kt0 + lq, nkv - 1)];
#pragma unroll
    for (int i = 0; i < TL; ++i) {
      const int c = i * 64 + l;
      kt[i] = kPos ? ld16(kb + (int64_t)min(kt0 + c / CPR, nkv - 1) * kv_stride + (c % CPR) * 8)
                   : bld16(rk, (uint32_t)(kt0 + c / CPR) * row_b + (c % CPR) * 16);
    }
#pragma unroll
    for (int i = 0; i < TL; ++i) {
      const int c = i * 64 + l;
      vt[i] = kPos ? ld16(vb + (int64_t)min(kt0 + c / CPR, nkv - 1) * kv_stride + (c % CPR) * 8)
                   : bld16(rv, (uint32_t)(kt0 + c / CPR) * row_b + (c % CPR) * 16);
    }
  };
  typedef short v4s __attribute__((ext_vector_type(4)));
  typedef v4s __attribute__((address_space(3))) * lds_v4s;
  f32x16 o[D / 32];
#pragma unroll
  for (int mb = 0; mb < D / 32; ++mb) o[mb] = f32x16{};
  // log2 units.  A padding lane never asks for a rescale, but its alpha in one is inf - inf: its
  // sum and O may be NaN, stay in its own column to the end (partials too) and are never used.
  float m = valid ? -1e30f : INFINITY;
  float ls = 0.f;
  if (t < t_hi) load(t * kKeys);
  // Q has to be there before the loop: the compiler's wait for it at the products would count
  // the next tile's loads too (1104-key probe 14.5 -> 13.8 us)
#pragma unroll
  for (int st = 0; st < D / 16; ++st) asm volatile("" : "+v"(qreg[st]));
  for (; t < t_hi; t += KW) {
    const int kt0 = t * kKeys;
#pragma unroll
    for (int i = 0; i < TL; ++i) {
      const int c = i * 64 + l;
      st16(kl + (c / CPR) * KSTR + (c % CPR) * 8, kt[i]);
      st16(vl + (c / CPR) * VSTR + (c % CPR) * 8, vt[i]);
    }
    const int kpc = kt0 + lq < nkv ? kp : INT_MAX;
    asm volatile("" ::: "memory");  // (a wave's LDS accesses execute in order)
    if (t + KW < t_hi) load(kt0 + KW * kKeys);  // in flight during this tile's work
    f32x16 s = f32x16{};
#pragma unroll
    for (int st = 0; st < D / 16; ++st)
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, ld16(krd + 16 * st)), qreg[st],
                                                  s, 0, 0, 0);
    // lane value v is key 8 (v >> 2) + 4 hi + (v & 3) of the tile
    const bool edge = kPos ? __ballot(kpc > wmin) != 0 : kt0 + kKeys > wmin || kt0 + kKeys > nkv;
    if (edge) {
      if (kPos) {
        if (hi == 0) kp_l[kPos ? w : 0][lq] = kpc;
        asm volatile("" ::: "memory");
      }
#pragma unroll
      for (int c = 0; c < 4; ++c) {
        int4 kk = make_int4(0, 0, 0, 0);
        if (kPos) kk = *reinterpret_cast<const int4*>(&kp_l[kPos ? w : 0][8 * c + 4 * hi]);
        const int ka[4] = {kk.x, kk.y, kk.z, kk.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int j = kt0 + 8 * c + 4 * hi + e;
          if (j >= nkv || (kPos ? ka[e] : j) > qpos) s[4 * c + e] = -INFINITY;
        }
      }
    }
    float mt = s[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) mt = fmaxf(mt, s[v]);
    mt = fmaxf(mt, __shfl_xor(mt, 32, 64)) * scale2;
    // lazy rescale: a stale max stays unless some row's max grew by more than 2^8
    if (__ballot(mt > m + 8.f)) {
      const float mn = fmaxf(m, mt);
      const float alpha = __builtin_amdgcn_exp2f(m - mn);
      ls *= alpha;
#pragma unroll
      for (int mb = 0; mb < D / 32; ++mb) o[mb] *= alpha;
      m = mn;
    }
    bf16x8 pb[2];
    float psum = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float p = __builtin_amdgcn_exp2f(fmaf(s[v], scale2, -m));
      psum += p;
      pb[v >> 3][v & 7] = (__bf16)p;
    }
    ls += psum;
#pragma unroll
    for (int k2 = 0; k2 < 2; ++k2)
#pragma unroll
      for (int mb = 0; mb < D / 32; ++mb) {
        const uint16_t* p0 = vrd + 16 * k2 * VSTR + 32 * mb;
        const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p0));
        const v4s up = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p0 + 8 * VSTR));
        const bf16x8 va = __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, up, 0, 1, 2, 3, 4, 5, 6, 7));
        o[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va, pb[k2], o[mb], 0, 0, 0);
      }
    asm volatile("" ::: "memory");
  }

  // sum over the waves: every wave leaves a half of its O (64 columns) in
  // LDS, lane for lane, and takes 8 / KW of that half's 8 column groups over all KW waves
  ls += __shfl_xor(ls, 32, 64);
  if (!valid) m = -1e30f;
  if (hi == 0) ml_l[w][lq] = make_float2(m, ls);
  __syncthreads();
  float mx = -1e30f, lt = 0.f, f[KW];
#pragma unroll
  for (int i = 0; i < KW; ++i) mx = fmaxf(mx, ml_l[i][lq].x);
#pragma unroll
  for (int i = 0; i < KW; ++i) {
    const float2 ml = ml_l[i][lq];
    f[i] = __builtin_amdgcn_exp2f(ml.x - mx);
    lt += f[i] * ml.y;
  }
  const float inv = lt > 0.f ? 1.f / lt : 0.f;
  // (with n_split > 1) this unit's partial slot
  const int64_t slot = (((int64_t)b * max_units + unit) * hkv + g) * n_split + split;
  float4* red = reinterpret_cast<float4*>(lds);
#pragma unroll
  for (int half = 0; half < D / 64; ++half) {
    if (half) __syncthreads();  // the previous half has been read
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const f32x16& x = o[2 * half + i / 4];
      const int v = 4 * (i & 3);
      red[(w * 8 + i) * 64 + l] = make_float4(x[v], x[v + 1], x[v + 2], x[v + 3]);
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 8 / KW; ++j) {
      const int i = w * (8 / KW) + j;
      float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int k = 0; k < KW; ++k) {
        const float4 x = red[(k * 8 + i) * 64 + l];
        a.x += f[k] * x.x;
        a.y += f[k] * x.y;
        a.z += f[k] * x.z;
        a.w += f[k] * x.w;
      }
      if (n_split > 1) {
        part_o[(slot * NG + half * 8 + i) * 64 + l] = a;
      } else if (valid) {
        uint16_t* op = out + (grow * hq + head) * D + 64 * half + 8 * i + 4 * hi;
        *reinterpret_cast<uint2*>(op) =
            make_uint2(pack_bf16x2(a.x * inv, a.y * inv), pack_bf16x2(a.z * inv, a.w * inv));
      }
    }
  }
  if (w == 0 && hi == 0) {
    if (n_split > 1) part_ml[slot * kQv + lq] = make_float2(mx, lt);
    else if (valid && lse) lse[grow * hq + head] = lt > 0.f ? (mx + log2f(lt)) * kLn2 : -INFINITY;
  }
}

// Sums the n_split partials of a 32-vector unit in split order.  One wave per (unit,
// group of 4 columns per lane); a group's loads are all in flight at once.
constexpr int kMaxSplit = 16;
template <int D>
__global__ __launch_bounds__(256) void attn_keysplit_merge_kernel(
    uint16_t* __restrict__ out, float* __restrict__ lse, int64_t n_rows,
    const int32_t* __restrict__ cu_rows, int max_units, int hkv, int hq, int lg, int n_split,
    const float4* __restrict__ part_o, const float2* __restrict__ part_ml) {
  constexpr int NG = D / 8;
  const int l = threadIdx.x & 63, lq = l & 31, hi = l >> 5;
  const int grp = (blockIdx.x % (NG / 4)) * 4 + (threadIdx.x >> 6);
  const int64_t u = blockIdx.x / (NG / 4);  // (request, unit, KV head)
  const int g = (int)(u % hkv);
  const int unit = (int)(u / hkv % max_units), b = (int)(u / hkv / max_units);
  const int64_t r0 = cu_rows[b];
  const int nr = cu_rows[b + 1] - (int)r0;
  const int64_t nqv = (int64_t)max(nr, 0) << lg;
  if ((int64_t)unit * kQv >= nqv) return;
  const int64_t qv = (int64_t)unit * kQv + lq;
  const int64_t grow = r0 + (qv >> lg);
  const int head = (g << lg) + (int)(qv & ((1 << lg) - 1));
  float4 x[kMaxSplit];
  float2 ml[kMaxSplit];
#pragma unroll
  for (int s = 0; s < kMaxSplit; ++s) {
    const int64_t slot = u * n_split + min(s, n_split - 1);
    ml[s] = part_ml[slot * kQv + lq];
    x[s] = part_o[(slot * NG + grp) * 64 + l];
  }
  float mx = -1e30f;
#pragma unroll
  for (int s = 0; s < kMaxSplit; ++s) mx = fmaxf(mx, ml[s].x);
  float lt = 0.f;
  float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
  for (int s = 0; s < kMaxSplit; ++s) {
    const float f = s < n_split ? __builtin_amdgcn_exp2f(ml[s].x - mx) : 0.f;
    lt += f * ml[s].y;
    a.x += f * x[s].x;
    a.y += f * x[s].y;
    a.z += f * x[s].z;
    a.w += f * x[s].w;
  }
  if (qv >= nqv || grow >= n_rows) return;
  const float inv = lt > 0.f ? 1.f / lt : 0.f;
  uint16_t* op = out + (grow * hq + head) * D + 8 * grp + 4 * hi;
  *reinterpret_cast<uint2*>(op) =
      make_uint2(pack_bf16x2(a.x * inv, a.y * inv), pack_bf16x2(a.z * inv, a.w * inv));
  if (lse && grp == 0 && hi == 0)
    lse[grow * hq + head] = lt > 0.f ? (mx + log2f(lt)) * kLn2 : -INFINITY;
}

}  // namespace

// 32-vector units of a call (per request, KV head and 32 query vectors; no request has more
// rows than there are, max_rows is only a bound) and key tiles of its longest request.
static void unit_counts(const AttnShape& s, int64_t n_rows, int64_t n_kv_rows, int64_t& per_req,
                        int64_t& units, int64_t& tiles) {
  int lg = 0;
  while ((1 << lg) < s.hq / s.hkv) ++lg;
  per_req = ((std::min<int64_t>(s.max_rows, n_rows) << lg) + kQv - 1) / kQv;
  units = per_req * s.hkv * s.batch;
  tiles = (std::min<int64_t>(s.max_kv, n_kv_rows) + kKeys - 1) / kKeys;
}

// Where splitting the keys over waves beats sharing tiles between them (whole calls, us, this
// kernel against the shared-tile one).
//  * Explicit key positions: 64 units x 35 tiles 14.5 / 65.6; 64 x 322 30 / 548; 256 x 36
//    16.1 / 66.6; 256 x 1028 228 / 1748; 1024 x 9 23.3 / 23.7, x 50 67 / 93; 2048 x 9 31.7 /
//    31.3; 4096 x 9 82 / 57; 4096 x 66 315 / 276.  Beyond 1024 units over long ranges the
//    shared-tile kernel's blocks come to fill the chip too (2048 units: one round of two per
//    CU): head size 128, 1536 x 66 120 / 137, 1792 x 66 138 / 137, x 100 191 / 203, x 200 368 /
//    408, 1920 x 66 156 / 138, 2048 x 66 161 / 138, x 100 214 / 203; head size 64, 2048 x 66
//    101 / 114, x 200 255 / 331.  Short ranges at head size 128, where blocks that
//    no longer fit the chip at once start for little work: 512 x 3 11.8 / 12.3, 720 x 6 17.7 /
//    16.7, 720 x 8 20.1 / 19.8, 1024 x 3 15.5 / 13.5, 720 x 12 24.9 / 26.5 (head size 64, smaller
//    blocks: 1024 x 3 7.7 / 10.3).
//  * Causal rows (half the tiles are visible on average; their shared-tile kernel adapts its
//    grid): units x tiles at head size 128 (with the re-positioning and scatter before it)
//    138 x 18 21 / 38; 523 x 50 45 / 49; 1024 x 16 37 / 41; 2560 x 4 46 / 49; 1152 x 34 60 /
//    53; 829 x 82 73 / 58.  At head size 64: 680 x 66 38 / 42; 1600 x 162 113 / 79.
bool use_keysplit(const AttnShape& s, int64_t n_rows, int64_t n_kv_rows, bool kv_pos) {
  int64_t per_req, units, tiles;
  unit_counts(s, n_rows, n_kv_rows, per_req, units, tiles);
  if (kv_pos) {
    if (s.d == 128 && units > 512 && tiles <= 8) return false;
    return units <= 1024 || (units <= (s.d == 64 ? 2048 : 1792) && tiles >= 64);
  }
  return (double)units * (double)tiles * s.d <= 28672.0 * 128;
}

// Waves per block: 8 where a wave gets several tiles; short key ranges take smaller blocks, which
// start and combine for fewer waves.  (At head size 64 they also fit beside each other on a CU;
// at 128 the smaller forms take more than 256 registers, accumulators included, so a SIMD holds
// one wave of them: one 4-wave or two 2-wave blocks per CU.)  2048 units x 9 tiles: 45.5, 42.6, 31.6 us with 8, 4, 2 waves;
// 64 x 9: 8.3, 8.2, 9.3; 64 x 35: 14.3, 16.2, 25.0; 371 x 34: 32.7, 35.0, 35.2.
int keysplit_waves(const AttnShape& s, int64_t n_rows, int64_t n_kv_rows) {
  int64_t per_req, units, tiles;
  unit_counts(s, n_rows, n_kv_rows, per_req, units, tiles);
  return tiles >= 32 ? 8 : units <= 512 ? 4 : 2;
}

hipError_t launch_attn_keysplit(void* out, float* lse, const void* q, const int32_t* row_pos,
                                int64_t n_rows, const int32_t* cu_rows, const void* k_cache,
                                const void* v_cache, int64_t n_kv_rows, int64_t kv_row_stride,
                                const int32_t* cu_kv, const int32_t* kv_pos, const AttnShape& s,
                                float scale, void* ws, hipStream_t stream,
                                const QueryRot& qrot) {
  int lg = 0;
  while ((1 << lg) < s.hq / s.hkv) ++lg;
  int64_t max_units, units, tiles;
  unit_counts(s, n_rows, n_kv_rows, max_units, units, tiles);
  const int KW = keysplit_waves(s, n_rows, n_kv_rows);
  // Key ranges are cut over blocks where units leave three quarters of the CUs idle and a
  // cut wave still has two tiles (64 units x 322 tiles: 69 -> 30 us with 4 cuts, 36 with 8;
  // 8 x 130: 20.7 -> 10.8; 64 x 35: no gain, the merge costs what it saves).  At most 256 partials:
  // the workspace that a call of more than 64 keys brings always holds them.
  int n_split = 1;
  if (units * 4 <= 256 && tiles >= 64)
    n_split = (int)std::min<int64_t>(std::min<int64_t>(kMaxSplit, 256 / units), tiles / 16);
  const size_t slots = (size_t)units * n_split;
  float4* part_o = static_cast<float4*>(ws);
  float2* part_ml = reinterpret_cast<float2*>(static_cast<char*>(ws) + slots * kQv * s.d * 4);
  const int64_t blocks = units * n_split;
  if (blocks > 0x7fffffff) return hipErrorInvalidConfiguration;
  const dim3 grid((unsigned)blocks);
  const bool rot = qrot.table != nullptr;
  const float2* rtab = reinterpret_cast<const float2*>(qrot.table);
#define QCF_KS(D, Q, P, R)                                                                         \
  attn_keysplit_kernel<D, Q, P, R><<<grid, Q * 64, 0, stream>>>(                                  \
      static_cast<uint16_t*>(out), lse, static_cast<const uint16_t*>(q), row_pos, n_rows, cu_rows,  \
      static_cast<const uint16_t*>(k_cache), static_cast<const uint16_t*>(v_cache), n_kv_rows,     \
      kv_row_stride, cu_kv, kv_pos, (int)max_units, s.hkv, s.hq, lg, scale * kLog2e, n_split,      \
      part_o, part_ml, qrot.src, qrot.n_src, rtab, (int)qrot.n_table)
#define QCF_KSK(D, Q)                                                                              \
  do {                                                                                             \
    if (kv_pos) QCF_KS(D, Q, true, false);                                                         \
    else if (rot) QCF_KS(D, Q, false, true);                                                       \
    else QCF_KS(D, Q, false, false);                                                               \
  } while (0)
#define QCF_KSD(D)                                                                                 \
  do {                                                                                             \
    if (KW == 8) QCF_KSK(D, 8);                                                                    \
    else if (KW == 4) QCF_KSK(D, 4);                                                               \
    else QCF_KSK(D, 2);                                                                            \
    if (n_split > 1)                                                                               \
      attn_keysplit_merge_kernel<D><<<dim3((unsigned)(units * (D / 32))), 256, 0,               \
                                      stream>>>(static_cast<uint16_t*>(out), lse, n_rows, cu_rows,  \
                                                (int)max_units, s.hkv, s.hq, lg, n_split,           \
                                                part_o, part_ml);                                  \
  } while (0)
  if (s.d == 64) QCF_KSD(64); else QCF_KSD(128);
#undef QCF_KSD
#undef QCF_KSK
#undef QCF_KS
  return hipGetLastError();
}

}  // namespace qcf
