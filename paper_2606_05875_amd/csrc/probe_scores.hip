// Per-token importance of a critical layer (eq. single_layer_importance) and
// its sum over the critical layers (eq. critical_layer_importance).
//
// I(t) = sum_{i,h} softmax_t(q_{i,h} . k_{t,g(h)} * scale) needs every query
// row's softmax denominator over all N context keys before any column can be
// summed, so the bf16 path runs in three launches over the same grid of
// (KV head, 256-query-vector tile, key split, request) blocks, the head
// fastest, with the splits chosen for about 512 blocks:
//   stats   : each of the 8 waves holds 32 query vectors of one KV-head group
//             in registers; the split's keys pass through LDS (128 at a time,
//             the next ones prefetched into registers; long splits: a ring of
//             64-key stages) in 32-key products, and every vector keeps an
//             online (max, sum); the split's base-2 log-sum-exp is written.
//   columns : the same tiles again.  Each vector's log-sum-exp over all splits
//             is merged once per block (its partials loaded together, folded
//             in split order); the logits are recomputed and each key's
//             probabilities 2^(logit - lse) summed over the tile's vectors
//             into a per-(head, tile) column buffer.
//   final   : scores[t] (+)= those column sums in (head, tile) order.
// Every block issues its loads together and waits once per K chunk: on this
// part a dependent round trip to memory costs microseconds under load.
// No block waits for another: the launches are the only global
// synchronisation.  QK^T runs on the matrix cores (v_mfma_f32_32x32x16_bf16)
// with the same operand registers either way round: the statistics take S^T =
// K Q^T (a lane owns one query vector, so its max and sum stay in the lane),
// the columns take S = Q K^T (a lane owns one key, so its sum over the query
// vectors is 16 in-lane additions and one lane swap).  The fp32 path is
// probe_scores_f32.hip.  Every reduction has a fixed order, so results are
// deterministic.
//
// With a rotation table (kRot) the keys come from the stored chunk caches and
// each is moved to its request offset on the fly (eq. pic_online): a thread
// loads rotate-half piece pairs of a key, turns them by the key's table row in
// float32 and rounds to bf16 before the LDS store -- the very bits a stored
// re-positioned key has -- so no re-positioned copy is read or waited for.
#include <math.h>

#include <algorithm>

#include "qcf_attn.h"
#include "qcf_device.h"
#include "qcf_launch.h"

namespace qcf {
namespace {

constexpr int kThreads = 256;      // final pass
constexpr int kW = 8;              // bf16 path: waves per block
constexpr int kQvTile = 32 * kW;   // query vectors per block
constexpr int kChunkKeys = 128;    // keys staged in LDS at a time
constexpr int kRing = 4;           // long splits: LDS stages of the key ring
constexpr int kRingKeys = 64;      // keys per stage
constexpr int kRingSplit = 512;    // shortest split that takes the ring
constexpr int kMaxSplits = 64;     // key splits per query tile
constexpr int kPassBlocks = 512;   // blocks aimed for when choosing the splits
constexpr int kCUs = 256;          // compute units of MI355X

struct WsLayout {
  size_t part_off, col_off, total;
  int n_qt, n_splits, split_keys, max_qv;
};

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

WsLayout ws_layout(const ProbeShape& s) {
  WsLayout w{};
  const int grp = s.hq / s.hkv;
  w.max_qv = s.max_q_len * grp;
  w.n_qt = (w.max_qv + kQvTile - 1) / kQvTile;
  // key splits of whole 32-key groups, about kPassBlocks blocks per pass -- or half as
  // many when rounding the splits to 32 keys would leave more of the last round of
  // kCUs-block slots idle (blocks of equal work then finish together)
  const int64_t per_split = (int64_t)std::max(1, w.n_qt) * s.hkv * std::max(1, s.batch);
  const int ctx = std::max(1, s.max_ctx_len);
  auto splits_for = [&](int64_t target, int& keys) {
    const int want = (int)std::min<int64_t>(
        kMaxSplits, std::max<int64_t>(1, (target + per_split - 1) / per_split));
    keys = ((ctx + want - 1) / want + 31) / 32 * 32;
    return (ctx + keys - 1) / keys;
  };
  auto idle = [&](int splits) {
    const int64_t blocks = per_split * splits;
    return (double)(((blocks + kCUs - 1) / kCUs) * kCUs - blocks) / (double)blocks;
  };
  int keys_a = 0, keys_b = 0;
  // a batch aims at four times as many blocks: the splits are cut from the longest context,
  // so shorter requests leave splits empty, and shorter splits even out the busy blocks
  // (ragged 16-request batch: scores + selection 0.34 -> 0.30 ms)
  const int64_t target = (int64_t)kPassBlocks * (s.batch > 1 ? 4 : 1);
  const int sa = splits_for(target, keys_a), sb = splits_for(target / 2, keys_b);
  const bool half = idle(sb) < idle(sa);
  w.split_keys = half ? keys_b : keys_a;
  w.n_splits = half ? sb : sa;
  const size_t nb = (size_t)s.batch * s.hkv;
  // both regions grow with the shape (the split region is sized for the most
  // splits), so a workspace sized for one call serves any smaller one
  w.part_off = 0;
  w.col_off = align256(nb * kMaxSplits * w.max_qv * sizeof(float));
  w.total = w.col_off + align256(nb * (size_t)w.n_qt * s.max_ctx_len * sizeof(float));
  return w;
}

__device__ __forceinline__ float2 combine_ml(float2 a, float2 b) {
  const float m = fmaxf(a.x, b.x);
  if (m == -INFINITY) return make_float2(-INFINITY, 0.f);
  return make_float2(m, a.y * exp2f(a.x - m) + b.y * exp2f(b.x - m));
}

// ---------------------------------------------------------------- bf16 passes
template <int D, bool kCols, bool kRot>
__global__ __launch_bounds__(kW * 64) void scores_pass_bf16(
    float* __restrict__ part, float* __restrict__ colp, const uint16_t* __restrict__ q,
    int64_t n_q_rows, const uint16_t* __restrict__ k, int64_t n_kv_rows, int64_t k_stride,
    const int32_t* __restrict__ key_rot, const float2* __restrict__ rot_tab, int n_rot,
    const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_kv,
    const int32_t* __restrict__ ctx_len, int hq, int hkv, int lg, int n_qt, int n_splits,
    int split_keys, int max_qv, int max_ctx, float scale2) {
  constexpr int KSTR = D + 8;                          // padded LDS row (conflict-free reads)
  constexpr int CPR = D / 8;                           // 16-byte pieces per K row
  constexpr int PER = kChunkKeys * CPR / (kW * 64);    // pieces per thread per chunk
  constexpr int SPL = kMaxSplits / 2;                  // splits per lane in the merge
  constexpr int HP = CPR / 2;                          // 16-byte pieces per rotate-half
  constexpr int PU = PER / 2;                          // piece pairs per thread per chunk
  static_assert(PER % 2 == 0, "rotation works on whole piece pairs");
  __shared__ __attribute__((aligned(16))) uint16_t k_lds[kChunkKeys * KSTR];
  __shared__ float lse_l[kCols ? kQvTile : 1];
  __shared__ float red[kCols ? kW : 1][kCols ? kChunkKeys : 1];

  // block -> (KV head, query tile, split, request) with the head fastest:
  // blocks are dealt to the XCDs in turn, so with 8 KV heads every block of a
  // head runs on one XCD and its Q and split statistics are shared in that L2
  const int g = blockIdx.x % hkv;
  const int rest = blockIdx.x / hkv;
  const int qt = rest % n_qt, split = (rest / n_qt) % n_splits, b = rest / (n_qt * n_splits);
  const int64_t q0 = cu_q[b];
  const int nqv = min((cu_q[b + 1] - (int)q0) << lg, max_qv);
  if (qt * kQvTile >= nqv) return;
  const int64_t k0 = cu_kv[b];
  const int N = ctx_len[b];
  const int key_lo = split * split_keys;
  const int key_hi = min(N, key_lo + split_keys);
  if (kCols && key_lo >= key_hi) return;  // no keys: no columns (an empty split's statistics are still written)
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l = threadIdx.x & 63, lq = l & 31, hi = l >> 5;
  const int qv = qt * kQvTile + 32 * w + lq;
  const int64_t qrow = q0 + (qv >> lg);
  const bool valid = qv < nqv && qrow < n_q_rows;
  const bool live = __ballot(valid) != 0;  // the wave has a real query vector
  const int head = g * (1 << lg) + (qv & ((1 << lg) - 1));

  // Every load below is unconditional, its indices clamped to real rows: a
  // load under a lane condition gets a wait of its own, which serialises the
  // round trips.  Keys past the split and query vectors past the tile are
  // masked where their products are used, so the rows read for them only
  // have to be finite.
  uint4 buf[PER];
  // with kRot a thread owns piece pairs (j .. j+7, j+D/2 .. j+D/2+7) of a key,
  // and the key's rotation-table row is loaded ahead of its pieces, so its
  // (cos, sin) can be fetched (fetch_cs) while the pieces are still in flight
  int rot_i[kRot ? PU : 1];
  uint4 csv[kRot ? 4 * PU : 1];
  auto fetch = [&](int c0) {
    if constexpr (kRot) {
      int64_t rows[PU];
#pragma unroll
      for (int i = 0; i < PU; ++i) {
        const int c = threadIdx.x + i * kW * 64;
        rows[i] = min(k0 + min(c0 + c / HP, key_hi - 1), n_kv_rows - 1);
        rot_i[i] = key_rot[rows[i]];
      }
#pragma unroll
      for (int i = 0; i < PU; ++i) {
        const int ch = (threadIdx.x + i * kW * 64) % HP;
        const uint16_t* kp = k + rows[i] * k_stride + (int64_t)g * D + ch * 8;
        buf[2 * i] = ld16(kp);
        buf[2 * i + 1] = ld16(kp + D / 2);
      }
    } else {
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const int c = threadIdx.x + i * kW * 64;
        const int key = min(c0 + c / CPR, key_hi - 1), ch = c % CPR;
        const int64_t row = min(k0 + key, n_kv_rows - 1);
        buf[i] = ld16(k + row * k_stride + (int64_t)g * D + ch * 8);
      }
    }
  };
  auto fetch_cs = [&]() {
    if constexpr (kRot) {
#pragma unroll
      for (int i = 0; i < PU; ++i) {
        const int ch = (threadIdx.x + i * kW * 64) % HP;
        const float2* cp = rot_tab + (int64_t)min(max(rot_i[i], 0), n_rot - 1) * (D / 2) + ch * 8;
#pragma unroll
        for (int v = 0; v < 4; ++v) csv[4 * i + v] = ld16(cp + 2 * v);
      }
    }
  };
  if (key_lo < key_hi) fetch(key_lo);
  bf16x8 qreg[D / 16];
  {
    const uint16_t* qp = q + min(qrow, n_q_rows - 1) * (int64_t)hq * D + (int64_t)head * D + 8 * hi;
#pragma unroll
    for (int st = 0; st < D / 16; ++st) qreg[st] = as_bf16x8(ld16(qp + 16 * st));
  }
  if (kRot && key_lo < key_hi) fetch_cs();
  float lse_v[kCols ? 16 : 1];
  if (kCols) {
    // the vector's base-2 log-sum-exp over every split: lanes l (even splits)
    // and l^32 (odd splits) fold theirs in split order, then even + odd; its
    // padding rows get a reference that sends every exponential to 0
    // (branch-free, so every load is issued before the first one is used;
    // an empty split's -inf and a masked slot count as a floor with weight 0)
    const float* pg = part + (int64_t)(b * hkv + g) * n_splits * max_qv + min(qv, max_qv - 1);
    float x[SPL];
#pragma unroll
    for (int j = 0; j < SPL; ++j) x[j] = pg[min(2 * j + hi, n_splits - 1) * max_qv];
    asm volatile("" ::: "memory");  // all of them in flight before the first is used
    constexpr float kFloor = -1e30f;
    float mx = kFloor, ls = 0.f;
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
      const bool ok = valid && 2 * j + hi < n_splits && x[j] > kFloor;
      const float xj = ok ? x[j] : kFloor;
      const float mn = fmaxf(mx, xj);
      ls = ls * __builtin_amdgcn_exp2f(mx - mn) + (ok ? __builtin_amdgcn_exp2f(xj - mn) : 0.f);
      mx = mn;
    }
    if (ls == 0.f) mx = -INFINITY;
    const float2 mine = make_float2(mx, ls);
    const float2 other = make_float2(__shfl_xor(mx, 32, 64), __shfl_xor(ls, 32, 64));
    const float2 ml = hi == 0 ? combine_ml(mine, other) : combine_ml(other, mine);
    if (hi == 0) lse_l[32 * w + lq] = (valid && ml.y > 0.f) ? ml.x + __builtin_amdgcn_logf(ml.y) : 1e30f;
    __syncthreads();
    // S layout: value v of a lane belongs to query vector 8(v>>2)+4hi+(v&3) of the wave
#pragma unroll
    for (int v = 0; v < 16; ++v) lse_v[v] = lse_l[32 * w + 8 * (v >> 2) + 4 * hi + (v & 3)];
  }
  float m = -INFINITY, ls = 0.f;
  for (int c0 = key_lo; c0 < key_hi; c0 += kChunkKeys) {
    if (c0 > key_lo) __syncthreads();  // the previous chunk (and its sums) are no longer read
    if constexpr (kRot) {
      // the re-positioned key, rounded to bf16 as a stored re-positioned key is
#pragma unroll
      for (int i = 0; i < PU; ++i) {
        const int c = threadIdx.x + i * kW * 64;
        float x1[8], x2[8], y1[8], y2[8];
        Vec16<uint16_t>::unpack(buf[2 * i], x1);
        Vec16<uint16_t>::unpack(buf[2 * i + 1], x2);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const uint4 cv = csv[4 * i + e / 2];
          const float2 cs = (e & 1) ? make_float2(__uint_as_float(cv.z), __uint_as_float(cv.w))
                                    : make_float2(__uint_as_float(cv.x), __uint_as_float(cv.y));
          rope_pair(x1[e], x2[e], cs, y1[e], y2[e]);
        }
        uint16_t* dst = &k_lds[(c / HP) * KSTR + (c % HP) * 8];
        st16(dst, Vec16<uint16_t>::pack(y1));
        st16(dst + D / 2, Vec16<uint16_t>::pack(y2));
      }
    } else {
#pragma unroll
      for (int i = 0; i < PER; ++i) {
        const int c = threadIdx.x + i * kW * 64;
        st16(&k_lds[(c / CPR) * KSTR + (c % CPR) * 8], buf[i]);
      }
    }
    __syncthreads();
    const bool more = c0 + kChunkKeys < key_hi;
    if (more) fetch(c0 + kChunkKeys);  // in flight during this chunk's work
    const int n_keys = min(key_hi - c0, kChunkKeys);
    const int n_grp = (n_keys + 31) / 32;
    for (int kg = 0; kg < n_grp; ++kg) {
      if (kRot && more && kg == 1) fetch_cs();  // the next chunk's rotations, behind its pieces
      if (!live) {
        // a wave whose 32 query vectors are all padding (the request's last tile is
        // partly filled) adds nothing: it only takes part in the loads and barriers
        if (kCols && hi == 0) red[w][kg * 32 + lq] = 0.f;
        continue;
      }
      bf16x8 a[D / 16];
#pragma unroll
      for (int st = 0; st < D / 16; ++st) a[st] = as_bf16x8(ld16(&k_lds[(kg * 32 + lq) * KSTR + 8 * hi + 16 * st]));
      const int kt0 = c0 + kg * 32;
      f32x16 sacc = f32x16{};
      if (!kCols) {
        // S^T: value v of this lane is key 8(v>>2)+4hi+(v&3) of the group for the
        // lane's query vector; logits go to the log2 domain, keys past the split
        // are masked
#pragma unroll
        for (int st = 0; st < D / 16; ++st)
          sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[st], qreg[st], sacc, 0, 0, 0);
        if (kt0 + 32 > key_hi) {
#pragma unroll
          for (int v = 0; v < 16; ++v)
            if (kt0 + 8 * (v >> 2) + 4 * hi + (v & 3) >= key_hi) sacc[v] = -INFINITY;
        }
        float mt = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) mt = fmaxf(mt, sacc[v]);
        const float mn = fmaxf(m, mt * scale2);
        if (mn != -INFINITY) {
          float acc = 0.f;
#pragma unroll
          for (int v = 0; v < 16; ++v) acc += __builtin_amdgcn_exp2f(fmaf(sacc[v], scale2, -mn));
          ls = ls * __builtin_amdgcn_exp2f(m - mn) + acc;
          m = mn;
        }
      } else {
        // S: this lane's key kt0 + lq, value v for query vector 8(v>>2)+4hi+(v&3)
#pragma unroll
        for (int st = 0; st < D / 16; ++st)
          sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qreg[st], a[st], sacc, 0, 0, 0);
        float cs = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) cs += __builtin_amdgcn_exp2f(fmaf(sacc[v], scale2, -lse_v[v]));
        const float cs_other = __shfl_xor(cs, 32, 64);
        if (hi == 0) red[w][kg * 32 + lq] = kt0 + lq < key_hi ? cs + cs_other : 0.f;
      }
    }
    if (kCols) {
      __syncthreads();
      if (threadIdx.x < n_keys) {
        float acc = 0.f;
#pragma unroll
        for (int ww = 0; ww < kW; ++ww) acc += red[ww][threadIdx.x];
        colp[((int64_t)(b * hkv + g) * n_qt + qt) * max_ctx + c0 + threadIdx.x] = acc;
      }
    }
  }
  if (!kCols) {
    // lanes l and l^32 hold disjoint keys of the same query vector; the split's
    // base-2 log-sum-exp log2(sum_t 2^(logit_t)) = max + log2(sum) (-inf: no keys)
    const float2 ml = combine_ml(make_float2(m, ls), make_float2(__shfl_xor(m, 32, 64), __shfl_xor(ls, 32, 64)));
    if (valid && hi == 0)
      part[((int64_t)(b * hkv + g) * n_splits + split) * max_qv + qv] =
          ml.y > 0.f ? ml.x + __builtin_amdgcn_logf(ml.y) : -INFINITY;
  }
}

// ---------------------------------------------------------------- bf16 passes, long splits
// The two passes for splits of 512 keys and more (stored keys only): the same tiles, sums and
// order, so the same bits.  Bound: a wave's vector instructions and products in turn -- the
// pass above issues a group's 8 dependent products in a burst and then its 16 exponentials,
// and on 4 waves per SIMD its time is the sum of both (86.7 us for 128 query rows, 64/8 heads,
// 32768 keys; 60 with one product of eight, 73 without the exponentials).  Here S of the next
// group is fenced in between the exponentials of this one, product by product, and the keys
// come through a 4-stage LDS ring (64 keys, buffer loads into LDS three stages ahead) instead
// of registers, which leaves room for both score tiles at two blocks per CU.  Scores and
// selection at that size 180 -> 170 us, a ragged 16-request batch 322 -> 287 us.  With 128-key
// stages (one block per CU) 188 and 371 us: nothing hides a block's start.  Where the line lies
// (score calls, us, the pass above / this one, 64/8 heads of 128): 128 query rows, splits of 64
// keys 26.9 / 28.9, 128 29.2 / 32.2, 192 34.9 / 35.6, 256 39.8 / 41.2, 384 47.6 / 47.1, 512 58.2 /
// 57.3, 768 74.9 / 73.5; one tile of 64 vectors, 768 keys 40.7 / 36.0, 1056 50.6 / 43.4; 8 requests,
// 96 keys 67 / 77; head size 64, 128 rows, 256 keys 32.8 / 33.9, 512 46.1 / 44.9.  So splits of 512
// keys and more; shorter ones keep the pass above, as do keys rotated on the fly.  (Its wait for Q
// stands inside the loop: moved before it, as here, those calls gain nothing, 39.5 / 39.9 us for
// 5120 keys rotated on the fly, 62.7 / 65.4 for four requests over 128-key splits.)
template <int D, bool kCols>
__global__ __launch_bounds__(kW * 64, 4) void scores_ring_bf16(  // (4 waves per SIMD: two blocks per CU)
    float* __restrict__ part, float* __restrict__ colp, const uint16_t* __restrict__ q,
    int64_t n_q_rows, const uint16_t* __restrict__ k, int64_t n_kv_rows, int64_t k_stride,
    const int32_t* __restrict__ cu_q, const int32_t* __restrict__ cu_kv,
    const int32_t* __restrict__ ctx_len, int hq, int hkv, int lg, int n_qt, int n_splits,
    int split_keys, int max_qv, int max_ctx, float scale2) {
  constexpr int CPR = D / 8;                // 16-byte pieces per K row
  constexpr int RB = D * 2;                 // bytes per LDS row
  constexpr int ST = kRingKeys * RB;        // bytes per stage
  constexpr int RPS = 64 / CPR;             // rows per 64-lane transfer
  constexpr int SPW = kRingKeys / RPS / kW;  // transfers per wave and chunk
  constexpr int SPL = kMaxSplits / 2;       // splits per lane in the merge
  __shared__ __attribute__((aligned(1024))) uint8_t k_lds[kRing * ST];
  __shared__ float lse_l[kCols ? kQvTile : 1];
  __shared__ float red[kCols ? 3 : 1][kCols ? kW : 1][kCols ? kRingKeys : 1];

  // block -> (KV head, query tile, split, request) with the head fastest:
  // blocks are dealt to the XCDs in turn, so with 8 KV heads every block of a
  // head runs on one XCD and its Q and split statistics are shared in that L2
  const int g = blockIdx.x % hkv;
  const int rest = blockIdx.x / hkv;
  const int qt = rest % n_qt, split = (rest / n_qt) % n_splits, b = rest / (n_qt * n_splits);
  const int64_t q0 = cu_q[b];
  const int nqv = min((cu_q[b + 1] - (int)q0) << lg, max_qv);
  if (qt * kQvTile >= nqv) return;
  const int64_t k0 = cu_kv[b];
  const int N = ctx_len[b];
  const int key_lo = split * split_keys;
  const int key_hi = min(N, key_lo + split_keys);
  if (kCols && key_lo >= key_hi) return;  // no keys: no columns (an empty split's statistics are still written)
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l = threadIdx.x & 63, lq = l & 31, hi = l >> 5;
  const int qv = qt * kQvTile + 32 * w + lq;
  const int64_t qrow = q0 + (qv >> lg);
  const bool valid = qv < nqv && qrow < n_q_rows;
  const bool live = __ballot(valid) != 0;  // the wave has a real query vector
  const int head = g * (1 << lg) + (qv & ((1 << lg) - 1));

  // Keys arrive by buffer loads with an LDS destination, three chunks ahead; the descriptor ends
  // at the last key that exists, past it rows read as zeros (keys past the split are masked
  // where their products are used).  Chunk c of LDS row r sits at c ^ (r % 16) (D = 64: c ^ (r /
  // 2 % 8)): conflict-free fragment reads without padding.
  const uint32_t row_b = (uint32_t)(k_stride * 2);
  const int n_chunk = key_lo < key_hi ? (key_hi - key_lo + kRingKeys - 1) / kRingKeys : 0;
  const int64_t kfirst = min(k0 + key_lo, n_kv_rows - 1);
  const int64_t kleft = min((int64_t)key_hi - key_lo, n_kv_rows - kfirst);
  const int dr = RPS * w + l / CPR, dc = l % CPR;  // transfer i fills rows dr + RPS kW i
  const uint32_t koff = (uint32_t)dr * row_b + (dc ^ (D == 128 ? dr & 15 : (dr >> 1) & 7)) * 16;
  const uint32_t k_base = lds_addr(k_lds);
  const uint16_t* kb = k + kfirst * k_stride + (int64_t)g * D;
  auto issue = [&](int c) {
    const int64_t rows = min(kleft - (int64_t)c * kRingKeys, (int64_t)kRingKeys);
    const i32x4 rk = make_rsrc(kb + (rows > 0 ? (int64_t)c * kRingKeys * k_stride : 0),
                               rows > 0 ? (uint32_t)(rows - 1) * row_b + RB : 0u);
#pragma unroll
    for (int i = 0; i < SPW; ++i) {
      const uint32_t soff = (uint32_t)(RPS * kW * i) * row_b;
      dma16(rk, koff + soff, k_base + (uint32_t)((c & (kRing - 1)) * ST + (w + kW * i) * 1024));
    }
  };
  if (n_chunk > 0) {
    issue(0);
    issue(1);
    issue(2);
  }
  bf16x8 qreg[D / 16];
  {
    const uint16_t* qp = q + min(qrow, n_q_rows - 1) * (int64_t)hq * D + (int64_t)head * D + 8 * hi;
#pragma unroll
    for (int st = 0; st < D / 16; ++st) qreg[st] = as_bf16x8(ld16(qp + 16 * st));
  }
  float lse_v[kCols ? 16 : 1];
  if (kCols) {
    // the vector's base-2 log-sum-exp over every split: lanes l (even splits)
    // and l^32 (odd splits) fold theirs in split order, then even + odd; its
    // padding rows get a reference that sends every exponential to 0
    // (branch-free, so every load is issued before the first one is used;
    // an empty split's -inf and a masked slot count as a floor with weight 0)
    // loads are unconditional, from clamped rows: a load under a lane condition gets a wait of its own
    const float* pg = part + (int64_t)(b * hkv + g) * n_splits * max_qv + min(qv, max_qv - 1);
    float x[SPL];
#pragma unroll
    for (int j = 0; j < SPL; ++j) x[j] = pg[min(2 * j + hi, n_splits - 1) * max_qv];
    asm volatile("" ::: "memory");  // all of them in flight before the first is used
    constexpr float kFloor = -1e30f;
    float mx = kFloor, ls = 0.f;
#pragma unroll
    for (int j = 0; j < SPL; ++j) {
      const bool ok = valid && 2 * j + hi < n_splits && x[j] > kFloor;
      const float xj = ok ? x[j] : kFloor;
      const float mn = fmaxf(mx, xj);
      ls = ls * __builtin_amdgcn_exp2f(mx - mn) + (ok ? __builtin_amdgcn_exp2f(xj - mn) : 0.f);
      mx = mn;
    }
    if (ls == 0.f) mx = -INFINITY;
    const float2 mine = make_float2(mx, ls);
    const float2 other = make_float2(__shfl_xor(mx, 32, 64), __shfl_xor(ls, 32, 64));
    const float2 ml = hi == 0 ? combine_ml(mine, other) : combine_ml(other, mine);
    if (hi == 0) lse_l[32 * w + lq] = (valid && ml.y > 0.f) ? ml.x + __builtin_amdgcn_logf(ml.y) : 1e30f;
    __syncthreads();
    // S layout: value v of a lane belongs to query vector 8(v>>2)+4hi+(v&3) of the wave
#pragma unroll
    for (int v = 0; v < 16; ++v) lse_v[v] = lse_l[32 * w + 8 * (v >> 2) + 4 * hi + (v & 3)];
  }
  // Q has to be there before the loop: the compiler's wait for it at the products would count
  // later loads too
#pragma unroll
  for (int st = 0; st < D / 16; ++st) asm volatile("" : "+v"(qreg[st]));
  float m = -INFINITY, ls = 0.f;
  constexpr int NS = D / 16;   // products per group
  constexpr int EG = 16 / NS;  // elements of a group per product
  const int ky = D == 128 ? lq & 15 : (lq >> 1) & 7;
  const int krd = lq * RB + (hi ^ (ky & 1)) * 16 + (ky >> 1) * 32;
  auto frag = [&](const uint8_t* kl, int st) { return as_bf16x8(ld16(kl + (krd ^ (st << 5)))); };
  auto mfma = [&](const bf16x8& a, int st, const f32x16& c) {
    return kCols ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(qreg[st], a, c, 0, 0, 0)
                 : __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qreg[st], c, 0, 0, 0);
  };
  // exponential argument of value v: statistics (S^T: key 8(v>>2)+4hi+(v&3) of the group, the
  // lane's vector) relative to the running reference, columns (S: the lane's key, vector
  // 8(v>>2)+4hi+(v&3)) to the vector's log-sum-exp
  auto arg = [&](const f32x16& s, int v, float nm) {
    return fmaf(s[v], scale2, kCols ? -lse_v[kCols ? v : 0] : nm);
  };
  // S(next) beside the exponentials of S(cur): groups fenced with sched_barrier, one product each,
  // with its K fragment read PF groups ahead, so the matrix cores and the vector ALUs run
  // side by side inside a wave; returns the sum of the exponentials.
  auto fused = [&](const uint8_t* kl, f32x16& sn, const f32x16& sc, float nm) {
    constexpr int PF = 4;
    bf16x8 a[NS];
#pragma unroll
    for (int i = 0; i < PF; ++i) a[i] = frag(kl, i);
    float x[16], p[16], sum = 0.f;
#pragma unroll
    for (int v = 0; v < EG; ++v) x[v] = arg(sc, v, nm);
#pragma unroll
    for (int i = 0; i < NS; ++i) {
      __builtin_amdgcn_sched_barrier(0);
      if (i + PF < NS) a[i + PF] = frag(kl, i + PF);
      sn = mfma(a[i], i, i == 0 ? f32x16{} : sn);
#pragma unroll
      for (int v = EG * (i + 1); v < EG * (i + 2) && v < 16; ++v) x[v] = arg(sc, v, nm);
#pragma unroll
      for (int v = EG * i; v < EG * (i + 1); ++v) {
        p[v] = __builtin_amdgcn_exp2f(x[v]);
        asm volatile("" : "+v"(p[v]));  // stays in its group
      }
      if (i > 0) {
#pragma unroll
        for (int v = EG * (i - 1); v < EG * i; ++v) sum += p[v];
      }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int v = EG * (NS - 1); v < 16; ++v) sum += p[v];
    return sum;
  };
  f32x16 s0, s1;
  auto colsum = [&](int c) {  // the column sums of chunk c over the waves, after a barrier
    if constexpr (kCols) {
      const int t = threadIdx.x, key = key_lo + c * kRingKeys + t;
      if (t < kRingKeys && key < key_hi) {
        float acc = 0.f;
#pragma unroll
        for (int ww = 0; ww < kW; ++ww) acc += red[c % 3][ww][t];
        colp[((int64_t)(b * hkv + g) * n_qt + qt) * max_ctx + key] = acc;
      }
    }
  };
  auto meet = [&]() {  // the next chunk has landed (two younger ones may be on their way); the block meets
    asm volatile("" ::: "memory");
    wait_vm_lgkm0<2 * SPW>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  if (kCols && !live) {  // a wave without real query vectors adds nothing: it only loads and meets
#pragma unroll
    for (int i = 0; i < (kCols ? 3 : 0); ++i) red[i][w][l] = 0.f;
  }
  if (n_chunk > 0) {
    meet();
    if (live) {
#pragma unroll
      for (int st = 0; st < NS; ++st) s0 = mfma(frag(k_lds, st), st, st == 0 ? f32x16{} : s0);
    }
  }
  // One 32-key group: its exponentials, beside the products of the wave's next group at kl.
  auto group = [&](int c, int kg, const uint8_t* kl, f32x16& sc, f32x16& sn) {
    const int kt0 = key_lo + c * kRingKeys + kg * 32;
    if constexpr (!kCols) {
      if (kt0 + 32 > key_hi) {  // keys past the split are masked
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (kt0 + 8 * (v >> 2) + 4 * hi + (v & 3) >= key_hi) sc[v] = -INFINITY;
      }
      float mt = -INFINITY;
#pragma unroll
      for (int v = 0; v < 16; ++v) mt = fmaxf(mt, sc[v]);
      const float mn = fmaxf(m, mt * scale2);
      const float sum = fused(kl, sn, sc, -mn);
      ls = mn != -INFINITY ? ls * __builtin_amdgcn_exp2f(m - mn) + sum : ls;
      m = mn;
    } else {
      const float sum = fused(kl, sn, sc, 0.f);
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(sum), __float_as_uint(sum), false, false);
      if (hi == 0) red[c % 3][w][kg * 32 + lq] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    }
  };
  // A chunk's two groups, each beside the products of the next one; the second multiplies into
  // the next chunk (past the last: zero rows, unused), so the block meets before it.
  for (int c = 0; c < n_chunk; ++c) {
    // (both stages' addresses up here: formed at their uses, the D = 128 statistics spill 20 registers)
    const uint8_t* kc = k_lds + (c & (kRing - 1)) * ST;
    const uint8_t* kn = k_lds + ((c + 1) & (kRing - 1)) * ST;
    issue(c + 3);  // into the stage of chunk c - 1, last read before the last barrier
    constexpr int GB = 32 * RB;  // LDS bytes of a group
    if (live) group(c, 0, kc + GB, s0, s1);
    meet();
    if (c > 0) colsum(c - 1);
    if (live) group(c, 1, kn, s1, s0);
  }
  wait_vm_lgkm0<0>();  // the last (zero-row) transfers, before the LDS is released
  if constexpr (kCols) {
    __syncthreads();
    if (n_chunk > 0) colsum(n_chunk - 1);
  } else {
    // lanes l and l^32 hold disjoint keys of the same query vector; the split's base-2
    // log-sum-exp is max + log2(sum) (-inf: no keys)
    const float2 ml = combine_ml(make_float2(m, ls), make_float2(__shfl_xor(m, 32, 64), __shfl_xor(ls, 32, 64)));
    if (valid && hi == 0)
      part[((int64_t)(b * hkv + g) * n_splits + split) * max_qv + qv] =
          ml.y > 0.f ? ml.x + __builtin_amdgcn_logf(ml.y) : -INFINITY;
  }
}

// ---------------------------------------------------------------- bf16 final
// scores[t] (+)= the column sums of every (KV head, query tile) of the request
// that has query vectors, head-major
__global__ __launch_bounds__(kThreads) void scores_final(float* __restrict__ scores, int accumulate,
                                                         const float* __restrict__ colp,
                                                         const int32_t* __restrict__ cu_q,
                                                         const int32_t* __restrict__ cu_kv,
                                                         const int32_t* __restrict__ ctx_len,
                                                         int64_t n_kv_rows, int hkv, int lg,
                                                         int n_qt, int max_qv, int max_ctx) {
  const int t = blockIdx.x * kThreads + threadIdx.x, b = blockIdx.y;
  if (t >= ctx_len[b]) return;
  const int64_t row = cu_kv[b] + t;
  if (row >= n_kv_rows) return;
  const int nqv = min((cu_q[b + 1] - cu_q[b]) << lg, max_qv);
  const int nt = (nqv + kQvTile - 1) / kQvTile;
  const float* cp = colp + (int64_t)b * hkv * n_qt * max_ctx + t;
  float acc = 0.f;
  for (int g = 0; g < hkv; ++g)
    for (int j = 0; j < nt; ++j) acc += cp[((int64_t)g * n_qt + j) * max_ctx];
  scores[row] = accumulate ? scores[row] + acc : acc;
}

}  // namespace

size_t probe_scores_workspace(const ProbeShape& s) {
  if (s.batch <= 0 || s.max_q_len <= 0 || s.max_ctx_len <= 0) return 256;
  const WsLayout w = ws_layout(s);
  const size_t f32 = align256((size_t)s.batch * s.hq * s.max_q_len * sizeof(float2));
  return w.total > f32 ? w.total : f32;
}

hipError_t launch_probe_scores(float* scores, int accumulate, const void* q, int64_t n_q_rows,
                               const void* k, int64_t n_kv_rows, int64_t k_row_stride,
                               const KeyRot& rot, bool bf16, const int32_t* cu_q,
                               const int32_t* cu_kv, const int32_t* ctx_len, const ProbeShape& s,
                               float scale, void* ws, hipStream_t stream, const SelectArgs* sel) {
  if (s.batch == 0 || s.max_ctx_len == 0) return hipSuccess;
  const float scale2 = scale * kLog2e;
  int lg = 0;
  while ((1 << lg) < s.hq / s.hkv) ++lg;
  const bool rt = rot.row != nullptr;
  const float2* tab = reinterpret_cast<const float2*>(rot.table);
  const int n_rot = rt ? (int)rot.n : 1;
  if (!bf16) {
    const hipError_t e = launch_scores_f32(scores, accumulate, static_cast<const float*>(q), n_q_rows,
                                           static_cast<const float*>(k), n_kv_rows, k_row_stride, rot,
                                           cu_q, cu_kv, ctx_len, s, scale, ws, stream);
    if (e != hipSuccess || !sel) return e;
    return launch_select_topk(sel->out_idx, sel->out_pos, sel->n_out, scores, n_kv_rows,
                              sel->n_seg, sel->seg_start, sel->seg_len, sel->seg_k,
                              sel->out_start, nullptr, sel->max_seg_len, stream, sel->seg_req,
                              cu_kv, s.batch);
  }
  const WsLayout w = ws_layout(s);
  if (s.batch > 65535) return hipErrorInvalidConfiguration;
  char* wb = static_cast<char*>(ws);
  float* part = reinterpret_cast<float*>(wb + w.part_off);
  float* colp = reinterpret_cast<float*>(wb + w.col_off);
  const uint16_t* qb = static_cast<const uint16_t*>(q);
  const uint16_t* kb = static_cast<const uint16_t*>(k);
  if (w.max_qv > 0 && n_q_rows > 0 && n_kv_rows > 0) {
    const int64_t nblk = (int64_t)s.hkv * w.n_qt * w.n_splits * s.batch;
    if (nblk > 0x7fffffff) return hipErrorInvalidConfiguration;
    dim3 grid((unsigned)nblk);
#define QCF_PASS(D, C, R)                                                                          \
  scores_pass_bf16<D, C, R><<<grid, kW * 64, 0, stream>>>(                                         \
      part, colp, qb, n_q_rows, kb, n_kv_rows, k_row_stride, rot.row, tab, n_rot, cu_q, cu_kv,     \
      ctx_len, s.hq, s.hkv, lg, w.n_qt, w.n_splits, w.split_keys, w.max_qv, s.max_ctx_len, scale2)
#define QCF_RING(D, C)                                                                             \
  scores_ring_bf16<D, C><<<grid, kW * 64, 0, stream>>>(                                            \
      part, colp, qb, n_q_rows, kb, n_kv_rows, k_row_stride, cu_q, cu_kv, ctx_len, s.hq, s.hkv,    \
      lg, w.n_qt, w.n_splits, w.split_keys, w.max_qv, s.max_ctx_len, scale2)
#define QCF_PASSES(D, R)     \
  do {                       \
    if (!R && ring) {        \
      QCF_RING(D, false);    \
      QCF_RING(D, true);     \
    } else {                 \
      QCF_PASS(D, false, R); \
      QCF_PASS(D, true, R);  \
    }                        \
  } while (0)
    // (a stage's byte offsets are 32-bit)
    const bool ring = w.split_keys >= kRingSplit && k_row_stride * 2 * kRingKeys < (int64_t)1 << 31;
    if (s.d == 64) {
      if (rt) QCF_PASSES(64, true); else QCF_PASSES(64, false);
    } else {
      if (rt) QCF_PASSES(128, true); else QCF_PASSES(128, false);
    }
#undef QCF_PASSES
#undef QCF_RING
#undef QCF_PASS
  }
  if (sel && sel->max_seg_len <= 1024) {
    // the column sums are added per key by the selection itself (same order)
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const ScoreCols c{colp, cu_q, cu_kv, ctx_len, n_kv_rows, s.batch, s.hkv, lg,
                      std::max(1, w.n_qt), w.max_qv, s.max_ctx_len, kQvTile, accumulate};
    return launch_select_topk_cols(scores, n_kv_rows, c, *sel, stream);
  }
  scores_final<<<dim3((s.max_ctx_len + kThreads - 1) / kThreads, s.batch), kThreads, 0, stream>>>(
      scores, accumulate, colp, cu_q, cu_kv, ctx_len, n_kv_rows, s.hkv, lg, std::max(1, w.n_qt),
      w.max_qv, s.max_ctx_len);
  if (sel) {
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return launch_select_topk(sel->out_idx, sel->out_pos, sel->n_out, scores, n_kv_rows,
                              sel->n_seg, sel->seg_start, sel->seg_len, sel->seg_k, sel->out_start,
                              nullptr, sel->max_seg_len, stream, sel->seg_req, cu_kv, s.batch);
  }
  return hipGetLastError();
}

}  // namespace qcf
