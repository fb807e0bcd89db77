// Causal attention of the recomputed rows on 4-wave blocks, two per CU (the wave step is
// that of attention.hip: 32 query vectors per wave, 64-key tiles through LDS, the same
// products in the same order, so the same bits).
//
// Why beside the 8-wave blocks: an 8-wave block fills a CU, so its start (positions, then Q and
// its rotation, while the first tiles travel: ~5 us) and its output stores (~2.5 us) leave the
// matrix cores idle, which a chunk-length block pays once per ~8 key steps and a block of a
// ragged batch once per ~44.  Two half-size blocks hide each other's ends, their waves drift
// out of step by themselves (one's products beside the other's exponentials), and a call has
// twice as many tiles to even out.  Each tile is loaded by twice as many blocks, which costs
// one very long request ~2% (its 8-wave blocks with work queues stay), and a block alone on its
// CU waits for its keys in every step (batches of few tiles take 8-wave blocks: attn_route).
// Bound: matrix cores and vector ALUs together.  A wave's step takes ~2600 cycles beside its
// neighbour's and ~2350 alone (1024 of them products: the two waves of a SIMD keep its matrix
// core ~78% busy).
//  * LDS rows are unpadded, chunks XORed by the row instead (K by row % 16, V by 4 (row % 4) at
//    head size 128), which keeps the fragment and transposing reads conflict-free: 32
//    transfers per step instead of 37, each on whole 64-byte pieces, one offset register each
//    for K and V instead of five, and no spills (padded: 4; a spill reload waits for every
//    transfer in flight).  Padded rows: 16-request batch +1.4%, 20 x 512-token layer +3.5%.
//  * Two stages each of K and V: step t requests K(t+2) and V(t+1), one transfer per two
//    products of S(t+1) (all at the head of the step: +0.5 to +1.3%), and ends by waiting
//    for them.
// Whole layer recompute, 8-wave blocks -> this kernel: 20 chunks of 512 offline 146 -> 126 us,
// 20 x 512 context at 30% 291 -> 283, 16-request batch 1835 -> 1801, 5 x 512 with 64/8 heads
// at 50% 105 -> 81, 16 x 1024 655 -> 646.
#include <limits.h>
#include <math.h>

#include <algorithm>

#include "qcf_attn.h"
#include "qcf_device.h"
#include "qcf_launch.h"

namespace qcf {
namespace {

constexpr int kW = 4;           // waves per block
constexpr int kQv = 32 * kW;    // query vectors per block
constexpr int kKT = 64;         // keys per tile

template <int D, bool kRot>
__global__ __launch_bounds__(kW * 64, 2) void attn_w4_kernel(
    uint16_t* __restrict__ out, float* __restrict__ lse, const uint16_t* __restrict__ q,
    const int32_t* __restrict__ row_pos, int64_t n_rows, const int32_t* __restrict__ cu_rows,
    const uint16_t* __restrict__ kc, const uint16_t* __restrict__ vc, int64_t n_kv_rows,
    int64_t kv_stride, const int32_t* __restrict__ cu_kv, int batch, int max_tiles, int hkv,
    int hq, int lg, float scale2, const int32_t* __restrict__ q_src, int64_t n_q_src,
    const float2* __restrict__ rtab, int n_tab) {
  constexpr int CH = D / 8;           // 16-byte chunks per LDS row
  constexpr int RPS = 64 / CH;        // rows per 64-lane transfer
  constexpr int RB = D * 2;           // bytes per LDS row
  constexpr int ST = kKT * RB;        // bytes per stage
  constexpr int SP = kKT / RPS / kW;  // transfers per wave, K or V
  __shared__ __attribute__((aligned(1024))) uint8_t k_lds[2 * ST];
  __shared__ __attribute__((aligned(1024))) uint8_t v_lds[2 * ST];
  __shared__ int red[kW];

  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int l = threadIdx.x & 63, lq = l & 31, hi = l >> 5;
  const int G = 1 << lg;
  const int rpb = kQv >> lg;
  const uint32_t k_base = lds_addr(k_lds), v_base = lds_addr(v_lds);
  const int qv = 32 * w + lq;
  const int g = blockIdx.x % hkv;
  const int rest = blockIdx.x / hkv;
  const int rank = rest / max_tiles;
  const int tile = max_tiles - 1 - (rest - rank * max_tiles);
  int b = rank;
  if (batch > 1 && batch <= 64) {
    // rank of lane j's request: requests with more keys, or as many and a lower index
    const int nk = l < batch ? cu_kv[l + 1] - cu_kv[l] : -1;
    int rk = 0;
    for (int x = 0; x < batch; ++x) {
      const int nx = __shfl(nk, x, 64);
      rk += (nx > nk || (nx == nk && x < l)) ? 1 : 0;
    }
    const uint64_t hit = __ballot(l < batch && rk == rank);
    b = __builtin_amdgcn_readfirstlane(hit ? (int)__builtin_ctzll(hit) : rank);
  }
  const int64_t r0 = cu_rows[b];
  const int nr = cu_rows[b + 1] - (int)r0;
  if (tile * rpb >= nr) return;
  const int64_t kv0 = cu_kv[b];
  int nkv = cu_kv[b + 1] - (int)kv0;
  if (kv0 + nkv > n_kv_rows) nkv = (int)(n_kv_rows - kv0);

  const uint32_t row_b = (uint32_t)(kv_stride * 2);
  const int tg = l >> 4, te = (l >> 2) & 3, tq = l & 3;
  // Chunk c of K row r sits at c ^ (r % 16) (D = 64: c ^ (r / 2 % 8)), chunk c of V row r at
  // c ^ 4 (r % 4) (D = 64: c ^ 4 (r / 2 % 2)).  A lane's K fragment st is then at krd ^ (st << 5),
  // its V column block mb at vrd ^ (mb << 6).
  const int ky = D == 128 ? lq & 15 : (lq >> 1) & 7;
  const int krd = lq * RB + (hi ^ (ky & 1)) * 16 + (ky >> 1) * 32;
  const int vrd = (4 * (tg >> 1) + te) * RB + (D == 128 ? te : te >> 1) * 64 + 32 * (tg & 1) + 8 * tq;
  typedef short v4s __attribute__((ext_vector_type(4)));
  typedef v4s __attribute__((address_space(3))) * lds_v4s;
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));

  const int rl = tile * rpb + (qv >> lg);
  const int head = g * G + (qv & (G - 1));
  const int64_t grow = r0 + rl;
  const bool valid = rl < nr && grow < n_rows;
  const uint32_t range = nkv > 0 ? (uint32_t)(nkv - 1) * row_b + D * 2 : 0u;
  const i32x4 rk = make_rsrc(kc + kv0 * kv_stride + (int64_t)g * D, range);
  const i32x4 rv = make_rsrc(vc + kv0 * kv_stride + (int64_t)g * D, range);
  const int dr = RPS * w + l / CH, dc = l % CH;  // transfer i of a wave fills rows dr + RPS kW i
  const uint32_t koff = (uint32_t)dr * row_b + (dc ^ (D == 128 ? dr & 15 : (dr >> 1) & 7)) * 16;
  const uint32_t voff = (uint32_t)dr * row_b + (dc ^ (4 * (D == 128 ? dr & 3 : (dr >> 1) & 1))) * 16;
  int nt = max(0, nkv + kKT - 1) / kKT;  // key tiles (until the largest row position is known)
  auto issue_k1 = [&](int r, int i) {
    const uint32_t soff = r < nt ? (uint32_t)(r * kKT + RPS * kW * i) * row_b : kOob;
    dma16(rk, koff + soff, k_base + (uint32_t)((r & 1) * ST + (w + kW * i) * 1024));
  };
  auto issue_v1 = [&](int r, int i) {
    const uint32_t soff = r < nt ? (uint32_t)(r * kKT + RPS * kW * i) * row_b : kOob;
    dma16(rv, voff + soff, v_base + (uint32_t)((r & 1) * ST + (w + kW * i) * 1024));
  };
  auto issue_k = [&](int r) {
#pragma unroll
    for (int i = 0; i < SP; ++i) issue_k1(r, i);
  };
  auto issue_v = [&](int r) {
#pragma unroll
    for (int i = 0; i < SP; ++i) issue_v1(r, i);
  };
  issue_k(0);
  issue_v(0);
  issue_k(1);
  const int64_t crow = min(grow, n_rows - 1);
  const int pos_raw = row_pos[crow];
  bf16x8 qreg[D / 16];
  {
    int64_t qrow = crow;
    if (kRot && q_src) qrow = min(max((int64_t)q_src[crow], (int64_t)0), n_q_src - 1);
    const uint16_t* qp = q + qrow * (int64_t)hq * D + (int64_t)head * D + 8 * hi;
#pragma unroll
    for (int st = 0; st < D / 16; ++st) qreg[st] = as_bf16x8(ld16(qp + 16 * st));
  }
  if (kRot) rotate_query<D>(qreg, rtab + (int64_t)min(max(pos_raw, 0), n_tab - 1) * (D / 2), hi);
  const int qpos = valid ? pos_raw : INT_MIN;
  const int wmax = wave_max_i(valid ? qpos : -1);
  const int wmin = wave_min_i(valid ? qpos : INT_MAX);
  if (l == 0) red[w] = wmax;
  __syncthreads();
  int bmax = red[0];
#pragma unroll
  for (int i = 1; i < kW; ++i) bmax = max(bmax, red[i]);
  nt = max(0, min(nkv, bmax + 1) + kKT - 1) / kKT;
  const int wave_end = min(nkv, wmax + 1);
  f32x16 o[D / 32];
#pragma unroll
  for (int mb = 0; mb < D / 32; ++mb) o[mb] = f32x16{};
  float m = valid ? -1e30f : INFINITY;
  float ls = 0.f;

  auto meet = [&]() {  // every transfer and LDS access so far is complete, then the block meets
    asm volatile("" ::: "memory");
    wait_vm_lgkm0<0>();
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  auto qk_half = [&](const uint8_t* kl, int hb, f32x16& sh) {
    bf16x8 kf[D / 16];
#pragma unroll
    for (int st = 0; st < D / 16; ++st) kf[st] = as_bf16x8(ld16(kl + hb * 32 * RB + (krd ^ (st << 5))));
    sh = f32x16{};
#pragma unroll
    for (int st = 0; st < D / 16; ++st)
      sh = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[st], qreg[st], sh, 0, 0, 0);
  };
  auto softmax_pre = [&](f32x16 (&sc)[2], int kt0) {
    if (kt0 + kKT > wmin || kt0 + kKT > nkv) {
#pragma unroll
      for (int hb = 0; hb < 2; ++hb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int j = kt0 + hb * 32 + 8 * (v >> 2) + 4 * hi + (v & 3);
          if (j >= nkv || j > qpos) sc[hb][v] = -INFINITY;
        }
    }
    float mt = sc[0][0];
#pragma unroll
    for (int hb = 0; hb < 2; ++hb)
#pragma unroll
      for (int v = 0; v < 16; ++v) mt = fmaxf(mt, sc[hb][v]);
    {
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mt), __float_as_uint(mt),
                                                       false, false);
      mt = fmaxf(mt, fmaxf(__uint_as_float(sw[0]), __uint_as_float(sw[1]))) * scale2;
    }
    if (__ballot(mt > m + 8.f)) {
      const float mn = fmaxf(m, mt);
      const float alpha = __builtin_amdgcn_exp2f(m - mn);
      ls *= alpha;
#pragma unroll
      for (int mb = 0; mb < D / 32; ++mb) o[mb] *= alpha;
      m = mn;
    }
  };
  auto softmax_exp = [&](f32x16 (&sc)[2], bf16x8 (&pb)[2][2]) {
    const float nm = -m;
    float psum = 0.f;
#pragma unroll
    for (int hb = 0; hb < 2; ++hb)
#pragma unroll
      for (int v = 0; v < 16; v += 2) {
        const float p0 = __builtin_amdgcn_exp2f(fmaf(sc[hb][v], scale2, nm));
        const float p1 = __builtin_amdgcn_exp2f(fmaf(sc[hb][v + 1], scale2, nm));
        psum += p0;
        psum += p1;
        const bf16x2_t pk = __builtin_convertvector((f32x2_t){p0, p1}, bf16x2_t);
        pb[hb][v >> 3][v & 7] = pk[0];
        pb[hb][v >> 3][(v & 7) + 1] = pk[1];
      }
    ls += psum;
  };
  // S(t+1) = K Q^T beside P(t) = exp2(S(t) * scale2 - m), one product per fenced group with its K
  // fragment read four groups ahead (attention.hip), and the next transfers in between
  auto qk_exp_fused = [&](const uint8_t* kl, f32x16 (&sn)[2], f32x16 (&sc)[2], bf16x8 (&pb)[2][2], int tt) {
    constexpr int NS = D / 16;    // products per 32-key half
    constexpr int NM = 2 * NS;    // products per tile
    constexpr int EG = 32 / NM;   // elements of the tile per group (2 at D = 128)
    constexpr int PF = 4;         // K fragments in flight
    constexpr int DSTEP = NM / (2 * SP);
    static_assert(EG % 2 == 0 && EG * NM == 32, "groups cover the tile in element pairs");
    auto kfrag = [&](int i) { return as_bf16x8(ld16(kl + (i / NS) * 32 * RB + (krd ^ ((i % NS) << 5)))); };
    bf16x8 kf[NM];
#pragma unroll
    for (int i = 0; i < PF; ++i) kf[i] = kfrag(i);
    const float nm = -m;
    float psum = 0.f;
    float x[32], p[32];  // element e = 16 hb + v of the tile
    auto arg = [&](int g) {
#pragma unroll
      for (int e = EG * g; e < EG * (g + 1); ++e) x[e] = fmaf(sc[e / 16][e % 16], scale2, nm);
    };
    auto sum_pack = [&](int g) {
#pragma unroll
      for (int e = EG * g; e < EG * (g + 1); e += 2) {
        const int v = e % 16;
        psum += p[e];
        psum += p[e + 1];
        const bf16x2_t pk = __builtin_convertvector((f32x2_t){p[e], p[e + 1]}, bf16x2_t);
        pb[e / 16][v >> 3][v & 7] = pk[0];
        pb[e / 16][v >> 3][(v & 7) + 1] = pk[1];
      }
    };
    arg(0);
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      __builtin_amdgcn_sched_barrier(0);
      if (i + PF < NM) kf[i + PF] = kfrag(i + PF);
      if (i % DSTEP == 0 && i / DSTEP < SP) issue_k1(tt + 2, i / DSTEP);
      else if (i % DSTEP == 0 && i / DSTEP < 2 * SP) issue_v1(tt + 1, i / DSTEP - SP);
      const int hb = i / NS, st = i % NS;
      sn[hb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[i], qreg[st], st == 0 ? f32x16{} : sn[hb],
                                                       0, 0, 0);
      if (i + 1 < NM) arg(i + 1);
#pragma unroll
      for (int e = EG * i; e < EG * (i + 1); ++e) p[e] = __builtin_amdgcn_exp2f(x[e]);
      if (i > 0) sum_pack(i - 1);
    }
    __builtin_amdgcn_sched_barrier(0);
    sum_pack(NM - 1);
    ls += psum;
  };
  // O += P V, one product per fenced group with its V fragment read four groups ahead
  auto pv = [&](const uint8_t* vl, bf16x8 (&pb)[2][2]) {
    constexpr int NB = D / 32;
    constexpr int NM = 4 * NB;  // products, ordered (hb, k2, mb)
    constexpr int PF = 4;       // V fragments in flight
    auto vfrag = [&](int j) {
      const int hb = j / (2 * NB), k2 = (j / NB) % 2, mb = j % NB;
      const uint8_t* p0 = vl + (hb * 32 + 16 * k2) * RB + (vrd ^ (mb << 6));
      const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p0));
      const v4s up = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p0 + 8 * RB));
      return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, up, 0, 1, 2, 3, 4, 5, 6, 7));
    };
    bf16x8 vf[NM];
#pragma unroll
    for (int j = 0; j < PF; ++j) vf[j] = vfrag(j);
#pragma unroll
    for (int j = 0; j < NM; ++j) {
      __builtin_amdgcn_sched_barrier(0);
      if (j + PF < NM) vf[j + PF] = vfrag(j + PF);
      const int hb = j / (2 * NB), k2 = (j / NB) % 2, mb = j % NB;
      o[mb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[j], pb[hb][k2], o[mb], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  f32x16 sa[2], sb[2];
  meet();
  if (nt > 0 && wave_end > 0) {
    qk_half(k_lds, 0, sa[0]);
    qk_half(k_lds, 1, sa[1]);
  }
  asm volatile("" ::: "memory");
  wait_vm_lgkm0<0>();
  __builtin_amdgcn_s_barrier();  // K(0) has been read before K(2) takes its place
  asm volatile("" ::: "memory");
  auto step = [&](int t, f32x16 (&sc)[2], f32x16 (&sn)[2]) {
    const int kt0 = t * kKT;
    const bool do_cur = kt0 < wave_end;
    const bool do_next = t + 1 < nt && kt0 + kKT < wave_end;
    bf16x8 pb[2][2];
    if (!do_next) {
      issue_k(t + 2);
      issue_v(t + 1);
    }
    if (do_cur) softmax_pre(sc, kt0);
    __builtin_amdgcn_s_setprio(1);
    if (do_next)
      qk_exp_fused(k_lds + ((t + 1) & 1) * ST, sn, sc, pb, t);
    else if (do_cur)
      softmax_exp(sc, pb);
    __builtin_amdgcn_s_setprio(0);
    if (do_cur) pv(v_lds + (t & 1) * ST, pb);
    meet();
  };
  for (int t = 0; t < nt; t += 2) {
    step(t, sa, sb);
    if (t + 1 < nt) step(t + 1, sb, sa);
  }
  const float lt = ls + __shfl_xor(ls, 32, 64);
  if (!valid) return;
  const float inv = lt > 0.f ? 1.f / lt : 0.f;
  uint16_t* op = out + grow * (int64_t)hq * D + (int64_t)head * D;
  if (lse && hi == 0) lse[grow * hq + head] = lt > 0.f ? (m + log2f(lt)) * kLn2 : -INFINITY;
#pragma unroll
  for (int mb = 0; mb < D / 32; ++mb)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *reinterpret_cast<uint2*>(op + 32 * mb + 8 * i + 4 * hi) =
          make_uint2(pack_bf16x2(o[mb][4 * i] * inv, o[mb][4 * i + 1] * inv),
                     pack_bf16x2(o[mb][4 * i + 2] * inv, o[mb][4 * i + 3] * inv));
}

}  // namespace

hipError_t launch_attn_w4(void* out, float* lse, const void* q, const int32_t* row_pos,
                          int64_t n_rows, const int32_t* cu_rows, const void* k_cache,
                          const void* v_cache, int64_t n_kv_rows, int64_t kv_row_stride,
                          const int32_t* cu_kv, const AttnShape& s, float scale,
                          hipStream_t stream, const QueryRot& qrot) {
  int lg = 0;
  while ((1 << lg) < s.hq / s.hkv) ++lg;
  const int rpb = kQv >> lg;
  const int max_tiles = (s.max_rows + rpb - 1) / rpb;  // row tiles of the longest request
  const int64_t blocks = (int64_t)max_tiles * s.batch * s.hkv;
  if (blocks > 0x7fffffff) return hipErrorInvalidConfiguration;
  const float2* rtab = reinterpret_cast<const float2*>(qrot.table);
#define QCF_W4(D, R)                                                                               \
  attn_w4_kernel<D, R><<<dim3((unsigned)blocks), kW * 64, 0, stream>>>(                            \
      static_cast<uint16_t*>(out), lse, static_cast<const uint16_t*>(q), row_pos, n_rows, cu_rows,  \
      static_cast<const uint16_t*>(k_cache), static_cast<const uint16_t*>(v_cache), n_kv_rows,     \
      kv_row_stride, cu_kv, s.batch, max_tiles, s.hkv, s.hq, lg, scale * kLog2e, qrot.src,          \
      qrot.n_src, rtab, (int)qrot.n_table)
  if (s.d == 64) {
    if (qrot.table) QCF_W4(64, true); else QCF_W4(64, false);
  } else {
    if (qrot.table) QCF_W4(128, true); else QCF_W4(128, false);
  }
#undef QCF_W4
  return hipGetLastError();
}

}  // namespace qcf
