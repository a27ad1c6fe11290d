// hs_attn.hip — split-K flash-decoding attention over the per-request KV
// cache (gfx950), and the combine of its splits.
//
// Each generated token attends over all cached positions of its request, so
// decode streams the KV cache from HBM once per token (§2); the cache holds
// 2 * L * n_kv * d_h * s_ctx elements per request (Eq. 1, §4.1).  Work is
// split along the positions so that short batches still fill the GPU.
#include "hs_device.h"

#include <cfloat>

namespace hs {
namespace {

using namespace dev;

// ---------------------------------------------------------------------------
// split-K flash-decoding attention
// ---------------------------------------------------------------------------
// Online-softmax state of one query head over a set of positions: running
// max m, sum l = sum_t e^(s_t - m) and unnormalised output o = sum_t e^(s_t - m) v_t.
__device__ __forceinline__ float merge_weight(float m_part, float m_all) {
  return m_part == -INFINITY ? 0.f : expf(m_part - m_all);
}

// element (row, c) of the combined output: rows of n_heads * head_dim, or the
// packed activation layout where the O projection reads it (gemm_x_packed)
__device__ __forceinline__ int64_t attn_out_at(const AttnArgs &a, int64_t row, int c, int hd) {
  const int K = a.n_heads * hd;
  return a.out_packed ? packed_x_index((int)row, c, (K / 8 + 15) / 16) : row * K + c;
}

// One work group = (split, KV head j, query).  Each of its NW waves walks
// its share of the split's positions (LPT lanes per position, one 16-byte
// chunk of the K row and of the V row per lane), requesting the chunks of UB
// position groups at once; the split policy sizes splits so that one such
// batch usually covers a wave's share.  Every position group keeps an online
// softmax for the G query heads of KV head j.  The groups are merged with
// lane shuffles, the waves through LDS.  With a single split the work group
// writes the normalised output; otherwise every split writes its unnormalised
// partial o, its max m and its sum l, a split past the query's positions
// writing the neutral (o = 0, m = -inf, l = 0).
// K/V are read through buffer ranges that end at the split's last position,
// so that no load sits behind a branch.  In a cache of several blocks per
// request (PAGED) a batch of loads always lies in one block and gets a range
// of its own, the block's start read one batch ahead.  In decode, work-group
// row z serves the z-th longest request (a.order).
template <int DT, int HD, int G, int NW, bool PAGED>
__global__ __launch_bounds__(64 * NW) void k_attn(AttnArgs a) {
  using S = typename Ty<DT>::S;
  constexpr int CE = Ty<DT>::CE;
  constexpr int SB = (int)sizeof(S);
  constexpr int LPT = HD / CE;
  constexpr int TPW = 64 / LPT;           // positions per wave-wide load
  constexpr int STEP = NW * TPW;          // positions per work-group iteration
  constexpr int UB = attn_batch(G);       // iterations per batch of loads
  // decode: the longest requests' work groups are dispatched first
  const int split = blockIdx.x, j = blockIdx.y, qi = a.order ? a.order[blockIdx.z] : (int)blockIdx.z;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tg = lane / LPT, c = lane % LPT;
  // the query chunks are requested first (also by a split past the end,
  // which does not use them) and unpacked once the batch's K/V loads are in
  // flight, so their latency overlaps the cache metadata and K/V loads
  u32x4 qraw[G];
#pragma unroll
  for (int h = 0; h < G; ++h) qraw[h] = ld16((const S *)a.q + (int64_t)qi * a.ld_q + (j * G + h) * HD + c * CE);
  // the request's length, capacity and (contiguous cache) first element,
  // requested together
  // (16-bit storage prefills through k_attn_prefill: here a.prefill is set
  // for fp32 alone, and the 16-bit kernels compile the decode path only)
  int req, last;  // last: the query's position
  if (DT != HS_F32 || !a.prefill) {
    req = PAGED ? a.kv.act[qi] : qi;
    last = a.kv.len[req];
  } else {
    const int i = packed_request(a.pk, qi);
    req = a.pk->req[i];
    last = qi - a.pk->cu[i];
  }
  const int cap = a.kv.cap[req];
  const int64_t b_req = PAGED ? 0 : a.kv.tab[req];
  // the three loads issued together, one wait (a paged cache reads its block
  // table in the loop, whose loads the pin would turn into vector loads)
  if constexpr (!PAGED) asm volatile("" ::"s"(last), "s"(cap), "s"(b_req));
  const int L = min(last + 1, cap);
  const int t0 = split * a.S;
  const int64_t qh = (int64_t)qi * a.n_heads + j * G;  // first (query, head) row of this group
  if (t0 >= L) {
    for (int idx = threadIdx.x; idx < G * HD; idx += 64 * NW) {
      const int h = idx / HD, e = idx - h * HD;
      a.part_o[((qh + h) * a.n_split + split) * HD + e] = 0.f;
      if (e == 0) {
        a.part_ml[((qh + h) * a.n_split + split) * 2] = -INFINITY;
        a.part_ml[((qh + h) * a.n_split + split) * 2 + 1] = 0.f;
      }
    }
    return;
  }
  const int n = min(a.S, L - t0);
  const int n_it = (n + STEP - 1) / STEP;
  // one block per request: the split's rows are one range.  Several blocks:
  // each batch of loads (a whole number of which fills a block) reads the
  // block holding it, whose start is read one batch ahead.
  int64_t ko = 0, vo = 0;
  int bt = 0, toff = 0;
  int64_t kin = 0, vin = 0, b_next = 0;
  if constexpr (PAGED) {
    bt = a.kv.bt[req];
    toff = a.kv.toff[req];
    kin = (int64_t)((a.layer * 2) * a.n_kv + j) * bt * HD;
    vin = kin + (int64_t)a.n_kv * bt * HD;
    b_next = a.kv.tab[toff + t0 / bt];
  } else {
    ko = b_req + ((int64_t)((a.layer * 2) * a.n_kv + j) * cap + t0) * HD;
    vo = ko + (int64_t)a.n_kv * cap * HD;
  }
  const uint32_t nbytes = (uint32_t)n * HD * SB;
  const rsrc_t kr = make_rsrc((const S *)a.kv.buf + max(ko, (int64_t)0), nbytes);
  const rsrc_t vr = make_rsrc((const S *)a.kv.buf + max(vo, (int64_t)0), nbytes);

  float qf[G][CE];

  float m[G], l[G], o[G][CE];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    m[h] = -INFINITY;
    l[h] = 0.f;
#pragma unroll
    for (int e = 0; e < CE; ++e) o[h][e] = 0.f;
  }
  for (int it0 = 0; it0 < n_it; it0 += UB) {
    // all K and V chunks of the batch are requested before any is used;
    // positions past the split read zeros
    u32x4 kc[UB], vc[UB];
    rsrc_t kb = kr, vb = vr;
    int rel = 0;
    bool blk_ok = true;  // a paged batch's block is held (a pool that ran dry leaves it unheld)
    if constexpr (PAGED) {
      const int64_t b0 = b_next;
      blk_ok = b0 >= 0;
      const int pb = t0 + it0 * STEP, pn = pb + UB * STEP;
      b_next = pn < t0 + n ? a.kv.tab[toff + pn / bt] : 0;
      const int64_t at = max(b0, (int64_t)0) + (int64_t)(pb % bt) * HD;
      const uint32_t bytes = b0 < 0 ? 0u : (uint32_t)min(UB * STEP, n - it0 * STEP) * HD * SB;
      kb = make_rsrc((const S *)a.kv.buf + at + kin, bytes);
      vb = make_rsrc((const S *)a.kv.buf + at + vin, bytes);
      rel = it0 * STEP;
    }
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const uint32_t off = (uint32_t)((it0 + u) * STEP - rel + wave * TPW + tg) * (HD * SB) + (uint32_t)c * 16u;
      kc[u] = bld16_stream(kb, off);
      vc[u] = bld16_stream(vb, off);
    }
    // opaque to the compiler: keeps the unpack (and its wait) here, behind the loads
#pragma unroll
    for (int h = 0; h < G; ++h) {
      asm volatile("" : "+v"(qraw[h]));
      unpack<DT>(qraw[h], qf[h]);
    }
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const int tt = (it0 + u) * STEP + wave * TPW + tg;
      const bool valid = tt < n && blk_ok;  // positions of an unheld block are masked
      float kf[CE], vf[CE];
      unpack<DT>(kc[u], kf);
      unpack<DT>(vc[u], vf);
#pragma unroll
      for (int h = 0; h < G; ++h) {
        float d = 0.f;
#pragma unroll
        for (int e = 0; e < CE; ++e) d += qf[h][e] * kf[e];
        d = group_sum<LPT>(d);
        // branch-free update: a position past the split (zero K/V rows)
        // leaves the state as it is (a branch here let the compiler move a
        // V load behind it, with a wait for every load in flight)
        const float sc = valid ? d * a.scale : -INFINITY;
        const float mn = fmaxf(m[h], sc);
        const float corr = merge_weight(m[h], mn);
        const float p = valid ? expf(sc - mn) : 0.f;
        l[h] = l[h] * corr + p;
#pragma unroll
        for (int e = 0; e < CE; ++e) o[h][e] = o[h][e] * corr + p * vf[e];
        m[h] = mn;
      }
    }
  }
  // merge the TPW position groups of the wave (lanes with the same chunk c)
#pragma unroll
  for (int off = LPT; off < 64; off <<= 1) {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const float m2 = __shfl_xor(m[h], off), l2 = __shfl_xor(l[h], off);
      const float mn = fmaxf(m[h], m2);
      const float w1 = merge_weight(m[h], mn), w2 = merge_weight(m2, mn);
      l[h] = l[h] * w1 + l2 * w2;
#pragma unroll
      for (int e = 0; e < CE; ++e) o[h][e] = o[h][e] * w1 + __shfl_xor(o[h][e], off) * w2;
      m[h] = mn;
    }
  }
  __shared__ float s_m[NW][G], s_l[NW][G];
  __shared__ float s_o[NW][G][HD];
  if (tg == 0)
#pragma unroll
    for (int h = 0; h < G; ++h)
#pragma unroll
      for (int e = 0; e < CE; ++e) s_o[wave][h][c * CE + e] = o[h][e];
  if (lane == 0)
#pragma unroll
    for (int h = 0; h < G; ++h) {
      s_m[wave][h] = m[h];
      s_l[wave][h] = l[h];
    }
  __syncthreads();

  for (int idx = threadIdx.x; idx < G * HD; idx += 64 * NW) {
    const int h = idx / HD, e = idx - h * HD;
    float M = s_m[0][h];
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, s_m[w][h]);
    float num = 0.f, den = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float wt = merge_weight(s_m[w][h], M);
      num += wt * s_o[w][h][e];
      den += wt * s_l[w][h];
    }
    if (a.n_split == 1) {
      st_elem<DT>(a.out, attn_out_at(a, qi, (j * G + h) * HD + e, HD), num / den);
    } else {
      a.part_o[((qh + h) * a.n_split + split) * HD + e] = num;
      if (e == 0) {
        a.part_ml[((qh + h) * a.n_split + split) * 2] = M;
        a.part_ml[((qh + h) * a.n_split + split) * 2 + 1] = den;
      }
    }
  }
}

// storage-dtype parts the softmax probabilities enter the PV product as
template <int DT>
constexpr int P_PARTS = DT == HS_BF16 ? 3 : 2;

// Attention for query-head groups of 4..16 heads on the matrix cores.  One
// work group = (split, KV head j, query), as above; each wave takes tiles of 16
// consecutive positions.  Per tile, the scores of the tile's positions for all
// heads of the group are S^T = K Q^T (16 positions x 16 head slots, MFMA
// 16x16x32: exact products of the stored 16-bit values, fp32 sums).  A lane
// then holds the scores of positions 4 q .. 4 q + 3 (q = lane / 16) for head
// lane % 16 -- exactly the B-operand layout of the 16x16x16 MFMA that updates
// O^T (d x heads) += V^T P^T, so the online-softmax probabilities feed the
// matrix cores from registers.  That MFMA takes 16-bit operands, so P enters
// as the sum of storage-dtype parts, p = hi + lo (+ lo2) with hi = R(p),
// lo = R(p - hi), lo2 = R(p - hi - lo), one MFMA each: the products with the
// stored V values are exact and p keeps ~22 (fp16, two parts) or ~24 (bf16,
// three parts) significant bits, against fp32 in the definition (a single
// rounding of p to bf16 doubled the error of o and, over 28 layers, the
// error of the residual stream; two bf16 parts left the Qwen-shaped logits
// 1.8 % from the oracle, three 1.2 %).  l sums the parts, so o stays a
// weighted mean of the V rows.  For the V^T operand a lane loads
// chunk c = lane % 16 of the 4 positions it covers, and output row c of d-tile
// dt is element d = 8 c + dt, which a lane gathers from its four chunks.
// The waves merge through LDS as in k_attn.
template <int DT, int HD, int G, int NW, bool PAGED>
__global__ __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(3))) void k_attn_mma(AttnArgs a) {
  static_assert(DT != HS_F32 && G <= 16 && (HD == 64 || HD == 128), "16-bit storage, at most 16 heads per group");
  constexpr int SB = 2;
  constexpr int CPR = HD / 8;         // 16-byte chunks per row
  constexpr int KK = HD / 32;         // 32-wide k steps of the scores
  constexpr int UB = ATTN_MMA_BATCH;  // tiles per batch of loads
  constexpr int STEP = NW * 16;       // positions per work-group iteration
  // decode: the longest requests' work groups are dispatched first
  const int split = blockIdx.x, j = blockIdx.y, qi = a.order ? a.order[blockIdx.z] : (int)blockIdx.z;
  // (16-bit storage prefills through k_attn_prefill: here a.prefill is set
  // for fp32 alone, and the 16-bit kernels compile the decode path only)
  int req, last;  // last: the query's position
  if (DT != HS_F32 || !a.prefill) {
    req = PAGED ? a.kv.act[qi] : qi;
    last = a.kv.len[req];
  } else {
    const int i = packed_request(a.pk, qi);
    req = a.pk->req[i];
    last = qi - a.pk->cu[i];
  }
  // the request's length, capacity and (contiguous cache) first element,
  // requested together, one wait
  const int cap = a.kv.cap[req];
  const int64_t b_req = PAGED ? 0 : a.kv.tab[req];
  if constexpr (!PAGED) asm volatile("" ::"s"(last), "s"(cap), "s"(b_req));  // as in k_attn
  const int L = min(last + 1, cap);
  const int t0 = split * a.S;
  const int64_t qh = (int64_t)qi * a.n_heads + j * G;
  if (t0 >= L) {
    for (int idx = threadIdx.x; idx < G * HD; idx += 64 * NW) {
      const int h = idx / HD, e = idx - h * HD;
      a.part_o[((qh + h) * a.n_split + split) * HD + e] = 0.f;
      if (e == 0) {
        a.part_ml[((qh + h) * a.n_split + split) * 2] = -INFINITY;
        a.part_ml[((qh + h) * a.n_split + split) * 2 + 1] = 0.f;
      }
    }
    return;
  }
  const int n = min(a.S, L - t0);
  const int n_it = (n + STEP - 1) / STEP;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lg = lane >> 4;
  // one block per request: the split's rows are one range.  Several blocks:
  // each batch of loads (a whole number of which fills a block) reads the
  // block holding it, whose start is read one batch ahead.
  int64_t ko = 0, vo = 0;
  int bt = 0, toff = 0;
  int64_t kin = 0, vin = 0, b_next = 0;
  if constexpr (PAGED) {
    bt = a.kv.bt[req];
    toff = a.kv.toff[req];
    kin = (int64_t)((a.layer * 2) * a.n_kv + j) * bt * HD;
    vin = kin + (int64_t)a.n_kv * bt * HD;
    b_next = a.kv.tab[toff + t0 / bt];
  } else {
    ko = b_req + ((int64_t)((a.layer * 2) * a.n_kv + j) * cap + t0) * HD;
    vo = ko + (int64_t)a.n_kv * cap * HD;
  }
  const uint32_t nbytes = (uint32_t)n * HD * SB;
  const rsrc_t kr = make_rsrc((const uint16_t *)a.kv.buf + max(ko, (int64_t)0), nbytes);
  const rsrc_t vr = make_rsrc((const uint16_t *)a.kv.buf + max(vo, (int64_t)0), nbytes);

  // Q^T operand: head lane % 16 of the group (zero past G), k = 32 kk + 8 q ..
  u32x4 qb[KK];
#pragma unroll
  for (int kk = 0; kk < KK; ++kk)
    qb[kk] = li < G ? ld16((const uint16_t *)a.q + (int64_t)qi * a.ld_q + (j * G + li) * HD + (kk * 4 + lg) * 8)
                    : u32x4{0u, 0u, 0u, 0u};

  float m = -INFINITY, l = 0.f;
  f32x4 o[8];
#pragma unroll
  for (int dt = 0; dt < 8; ++dt) o[dt] = f32x4{0.f, 0.f, 0.f, 0.f};

  // A ring of UB tiles per wave: a tile's registers are requested again, for
  // the tile UB iterations on, as soon as its products are issued, so that
  // loads are in flight while the wave computes.  Positions past the split
  // read zeros.
  u32x4 kc[UB][KK], vc[UB][4];
  bool blk_ok[UB];  // as in k_attn
  auto request = [&](int u, int it) {
    rsrc_t kb = kr, vb = vr;
    int p0 = (it * NW + wave) * 16;
    blk_ok[u] = true;
    if constexpr (PAGED) {  // an iteration's positions lie in one block
      const int64_t b0 = b_next;
      blk_ok[u] = b0 >= 0;
      const int pb = t0 + it * STEP, pn = pb + STEP;
      b_next = pn < t0 + n ? a.kv.tab[toff + pn / bt] : 0;
      const int64_t at = max(b0, (int64_t)0) + (int64_t)(pb % bt) * HD;
      const uint32_t bytes = b0 < 0 || it >= n_it ? 0u : (uint32_t)min(STEP, n - it * STEP) * HD * SB;
      kb = make_rsrc((const uint16_t *)a.kv.buf + at + kin, bytes);
      vb = make_rsrc((const uint16_t *)a.kv.buf + at + vin, bytes);
      p0 -= it * STEP;
    }
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
      kc[u][kk] = bld16_stream(kb, (uint32_t)((p0 + li) * HD + (kk * 4 + lg) * 8) * SB);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      vc[u][i] = bld16_stream(vb, li < CPR ? (uint32_t)((p0 + 4 * lg + i) * HD + li * 8) * SB : BUF_OOB);
  };
#pragma unroll
  for (int u = 0; u < UB; ++u) request(u, u);
  for (int it0 = 0; it0 < n_it; it0 += UB) {
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const int p0 = ((it0 + u) * NW + wave) * 16;
      f32x4 sv = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) sv = mma<DT>(kc[u][kk], qb[kk], sv);
      float tmax = -INFINITY;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        sv[i] = p0 + 4 * lg + i < n && blk_ok[u] ? sv[i] * a.scale : -INFINITY;
        tmax = fmaxf(tmax, sv[i]);
      }
      tmax = fmaxf(tmax, __shfl_xor(tmax, 16));
      tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
      const float mn = fmaxf(m, tmax);
      const float corr = m == -INFINITY ? 0.f : __expf(m - mn);
      m = mn;
      l *= corr;  // this lane's positions only
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) o[dt] *= corr;
      // the PV operands: p = hi + lo (+ lo2 in bf16) in the storage dtype;
      // l sums the parts
      u32x2 ph, pl, pt{};
#pragma unroll
      for (int x = 0; x < 2; ++x) {
        float p[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) p[e] = sv[2 * x + e] == -INFINITY ? 0.f : __expf(sv[2 * x + e] - m);
        ph[x] = pack2<DT>(p[0], p[1]);
        const float h0 = lo_f32<DT>(ph[x]), h1 = hi_f32<DT>(ph[x]);
        pl[x] = pack2<DT>(p[0] - h0, p[1] - h1);
        const float l0 = lo_f32<DT>(pl[x]), l1 = hi_f32<DT>(pl[x]);
        if constexpr (P_PARTS<DT> == 3) {
          pt[x] = pack2<DT>(p[0] - h0 - l0, p[1] - h1 - l1);
          l += (h0 + l0 + lo_f32<DT>(pt[x])) + (h1 + l1 + hi_f32<DT>(pt[x]));
        } else {
          l += (h0 + l0) + (h1 + l1);
        }
      }
#pragma unroll
      for (int d0 = 0; d0 < 8; d0 += 2) {
        // V^T rows: the 16-bit elements d0 and d0 + 1 of chunk lane % 16 of the 4 positions
        const int w = d0 >> 1;
        u32x2 av[2];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          const uint32_t sel = e ? 0x07060302u : 0x05040100u;
          av[e][0] = __builtin_amdgcn_perm(vc[u][1][w], vc[u][0][w], sel);
          av[e][1] = __builtin_amdgcn_perm(vc[u][3][w], vc[u][2][w], sel);
        }
#pragma unroll
        for (int part = 0; part < P_PARTS<DT>; ++part)
#pragma unroll
          for (int e = 0; e < 2; ++e) o[d0 + e] = mma16<DT>(av[e], part == 0 ? ph : part == 1 ? pl : pt, o[d0 + e]);
      }
      // kept apart: the compiler gathers both tiles' operands first and sinks the requests to the loop's end
      __builtin_amdgcn_sched_barrier(0);
      request(u, it0 + u + UB);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);

  __shared__ float s_m[NW][16], s_l[NW][16];
  __shared__ float s_o[NW][16][HD + 1];
  if (lg == 0) {
    s_m[wave][li] = m;
    s_l[wave][li] = l;
  }
#pragma unroll
  for (int dt = 0; dt < 8; ++dt)
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int d = (4 * lg + i) * 8 + dt;
      if (d < HD) s_o[wave][li][d] = o[dt][i];
    }
  __syncthreads();
  for (int idx = threadIdx.x; idx < G * HD; idx += 64 * NW) {
    const int h = idx / HD, e = idx - h * HD;
    float M = s_m[0][h];
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, s_m[w][h]);
    float num = 0.f, den = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float wt = merge_weight(s_m[w][h], M);
      num += wt * s_o[w][h][e];
      den += wt * s_l[w][h];
    }
    if (a.n_split == 1) {
      st_elem<DT>(a.out, attn_out_at(a, qi, (j * G + h) * HD + e, HD), num / den);
    } else {
      a.part_o[((qh + h) * a.n_split + split) * HD + e] = num;
      if (e == 0) {
        a.part_ml[((qh + h) * a.n_split + split) * 2] = M;
        a.part_ml[((qh + h) * a.n_split + split) * 2 + 1] = den;
      }
    }
  }
}

// Prefill attention on the matrix cores (causal: row r of the request attends
// to rows 0..r).  The 16 MFMA columns of a query tile hold QPT = 16 / G
// consecutive query rows x the G query heads of KV head j.  A work group takes
// NW x QT consecutive query tiles of one request, QT per wave; its waves walk
// the request's key tiles of 16 positions together, KT per step, which they
// copy straight into LDS in MFMA operand order (K: four lanes' chunks of a
// position apart; V: four positions of a channel chunk), one step ahead.  So a
// K/V row read from L2 serves NW x QT x QPT query rows, and each wave keeps the
// whole online softmax of its own columns.  Keys past a row are masked only in
// the steps that reach the wave's rows, and steps past them are skipped.  The
// probabilities are split into storage-dtype parts as in k_attn_mma; two key
// tiles together make the k range of one 16x16x32 MFMA.
//
// What bounds it: the softmax arithmetic (about 12 vector instructions a
// score) and the products (the parts double or triple those of PV) in turn:
// over sixteen requests (bf16, group 7, 14370 rows, 274-283 us) the vector
// units are busy half of the time and the matrix cores 43 %, LDS 11 % without
// bank conflicts.  One request of 640 rows (25-26 us, 320 work groups) is a
// chain of its longest groups' steps, the matrix cores 7 % busy.
//
// Slack, in units of the base-2 exponent, by which a column's scores may pass
// the running maximum before it is raised: exp2(s - m) stays below 2^11.5.
constexpr float RESCALE_SLACK = 11.5f;
// From this maximum on, scores are rounded before the maximum is subtracted.
// Below, one fma of the unrounded product leaves s - m off by at most half an
// ulp of m, 2^-5 (p up to 2 % more, the same factor in o and l); from here the
// ulp grows past whole units of the exponent: at 2^34 p of the largest score
// itself would be 2^+-1024.
constexpr float ROUND_FROM = 0x1p20f;

template <int DT, int HD, int G, int NW, int QT>
__global__ __launch_bounds__(64 * NW, 2) void k_attn_prefill(AttnArgs a) {
  static_assert(DT != HS_F32 && G <= 16 && (HD == 64 || HD == 128), "16-bit storage, at most 16 heads per group");
  constexpr int KT = NW;         // key tiles per step: one copied by each wave
  constexpr int CPR = HD / 8;    // 16-byte chunks per row
  constexpr int KK = HD / 32;    // 1 KB sub-blocks of a K tile
  constexpr int TB = KK + 4;     // sub-blocks of a key tile (K, then V)
  constexpr int QPT = 16 / G;    // query rows per tile
  static_assert(KT % 2 == 0, "key tiles in pairs");
  __shared__ __align__(1024) unsigned char s_kv[2][KT][TB * 1024];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lg = lane >> 4;
  // The work group's item: KV head j and group `grp` of one request's query
  // tiles.  Work groups are dealt to the 8 XCDs round robin; an XCD
  // serves every xh-th head (xh = gcd(n_kv, 8); 8 / xh XCDs share a head's
  // groups), so that the groups that read the same K/V rows share its L2, and
  // takes the groups of all requests in the order of their length, longest
  // first: in request order the last long groups ran alone at the end, and
  // the XCDs got unequal shares.
  const int per = a.n_kv / a.prefill_xh, share = 8 / a.prefill_xh;
  const int xcd = (int)blockIdx.x & 7, item = (int)blockIdx.x >> 3;
  const int j = xcd % a.prefill_xh + a.prefill_xh * (item % per);
  const int rank = item / per * share + xcd / a.prefill_xh;
  if (rank >= a.prefill_groups) return;
  const PrefillGroup pg = a.prefill_order[rank];
  const int grp = __builtin_amdgcn_readfirstlane(pg.group), req = __builtin_amdgcn_readfirstlane(pg.req);
  const int roff = __builtin_amdgcn_readfirstlane(pg.row0), nrows = __builtin_amdgcn_readfirstlane(pg.rows);
  const int t0 = (grp * NW + wave) * QT;                 // the wave's first query tile
  const int sh = li % G;                                 // the lane column's head
  int sq[QT];
  bool slot[QT];
#pragma unroll
  for (int s = 0; s < QT; ++s) {
    sq[s] = (t0 + s) * QPT + li / G;  // the lane column's query position in tile s
    slot[s] = li < QPT * G && sq[s] < nrows;
  }
  // columns without a query compute a row of zeros that is not stored
  const int wfirst = t0 * QPT;                                          // the wave's first row
  const int wlast = wfirst < nrows ? min((t0 + QT) * QPT, nrows) - 1 : -1;  // and its last
  const int glast = min((t0 - wave * QT + NW * QT) * QPT, nrows) - 1;   // the work group's last row
  const int n_steps = glast / (16 * KT) + 1, last_kt = glast / 16;
  // key tiles are read block by block (a block holds a whole number of tiles)
  const int bt = __builtin_amdgcn_readfirstlane(a.kv.bt[req]), toff = __builtin_amdgcn_readfirstlane(a.kv.toff[req]);
  const int64_t kin = (int64_t)((a.layer * 2) * a.n_kv + j) * bt * HD, vin = (int64_t)a.n_kv * bt * HD;
  const uint16_t *buf = (const uint16_t *)a.kv.buf;

  u32x4 qb[QT][KK];
#pragma unroll
  for (int s = 0; s < QT; ++s)
#pragma unroll
    for (int kk = 0; kk < KK; ++kk)
      qb[s][kk] = slot[s] ? ld16((const uint16_t *)a.q + (int64_t)(roff + sq[s]) * a.ld_q + (j * G + sh) * HD +
                                 (kk * 4 + lg) * 8)
                          : u32x4{0u, 0u, 0u, 0u};

  // This wave's key tile of step s: past the group's last tile the last one
  // again, past its last row that row again (finite values for probabilities
  // that are zero).  A block that is not allocated reads as zeros.
  // (same: values equal in every lane, of which the compiler cannot tell)
  auto same = [](int64_t v) {
    return (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) |
                     (uint32_t)__builtin_amdgcn_readfirstlane((int)v));
  };
  auto tile_base = [&](int s) { return a.kv.tab[toff + min(s * KT + wave, last_kt) * 16 / bt]; };
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_addr(&s_kv[0][wave][0]));
  auto issue = [&](int s, int64_t base) {
    const int64_t b0 = same(base);
    const int p0 = min(s * KT + wave, last_kt) * 16, pb = p0 % bt;
    const int top = min(16, glast + 1 - p0) - 1;  // the tile's last row
    const uint32_t dst = lds0 + (s & 1) * KT * TB * 1024;
    if (b0 < 0) {
#pragma unroll
      for (int x = 0; x < TB; ++x) *(u32x4 *)(&s_kv[s & 1][wave][x * 1024] + lane * 16) = u32x4{0u, 0u, 0u, 0u};
      return;
    }
    const uint64_t kp = (uint64_t)same((int64_t)(buf + b0 + kin + (int64_t)pb * HD));
    const uint64_t vp = kp + (uint64_t)same(vin) * 2u;
    constexpr uint32_t ROW = HD * 2, RANGE = 16 * ROW;
    const u32x4 kr{(uint32_t)kp, (uint32_t)(kp >> 32), RANGE, (uint32_t)BUF_WORD3};
    const u32x4 vr{(uint32_t)vp, (uint32_t)(vp >> 32), RANGE, (uint32_t)BUF_WORD3};
    const uint32_t ko = (uint32_t)min(li, top) * ROW + lg * 16;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) dma_1k(kr, ko + kk * 64, 0, dst + kk * 1024);
#pragma unroll
    for (int i = 0; i < 4; ++i)
      dma_1k(vr, (uint32_t)min(4 * lg + i, top) * ROW + (li % CPR) * 16, 0, dst + (KK + i) * 1024);
  };

  // Running maximum (base-2 units) and this lane's share of the sum.  The
  // maximum starts at the lowest finite number, which every finite score
  // raises or equals, so that s - m is a number for s = -inf too.
  float m[QT], l[QT];
  bool big[QT];  // some column's |m| >= ROUND_FROM (wave-uniform)
  f32x4 o[QT][8];
#pragma unroll
  for (int s = 0; s < QT; ++s) {
    m[s] = -FLT_MAX;
    l[s] = 0.f;
    big[s] = true;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) o[s][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const float c2 = a.scale * 1.44269504088896341f;
  issue(0, tile_base(0));
  int64_t nb = tile_base(1);
  for (int st = 0; st < n_steps; ++st) {
    dma_sync<0>();  // this step's tiles are in LDS, and the other half is free
    if (st + 1 < n_steps) {
      issue(st + 1, nb);
      nb = tile_base(st + 2);
    }
    const int k0 = st * KT * 16;  // the step's first key
    if (k0 > wlast) continue;
    const unsigned char *kv = &s_kv[st & 1][0][0] + lane * 16;
    // independent products next to each other: an MFMA waits for the previous
    // one on its accumulator
    f32x4 sc[QT][KT];
#pragma unroll
    for (int u = 0; u < KT; u += 2) {
#pragma unroll
      for (int kk = 0; kk < KK; ++kk)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const u32x4 kc = *(const u32x4 *)(kv + ((u + t) * TB + kk) * 1024);
#pragma unroll
          for (int s = 0; s < QT; ++s)
            sc[s][u + t] = mma<DT>(kc, qb[s][kk], kk ? sc[s][u + t] : f32x4{0.f, 0.f, 0.f, 0.f});
        }
    }
    if (k0 + KT * 16 - 1 > wfirst) {
#pragma unroll
      for (int s = 0; s < QT; ++s)
#pragma unroll
        for (int u = 0; u < KT; ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (k0 + u * 16 + 4 * lg + i > sq[s]) sc[s][u][i] = -INFINITY;
    }
    // o / l does not depend on the reference m as long as exp2(s - m) stays
    // in range.  m, the same for the four lanes of a column, is raised to the
    // column's maximum (and o, l rescaled) only when some score of the wave
    // passes it by more than RESCALE_SLACK.
#pragma unroll
    for (int s = 0; s < QT; ++s) {
      float tmax = -INFINITY;
#pragma unroll
      for (int u = 0; u < KT; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i) tmax = fmaxf(tmax, sc[s][u][i]);
      tmax *= c2;
      if (__ballot(tmax > m[s] + RESCALE_SLACK)) {
        tmax = fmaxf(tmax, __shfl_xor(tmax, 16));
        tmax = fmaxf(tmax, __shfl_xor(tmax, 32));
        const float mn = fmaxf(m[s], tmax);
        const float corr = __builtin_amdgcn_exp2f(m[s] - mn);
        l[s] *= corr;
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) o[s][dt] *= corr;
        m[s] = mn;
        big[s] = __ballot(fabsf(mn) >= ROUND_FROM) != 0;
      }
    }
    float mul[QT], sub[QT];  // p = exp2(score * mul - sub)
#pragma unroll
    for (int s = 0; s < QT; ++s) {
      mul[s] = big[s] ? 1.f : c2;
      sub[s] = big[s] ? 0.f : m[s];
      if (big[s]) {
#pragma clang fp contract(off)
#pragma unroll
        for (int u = 0; u < KT; ++u)
#pragma unroll
          for (int i = 0; i < 4; ++i) sc[s][u][i] = sc[s][u][i] * c2 - m[s];
      }
    }
#pragma unroll
    for (int u = 0; u < KT; u += 2) {
      u32x4 ph[QT], pl[QT], pt[QT];
#pragma unroll
      for (int s = 0; s < QT; ++s)
#pragma unroll
        for (int x = 0; x < 4; ++x) {  // elements 2 x, 2 x + 1 of the pair's eight keys
          float p[2];
#pragma unroll
          for (int e = 0; e < 2; ++e) {
            p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[s][u + (x >> 1)][2 * (x & 1) + e], mul[s], -sub[s]));
            l[s] += p[e];
          }
          ph[s][x] = pack2<DT>(p[0], p[1]);
          p[0] -= lo_f32<DT>(ph[s][x]);
          p[1] -= hi_f32<DT>(ph[s][x]);
          pl[s][x] = pack2<DT>(p[0], p[1]);
          if constexpr (P_PARTS<DT> == 3)
            pt[s][x] = pack2<DT>(p[0] - lo_f32<DT>(pl[s][x]), p[1] - hi_f32<DT>(pl[s][x]));
        }
      u32x4 vc[2][4];
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) vc[t][i] = *(const u32x4 *)(kv + ((u + t) * TB + KK + i) * 1024);
#pragma unroll
      for (int d0 = 0; d0 < 8; d0 += 2) {
        // the 16-bit elements d0 and d0 + 1 of keys 4 lg .. 4 lg + 3 of both tiles, low half first
        const int w2 = d0 >> 1;
        u32x4 av[2];
#pragma unroll
        for (int e = 0; e < 2; ++e)
#pragma unroll
          for (int t = 0; t < 2; ++t) {
            const uint32_t sel = e ? 0x07060302u : 0x05040100u;
            av[e][2 * t] = __builtin_amdgcn_perm(vc[t][1][w2], vc[t][0][w2], sel);
            av[e][2 * t + 1] = __builtin_amdgcn_perm(vc[t][3][w2], vc[t][2][w2], sel);
          }
#pragma unroll
        for (int part = 0; part < P_PARTS<DT>; ++part)
#pragma unroll
          for (int e = 0; e < 2; ++e)
#pragma unroll
            for (int s = 0; s < QT; ++s)
              o[s][d0 + e] = mma<DT>(av[e], part == 0 ? ph[s] : part == 1 ? pl[s] : pt[s], o[s][d0 + e]);
      }
    }
  }
  // lane (c, q) holds rows d = (4 q + i) * 8 + dt of its column's output: row
  // i's elements dt = 0..7 are one 16-byte chunk, in either layout of the
  // output.  The column's sum adds its four lanes.
#pragma unroll
  for (int s = 0; s < QT; ++s) {
    l[s] += __shfl_xor(l[s], 16);
    l[s] += __shfl_xor(l[s], 32);
    if (!slot[s]) continue;
    const float r = 1.0f / l[s];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int d = (4 * lg + i) * 8;
      float e[8];
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) {  // o / l, the product by 1 / l corrected by its remainder
        const float v = o[s][dt][i] * r;
        e[dt] = __builtin_fmaf(__builtin_fmaf(-v, l[s], o[s][dt][i]), r, v);
      }
      if (d < HD) *(u32x4 *)((uint16_t *)a.out + attn_out_at(a, roff + sq[s], (j * G + sh) * HD + d, HD)) = pack<DT>(e);
    }
  }
}

// o = sum_s e^(m_s - M) o_s / sum_s e^(m_s - M) l_s over the n_split splits
// of one (query, head), in split order (empty splits have weight zero);
// rounded to the storage dtype.  NSF > 0: at most NSF splits, whose partials
// are all requested at once.
template <int DT, int HD, int NSF>
__global__ __launch_bounds__(HD) void k_combine(AttnArgs a) {
  const int h = blockIdx.x, qi = blockIdx.y, e = threadIdx.x;
  const int ns = a.n_split;
  const int64_t base = ((int64_t)qi * a.n_heads + h) * ns;
  float num = 0.f, den = 0.f;
  if constexpr (NSF > 0) {
    const rsrc_t mr = make_rsrc(a.part_ml + base * 2, (uint32_t)ns * 8u);
    const rsrc_t orr = make_rsrc(a.part_o + base * HD, (uint32_t)ns * HD * 4u);
    float m[NSF], l[NSF], o[NSF];
#pragma unroll
    for (int sp = 0; sp < NSF; ++sp) {
      const u32x2 ml = bld8(mr, (uint32_t)sp * 8u);
      m[sp] = sp < ns ? __uint_as_float(ml[0]) : -INFINITY;  // past the splits: weight zero, no branch
      l[sp] = __uint_as_float(ml[1]);                        // (one would let its loads be put behind it)
      o[sp] = __uint_as_float(bld4(orr, (uint32_t)(sp * HD + e) * 4u));
    }
    float M = -INFINITY;
#pragma unroll
    for (int sp = 0; sp < NSF; ++sp) M = fmaxf(M, m[sp]);
#pragma unroll
    for (int sp = 0; sp < NSF; ++sp) {
      const float w = expf(m[sp] - M);
      den += w * l[sp];
      num += w * o[sp];
    }
  } else {
    __shared__ float s_m[ATTN_MAX_SPLITS], s_w[ATTN_MAX_SPLITS];
    for (int sp = e; sp < ns; sp += HD) s_m[sp] = a.part_ml[(base + sp) * 2];
    __syncthreads();
    float M = -INFINITY;
    for (int sp = 0; sp < ns; ++sp) M = fmaxf(M, s_m[sp]);
    for (int sp = e; sp < ns; sp += HD) s_w[sp] = expf(s_m[sp] - M);
    __syncthreads();
    for (int sp = 0; sp < ns; ++sp) {
      den += s_w[sp] * a.part_ml[(base + sp) * 2 + 1];
      num += s_w[sp] * a.part_o[(base + sp) * HD + e];
    }
  }
  st_elem<DT>(a.out, attn_out_at(a, qi, h * HD + e, HD), num / den);
}

template <int DT, int HD, bool PAGED>
hipError_t attn_hd(int group, int nq, const AttnArgs &a, hipStream_t st) {
  if (DT != HS_F32 && a.prefill) return hipErrorInvalidValue;  // 16-bit prefill runs k_attn_prefill
  const dim3 grid(a.n_split, a.n_kv, nq), block(64 * ATTN_WAVES);
  switch (group) {
    case 1: HS_LAUNCH((k_attn<DT, HD, 1, ATTN_WAVES, PAGED>), grid, block, 0, st, a); break;
    case 2: HS_LAUNCH((k_attn<DT, HD, 2, ATTN_WAVES, PAGED>), grid, block, 0, st, a); break;
    case 4:
      if constexpr (DT == HS_F32) HS_LAUNCH((k_attn<DT, HD, 4, ATTN_WAVES, PAGED>), grid, block, 0, st, a);
      else HS_LAUNCH((k_attn_mma<DT, HD, 4, ATTN_WAVES, PAGED>), grid, block, 0, st, a);
      break;
    case 7:
      if constexpr (DT == HS_F32) HS_LAUNCH((k_attn<DT, HD, 7, ATTN_WAVES, PAGED>), grid, block, 0, st, a);
      else HS_LAUNCH((k_attn_mma<DT, HD, 7, ATTN_WAVES, PAGED>), grid, block, 0, st, a);
      break;
    case 8:
      if constexpr (DT == HS_F32) HS_LAUNCH((k_attn<DT, HD, 8, ATTN_WAVES, PAGED>), grid, block, 0, st, a);
      else HS_LAUNCH((k_attn_mma<DT, HD, 8, ATTN_WAVES, PAGED>), grid, block, 0, st, a);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int DT>
hipError_t attn_dt(int head_dim, int group, int nq, const AttnArgs &a, hipStream_t st) {
  // pooled caches hold 16-bit storage only
  if constexpr (DT != HS_F32) {
    if (a.kv.paged) {
      if (head_dim == 64) return attn_hd<DT, 64, true>(group, nq, a, st);
      if (head_dim == 128) return attn_hd<DT, 128, true>(group, nq, a, st);
      return hipErrorInvalidValue;
    }
  }
  if (head_dim == 64) return attn_hd<DT, 64, false>(group, nq, a, st);
  if (head_dim == 128) return attn_hd<DT, 128, false>(group, nq, a, st);
  return hipErrorInvalidValue;
}

template <int DT, int HD>
hipError_t combine_hd(int nq, const AttnArgs &a, hipStream_t st) {
  const dim3 grid(a.n_heads, nq), block(HD);
  if (a.n_split <= 8) HS_LAUNCH((k_combine<DT, HD, 8>), grid, block, 0, st, a);
  else if (a.n_split <= 16) HS_LAUNCH((k_combine<DT, HD, 16>), grid, block, 0, st, a);
  else HS_LAUNCH((k_combine<DT, HD, 0>), grid, block, 0, st, a);
  return hipGetLastError();
}

template <int DT>
hipError_t combine_dt(int head_dim, int nq, const AttnArgs &a, hipStream_t st) {
  if (head_dim == 64) return combine_hd<DT, 64>(nq, a, st);
  if (head_dim == 128) return combine_hd<DT, 128>(nq, a, st);
  return hipErrorInvalidValue;
}

template <int DT, int HD, int QT>
hipError_t prefill_hd(int group, const AttnArgs &a, hipStream_t st) {
  const int share = 8 / a.prefill_xh;
  const dim3 grid((a.prefill_groups + share - 1) / share * (a.n_kv / a.prefill_xh) * 8), block(64 * PREFILL_WAVES);
  switch (group) {
    case 1: HS_LAUNCH((k_attn_prefill<DT, HD, 1, PREFILL_WAVES, QT>), grid, block, 0, st, a); break;
    case 2: HS_LAUNCH((k_attn_prefill<DT, HD, 2, PREFILL_WAVES, QT>), grid, block, 0, st, a); break;
    case 4: HS_LAUNCH((k_attn_prefill<DT, HD, 4, PREFILL_WAVES, QT>), grid, block, 0, st, a); break;
    case 7: HS_LAUNCH((k_attn_prefill<DT, HD, 7, PREFILL_WAVES, QT>), grid, block, 0, st, a); break;
    case 8: HS_LAUNCH((k_attn_prefill<DT, HD, 8, PREFILL_WAVES, QT>), grid, block, 0, st, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <int DT>
hipError_t prefill_dt(int head_dim, int group, const AttnArgs &a, hipStream_t st) {
  const bool two = a.prefill_qt == 2;
  if (!two && a.prefill_qt != 1) return hipErrorInvalidValue;
  if (head_dim == 64) return two ? prefill_hd<DT, 64, 2>(group, a, st) : prefill_hd<DT, 64, 1>(group, a, st);
  if (head_dim == 128) return two ? prefill_hd<DT, 128, 2>(group, a, st) : prefill_hd<DT, 128, 1>(group, a, st);
  return hipErrorInvalidValue;
}

}  // namespace

bool attn_prefill_on_mma(int dtype) { return dtype != HS_F32; }

// Query tiles per wave: two (each K/V tile read from LDS once for both) where
// that leaves enough work groups, else one.
constexpr int PREFILL_TWO_FROM = 512;
int attn_prefill_groups(int group, int n_kv, int n, const int *cu, int *groups) {
  const int qpt = 16 / group;
  for (int qt = 2;; qt = 1) {
    const int rows = PREFILL_WAVES * qt * qpt;
    int64_t sum = 0;
    for (int i = 0; i < n; ++i) sum += groups[i] = (cu[i + 1] - cu[i] + rows - 1) / rows;
    if (qt == 1 || sum * n_kv >= PREFILL_TWO_FROM) return qt;
  }
}

hipError_t launch_attention_prefill(int dtype, int head_dim, int group, int nrows, const AttnArgs &a,
                                    hipStream_t st) {
  if (nrows <= 0 || a.prefill_groups <= 0) return hipSuccess;
  if (a.prefill_xh <= 0 || 8 % a.prefill_xh || a.n_kv % a.prefill_xh || !a.prefill_order) return hipErrorInvalidValue;
  if (dtype == HS_F16) return prefill_dt<HS_F16>(head_dim, group, a, st);
  if (dtype == HS_BF16) return prefill_dt<HS_BF16>(head_dim, group, a, st);
  return hipErrorInvalidValue;
}

bool attn_supported(int dtype, int head_dim, int group) {
  (void)dtype;
  return (head_dim == 64 || head_dim == 128) && (group == 1 || group == 2 || group == 4 || group == 7 || group == 8);
}

hipError_t launch_attention(int dtype, int head_dim, int group, int nq, const AttnArgs &a, hipStream_t st) {
  if (nq <= 0) return hipSuccess;
  switch (dtype) {
    case HS_F32: return attn_dt<HS_F32>(head_dim, group, nq, a, st);
    case HS_F16: return attn_dt<HS_F16>(head_dim, group, nq, a, st);
    case HS_BF16: return attn_dt<HS_BF16>(head_dim, group, nq, a, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_combine(int dtype, int head_dim, int nq, const AttnArgs &a, hipStream_t st) {
  if (nq <= 0 || a.n_split <= 1) return hipSuccess;
  switch (dtype) {
    case HS_F32: return combine_dt<HS_F32>(head_dim, nq, a, st);
    case HS_F16: return combine_dt<HS_F16>(head_dim, nq, a, st);
    case HS_BF16: return combine_dt<HS_BF16>(head_dim, nq, a, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace hs
