// hs_gemm_dma.h — GEMM over more than 32 columns in 16-bit storage (large
// decode batches, prefill rows), both operands copied from memory straight
// into LDS.
#pragma once

#include "hs_gemm_epi.h"
#include "hs_gemm_plan.h"

#include <type_traits>
#include <utility>

namespace hs {
namespace dev {

// NR LDS reads spread over NM MFMAs
template <int I, int NR, int NM>
__device__ __forceinline__ void dma_sched() {
  if constexpr (I < NR) {
    __builtin_amdgcn_sched_group_barrier(0x008, NM * (I + 1) / (NR + 1) - NM * I / (NR + 1), 0);
    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    dma_sched<I + 1, NR, NM>();
  } else {
    __builtin_amdgcn_sched_group_barrier(0x008, NM - NM * NR / (NR + 1), 0);
  }
}

// lane row q (lanes 16 q .. 16 q + 15) holds word q of four chunks, chunk i's
// in x_i; afterwards it holds chunk q
__device__ __forceinline__ u32x4 transpose4(uint32_t x0, uint32_t x1, uint32_t x2, uint32_t x3) {
  const auto a = __builtin_amdgcn_permlane16_swap(x0, x1, false, false);
  const auto b = __builtin_amdgcn_permlane16_swap(x2, x3, false, false);
  const auto c = __builtin_amdgcn_permlane32_swap(a[0], b[0], false, false);
  const auto d = __builtin_amdgcn_permlane32_swap(a[1], b[1], false, false);
  return u32x4{c[0], d[0], c[1], d[1]};
}

// f(0, 1, ...) with the numbers as types
template <class F, int... T>
__device__ __forceinline__ void dma_each(F f, std::integer_sequence<int, T...>) {
  f(std::integral_constant<int, T>{}...);
}

// four consecutive values in the storage dtype, 8 bytes
template <int DT>
__device__ __forceinline__ u32x2 pack4(float a, float b, float c, float d) {
  return u32x2{pack2<DT>(a, b), pack2<DT>(c, d)};
}

// Work unit u of one K range -> row group and column group: super rows of SH
// row groups, in each the column groups in turn, in each of these the row
// groups, so that the units an XCD runs at a time share operands in its L2.
__device__ __forceinline__ void dma_unit(int u, int nrg, int ncg, int &rg, int &cg) {
  constexpr int SH = 8;
  const int sr = u / (SH * ncg), sh = min(SH, nrg - sr * SH), v = u - sr * SH * ncg;
  rg = sr * SH + v % sh;
  cg = v / sh;
}

// row tile t of row group rg -> matrix and first row
template <int EPI, int TR, int RTW>
__device__ __forceinline__ void dma_tile(const GemmArgs &a, int rg, int t, int &m, int &r0) {
  if constexpr (EPI == EPI_SWIGLU) {
    constexpr int H = RTW / 2;
    const int w = t / RTW, k = t % RTW;
    m = k < H ? 0 : 1;
    r0 = 16 * (rg * (TR / 2) + w * H + k % H);
  } else {
    int u = rg * TR + t;
    m = 0;
    if (a.rows[1] > 0) {  // q, k, v in turn
      const int tq = a.rows[0] / 16, tk = a.rows[1] / 16;
      if (u >= tq) {
        u -= tq;
        m = 1;
        if (u >= tk) {
          u -= tk;
          m = 2;
        }
      }
    }
    r0 = 16 * u;  // past the rows in a partial last group
  }
}

// The q/k/v epilogue of a whole work group: bias, RoPE, R(q) and the K/V
// append.  A column's request, position, block and RoPE positions are a chain
// of four dependent reads, so the work group makes it once, one column per
// thread, into LDS (free after the main loop; walking it per column tile in
// every wave cost ~60 us of each 12 x 20 tile).  The four lanes that hold one
// column's 16 packed rows of a tile, 8 channels of each head half in 4-byte
// words, exchange words with those of three more tiles or halves (a 4 x 4
// transpose by row swaps), so that every lane stores one whole 16-byte chunk.
template <int DT, int NW, int TR, int TC, int RTW, int CTW>
__device__ __forceinline__ void dma_qkv(const GemmArgs &a, unsigned char *s_mem, int rg, int wtile0, int gcol0, int wcol0,
                                        const int *mat, const int *row0, const f32x4 (&acc)[RTW][CTW]) {
  static_assert(RTW % 2 == 0, "chunks in groups of four");
  constexpr int NC = TC * 16;
  int64_t *s_kv = (int64_t *)s_mem;            // K row of head 0 of this layer at the column's position (negative: none)
  int *s_bh = (int *)(s_mem + NC * 8);         // elements from one KV head to the next
  int *s_pos = s_bh + NC;                      // RoPE positions [3][NC], one per section
  const int hd = a.head_dim, half = hd >> 1;
  const bool per_sec = a.prefill && a.rope_m3;
  for (int t = threadIdx.x; t < NC; t += 64 * NW) {
    const int col = gcol0 + t;
    const bool ok = col < a.ncols;
    int pos, cap, bt, req;
    int64_t base;
    if (a.kv.paged) req = qkv_fetch_row<true>(a, ok ? col : 0, ok, pos, cap, bt, base);
    else req = qkv_fetch_row<false>(a, ok ? col : 0, ok, pos, cap, bt, base);
    const rsrc_t pr = qkv_pos_rsrc(a);
    uint32_t p[3];
#pragma unroll
    for (int s = 0; s < 3; ++s)
      p[s] = bld4(pr, ok ? (uint32_t)(per_sec ? s * a.rope_ld + col : req) * 4u : BUF_OOB);
#pragma unroll
    for (int s = 0; s < 3; ++s)
      s_pos[s * NC + t] = min(max(!a.prefill || a.rope_m3 ? (int)p[s] : pos, 0), a.rope_max - 1);
    s_kv[t] = base < 0 ? -1 : base + ((int64_t)a.layer * 2 * a.n_kv * bt + (a.kv.paged ? pos % bt : pos)) * hd;
    s_bh[t] = bt * hd;
  }
  const int lane = threadIdx.x & 63, li = lane & 15, lq = lane >> 4, rr = 4 * lq;
  // this lane's biases (elements j0, j0 + 1 of both head halves) and table
  // entries of every tile; where the sections split a pair of neighbours,
  // each has its own position
  uint32_t bias[RTW][2];
  int j0[RTW], sec[RTW];
  const bool odd_sec = per_sec && ((a.sec0 | a.sec1) & 1);
#pragma unroll
  for (int r = 0; r < RTW; ++r) {
    const int m = mat[r], head = row0[r] / hd;
    const bool live = row0[r] < a.rows[m];
    j0[r] = (row0[r] - head * hd + rr) >> 1;
    sec[r] = j0[r] < a.sec0 ? 0 : (j0[r] < a.sec1 ? 1 : 2);
    const rsrc_t bq = make_rsrc(a.bias[m], a.bias[m] ? (uint32_t)a.rows[m] * 2u : 0u);
    bias[r][0] = bld4(bq, live ? (uint32_t)(head * hd + j0[r]) * 2u : BUF_OOB);
    bias[r][1] = bld4(bq, live ? (uint32_t)(head * hd + half + j0[r]) * 2u : BUF_OOB);
  }
  // store group s: chunks of four (tile, half) items, item lq this lane's;
  // whole groups of four tiles take one half each, two last tiles both halves
  constexpr int NS = RTW / 2;
  int s_m[NS], s_head[NS], s_ch[NS];  // matrix (-1: past the rows), K/V slab, first channel
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const bool quad = s / 2 * 4 + 4 <= RTW;
    const int r = quad ? s / 2 * 4 + lq : RTW - 2 + (lq & 1), h = quad ? s & 1 : lq >> 1;
    int m, r0;
    dma_tile<EPI_QKV, TR, RTW>(a, rg, wtile0 + r, m, r0);
    const int head = r0 / hd;
    s_m[s] = r0 < a.rows[m] ? m : -1;
    s_head[s] = m == 2 ? a.n_kv + head : head;
    s_ch[s] = (r0 - head * hd) / 2 + h * half;
  }
  __syncthreads();
  const float *tab = a.rope_tab;
  // cos, sin of pairs j0 and j0 + 1, one column tile ahead where the registers allow it
  constexpr int AHEAD = RTW * CTW < 32 ? 1 : 0;
  f32x4 cs[1 + AHEAD][RTW];
  auto fetch = [&](int c, f32x4 *out) {
    const int t = wcol0 + c * 16 + li;
#pragma unroll
    for (int r = 0; r < RTW; ++r) {
      if (mat[r] == 2 || row0[r] >= a.rows[mat[r]]) continue;  // wave-uniform
      out[r] = *(const f32x4 *)(tab + 2 * ((int64_t)s_pos[sec[r] * NC + t] * half + j0[r]));
      if (odd_sec) {
        const int i = j0[r] + 1, s1 = i < a.sec0 ? 0 : (i < a.sec1 ? 1 : 2);
        const float *e = tab + 2 * ((int64_t)s_pos[s1 * NC + t] * half + i);
        out[r][2] = e[0];
        out[r][3] = e[1];
      }
    }
  };
  if (AHEAD) fetch(0, cs[0]);
#pragma unroll
  for (int c = 0; c < CTW; ++c) {
    if (!AHEAD) fetch(c, cs[0]);
    else if (c + 1 < CTW) fetch(c + 1, cs[(c + 1) & AHEAD]);
    const int t = wcol0 + c * 16 + li, col = gcol0 + t;
    uint32_t w[RTW][2];
#pragma unroll
    for (int r = 0; r < RTW; ++r) {
      float o1[2], o2[2];
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const uint32_t h1 = (bias[r][0] >> (16 * e)) & 0xFFFFu, h2 = (bias[r][1] >> (16 * e)) & 0xFFFFu;
        const float v1 = acc[r][c][2 * e] + (DT == HS_F16 ? f16_to_f32(h1) : bf16_to_f32(h1));
        const float v2 = acc[r][c][2 * e + 1] + (DT == HS_F16 ? f16_to_f32(h2) : bf16_to_f32(h2));
        o1[e] = v1;
        o2[e] = v2;
        if (mat[r] < 2) {
          const float co = cs[c & AHEAD][r][2 * e], si = cs[c & AHEAD][r][2 * e + 1];
          o1[e] = v1 * co - v2 * si;
          o2[e] = v2 * co + v1 * si;
        }
      }
      const u32x2 p = pack4<DT>(o1[0], o1[1], o2[0], o2[1]);
      w[r][0] = p[0];
      w[r][1] = p[1];
    }
    const int64_t kv = s_kv[t];
    const int bh = s_bh[t];
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int g = s / 2 * 4;
      u32x4 x;
      if (g + 4 <= RTW) x = transpose4(w[g][s & 1], w[g + 1][s & 1], w[g + 2][s & 1], w[g + 3][s & 1]);
      else x = transpose4(w[RTW - 2][0], w[RTW - 1][0], w[RTW - 2][1], w[RTW - 1][1]);
      if (col < a.ncols) {
        if (s_m[s] == 0) *(u32x4 *)((uint16_t *)a.out + (int64_t)col * a.ld_out + s_head[s] * hd + s_ch[s]) = x;
        else if (s_m[s] > 0 && kv >= 0) *(u32x4 *)((uint16_t *)a.kv.buf + kv + (int64_t)s_head[s] * bh + s_ch[s]) = x;
      }
    }
  }
}

// Y[c][n] = sum_k X[c][k] W[n][k].  Weights and activations sit in the packed
// layout (16 rows or columns x 32 elements = 1 KB in MFMA operand order), so
// one wave-wide 16-byte buffer load to LDS moves one sub-block, lane l's 16
// bytes to LDS byte 16 l, and a wave reads an MFMA operand back with one
// conflict-free ds_read_b128.  No register and no write instruction stages the
// data.
//
// A work group of WR x WC waves owns TR = WR RTW row tiles and TC = WC CTW
// column tiles; wave (wr, wc) computes RTW x CTW of them over the work group's
// K range.  K advances in stages of KS sub-blocks through a ring of ST stages
// in LDS.  A wave reads the operands of the next sub-block while it issues the
// MFMAs of the present one, the reads spread between them.  At a stage's last
// sub-block it waits for its own loads of the next stage (the counter then
// still covers ST - 2 stages), meets the others at one barrier, and requests
// the stage ST on into the slot that this one leaves (its operands are in
// registers by then).
//
// The shapes of decode batches take two sub-blocks per stage: half the
// barriers, and 2 KB of a row tile requested at a time; where a single column
// group reads the weights, they are loaded with the non-temporal hint.  Decode
// layer: 120 requests 297 -> 277 us, 75 326 -> 314, 256 623 -> 610; gate/up
// over 75 columns (22016 x 4096) 52.9 -> 42.9 us (traced alone 44.8), over 120
// (37888 x 3584) 60.7 -> 54.7 (57.1), over 256 85.6 -> 80.2 (81.4).  The loads
// alone, in this order without the arithmetic, take 35-37 us over 75 columns
// and 48 over 120.
//
// What bounds it.  In decode about 36-40 B/ns of operands pass per CU: weights
// from HBM (in this order loads alone reach 6.1 TB/s, 24 B/ns per CU; a plain
// read of 4 GiB reaches 7.0) and activations from L2 (loads alone 128 B/ns)
// together, so a tile's time is about its bytes, 1 KB x (TR + TC) per
// sub-block, and the launcher takes the shape with the fewest bytes per CU that
// still fills the chip.  The largest tile (16 x 16) is bound by the clock that
// the power limit leaves and by the waits at its stages: 37888 x 3584 over
// 14370 columns runs 3.0-3.2 ms (1220-1310 TFLOP/s; hipBLASLt 3.15), at
// 1.85 GHz, its MFMAs 64 % busy, its waves waiting 28 % of their time, LDS 24 %
// busy without bank conflicts; with both operands staged through registers it
// took 4.05 ms.  A 4-wave variant with wave tiles of 8 x 8 (one wave per SIMD,
// a quarter fewer LDS reads) took 3.82 ms.  One round of 230-240 work groups
// (640 rows) keeps its MFMAs 35-50 % busy: each group fills its ring, runs and
// stores with nothing beside it.
//
// EPI: EPI_SWIGLU; EPI_QKV (bias, RoPE, R(q), K/V append; K not split); or
// EPI_STORE, fp32 rows by a.f32_out: logits, K-split partials (residual rows,
// or q|k|v rows in turn), or the residual add
template <int DT, int WR, int WC, int RTW, int CTW, int KS, int ST, int EPI, bool NT>
__global__ __launch_bounds__(64 * WR * WC) __attribute__((amdgpu_waves_per_eu(WR * WC / 4, 2)))
void k_gemm_dma(GemmArgs a) {
  constexpr int NW = WR * WC, TR = WR * RTW, TC = WC * CTW;
  constexpr int NB = (TR + TC) * KS;        // sub-blocks per stage
  // Of them moved per wave: row tiles' first, column tiles' after.  With
  // several sub-blocks per stage each kind is dealt out by itself (LA and LB
  // loads per wave), so that a load's kind, and with it the cache hint, is
  // known at compile time; some waves may move empty ones (their counters
  // agree).
  constexpr bool APART = KS > 1;
  constexpr int LA = APART ? (TR * KS + NW - 1) / NW : 0, LB = APART ? (TC * KS + NW - 1) / NW : (NB + NW - 1) / NW;
  constexpr int LPW = LA + LB;
  constexpr bool PAD = APART ? LA * NW > TR * KS || LB * NW > TC * KS : LB * NW > NB;
  static_assert((KS > 1 ? KS % 2 == 0 : ST % 2 == 0) && (ST - 1) * LPW <= 63, "ring depth");
  static_assert(!NT || APART, "the hint needs the kinds apart");
  static_assert(EPI != EPI_SWIGLU || RTW % 2 == 0, "gate/up pairs per wave");
  __shared__ __align__(1024) unsigned char s_mem[(ST * NB + (PAD ? 1 : 0)) * 1024];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wr = wave / WC, wc = wave % WC, li = lane & 15, lq = lane >> 4;
  const int nsb = (a.K / 8 + 15) / 16 * 4;  // sub-blocks of a packed row or column tile

  // Work units in the order (K split, unit); each XCD (work groups are dealt
  // to the 8 of them round robin) takes one run of them.  The units of a split
  // tail follow, a unit's K ranges one after another.
  const int nrg = a.n_groups, ncg = a.n_colg, per = nrg * ncg;
  const int total = a.tail_split > 1 ? a.tail_from : per * a.k_split;
  const int q8 = total >> 3, r8 = total & 7, xcd = (int)blockIdx.x & 7, behind = (int)blockIdx.x - total;
  const bool tail = EPI == EPI_STORE && behind >= 0;
  const int unit = tail ? total + behind / a.tail_split
                        : (xcd < r8 ? xcd * (q8 + 1) : r8 * (q8 + 1) + (xcd - r8) * q8) + ((int)blockIdx.x >> 3);
  const int nks = tail ? a.tail_split : a.k_split, sp = tail ? behind % a.tail_split : unit / per;
  int rg, cg;
  dma_unit(tail ? unit : unit - sp * per, nrg, ncg, rg, cg);
  // this split's sub-blocks [g0, g0 + ns), whole k-blocks of 4, in n stages, at least ST (the launcher sees to it)
  const int kper = (nsb / 4 + nks - 1) / nks * 4;
  const int g0 = sp * kper, ns = min(nsb, g0 + kper) - g0, n = ns / KS;

  // this wave's LPW sub-blocks of every stage; tiles past the data have an
  // empty range (nothing is read, and what their operands hold reaches only
  // outputs that are not stored)
  u32x4 rs[LPW];
  uint32_t live[LPW], ldst[LPW];
  const int n_ct = (a.ncols + 15) >> 4;
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int b = !APART ? wave * LPW + i : i < LA ? wave * LA + i : TR * KS + wave * LB + i - LA;
    const bool row = APART ? i < LA : b < TR;
    const bool pad = b >= (row ? TR * KS : NB);
    const int t = pad ? 0 : b / KS, k = b % KS;
    uint64_t p;
    bool in;
    if (row) {
      int m, r0;
      dma_tile<EPI, TR, RTW>(a, rg, t, m, r0);
      in = r0 < a.rows[m];
      p = (uint64_t)a.w[m] + ((uint64_t)(in ? r0 >> 4 : 0) * nsb + g0 + k) * 1024u;
    } else {
      const int ct = cg * TC + t - TR;
      in = !pad && ct < n_ct;
      p = (uint64_t)a.x + ((uint64_t)(in ? ct : 0) * nsb + g0 + k) * 1024u;
    }
    in = in && !pad;
    rs[i] = u32x4{(uint32_t)p, (uint32_t)(p >> 32), in ? (uint32_t)(ns - k) * 1024u : 0u, (uint32_t)BUF_WORD3};
    live[i] = in ? ~0u : 0u;
    ldst[i] = PAD && pad ? ~0u : (uint32_t)b * 1024u;
  }
  const uint32_t lds0 = lds_addr(s_mem);
  const uint32_t vo = (uint32_t)lane * 16u;
  // With one column group each work group starts its K range at another stage
  // (wrapping round), so that the chip's row tiles do not walk the same
  // address bits in step: 37888 x 3584 over 256 columns 84 -> 76 us, 4096 x
  // 11008 in 8 splits over 64 columns 20.4 -> 18.5 us.  With several column
  // groups the stages stay in step for the L2.
  const int rot = ncg == 1 ? (int)(((uint32_t)unit * 37u) % (uint32_t)n) : 0;
  auto issue = [&](int s, int slot) {
    int g = s + rot;
    g -= g >= n ? n : 0;
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
      const uint32_t dst = PAD && ldst[i] == ~0u ? (uint32_t)(ST * NB) * 1024u : (uint32_t)(slot * NB) * 1024u + ldst[i];
      if (NT && i < LA) dma_1k_stream(rs[i], vo, (uint32_t)g * (KS * 1024u) & live[i], lds0 + dst);
      else dma_1k(rs[i], vo, (uint32_t)g * (KS * 1024u) & live[i], lds0 + dst);
    }
  };

  f32x4 acc[RTW][CTW];
#pragma unroll
  for (int r = 0; r < RTW; ++r)
#pragma unroll
    for (int c = 0; c < CTW; ++c) acc[r][c] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < ST; ++s) issue(s, s);
  u32x4 av[2][RTW], bv[2][CTW];
  const unsigned char *la = s_mem + wr * RTW * KS * 1024 + lane * 16;
  const unsigned char *lb = s_mem + (TR + wc * CTW) * KS * 1024 + lane * 16;
  dma_sync<(ST - 1) * LPW>();
#pragma unroll
  for (int r = 0; r < RTW; ++r) av[0][r] = *(const u32x4 *)(la + r * KS * 1024);
#pragma unroll
  for (int c = 0; c < CTW; ++c) bv[0][c] = *(const u32x4 *)(lb + c * KS * 1024);
  int slot = 0;
  // the MFMAs of the operands in set `cur`, and meanwhile the reads of the
  // sub-block at `at` (bytes into a tile's place in the ring) into the other
  auto step = [&](auto CUR, auto NEXT, int at) {
    constexpr int cur = decltype(CUR)::value;
    if constexpr (decltype(NEXT)::value) {
#pragma unroll
      for (int c = 0; c < CTW; ++c) bv[cur ^ 1][c] = *(const u32x4 *)(lb + at + c * KS * 1024);
#pragma unroll
      for (int r = 0; r < RTW; ++r) av[cur ^ 1][r] = *(const u32x4 *)(la + at + r * KS * 1024);
    }
#pragma unroll
    for (int r = 0; r < RTW; ++r)
#pragma unroll
      for (int c = 0; c < CTW; ++c) acc[r][c] = mma<DT>(av[cur][r], bv[cur][c], acc[r][c]);
    if constexpr (decltype(NEXT)::value) dma_sched<0, RTW + CTW, RTW * CTW>();
  };
  using std::integral_constant;
  using Yes = std::true_type;
  using No = std::false_type;
  // CUR: the register set of the stage's first sub-block; LEFT: loads that may
  // stay in flight at its barrier; MORE: a stage to request; NEXT: a stage
  // whose first operands to read.  The barrier stands before the last
  // sub-block's MFMAs: by then every wave has the stage's operands in
  // registers.
  auto stage = [&](int s, auto CUR, auto LEFT, auto MORE, auto NEXT) {
    constexpr int cur = decltype(CUR)::value;
    dma_each(
        [&](auto... T) { (step(integral_constant<int, (cur + decltype(T)::value) & 1>{}, Yes{}, (slot * NB + decltype(T)::value + 1) * 1024), ...); },
        std::make_integer_sequence<int, KS - 1>{});
    dma_sync<decltype(LEFT)::value>();
    const int nx = slot + 1 == ST ? 0 : slot + 1;
    if constexpr (decltype(MORE)::value) issue(s + ST, slot);
    step(integral_constant<int, (cur + KS - 1) & 1>{}, NEXT, nx * NB * 1024);
    slot = nx;
  };
  constexpr int ODD = KS % 2;  // with one sub-block per stage the register sets change from stage to stage
  int s = 0;
  for (; s < n - ST; s += 1 + ODD) {  // ODD: n and ST are even
    stage(s, integral_constant<int, 0>{}, integral_constant<int, (ST - 2) * LPW>{}, Yes{}, Yes{});
    if constexpr (ODD)
      stage(s + 1, integral_constant<int, 1>{}, integral_constant<int, (ST - 2) * LPW>{}, Yes{}, Yes{});
  }
  // the last ST stages, all requested
  dma_each(
      [&](auto... T) {
        (stage(s + decltype(T)::value, integral_constant<int, decltype(T)::value & ODD>{},
               integral_constant<int, (ST - 2 > decltype(T)::value ? ST - 2 - decltype(T)::value : 0) * LPW>{}, No{},
               std::bool_constant<(decltype(T)::value < ST - 1)>{}),
         ...);
      },
      std::make_integer_sequence<int, ST>{});

  // lane (li, lq) holds rows 4 lq .. 4 lq + 3 of each row tile for column li of each column tile
  int mat[RTW], row0[RTW];
#pragma unroll
  for (int r = 0; r < RTW; ++r) dma_tile<EPI, TR, RTW>(a, rg, wr * RTW + r, mat[r], row0[r]);
  const int rr = 4 * lq;
  if constexpr (EPI == EPI_QKV) {
    dma_qkv<DT, NW, TR, TC, RTW, CTW>(a, s_mem, rg, wr * RTW, cg * TC * 16, wc * CTW * 16, mat, row0, acc);
    return;
  }
#pragma unroll
  for (int c = 0; c < CTW; ++c) {
    const int col = (cg * TC + wc * CTW + c) * 16 + li;
    if (col >= a.ncols) continue;
    if constexpr (EPI == EPI_SWIGLU) {
      constexpr int H = RTW / 2;
      const int nkb_o = (a.rows[0] / 8 + 15) / 16;
#pragma unroll
      for (int r = 0; r < H; ++r) {
        const int j = row0[r] + rr;
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float g = acc[r][c][e], u = acc[r + H][c][e];
          o[e] = g / (1.0f + expf(-g)) * u;
        }
        // rows[0] is a multiple of 8: the four rows are in or out together, and 8-byte aligned
        const int64_t at = a.out_packed ? packed_x_index(col, j, nkb_o) : (int64_t)col * a.ld_out + j;
        if (j < a.rows[0]) *(u32x2 *)((uint16_t *)a.out + at) = pack4<DT>(o[0], o[1], o[2], o[3]);
      }
    } else if (a.f32_out == F32_LOGITS) {
      float *o = (float *)a.out + (int64_t)col * a.ld_out;
      const bool vec = (a.ld_out & 3) == 0 && ((uintptr_t)a.out & 15) == 0;  // the caller's buffer
#pragma unroll
      for (int r = 0; r < RTW; ++r) {
        const int row = row0[r] + rr;
        if (vec && row + 3 < a.rows[0]) {
          *(f32x4 *)(o + row) = acc[r][c];
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (row + e < a.rows[0]) o[row + e] = acc[r][c][e];
        }
      }
    } else {
      // fp32 rows of which there is a multiple of 4, 16-byte aligned
      const bool add = a.f32_out == F32_RESID && !tail;
      const int nrow = a.rows[0] + a.rows[1] + a.rows[2];
      float *o = add ? a.resid + (int64_t)col * a.ld_resid : a.splitk_ws + ((int64_t)sp * a.ncols + col) * nrow;
      if (tail)  // rows and columns of the work-group tile
        o = a.splitk_ws - rg * TR * 16 +
            (((int64_t)sp * (per - total) + unit - total) * (TC * 16) + col - cg * TC * 16) * (TR * 16);
#pragma unroll
      for (int r = 0; r < RTW; ++r) {
        const int row = 16 * (rg * TR + wr * RTW + r) + rr;
        if (row < nrow) {
          f32x4 v = acc[r][c];
          if (add) v += *(const f32x4 *)(o + row);
          *(f32x4 *)(o + row) = v;
        }
      }
    }
  }
}

// x += the partials of a split tail's unit blockIdx.y, in split order; four
// rows of one column per thread
__global__ __launch_bounds__(256) void k_dma_tail_sum(GemmArgs a, int tr, int tc) {
  const int nu = a.n_groups * a.n_colg - a.tail_from, r4 = tr * 4, i = (int)blockIdx.x * 256 + threadIdx.x;
  int rg, cg;
  dma_unit(a.tail_from + (int)blockIdx.y, a.n_groups, a.n_colg, rg, cg);
  const int lc = i / r4, lr = i % r4 * 4, col = cg * tc * 16 + lc, row = rg * tr * 16 + lr;
  if (lc >= tc * 16 || col >= a.ncols || row >= a.rows[0]) return;
  const int64_t slice = (int64_t)nu * tc * tr * 256;
  const float *p = a.splitk_ws + ((int64_t)blockIdx.y * tc * 16 + lc) * (tr * 16) + lr;
  f32x4 s = *(const f32x4 *)p;
  for (int k = 1; k < a.tail_split; ++k) s += *(const f32x4 *)(p + k * slice);
  *(f32x4 *)(a.resid + (int64_t)col * a.ld_resid + row) += s;
}

template <int DT, int WR, int WC, int RTW, int CTW, int KS, int ST, int EPI>
hipError_t dma_start(const GemmArgs &g, hipStream_t st) {
  const int n = g.n_groups * g.n_colg;
  const dim3 units(g.tail_split > 1 ? g.tail_from + (n - g.tail_from) * g.tail_split : n * g.k_split), block(64 * WR * WC);
  // weights that one column group reads alone are not kept in the caches
  bool alone = false;
  if constexpr (KS > 1) {
    alone = g.n_colg == 1;
    if (alone) HS_LAUNCH((k_gemm_dma<DT, WR, WC, RTW, CTW, KS, ST, EPI, true>), units, block, 0, st, g);
  }
  if (!alone) HS_LAUNCH((k_gemm_dma<DT, WR, WC, RTW, CTW, KS, ST, EPI, false>), units, block, 0, st, g);
  const hipError_t e = hipGetLastError();
  if (EPI != EPI_STORE || e != hipSuccess || g.tail_split <= 1) return e;
  constexpr int TR = WR * RTW, TC = WC * CTW;
  HS_LAUNCH(k_dma_tail_sum, dim3((TR * TC * 64 + 255) / 256, n - g.tail_from), dim3(256), 0, st, g, TR, TC);
  return hipGetLastError();
}

template <int DT>
hipError_t gemm_dma(int epi, const GemmArgs &a, int tiles16, int *parts, hipStream_t st) {
  *parts = 0;
  DmaPlan p;
  if (!a.x_packed || !dma_plan(epi, a, tiles16, &p)) return hipErrorInvalidValue;
  GemmArgs g = a;
  g.k_split = p.k_split;
  g.n_groups = p.n_groups;
  g.n_colg = p.n_colg;
  g.tail_from = p.tail_from;
  g.tail_split = p.tail_split;
  g.f32_out = p.partial ? F32_PARTS : epi == EPI_RESID ? F32_RESID : F32_LOGITS;
  if (p.partial) *parts = p.k_split;
  const bool direct_qkv = epi_qkv(epi) && !p.partial;
  switch (p.shape) {
#define HS_DMA_CASE(I, WR, WC, RTW, CTW, KS, ST)                                                    \
  case I:                                                                                           \
    if (epi == EPI_SWIGLU) return dma_start<DT, WR, WC, RTW, CTW, KS, ST, EPI_SWIGLU>(g, st);           \
    if constexpr (I >= DMA_WIDE_FROM)                                                               \
      if (direct_qkv) return dma_start<DT, WR, WC, RTW, CTW, KS, ST, EPI_QKV>(g, st);                   \
    if (direct_qkv) return hipErrorInvalidValue;                                                    \
    return dma_start<DT, WR, WC, RTW, CTW, KS, ST, EPI_STORE>(g, st);
    HS_DMA_SHAPES(HS_DMA_CASE)
#undef HS_DMA_CASE
  }
  return hipErrorInvalidValue;
}

}  // namespace dev
}  // namespace hs
