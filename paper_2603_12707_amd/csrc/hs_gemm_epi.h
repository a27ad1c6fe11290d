// hs_gemm_epi.h — row-tile maps and epilogues shared by the GEMM kernels: logits, residual add, SwiGLU, and the
// q/k/v epilogue (bias, RoPE, R(q), K/V append).
#pragma once

#include "hs_device.h"

namespace hs {
namespace dev {

// ---------------------------------------------------------------------------
// row tiles
// ---------------------------------------------------------------------------
// q/k/v: R consecutive tiles of the q, k, v matrices taken in turn (their
// rows packed in head-paired order); SwiGLU pairs row j of the gate and of
// the up projection; the other epilogues take R consecutive tiles.
// rows of a K-split GEMM's partials: the residual rows, or q|k|v rows in turn
__host__ __device__ inline int split_rows(const GemmArgs &a, int epi) {
  return epi_qkv(epi) ? (a.n_heads + 2 * a.n_kv) * a.head_dim : a.rows[0];
}

template <int EPI, int R>
__device__ __forceinline__ void tile_map(const GemmArgs &a, int g, int *mat, int *row0) {
  if constexpr (epi_qkv(EPI)) {
    const int tq = a.n_heads * a.head_dim / 16, tk = a.n_kv * a.head_dim / 16;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      int m = 0, t = g * R + r;
      if (t >= tq) {
        t -= tq;
        m = 1;
        if (t >= tk) {
          t -= tk;
          m = 2;
        }
      }
      mat[r] = m;
      row0[r] = 16 * t;  // past the v rows for a partial last group
    }
  } else if constexpr (EPI == EPI_SWIGLU) {
    mat[0] = 0;
    mat[1] = 1;
    row0[0] = row0[1] = 16 * g;
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r) {
      mat[r] = 0;
      row0[r] = 16 * (R * g + r);
    }
  }
}

// PK: the SwiGLU output goes to the packed activation layout where a.out_packed
// says so (the down projection reads it so): k_gemm's, up to 32 columns.
// k_gemm_dma stores that layout in its own epilogue, and the fp32 kernels for
// wider GEMMs never write it.
template <int DT, int EPI, int R, bool PK = false>
__device__ __forceinline__ void gemm_epilogue(const GemmArgs &a, const int *mat, const int *row0, const f32x4 *v,
                                              int col, int rr) {
  if constexpr (EPI == EPI_STORE) {
    float *o = (float *)a.out + (int64_t)col * a.ld_out;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = row0[r] + rr + e;
        if (row < a.rows[mat[r]]) o[row] = v[r][e];
      }
  } else if constexpr (EPI == EPI_RESID) {
    float *x = a.resid + (int64_t)col * a.ld_resid;
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int row = row0[r] + rr + e;
        if (row < a.rows[mat[r]]) x[row] += v[r][e];
      }
  } else if constexpr (EPI == EPI_SWIGLU) {
    const bool packed = PK && a.out_packed;
    const int nkb_o = (a.rows[0] / 8 + 15) / 16;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int j = row0[0] + rr + e;
      if (j < a.rows[0]) {
        const float g = v[0][e], u = v[1][e];
        const int64_t at = packed ? packed_x_index(col, j, nkb_o) : (int64_t)col * a.ld_out + j;
        st_elem<DT>(a.out, at, g / (1.0f + expf(-g)) * u);
      }
    }
  }
}

// q/k/v epilogue inputs of one thread (one output column, packed rows
// rr..rr+3 of each of its R tiles: RoPE pairs (j, j + d_h/2) and
// (j + 1, j + 1 + d_h/2)), read ahead of the main loop: the KV position,
// capacity and base of the column's request and the RoPE position of each
// pair first; the cos/sin entries and the biases once those positions are in.
// Every read goes through a buffer range, so none sits behind a branch.
template <int R>
struct QkvIn {
  int pos, cap, bt;
  int64_t base;  // start of the block holding pos (negative: none)
  int p[R][2];
  float cs[R][2], sn[R][2], b1[R][2], b2[R][2];
};

// column col's request, position, capacity and block; returns the request
template <bool PAGED>
__device__ __forceinline__ int qkv_fetch_row(const GemmArgs &a, int col, bool ok, int &pos, int &cap, int &bt,
                                             int64_t &base) {
  const bool dec = !a.prefill;
  const KvRef &kv = a.kv;
  // decode: column col is request act[col]; prefill: the packed row's request
  // and its position in that request
  int req = 0, ppos = 0;
  if (!dec) {
    const int i = packed_request(a.pk, col);
    req = a.pk->req[i];
    ppos = col - a.pk->cu[i];
  }
  const uint32_t nb = (uint32_t)kv.nreq * 4u;
  if constexpr (PAGED) {
    const rsrc_t ar = make_rsrc(kv.act, dec ? (uint32_t)a.ncols * 4u : 0u);
    if (dec) req = (int)bld4(ar, ok ? (uint32_t)col * 4u : BUF_OOB);
  } else if (dec) {
    req = col;
  }
  const rsrc_t lr = make_rsrc(kv.len, dec ? nb : 0u), cr = make_rsrc(kv.cap, nb);
  const rsrc_t br = make_rsrc(kv.tab, (uint32_t)kv.ntab * 8u);
  const uint32_t ro = ok ? (uint32_t)req * 4u : BUF_OOB;
  const uint32_t pl = bld4(lr, dec ? ro : BUF_OOB);
  cap = (int)bld4(cr, ro);
  if constexpr (PAGED) {  // the block holding the position
    const rsrc_t or_ = make_rsrc(kv.toff, nb), tr = make_rsrc(kv.bt, nb);
    const int toff = (int)bld4(or_, ro);
    bt = max(1, (int)bld4(tr, ro));
    pos = dec ? (int)pl : ppos;
    const u32x2 bb = bld8(br, ok && pos < cap ? (uint32_t)(toff + pos / bt) * 8u : BUF_OOB);
    base = ok && pos < cap ? (int64_t)(((uint64_t)bb[1] << 32) | bb[0]) : -1;
  } else {  // one block per request: its start, read beside the length
    const u32x2 bb = bld8(br, ok ? (uint32_t)req * 8u : BUF_OOB);
    bt = cap;
    pos = dec ? (int)pl : ppos;
    base = ok && pos < cap ? (int64_t)(((uint64_t)bb[1] << 32) | bb[0]) : -1;
  }
  return req;
}
// the RoPE positions: of the requests (decode), of the packed rows per section (prefill M-RoPE), or not read
__device__ __forceinline__ rsrc_t qkv_pos_rsrc(const GemmArgs &a) {
  return make_rsrc(a.rope_pos, !a.prefill ? (uint32_t)a.kv.nreq * 4u : (a.rope_m3 ? 3u * a.rope_ld * 4u : 0u));
}

template <int DT, int R, bool PAGED>
__device__ __forceinline__ void qkv_fetch_ids(const GemmArgs &a, const int *mat, const int *row0, int col, int rr,
                                              bool ok, QkvIn<R> &in) {
  const bool dec = !a.prefill;
  const rsrc_t pr = qkv_pos_rsrc(a);
  const int req = qkv_fetch_row<PAGED>(a, col, ok, in.pos, in.cap, in.bt, in.base);
  const int hd = a.head_dim;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int j0 = (row0[r] % hd + rr) >> 1;
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int i = j0 + e, sec = i < a.sec0 ? 0 : (i < a.sec1 ? 1 : 2);
      const bool rot = ok && mat[r] < 2 && (dec || a.rope_m3);
      const uint32_t pv = bld4(pr, rot ? (uint32_t)(dec ? req : sec * a.rope_ld + col) * 4u : BUF_OOB);
      in.p[r][e] = (dec || a.rope_m3) ? (int)pv : in.pos;
    }
  }
}

template <int DT, int R>
__device__ __forceinline__ void qkv_fetch_tab(const GemmArgs &a, const int *mat, const int *row0, int rr, bool ok,
                                              QkvIn<R> &in) {
  const int hd = a.head_dim, half = hd >> 1;
  const rsrc_t tr = make_rsrc(a.rope_tab, (uint32_t)a.rope_max * half * 8u);
  constexpr int SB = DT == HS_F32 ? 4 : 2;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int m = mat[r], head = row0[r] / hd, j0 = (row0[r] - head * hd + rr) >> 1;
    const bool live = ok && row0[r] < a.rows[m];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int p = min(max(in.p[r][e], 0), a.rope_max - 1);
      const u32x2 t = bld8(tr, live && m < 2 ? (uint32_t)(p * half + j0 + e) * 8u : BUF_OOB);
      in.cs[r][e] = __uint_as_float(t[0]);
      in.sn[r][e] = __uint_as_float(t[1]);
    }
    const rsrc_t bq = make_rsrc(a.bias[m], a.bias[m] ? (uint32_t)a.rows[m] * SB : 0u);
    const uint32_t o1 = (uint32_t)(head * hd + j0) * SB, o2 = (uint32_t)(head * hd + half + j0) * SB;
    if constexpr (DT == HS_F32) {
      const u32x2 v1 = bld8(bq, live ? o1 : BUF_OOB), v2 = bld8(bq, live ? o2 : BUF_OOB);
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        in.b1[r][e] = __uint_as_float(v1[e]);
        in.b2[r][e] = __uint_as_float(v2[e]);
      }
    } else {
      const uint32_t v1 = bld4(bq, live ? o1 : BUF_OOB), v2 = bld4(bq, live ? o2 : BUF_OOB);
#pragma unroll
      for (int e = 0; e < 2; ++e) {
        const uint32_t h1 = (v1 >> (16 * e)) & 0xFFFFu, h2 = (v2 >> (16 * e)) & 0xFFFFu;
        in.b1[r][e] = DT == HS_F16 ? f16_to_f32(h1) : bf16_to_f32(h1);
        in.b2[r][e] = DT == HS_F16 ? f16_to_f32(h2) : bf16_to_f32(h2);
      }
    }
  }
}

// bias, RoPE on q and k, then R(q) to the q workspace and k, v rows appended
// to the cache at the request's position
template <int DT, int R, bool PAGED>
__device__ __forceinline__ void qkv_store(const GemmArgs &a, const int *mat, const int *row0, const f32x4 *v, int col,
                                          int rr, const QkvIn<R> &in) {
  constexpr int B = DT == HS_F32 ? 4 : 2;
  const int hd = a.head_dim, half = hd >> 1;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int m = mat[r];
    if (row0[r] >= a.rows[m]) continue;
    const int head = row0[r] / hd, j0 = (row0[r] - head * hd + rr) >> 1;
    float w1[2], w2[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const float v1 = v[r][2 * e] + in.b1[r][e], v2 = v[r][2 * e + 1] + in.b2[r][e];
      float o1 = v1, o2 = v2;
      if (m < 2) {
        o1 = v1 * in.cs[r][e] - v2 * in.sn[r][e];
        o2 = v2 * in.cs[r][e] + v1 * in.sn[r][e];
      }
      w1[e] = o1;
      w2[e] = o2;
    }
    // pairs j0 and j0 + 1 (j0 is even): two neighbouring elements of each half
    if (m == 0) {
      void *q = (char *)a.out + ((int64_t)col * a.ld_out + head * hd) * B;
      st_elem2<DT>(q, j0, w1[0], w1[1]);
      st_elem2<DT>(q, j0 + half, w2[0], w2[1]);
    } else if (in.base >= 0) {
      const int pin = PAGED ? in.pos % in.bt : in.pos;  // position within its block
      const int64_t off = in.base + ((int64_t)((a.layer * 2 + (m == 2 ? 1 : 0)) * a.n_kv + head) * in.bt + pin) * hd;
      st_elem2<DT>(a.kv.buf, off + j0, w1[0], w1[1]);
      st_elem2<DT>(a.kv.buf, off + j0 + half, w2[0], w2[1]);
    }
  }
}

}  // namespace dev
}  // namespace hs
