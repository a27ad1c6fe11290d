// hs_gemm_plan.h — the launch rule of the many-column GEMM (k_gemm_dma): its
// work-group tiles and the choice of tile and K split.  Host code alone.
#pragma once

#include <algorithm>

#include "hs_internal.h"

namespace hs {
namespace dev {

// ---------------------------------------------------------------------------
// the shape of a launch
// ---------------------------------------------------------------------------
// Work-group tiles, TR x TC row x column tiles.  Up to 16 column tiles a
// single column group reads every weight once from HBM; TR then follows the
// number of row tiles, so that they make close to a whole number of work
// groups per CU.  The wide ones are for prefill rows.
#define HS_DMA_SHAPES(X)   \
  X(0, 1, 4, 6, 1, 2, 4)   \
  X(1, 1, 4, 8, 1, 2, 4)   \
  X(2, 1, 4, 10, 1, 2, 4)  \
  X(3, 1, 4, 6, 2, 2, 4)   \
  X(4, 1, 4, 8, 2, 2, 4)   \
  X(5, 1, 4, 10, 2, 2, 4)  \
  X(6, 1, 8, 6, 2, 2, 3)   \
  X(7, 1, 8, 8, 2, 2, 3)   \
  X(8, 1, 8, 10, 2, 2, 3)  \
  X(9, 2, 4, 4, 5, 1, 4)   \
  X(10, 2, 4, 6, 5, 1, 4)  \
  X(11, 2, 4, 8, 2, 1, 6)  \
  X(12, 2, 4, 8, 4, 1, 4)
constexpr int DMA_WIDE_FROM = 9;  // shapes with a q/k/v epilogue of their own

struct DmaShape {
  int tr, tc, fill;  // fill: sub-blocks of K that fill the ring
};
struct DmaPlan {
  int shape, k_split;
  bool partial;  // fp32 partials for split_finish
  int n_groups, n_colg;
  int tail_from, tail_split;
};

// Takes the shape and K split with the least estimated time.  A CU passes
// about 40 B/ns of operands, so a work group takes 25 ns per stage and
// sub-block (or, on few columns per row tile, what its MFMAs take), plus ~2.5
// us to fill and drain its ring; the chip takes as many rounds of work groups
// as 256 CUs need.  fp32 partials cost their bytes written and read once and
// a launch.  A residual projection's last round, where it leaves half the CUs
// idle or more, is cut over K instead into as many ranges as give every CU one:
// 3584 x 18944 over 14370 columns, 798 tiles of 16 x 16, takes three rounds and
// an eighth instead of four (O and down, both layers: 4270 -> 3770 us).
// How far the choice is from the best: every shape and split timed for each
// GEMM of both 7B-shaped models at 33, 48, 64, 75, 96, 120, 160, 200, 256, 320,
// 512 and 640 columns, weights from HBM.  Of the 120, 93 are within 6 % of the
// best and 113 within 15 %, 3 % in the sum.  The worst are O over 75-120
// columns (4096 x 4096 over 120: 22.0 us with 8 splits of 8 x 8 tiles, 17.0 with
// 4 of 8 x 4) and down over 320 (52.6 against 44.3; 74.9 against 63.4); q/k/v is
// up to 14 % off, the LM head 13 %, gate/up 5 %.  (O and q/k/v of 64-160 columns
// would do with half the splits.)
inline bool dma_plan(int epi, const GemmArgs &a, int tiles16, DmaPlan *best) {
  static constexpr DmaShape shapes[] = {
#define HS_DMA_ENTRY(I, WR, WC, RTW, CTW, KS, ST) {WR * RTW, WC * CTW, KS * ST},
      HS_DMA_SHAPES(HS_DMA_ENTRY)
#undef HS_DMA_ENTRY
  };
  constexpr int n_shapes = (int)(sizeof(shapes) / sizeof(shapes[0]));
  const int nsb = (a.K / 8 + 15) / 16 * 4, n_ct = (a.ncols + 15) / 16;
  const bool qkv = epi_qkv(epi), resid = epi == EPI_RESID;
  const int64_t prows = qkv ? (int64_t)a.rows[0] + a.rows[1] + a.rows[2] : a.rows[0];
  double least = 0.0;
  bool found = false;
  for (int i = 0; i < n_shapes; ++i) {
    const DmaShape &sh = shapes[i];
    const int rows_per = epi == EPI_SWIGLU ? sh.tr / 2 : sh.tr;
    const int nrg = (tiles16 + rows_per - 1) / rows_per, ncg = (n_ct + sh.tc - 1) / sh.tc;
    const double load = 25.0 * (sh.tr + (double)n_ct / ncg), mfma = 2.4 * sh.tr * sh.tc;
    for (int ks = 1; ks <= DMA_SPLIT_MAX; ++ks) {
      const int kper = (nsb / 4 + ks - 1) / ks * 4, last = nsb - (ks - 1) * kper;
      if (last < sh.fill) break;  // every split fills the ring
      const bool partial = (resid && ks > 1) || (qkv && (ks > 1 || i < DMA_WIDE_FROM));
      if (ks > 1 && !partial) break;
      const int64_t floats = (int64_t)ks * a.ncols * prows;
      if (partial && (!a.splitk_ws || prows % 4 || floats > a.splitk_cap || floats > DMA_SPLIT_FLOATS)) continue;
      const int64_t units = (int64_t)nrg * ncg * ks;
      double t = (double)((units + 255) / 256) * (kper * (load > mfma ? load : mfma) + 2500.0);
      if (partial) t += 4000.0 + (double)floats * 8.0 / 5000.0;
      if (!found || t < least) {
        found = true;
        least = t;
        *best = DmaPlan{i, ks, partial, nrg, ncg, 0, 1};
      }
      const int64_t rest = units % 256;
      const int ts = resid && !partial && units > 256 && rest && prows % 4 == 0 && a.splitk_ws
                         ? (int)std::min<int64_t>(DMA_SPLIT_MAX, 256 / rest) : 1;
      if (ts > 1) {
        const int tk = (nsb / 4 + ts - 1) / ts * 4;
        const int64_t tf = ts * rest * sh.tr * sh.tc * 256;
        if (nsb - (ts - 1) * tk >= sh.fill && tf <= a.splitk_cap && tf <= DMA_SPLIT_FLOATS) {
          const double each = load > mfma ? load : mfma;
          t = (double)(units / 256) * (kper * each + 2500.0) + tk * each + 6500.0 + (double)tf * 8.0 / 5000.0;
          if (t < least) {
            least = t;
            *best = DmaPlan{i, ks, partial, nrg, ncg, (int)(units - rest), ts};
          }
        }
      }
    }
  }
  return found;
}

}  // namespace dev
}  // namespace hs
