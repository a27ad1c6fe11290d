// The launch rule of the many-column GEMM as a host library, for the tests.
#include "hs_gemm_plan.h"

extern "C" int plan_gemm(int epi, int rows0, int rows1, int rows2, int K, int ncols, int64_t cap, int32_t *out) {
  static float ws;  // only whether there is a workspace counts
  hs::GemmArgs a{};
  a.rows[0] = rows0;
  a.rows[1] = rows1;
  a.rows[2] = rows2;
  a.K = K;
  a.ncols = ncols;
  a.splitk_ws = cap > 0 ? &ws : nullptr;
  a.splitk_cap = cap;
  const int tiles16 = hs::epi_qkv(epi) ? (rows0 + rows1 + rows2) / 16 : (rows0 + 15) / 16;
  hs::dev::DmaPlan p{};
  if (!hs::dev::dma_plan(epi, a, tiles16, &p)) return 0;
  const int32_t v[] = {p.shape, p.k_split, p.partial, p.n_groups, p.n_colg, p.tail_from, p.tail_split};
  for (int i = 0; i < 7; ++i) out[i] = v[i];
  return 1;
}
