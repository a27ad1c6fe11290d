// The launch rule of the many-column GEMM and the scratch of a decode step as a host library, for the tests.
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

// out: bytes of the layers' scratch, of the logits and of SPLITK_MAX splits of the widest GEMM, floats of partials
extern "C" void plan_step(int d, int n_heads, int n_kv, int head_dim, int ffn, int vocab, int dtype, int n, int n_split,
                          int64_t *out) {
  hs_config c{};
  c.d_model = d;
  c.n_heads = n_heads;
  c.n_kv_heads = n_kv;
  c.head_dim = head_dim;
  c.ffn_dim = ffn;
  c.vocab = vocab;
  c.dtype = dtype;
  const hs::StepScratch s = hs::step_scratch(c, n, n_split);
  out[0] = (int64_t)s.layers();
  out[1] = (int64_t)s.logits;
  out[2] = (int64_t)hs::whole256(hs::SPLITK_MAX * n * hs::splitk_rows(c) * 4);
  out[3] = hs::step_splitk_floats(c, n, n_split);
}
