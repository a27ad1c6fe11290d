"""Every work-group tile of the many-column GEMM with every way it stores, at the real projection sizes: one decode step
of one LLaVA-1.5-7B- or Qwen2.5-VL-7B-shaped layer with its LM head, at batches chosen so that the launch rule takes each
of them (gemm_plan.SHAPE_CASES; test_gemm_plan.py checks that it does).  Requests repeat seven patterns of token, cache
rows, length and RoPE position, so that all columns of a batch are compared with seven oracle steps: logits, token,
residual stream and the appended K/V rows.

fp32 storage has GEMMs of its own (k_gemm_lds and k_gemm_tile by the number of work groups), here with 1024-wide rows,
192 / 64 / 2 x 344 / 64 / 512 row tiles (q/k/v, O, gate/up, down, head), over
  48 columns:   k_gemm_tile for the head (64 groups of 8 x 8), 8 x 8 tiles for gate/up (86), K splits for the others;
  300:          8 x 8 tiles for gate/up (264 groups) and the head (192), K splits for the others;
  900:          16 x 8 for gate/up (384) and the head (256), 8 x 8 without a split for q/k/v (192);
  2049:         16 x 16 for gate/up (432) and the head (288), 16 x 8 for q/k/v (272), 8 x 8 for O and down (136);
  3400:         16 x 16 for q/k/v (224), 16 x 8 for O and down (216)."""
from __future__ import annotations

import gc

import pytest
import torch

import gemm_plan as G
from helpers import KV_ROW0_TOL, LOGIT_TOL
from oracle import oracle as O
from workload import synth

pytestmark = pytest.mark.gpu
PATTERNS, CAP = 7, 4  # 7: prime to the 16 columns of a tile
CASES = dict(G.SHAPE_CASES, f32=[48, 300, 900, 2049, 3400])
# fp32: sums of up to 5504 products of either sign, sqrt(5504) 2^-24 = 4e-6 of their size each, a handful in a row
F32_TOL = 1e-4


def _pattern(p):
    return 1 + p % 3, 2 + 3 * p  # length, RoPE position


class Case:
    def __init__(self, name):
        import paper_2603_12707_amd as hs
        self.cfg = cfg = G.shape_cfg(name)
        cpu, self.gpu = {}, {}
        for n in synth.weight_names(cfg):
            t = synth.make_weight(cfg, n, device="cuda")
            cpu[n] = t.cpu()
            self.gpu[n] = hs.pack_weight(cfg, n, t)
            del t
        ora = O.Model(cfg, cpu)
        nkv, hd = cfg["n_kv_heads"], cfg["head_dim"]
        self.tok = synth.uniform_int(11, "tok", PATTERNS, 0, cfg["vocab"] - 1)
        self.kv = synth.normal(11, "kv", (PATTERNS, 2, nkv, CAP, hd), 1.0, cfg["dtype"])
        self.logits, self.hidden, self.next, self.rows = [], [], [], []
        for p in range(PATTERNS):
            length, rope = _pattern(p)
            seq = ora.new_seq(CAP)
            for sel in range(2):
                for h in range(nkv):
                    seq.write_kv(0, sel, h, 0, self.kv[p, sel, h, :length].float())
            seq.set_len(length, rope)
            logits, hidden, tok = seq.decode(int(self.tok[p]))
            self.logits.append(torch.from_numpy(logits.copy()))
            self.hidden.append(torch.from_numpy(hidden.copy()))
            self.next.append(tok)
            self.rows.append(torch.stack([torch.stack([torch.from_numpy(seq.read_kv(0, sel, h, length, 1)[0].copy())
                                                       for h in range(nkv)]) for sel in range(2)]))
        for k in ("logits", "hidden", "rows"):
            setattr(self, k, torch.stack(getattr(self, k)).cuda())
        self.next = torch.tensor(self.next, device="cuda")


@pytest.fixture(scope="module")
def made():
    kept = {}
    yield kept
    kept.clear()
    gc.collect()
    torch.cuda.empty_cache()


@pytest.fixture
def case(request, made):
    """The model's case, made once (one model at a time: the cases are in model order)."""
    if request.param not in made:
        made.clear()
        gc.collect()
        torch.cuda.empty_cache()
        made[request.param] = Case(request.param)
    return made[request.param]


def _worst(got, ref):
    """largest over the rows of max |got - ref| / max |ref|"""
    err = (got - ref).abs().flatten(1).amax(1) / ref.abs().flatten(1).amax(1)
    assert torch.isfinite(err).all()
    return float(err.max())


@pytest.mark.timeout(300)
@pytest.mark.parametrize("case,batch", [(m, n) for m, ns in CASES.items() for n in ns], indirect=["case"])
def test_decode_batches_of_every_shape(case, batch):
    import paper_2603_12707_amd as hs
    cfg = case.cfg
    tol, row_tol = (F32_TOL, F32_TOL) if cfg["dtype"] == "f32" else (LOGIT_TOL, KV_ROW0_TOL)
    model = hs.Model(cfg, case.gpu, max_batch=batch, max_ctx=32, packed=True)
    which = torch.arange(batch) % PATTERNS
    buf = case.kv[which].cuda()  # request r: its own copy of pattern r % 7
    kv = hs.KVCache(model, [0] * batch, [CAP] * batch, buf.view(-1).view(torch.uint8))
    for r in range(batch):
        kv.set_length(r, *_pattern(r % PATTERNS))
    tin = case.tok[which].to(torch.int32).cuda()
    tout = torch.full_like(tin, -1)
    logits = torch.full((batch, cfg["vocab"]), float("nan"), device="cuda")
    hidden = torch.full((batch, cfg["d_model"]), float("nan"), device="cuda")
    kv.decode(tin, tout, logits, hidden)
    torch.cuda.synchronize()
    assert model.status() == 0
    at = torch.tensor([_pattern(r % PATTERNS)[0] for r in range(batch)], device="cuda")
    which = which.cuda()
    appended = buf[torch.arange(batch, device="cuda"), :, :, at].float()  # [batch, K|V, head, channel]
    per_row = (appended - case.rows[which]).flatten(0, 2), case.rows[which].flatten(0, 2)
    assert float((per_row[0].abs().amax(1) / per_row[1].abs().amax(1)).max()) <= row_tol
    assert _worst(hidden, case.hidden[which]) <= tol
    ref = case.logits
    for lo in range(0, batch, 512):  # (a chunk of columns at a time: 152064 words)
        w, got = which[lo:lo + 512], logits[lo:lo + 512]
        assert _worst(got, ref[w]) <= tol
        # the token: the oracle's, or one within twice the largest difference of it
        tok = tout[lo:lo + 512].long()
        gap = ref[w].gather(1, case.next[w, None]) - ref[w].gather(1, tok[:, None])
        assert bool((gap[:, 0] <= 2 * (got - ref[w]).abs().amax(1)).all())
    kv.close()
    model.close()
