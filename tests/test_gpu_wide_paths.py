"""Small cases at the edges of the wide GEMM's work-group tiles and of the prefill attention's work groups, against the
oracle: the q/k/v epilogue that walks a column's metadata once per work group (RoPE sections that split a pair of
neighbours, biases, ragged columns, contiguous and pooled caches), decode batches around its column tiles, and key
steps, query tiles and requests that end inside a step."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from helpers import KV_ROW0_TOL, LOGIT_TOL, Pair, rel_err, small_cfg, to_device, token_ok
from workload import synth

pytestmark = pytest.mark.gpu
TDT = {"f16": torch.float16, "bf16": torch.bfloat16}


def _prefill(cfg, shapes, pool, weights=None):
    """Prefills the requests (n_v, s_text) in one pass; returns the cache, the oracle's sequences and their tokens
    after checking every request's logits, first token and layer-0 K/V rows."""
    import paper_2603_12707_amd as hs
    n = len(shapes)
    caps = [a + b + 4 for a, b in shapes]
    pair = Pair(cfg, max_batch=n, max_ctx=max(caps), weights_cpu=weights)
    pair.gpu.reserve_rows(sum(a + b for a, b in shapes))
    if pool:
        kv = hs.KVPool(pair.gpu, n, 256, sum(-(-c // 256) for c in caps))
        for r, (n_v, _) in enumerate(shapes):
            kv.admit(r, n_v, caps[r])
    else:
        kv = hs.KVCache(pair.gpu, [a for a, _ in shapes], caps)
    ins = [pair.request_inputs(r, a, b) for r, (a, b) in enumerate(shapes)]
    embs, ids = [e for e, _, _ in ins if e.shape[0]], [i for _, i, _ in ins if i.shape[0]]
    pos = torch.cat([p for _, _, p in ins], dim=1).contiguous().cuda() if cfg["rope_kind"] == 1 else None
    logits = torch.empty(n, cfg["vocab"], dtype=torch.float32, device="cuda")
    toks = kv.prefill_batch(list(range(n)), torch.cat(embs).cuda() if embs else None,
                            torch.cat(ids).cuda() if ids else None, [b for _, b in shapes], pos, last_logits=logits)
    torch.cuda.synchronize()
    toks, got = toks.cpu().tolist(), logits.cpu().numpy()
    seqs, nxt = [], []
    for r, (n_v, s_text) in enumerate(shapes):
        s = pair.ora.new_seq(caps[r])
        emb, i, p = ins[r]
        ref, tok = s.prefill(emb if n_v else None, i, p)
        assert rel_err(got[r], ref) <= LOGIT_TOL, (r, rel_err(got[r], ref))
        assert token_ok(toks[r], got[r], ref)[0], (r, toks[r], tok)
        for at in {0, (n_v + s_text) // 2, n_v + s_text - 1}:
            for h in {0, cfg["n_kv_heads"] - 1}:
                for sel in range(2):
                    row = torch.empty(1, cfg["head_dim"], dtype=TDT[cfg["dtype"]], device="cuda")
                    kv.read(r, 0, sel, h, at, 1, row)
                    err = rel_err(row.float().cpu().numpy(), s.read_kv(0, sel, h, at, 1))
                    assert err <= KV_ROW0_TOL, (r, at, h, sel, err)
        seqs.append(s)
        nxt.append(tok)
    return pair, kv, seqs, nxt


# (heads, KV heads, head_dim, M-RoPE sections or None, bias, dtype, pooled)
PREFILLS = {
    "mha_f16": (8, 8, 128, None, 0, "f16", False),
    "gqa7_odd_sections_bf16_pool": (14, 2, 128, (15, 26, 23), 1, "bf16", True),
    "gqa4_hd64_f16_pool": (8, 2, 64, (7, 12, 13), 0, "f16", True),
    "gqa8_bf16": (8, 1, 128, None, 1, "bf16", False),
    "gqa2_hd64_bf16": (6, 3, 64, (8, 12, 12), 1, "bf16", False),
}


@pytest.mark.parametrize("name", list(PREFILLS))
@pytest.mark.parametrize("shapes", [[(33, 1)], [(1, 63), (0, 65), (40, 88), (0, 1)], [(250, 63), (17, 3), (129, 128)]],
                         ids=["one_34", "mixed_258", "ragged_590"])
def test_prefill_edges(name, shapes):
    nh, nkv, hd, sec, bias, dtype, pool = PREFILLS[name]
    cfg = small_cfg(n_layers=1, d_model=512, n_heads=nh, n_kv_heads=nkv, head_dim=hd, ffn_dim=520, vocab=307,
                    dtype=dtype, qkv_bias=bias, rope_kind=1 if sec else 0, mrope_section=sec or (0, 0, 0))
    pair, kv, _, _ = _prefill(cfg, shapes, pool)
    assert pair.gpu.status() == 0
    kv.close()
    pair.gpu.close()


@pytest.mark.parametrize("sign", [1, -1], ids=["high", "low"])
@pytest.mark.parametrize("dtype,size", [("f16", 250.0), ("f16", 4e4), ("bf16", 250.0), ("bf16", 1e17)])
@pytest.mark.parametrize("nh,nkv,hd", [(4, 4, 64), (14, 2, 128)])
def test_prefill_scores_of_any_size(nh, nkv, hd, dtype, size, sign):
    """q rows that are all `size` and k rows that are all sign * size before RoPE (zero projections, constant biases):
    scores of either sign up to 1e11 (f16) and 1e36 (bf16), far past where the rounding of a score alone spans many
    units of its exponent.  The score at distance t is sign * size^2 * sum_i 2 cos(t theta_i): of positive ones the
    row's own is the largest by 3 %, of negative ones, at these context lengths, one is larger than every other by 2 %
    of the range, so that the softmax picks one position whatever the order of the sums."""
    cfg = small_cfg(n_layers=1, d_model=512, n_heads=nh, n_kv_heads=nkv, head_dim=hd, ffn_dim=520, vocab=307,
                    dtype=dtype, qkv_bias=1)
    w = synth.make_weights(cfg)
    for leaf, v in (("q", size), ("k", sign * size)):
        w["layers.0.w" + leaf].zero_()
        w["layers.0.b" + leaf].fill_(v)
    pair, kv, _, _ = _prefill(cfg, [(0, 1), (0, 4), (70, 2), (120, 9)], False, w)
    assert pair.gpu.status() == 0
    kv.close()
    pair.gpu.close()


def test_reserved_rows_run_as_created_ones():
    """Eight requests of 64 rows in one pass: a model whose rows were reserved after its creation gives, bit for bit,
    what one created for as many rows gives (the down projection splits K by the size of the workspace)."""
    import paper_2603_12707_amd as hs
    cfg = small_cfg(n_layers=1, d_model=1024, n_heads=8, n_kv_heads=8, head_dim=128, ffn_dim=4096, vocab=307,
                    dtype="f16")
    w = to_device(synth.make_weights(cfg))
    ids = torch.cat([synth.text_ids(cfg, r, 64) for r in range(8)]).cuda()
    got = []
    for max_ctx in (512, 64):
        model = hs.Model(cfg, w, max_batch=8, max_ctx=max_ctx)
        model.reserve_rows(512)
        kv = hs.KVCache(model, [0] * 8, [64] * 8)
        logits = torch.empty(8, cfg["vocab"], dtype=torch.float32, device="cuda")
        kv.prefill_batch(list(range(8)), None, ids, [64] * 8, None, last_logits=logits)
        torch.cuda.synchronize()
        got.append(logits)
        kv.close()
        model.close()
    assert torch.equal(got[0], got[1])


@pytest.mark.parametrize("batch", [33, 65, 129])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_decode_batches(batch, dtype):
    """One decode step over batches just past a column tile: K ranges of whole and of a partial k-block (d 640, F 1000),
    with their splits, after a packed prefill of as many requests."""
    cfg = small_cfg(n_layers=1, d_model=640, n_heads=8, n_kv_heads=2, head_dim=64, ffn_dim=1000, vocab=301, dtype=dtype,
                    qkv_bias=1)
    shapes = [(r % 5, 1 + r % 3) for r in range(batch)]
    pair, kv, seqs, nxt = _prefill(cfg, shapes, False)
    tin = torch.tensor(nxt, dtype=torch.int32, device="cuda")
    tout = torch.empty_like(tin)
    logits = torch.empty(batch, cfg["vocab"], dtype=torch.float32, device="cuda")
    kv.decode(tin, tout, logits)
    torch.cuda.synchronize()
    got, toks = logits.cpu().numpy(), tout.cpu().tolist()
    for r in range(batch):
        ref, _, tok = seqs[r].decode(nxt[r])
        assert rel_err(got[r], ref) <= LOGIT_TOL, (r, rel_err(got[r], ref))
        assert token_ok(toks[r], got[r], ref)[0], (r, toks[r], tok)
    assert pair.gpu.status() == 0
    kv.close()
    pair.gpu.close()


def test_release_keeps_the_other_requests():
    """Admission, a packed prefill, releases in any order and a second pass in the freed slots: the decode columns that
    stay are those of the requests that stay."""
    cfg = small_cfg(n_layers=1, d_model=512, n_heads=8, n_kv_heads=8, head_dim=64, ffn_dim=520, vocab=307, dtype="f16")
    shapes = [(5, 4), (0, 30), (300, 7), (2, 2)]
    pair, kv, seqs, nxt = _prefill(cfg, shapes, True)
    for gone in (2, 0):
        kv.release(gone)
    live = [1, 3]
    assert [n > 0 for n in kv.lengths()] == [r in live for r in range(4)]
    tin = torch.tensor([nxt[r] if r in live else 0 for r in range(4)], dtype=torch.int32, device="cuda")
    tout = torch.full_like(tin, -7)
    logits = torch.empty(2, cfg["vocab"], dtype=torch.float32, device="cuda")
    kv.decode(tin, tout, logits)
    torch.cuda.synchronize()
    got, toks = logits.cpu().numpy(), tout.cpu().tolist()
    for k, r in enumerate(live):
        ref, _, tok = seqs[r].decode(nxt[r])
        assert rel_err(got[k], ref) <= LOGIT_TOL
        assert token_ok(toks[r], got[k], ref)[0], (r, toks[r], tok)
    assert toks[0] == toks[2] == -7
    kv.release(3)
    kv.release(1)
    free, total = kv.blocks()
    assert free == total and kv.lengths() == [0, 0, 0, 0]
    kv.close()
    pair.gpu.close()


def test_residual_split_tail():
    """8934 rows at d 2048: 280 work-group tiles of O and down, whose last 24 (the last columns) are split eight ways over
    K.  The short requests in those columns against the oracle, a long one against its own prefill alone (another K order
    in fp32 moves a stored fp16 value by at most one rounding, 2^-11, at each of the layer's five; 2^-8 covers them)."""
    cfg = small_cfg(n_layers=1, d_model=2048, n_heads=16, n_kv_heads=16, head_dim=128, ffn_dim=2048, vocab=307,
                    dtype="f16")
    import paper_2603_12707_amd as hs
    shapes = [(300, 6)] * 29 + [(11, 9)] * 3
    pair = Pair(cfg, max_batch=len(shapes), max_ctx=310)
    pair.gpu.reserve_rows(sum(a + b for a, b in shapes))
    ins = [pair.request_inputs(r, a, b) for r, (a, b) in enumerate(shapes)]

    def run(reqs):
        kv = hs.KVCache(pair.gpu, [a for a, _ in shapes], [310] * len(shapes))
        logits = torch.empty(len(reqs), cfg["vocab"], dtype=torch.float32, device="cuda")
        kv.prefill_batch(reqs, torch.cat([ins[r][0] for r in reqs]).cuda(), torch.cat([ins[r][1] for r in reqs]).cuda(),
                         [shapes[r][1] for r in reqs], None, last_logits=logits)
        torch.cuda.synchronize()
        kv.close()
        return logits.cpu().numpy()

    got = run(list(range(len(shapes))))
    for r in (29, 30, 31):
        ref, _ = pair.ora.new_seq(30).prefill(ins[r][0], ins[r][1], None)
        assert rel_err(got[r], ref) <= LOGIT_TOL, (r, rel_err(got[r], ref))
    for r in (0, 28):
        assert rel_err(got[r], run([r])[0]) <= 2.0 ** -8, r
    pair.gpu.close()
