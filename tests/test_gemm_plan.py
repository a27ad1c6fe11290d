"""The launch rule of the many-column GEMM, on the host: whatever the sizes, the plan it returns covers every row,
column and K range, fills its ring in each of them and keeps its partials inside the workspace."""
from __future__ import annotations

import itertools
import os
import random

import pytest

import gemm_plan as G

pytestmark = pytest.mark.skipif(not os.path.exists("/opt/rocm/include/hip/hip_runtime.h"), reason="no HIP headers")


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return G.build(str(tmp_path_factory.mktemp("plan") / "plan.so"))


def _cases():
    r = random.Random(7)
    dims = [8, 64, 128, 136, 256, 640, 688, 1000, 1024, 2048, 3584, 4096, 4608, 11008, 18944]
    cols = [33, 40, 48, 49, 64, 75, 96, 97, 120, 128, 129, 160, 192, 200, 256, 257, 320, 321, 512, 640, 2048, 3509,
            8934, 14370, 65536]
    for epi in G.EPI:
        for K, n in itertools.product(dims, cols):
            rows = {"store": (r.choice([1, 17, 301, 1024, 32000, 152064]),), "resid": (r.choice(dims),),
                    "swiglu": (r.choice(dims),) * 2}.get(epi)
            if epi == "qkv":
                hd, nkv = r.choice([64, 128]), r.choice([1, 2, 4, 8, 32])
                rows = (hd * nkv * r.choice([1, 2, 4, 7, 8]), hd * nkv, hd * nkv)
            for cap in (0, 4 * n * sum(rows) // 3, 1 << 20, 16 << 20):
                yield epi, rows, K, n, cap


def test_plans_of_all_sizes(lib):
    seen = set()
    for epi, rows, K, n, cap in _cases():
        p = G.plan(lib, epi, rows, K, n, cap)
        what = (epi, rows, K, n, cap, p)
        assert p is not None, what
        tr, tc, fill = G.SHAPES[p.shape]
        seen.add((p.shape, epi))
        tiles16 = sum(rows) // 16 if epi == "qkv" else (rows[0] + 15) // 16
        per_row = tr // 2 if epi == "swiglu" else tr
        assert (p.n_groups - 1) * per_row < tiles16 <= p.n_groups * per_row, what
        assert (p.n_colg - 1) * tc * 16 < n <= p.n_colg * tc * 16, what
        blocks = (K // 8 + 15) // 16  # k-blocks of four sub-blocks

        def ranges(parts):
            per = -(-blocks // parts) * 4
            return [min(4 * blocks, (i + 1) * per) - i * per for i in range(parts)]
        assert min(ranges(p.k_split)) >= fill, what
        assert p.k_split == 1 or p.partial, what  # split sums go through the workspace
        out_rows = sum(rows) if epi == "qkv" else rows[0]
        if p.partial:
            assert epi in ("resid", "qkv") and out_rows % 4 == 0, what
            assert p.k_split * n * out_rows <= min(cap, 16 << 20), what
        if epi == "qkv" and not p.partial:
            assert p.shape >= 9, what  # the shapes with a q/k/v epilogue of their own
        if p.tail_split > 1:
            units = p.n_groups * p.n_colg
            assert epi == "resid" and p.k_split == 1 and not p.partial, what
            assert 0 < p.tail_from < units and p.tail_from % 256 == 0, what
            assert min(ranges(p.tail_split)) >= fill, what
            tail = units - p.tail_from
            assert tail * p.tail_split <= 256 and tail * p.tail_split * tr * tc * 256 <= cap, what
    assert {s for s, _ in seen} == set(range(len(G.SHAPES)))


def test_step_scratch_of_all_sizes(lib):
    """A decode step's K-split partials: the static array holds them beside the layers' scratch whenever it accepts the
    step, they hold SPLITK_MAX splits of the widest GEMM, and the q/k/v, O and down plans find room."""
    import ctypes
    r = random.Random(3)
    static, less_seen = 64 << 20, 0
    for _ in range(4000):
        hd, nkv, g = r.choice([64, 128]), r.choice([1, 2, 4, 8, 32]), r.choice([1, 2, 4, 7, 8])
        d, F = 8 * r.randint(1, 700), 8 * r.randint(1, 2500)
        V, n, ns = r.choice([301, 32000, 152064]), r.randint(1, 700), r.choice([1, 1, 2, 8, 40])
        out = (ctypes.c_int64 * 4)()
        lib.plan_step(d, nkv * g, nkv, hd, F, V, r.randint(0, 2), n, ns, out)
        layers, logits, few, floats = out
        what = (d, nkv * g, nkv, hd, F, V, n, ns, list(out))
        rows = max(d, (g + 2) * nkv * hd)
        assert few == -(-16 * n * rows // 256) * 256 and floats >= 4 * n * rows, what
        assert floats <= max(4 * n * rows, min(8 * n * rows, 16 << 20)), what
        if layers + few <= static:  # accepted, with the caller's logits or (logits in the layers' place) its own
            assert layers + -(-4 * floats // 256) * 256 <= static, what
        less_seen += floats < min(8 * n * rows, 16 << 20)
    assert less_seen > 50


def test_shape_cases_run_every_kind(lib):
    """The decode batches that the GPU tests compare with the oracle (test_gpu_gemm_shapes.py) reach whatever the rule
    chooses over the batches below 4100."""
    want, got = {}, set()
    for model, batches in G.SHAPE_CASES.items():
        cfg = G.shape_cfg(model)
        for n in itertools.chain(range(33, 700), range(700, 4100, 7)):
            for g, kind in G.step_kinds(lib, cfg, n).items():
                want.setdefault(kind, (model, g, n))
        for n in batches:
            got |= set(G.step_kinds(lib, cfg, n).values())
    missing = {k: w for k, w in want.items() if k not in got}
    assert not missing, missing
    assert {s for s, kind, _ in got if kind == "swiglu"} >= {0, 2, 3, 5, 6, 8, 10, 12}
    assert {s for s, _, _ in got} == set(range(len(G.SHAPES)))


def test_shapes_table(lib):
    """SHAPES repeats the library's table."""
    import re
    with open(os.path.join(G.ROOT, "paper_2603_12707_amd", "csrc", "hs_gemm_plan.h")) as f:
        rows = re.findall(r"X\((\d+), (\d+), (\d+), (\d+), (\d+), (\d+), (\d+)\)", f.read())
    got = [(wr * rtw, wc * ctw, ks * st) for _, wr, wc, rtw, ctw, ks, st in (map(int, r) for r in rows)]
    assert got == G.SHAPES
