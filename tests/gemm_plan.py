"""The library's launch rule of the many-column GEMM, compiled for the host (tests/plan/plan_query.cpp)."""
from __future__ import annotations

import collections
import ctypes
import os
import subprocess

from workload import configs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
EPI = {"store": 0, "resid": 1, "swiglu": 2, "qkv": 3}
# row tiles, column tiles and ring depth (sub-blocks of 32 elements of K) of the shapes
SHAPES = [(6, 4, 8), (8, 4, 8), (10, 4, 8), (6, 8, 8), (8, 8, 8), (10, 8, 8), (6, 16, 6), (8, 16, 6), (10, 16, 6),
          (8, 20, 4), (12, 20, 4), (16, 8, 6), (16, 16, 4)]
Plan = collections.namedtuple("Plan", "shape k_split partial n_groups n_colg tail_from tail_split")


def build(path: str) -> ctypes.CDLL:
    csrc = os.path.join(ROOT, "paper_2603_12707_amd", "csrc")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-Wall", "-D__HIP_PLATFORM_AMD__",
                           "-I", os.path.join(ROOT, "include"), "-I", csrc, "-I", "/opt/rocm/include",
                           os.path.join(ROOT, "tests", "plan", "plan_query.cpp"), "-o", path])
    lib = ctypes.CDLL(path)
    lib.plan_gemm.argtypes = [ctypes.c_int] * 6 + [ctypes.c_int64, ctypes.POINTER(ctypes.c_int32)]
    return lib


def plan(lib, epi: str, rows, K: int, ncols: int, cap: int = 16 << 20):
    """The Plan for rows (of up to three matrices) x K weights over ncols columns with a workspace of cap floats, or
    None."""
    out = (ctypes.c_int32 * 7)()
    r = list(rows) + [0] * (3 - len(rows))
    return Plan(*out) if lib.plan_gemm(EPI[epi], *r, K, ncols, cap, out) else None


def gemms(cfg: dict) -> dict:
    """(epilogue, rows, K) of the projections of one layer and of the LM head"""
    d, F = cfg["d_model"], cfg["ffn_dim"]
    q, k = cfg["n_heads"] * cfg["head_dim"], cfg["n_kv_heads"] * cfg["head_dim"]
    return {"qkv": ("qkv", (q, k, k), d), "o": ("resid", (d,), q), "gateup": ("swiglu", (F, F), d),
            "down": ("resid", (d,), F), "head": ("store", (cfg["vocab"],), d)}


def step_floats(lib, cfg: dict, n: int) -> int:
    """Floats of K-split partials of a decode step over n columns (attention in one split)."""
    out = (ctypes.c_int64 * 4)()
    lib.plan_step(*(cfg[k] for k in ("d_model", "n_heads", "n_kv_heads", "head_dim", "ffn_dim", "vocab")),
                  configs.DTYPE_CODE[cfg["dtype"]], n, 1, out)
    return out[3]


def step_kinds(lib, cfg: dict, n: int) -> dict:
    """projection -> (shape, how it stores, whether one column group covers the batch) of a decode step over n columns"""
    kinds = {}
    for g, (epi, rows, K) in gemms(cfg).items():
        p = plan(lib, epi, rows, K, n, step_floats(lib, cfg, n))
        kinds[g] = (p.shape, epi + ("_part" if p.partial else "_tail" if p.tail_split > 1 else ""), p.n_colg == 1)
    return kinds


# Decode batches of one layer and the LM head that run, between them, every (shape, store, column groups) that the rule
# chooses for the two 7B-shaped models over batches below 4100 (a pooled cache holds up to 4096 requests).
SHAPE_CASES = {
    "llava7b_b1": [33, 65, 123, 129, 257, 513, 641, 903, 1540, 2063, 2247, 2821],
    "qwen7b_b16": [33, 65, 113, 129, 150, 304, 560, 641, 1253, 1414, 2884],
}


def shape_cfg(model: str) -> dict:
    if model == "f32":  # (fp32 storage runs other GEMMs; see test_gpu_gemm_shapes.py)
        return dict(configs.get("tiny", n_layers=1), d_model=1024, n_heads=16, n_kv_heads=16, ffn_dim=5504, vocab=8192)
    return configs.get(model, n_layers=1)
