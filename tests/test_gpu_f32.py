"""The float32 matrix-core kernels (attention, dq, dk/dv) at the edges of their
tiles, against the float64 oracle (1e-5) and the scalar float32 kernels."""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_19920_amd import h2o as H
from paper_2608_19920_amd import workloads as W
import _gpu as U

pytestmark = pytest.mark.gpu

CASES = [  # B, Hq, Hkv, d, M, T, cache
    (1, 1, 1, 64, 0, 1, False),        # one row, one key
    (1, 2, 2, 128, 15, 1, False),      # 16 keys: one step, seven waves without one
    (2, 7, 1, 64, 131, 5, False),      # G = 7, 35 rows: a 3-row remainder
    (1, 8, 2, 128, 128, 33, False),    # 132 rows, keys past one step per wave
    (3, 4, 1, 128, 257, 16, True),     # cache mode, one key in the last step
    (1, 4, 4, 64, 40, 40, True),       # every cached slot a chunk token
    (4, 64, 16, 64, 70, 32, False),    # 256 blocks of 32 rows
    (4, 64, 16, 128, 70, 32, True),
]


def _inputs(B, Hq, Hkv, d, M, T, cache):
    wl = W.custom("f32", B=B, Hq=Hq, Hkv=Hkv, d=d, M=max(M, 1), T=T, dtype="f32", heavy_frac=0.02)
    x = W.make_inputs(wl, seed=7)
    for n in ("k_cache", "v_cache"):
        x[n] = x[n][:, :, :M]
    rng = np.random.default_rng(3)
    x["dout"] = rng.standard_normal(x["q"].shape).astype(np.float32)
    x["tp"] = rng.integers(-3, M + T, size=(B, Hkv, M)).astype(np.int32)
    return x, float(x["scale"])


def _run(x, scale, B, Hq, Hkv, d, M, T, cache, pos0):
    dev = {n: U.to_dev(x[n], torch.float32) for n in ("q", "k_cache", "v_cache", "k_new", "v_new",
                                                     "dout")}
    tp = U.to_dev(x["tp"], torch.int32)
    b = H.alloc_step(B, Hq, Hkv, T, M, d, torch.float32, insert_first=cache)
    if cache:
        H.h2o_sdpa_cache(dev["q"], dev["k_cache"], dev["v_cache"], tp, b["out"], b["lse"],
                         b["wsum"], b["workspace"], pos0, scale)
    else:
        H.h2o_sdpa_chunk(dev["q"], dev["k_cache"], dev["v_cache"], dev["k_new"], dev["v_new"],
                         b["out"], b["lse"], b["wsum"], b["workspace"], scale)
    names = ("q", "k_cache", "v_cache") + (() if cache else ("k_new", "v_new"))
    g = {n: torch.empty_like(dev[n]) for n in names}
    ws = torch.empty(max(H.h2o_backward_workspace_bytes(B, Hq, Hkv, T, M, d, torch.float32), 16),
                     dtype=torch.uint8, device="cuda")
    H.h2o_sdpa_chunk_backward(dev["q"], dev["k_cache"], dev["v_cache"], dev["k_new"],
                              dev["v_new"], b["lse"], dev["dout"], g["q"], g["k_cache"],
                              g["v_cache"], g.get("k_new"), g.get("v_new"), ws, scale,
                              token_pos=tp if cache else None, pos0=pos0)
    torch.cuda.synchronize()
    return {**{n: U.to_np(b[n]) for n in ("out", "lse", "wsum")},
            **{"d_" + n: U.to_np(t) for n, t in g.items()}}


@pytest.mark.parametrize("case", CASES, ids=["-".join(map(str, c)) for c in CASES])
def test_f32_matrix_core_kernels(case):
    B, Hq, Hkv, d, M, T, cache = case
    x, scale = _inputs(*case)
    pos0 = M // 2
    got = _run(x, scale, *case, pos0)
    if cache:
        out, lse, wsum = oracle.sdpa_cache(x["q"], x["k_cache"], x["v_cache"], x["tp"], pos0, scale)
    else:
        out, lse, wsum = oracle.sdpa_chunk(x["q"], x["k_cache"], x["v_cache"], x["k_new"],
                                           x["v_new"], scale)
    U.check("f32", out=(got["out"], out), lse=(got["lse"], lse), wsum=(got["wsum"], wsum))
    try:
        H.h2o_debug_force_path(0)
        ref = _run(x, scale, *case, pos0)
    finally:
        H.h2o_debug_force_path(-1)
    for n, r in ref.items():
        # gradients: sums of products whose terms carry exp()'s relative error
        # (a logit of up to ~50 rounded to 2^-24 of it: 3e-6), against the
        # gradient's own norm; both sides carry it. Where a gradient cancels
        # (one key: dP = D, an exact 0) what is left is the rounding of dP, a
        # sum of d products of normal draws: 2^-24 scale sum |dO V| |K|, about
        # 2^-24 d/sqrt(d) < 2^-20 an element
        seen = np.isfinite(r)
        err = np.linalg.norm(np.where(seen, got[n] - r, 0.0))
        assert np.array_equal(np.isfinite(got[n]), seen), n
        assert err <= 2e-5 * np.linalg.norm(r[seen]) + 2.0 ** -20 * np.sqrt(r.size), (n, err)
