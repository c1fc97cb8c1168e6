"""Token steps for every group size of the decode kernels, at cache lengths
around the edges of the finish's single pass (4,096 slots), the combine's
blocks (2,048) and the insert-first scan's rounds (4,096 slots; rows of M % 4 != 0
are read by single loads): fused against the separate calls bit for bit, and
against the float64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_19920_amd import h2o as H
from paper_2608_19920_amd import workloads as W
import _gpu as U

pytestmark = pytest.mark.gpu

STEP = [  # B, Hq, Hkv, d, M
    (1, 7, 1, 128, 4097), (2, 16, 2, 128, 6145), (1, 3, 1, 64, 4096), (1, 10, 2, 64, 4099),
    (1, 6, 1, 128, 33), (1, 7, 1, 64, 8192), (1, 8, 1, 128, 1), (1, 5, 1, 128, 2049),
    (1, 2, 2, 128, 140000),           # over 64 candidate blocks a head; 143 MB: non-temporal loads
    (1, 14, 2, 128, 98304),           # 96 MiB of K and V, the least with non-temporal loads
]
INSERT = [(1, 7, 1, 128, 4097), (2, 14, 2, 64, 8200), (1, 16, 2, 128, 12289), (1, 4, 1, 128, 4096),
          (1, 8, 2, 128, 98305)]   # non-temporal loads


def _inputs(B, Hq, Hkv, d, M):
    wl = W.custom("g", B=B, Hq=Hq, Hkv=Hkv, d=d, M=M, T=1, heavy_frac=0.02)
    x = W.make_inputs(wl, seed=M)
    x["scores"][..., -1] = x["scores"].min(-1)   # a tie for the smallest: the lower slot wins
    return x


def _step(x, how):
    B, Hq, T, d = x["q"].shape
    Hkv, M = x["k_cache"].shape[1:3]
    st = U.device_state(x, "bf16")
    q, kn, vn = (U.to_dev(x[n], torch.bfloat16) for n in ("q", "k_new", "v_new"))
    first = how.startswith("insert")
    b = H.alloc_step(B, Hq, Hkv, T, M, d, torch.bfloat16, insert_first=first)
    pos0, scale = int(x["pos0"]), float(x["scale"])
    args = (q, st["k_cache"], st["v_cache"], st["scores"], st["token_pos"], kn, vn, b["out"],
            b["lse"], b["wsum"], b["evict_idx"], b["workspace"], pos0, scale)
    if how == "insert":
        H.h2o_chunk_step_insert_first(*args)
    elif how == "insert_parts":
        zero = torch.zeros(B, Hkv, M + 1, device="cuda")
        H.h2o_evict_insert(st["k_cache"], st["v_cache"], st["scores"], st["token_pos"], kn, vn,
                           zero, b["evict_idx"], pos0)
        H.h2o_sdpa_cache(q, st["k_cache"], st["v_cache"], st["token_pos"], b["out"], b["lse"],
                         b["wsum"], b["workspace"], pos0, scale)
        st["scores"] += b["wsum"]
    elif how == "halves":
        H.h2o_chunk_step(*args, part="attend")
        H.h2o_chunk_step(*args, part="evict")
    else:
        H.step(st, q, kn, vn, b, pos0, scale, fused=how == "fused")
    torch.cuda.synchronize()
    return {**{n: U.to_np(b[n]) for n in ("out", "lse", "wsum", "evict_idx")},
            **{n: U.to_np(st[n]) for n in ("k_cache", "v_cache", "scores", "token_pos")}}


@pytest.mark.parametrize("shape", STEP, ids=str)
def test_token_step(shape):
    x = _inputs(*shape)
    got = _step(x, "fused")
    for how in ("calls", "halves"):
        ref = _step(x, how)
        for n in ref:
            np.testing.assert_array_equal(got[n], ref[n], err_msg=f"{how}: {n}")
    out, lse, wsum = oracle.sdpa_chunk(x["q"], x["k_cache"], x["v_cache"], x["k_new"],
                                       x["v_new"], x["scale"])
    U.check("bf16", out=(got["out"], out), lse=(got["lse"], lse), wsum=(got["wsum"], wsum))
    acc = oracle.accumulate_scores(x["scores"], got["wsum"])
    np.testing.assert_array_equal(got["evict_idx"], oracle.bottomk(acc, 1))


@pytest.mark.parametrize("shape", INSERT, ids=str)
def test_token_step_insert_first(shape):
    x = _inputs(*shape)
    got, ref = _step(x, "insert"), _step(x, "insert_parts")
    for n in ref:
        np.testing.assert_array_equal(got[n], ref[n], err_msg=n)
    np.testing.assert_array_equal(got["evict_idx"], oracle.bottomk(x["scores"], 1))
