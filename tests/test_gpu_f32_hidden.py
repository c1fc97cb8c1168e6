"""Float32 kernels with Inf and NaN in what a query does not see: the values of a
later chunk token, the keys and values of a slot of a later position, the output
gradient of an earlier query. Wherever the scalar kernels, which skip such pairs,
give a finite result, the matrix-core kernels give the same one."""
import numpy as np
import pytest
import torch

from paper_2608_19920_amd import h2o as H
import _gpu as U
from test_gpu_f32 import _inputs, _run

pytestmark = pytest.mark.gpu

CASES = [  # B, Hq, Hkv, d, M, T, cache
    (1, 7, 1, 64, 131, 5, False),      # G = 7, a 3-row remainder
    (1, 8, 2, 128, 40, 33, False),     # three steps of chunk keys
    (1, 2, 2, 64, 0, 17, False),       # chunk keys only
    (4, 64, 16, 64, 70, 32, False),    # blocks of 32 rows
    (2, 8, 2, 64, 90, 20, True),
    (4, 64, 16, 128, 70, 32, True),    # blocks of 32 rows
]


@pytest.mark.parametrize("poison", ["keys", "rows"])
@pytest.mark.parametrize("case", CASES, ids=["-".join(map(str, c)) for c in CASES])
def test_hidden_pairs_contribute_nothing(case, poison):
    B, Hq, Hkv, d, M, T, cache = case
    x, scale = _inputs(*case)
    pos0 = M // 2
    if poison == "rows":                        # position 0 of one head
        x["dout"][0, 0, 0, 3], x["dout"][0, 0, 0, d - 1] = np.inf, np.nan
    elif cache:                                 # slots nobody sees, one the last query sees
        x["tp"][:, :, 5], x["tp"][:, :, M - 1] = pos0 + T, pos0 + T + 7
        x["tp"][0, 0, 33] = pos0 + T - 1
        x["k_cache"][:, :, 5], x["v_cache"][:, :, M - 1] = np.nan, np.inf
        x["v_cache"][:, :, 5, 1] = -np.inf
        x["v_cache"][0, 0, 33, 2] = np.inf
    else:                                       # the last chunk tokens of one head
        x["v_new"][0, 0, T - 1, 0], x["v_new"][0, 0, T - 3, d - 2] = np.inf, np.nan
    got = _run(x, scale, *case, pos0)
    try:
        H.h2o_debug_force_path(0)
        ref = _run(x, scale, *case, pos0)
    finally:
        H.h2o_debug_force_path(-1)
    bad = 0
    for n, r in ref.items():
        # tolerance as for finite inputs: exp()'s relative error, and the rounding
        # of a gradient that cancels (2^-20 an element)
        seen = np.isfinite(r)
        bad += r.size - seen.sum()
        if not seen.any():
            continue
        # (a query that sees no slot has lse -inf on both sides)
        assert np.isfinite(got[n][seen]).all(), (n, int((~np.isfinite(got[n][seen])).sum()))
        err = np.linalg.norm(got[n][seen] - r[seen])
        assert err <= 2e-5 * np.linalg.norm(r[seen]) + 2.0 ** -20 * np.sqrt(r.size), (n, err)
    assert bad > 0
    assert np.isfinite(ref["out"]).mean() > 0.1 and np.isfinite(ref["d_v_cache"]).any() or M == 0
