"""Evictions of one token (argmin and insert in one launch) and h2o_norm's
ranking with its insert, bit-exact against the oracle where the argmin changes
its block shape or starts another round of loads."""
import pytest

from test_gpu_variants import POLICIES, _assert_same, _evict_inputs, _expect, _run_evict
from _gpu import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("policy", POLICIES)
@pytest.mark.parametrize("M", [255, 257, 4096, 4097, 16384, 16385, 33001])
@pytest.mark.parametrize("quant", [None, 2])
def test_one_token_edges(M, quant, policy):
    """256 x 16 slots are one round of the small block, 1,024 x 16 of the
    large one; with quant the row has many equal keys and the lowest slot
    wins."""
    B, Hkv, T, d = 2, 3, 1, 64
    say(f"argmin {policy} M{M} quant {quant}")
    x = _evict_inputs(B, Hkv, M, T, d, "bf16", quant, seed=M)
    _assert_same(_run_evict(x, T, "bf16", policy), _expect(x, T, policy), policy)


@pytest.mark.parametrize("M,T", [(5, 2), (33, 33), (4096, 4096), (4200, 4097), (20000, 7)])
def test_norm_rows_edges(M, T):
    """h2o_norm, several tokens: ranking and insert in one launch up to the
    select kernel's 4,096 bins, in two above."""
    B, Hkv, d, dt = 3, 2, 128, "f32"
    say(f"norm M{M} T{T}")
    x = _evict_inputs(B, Hkv, M, T, d, dt, 1, seed=M + T)
    _assert_same(_run_evict(x, T, dt, "h2o_norm"), _expect(x, T, "h2o_norm"), "h2o_norm")
