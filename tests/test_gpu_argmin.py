"""Evictions of one token (argmin and insert in one launch) and rankings of
several tokens that share a launch with their insert, bit-exact against the oracle where the kernels
change their block shape, start another round of loads or stop applying."""
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


@pytest.mark.parametrize("M,T,d,dt", [
    (2, 2, 64, "bf16"), (600, 128, 64, "bf16"), (600, 129, 64, "bf16"),
    (300, 64, 128, "bf16"), (300, 65, 128, "bf16"), (32, 32, 128, "f32"), (200, 33, 128, "f32"),
    (32768, 40, 64, "bf16"), (32769, 40, 64, "bf16"), (1027, 3, 128, "f32"),
])
def test_scores_ranked_in_place(M, T, d, dt):
    """h2o: one launch while the chunk is one 16-byte vector per thread (1,024) and
    the row fits LDS (32,768 slots), two beyond."""
    say(f"in place M{M} T{T} d{d} {dt}")
    for quant in (None, 1):
        x = _evict_inputs(2, 3, M, T, d, dt, quant, seed=M + T)
        _assert_same(_run_evict(x, T, dt, "h2o"), _expect(x, T, "h2o"), "h2o")
