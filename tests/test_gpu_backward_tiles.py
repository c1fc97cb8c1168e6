"""bf16 backward at the edges of the keys pass's two row tiles: 32 packed rows
(G * T) and one more at d = 128, 1,536 and one more at d = 64, both modes, with
the checks and tolerances of the general backward tests."""
import pytest

import test_gpu_backward as B
from paper_2608_19920_amd import h2o as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    (1, 4, 2, 64, 130, 768, "bf16"),      # 1,536 rows
    (1, 1, 1, 64, 70, 1537, "bf16"),
    (2, 4, 2, 128, 333, 16, "bf16"),      # 32 rows
    (1, 3, 1, 128, 200, 11, "bf16"),      # 33
    (3, 16, 16, 64, 150, 14, "bf16"),     # one part-filled tile
])
@pytest.mark.parametrize("mode", ["chunk", "cache"])
def test_keys_pass_tile_edges(shape, mode):
    if mode == "cache":                   # the chunk sits in the cache
        shape = shape[:4] + (shape[4] + shape[5],) + shape[5:]
    run = B.test_backward_chunk_mode if mode == "chunk" else B.test_backward_cache_mode
    try:
        run(shape, -1, None)
    finally:
        H.h2o_debug_force_path(-1)
