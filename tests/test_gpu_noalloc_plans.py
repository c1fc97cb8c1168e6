"""h2o_chunk_step_noalloc on shapes whose preferred workspace exceeds the fixed
scratch: the plan that runs in its place is still a split one (or, in float32,
one of the matrix-core kernels) where such a plan fits, and its results hold
against the oracle on sampled heads."""
import numpy as np
import pytest
import torch

import oracle
from paper_2608_19920_amd import h2o as H
from paper_2608_19920_amd import workloads as W
import _gpu as U

pytestmark = pytest.mark.gpu

CASES = [  # B, Hq, Hkv, d, M, T, dtype, a kernel that runs, one that does not
    (1, 32, 4, 64, 13130, 598, "bf16", "split_reduce", "colsum_reduce"),   # 5 splits wanted, 3 fit
    (4, 16, 8, 128, 3919, 190, "bf16", "split_reduce", "colsum_reduce"),   # 5 of 128 rows; 4 of 256
    (1, 64, 8, 64, 131100, 1, "bf16", "mfma_main", "decode_split"),     # the stored logits do not fit
    (1, 32, 4, 64, 18946, 229, "f32", "f32_attend", "generic_main"),    # 16-row partials do not, 32 do
    (8, 32, 4, 64, 1407, 599, "f32", "generic_main", "f32_attend"),     # only 64-row partials do
]


@pytest.mark.parametrize("case", CASES, ids=["-".join(map(str, c[:7])) for c in CASES])
def test_plan_within_the_scratch(case):
    B, Hq, Hkv, d, M, T, dt, runs, idle = case
    G, tdt = Hq // Hkv, U.TDT[dt]
    assert H.h2o_workspace_bytes(B, Hq, Hkv, T, M, d, tdt) > H.h2o_noalloc_scratch_bytes()
    U.say(f"noalloc {case}")
    x = W.make_inputs(W.custom("na", B=B, Hq=Hq, Hkv=Hkv, d=d, M=M, T=T, dtype=dt,
                               heavy_frac=0.02), seed=11)
    q, kn, vn = (U.to_dev(x[n], tdt) for n in ("q", "k_new", "v_new"))
    st = U.device_state(x, dt)
    new = lambda *s, t=torch.float32: torch.empty(*s, dtype=t, device="cuda")
    out, lse, wsum = new(B, Hq, T, d, t=tdt), new(B, Hq, T), new(B, Hkv, M + T)
    idx = new(B, Hkv, T, t=torch.int32)
    pos0, scale = int(x["pos0"]), float(x["scale"])
    try:
        H.h2o_debug_timing(True)
        H.h2o_chunk_step_noalloc(q, st["k_cache"], st["v_cache"], st["scores"], st["token_pos"],
                                 kn, vn, out, lse, wsum, idx, pos0, scale)
        torch.cuda.synchronize()
        counts = {k: H.h2o_debug_kernel_time(k)[1] for k in (runs, idle)}
    finally:
        H.h2o_debug_timing(False)
    assert counts == {runs: 1, idle: 0}
    for b, h in ((0, 0), (B - 1, Hkv - 1)):
        sl = np.s_[b:b + 1, h:h + 1]
        qs = np.s_[b:b + 1, h * G:(h + 1) * G]
        ref = oracle.sdpa_chunk(x["q"][qs], x["k_cache"][sl], x["v_cache"][sl], x["k_new"][sl],
                                x["v_new"][sl], x["scale"])
        U.check(dt, *((U.to_np(g)[s], r) for g, s, r in zip((out, lse, wsum), (qs, qs, sl), ref)),
                extra=f"head {(b, h)}")
    # the eviction and the insert, on the call's own summed weights
    w = wsum.cpu().numpy()
    acc = x["scores"].astype(np.float32) + w[..., :M]
    e = idx.cpu().numpy()
    np.testing.assert_array_equal(e, oracle.bottomk(acc, T))
    np.put_along_axis(acc, e, w[..., M:], -1)
    np.testing.assert_array_equal(st["scores"].cpu().numpy(), acc)
    pos = x["token_pos"].astype(np.int32)
    np.put_along_axis(pos, e, np.broadcast_to(pos0 + np.arange(T, dtype=np.int32), e.shape), -1)
    np.testing.assert_array_equal(st["token_pos"].cpu().numpy(), pos)
    for cache, rows in (("k_cache", kn), ("v_cache", vn)):
        want = U.to_dev(x[cache], tdt).scatter_(
            2, idx.long().unsqueeze(-1).expand(-1, -1, -1, d), rows)
        assert torch.equal(st[cache], want), cache
