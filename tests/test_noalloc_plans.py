"""The scratch limit of h2o_chunk_step_noalloc: a shape that some kernel path
fits into the 32 MiB array is not refused because a faster path's workspace
does not (host side only)."""
import itertools

import pytest
import torch

from paper_2608_19920_amd import h2o as H

LIMIT = 32 << 20


@pytest.fixture(scope="module")
def L():
    return H.lib()


def _align(n):
    return (n + 255) // 256 * 256


def _generic_f32(B, Hkv, G, T, M):
    """Workspace of the scalar float32 kernels: row statistics, column partials
    of 64-row blocks, the ranking copy."""
    BH, R, Nk = B * Hkv, G * T, M + T
    return _align(8 * BH * R) + _align(4 * -(-R // 64) * BH * Nk) + _align(4 * BH * M)


def _prefill(B, Hkv, G, T, M, d):
    """The least workspace of the prefill kernels: row statistics, column
    partials of 256-row blocks (128 at d = 64), the ranking copy."""
    BH, Nk, R, rows = B * Hkv, M + T, G * T, 256 if d == 128 else 128
    return (_align(8 * BH * R) + _align(4 * -(-R // rows) * BH * (-(-Nk // 32) * 32)) +
            _align(4 * BH * M))


@pytest.mark.skipif(torch.cuda.device_count() > 0, reason="a device is visible")
def test_accepted_shapes_stay_accepted(L):
    P, seen = 4096, 0
    for B, (Hq, Hkv), d, M, T, dt in itertools.product(
            (1, 4, 8), ((32, 8), (28, 4), (32, 4), (16, 16), (48, 4)), (64, 128),
            (300, 4096, 12288, 32768, 100000), (1, 64, 300), (0, 1)):
        if M < T:
            continue
        G = Hq // Hkv
        least = _generic_f32(B, Hkv, G, T, M) if dt == 0 else _prefill(B, Hkv, G, T, M, d)
        rc = L.h2o_chunk_step_noalloc(P, P, P, P, P, P, P, P, P, P, P, B, Hq, Hkv, T, M, d, 0.125,
                                      M, dt, None)
        if least <= LIMIT or L.h2o_workspace_bytes(B, Hq, Hkv, T, M, d, dt) <= LIMIT:
            assert rc == H.H2O_ENODEVICE, (B, Hq, Hkv, d, M, T, dt)
            seen += least <= LIMIT < L.h2o_workspace_bytes(B, Hq, Hkv, T, M, d, dt)
        else:
            assert rc == H.H2O_EWORKSPACE, (B, Hq, Hkv, d, M, T, dt)
    assert seen > 8   # the fallbacks were reached
