"""Logits that are NaN or infinite: the selection is by the total order that the header states, the same for every number of experts and
tokens, so that k different experts are chosen and the tables are whole whatever the bits are."""
import numpy as np
import pytest

from gpu_helpers import gpu_route

pytestmark = pytest.mark.gpu


def _chosen(lg, k):
    """positive NaN first, then by value from +infinity to -infinity, negative NaN last; NaN by their bits, ties to the lower index"""
    u = np.ascontiguousarray(lg, np.float32).view(np.uint32).astype(np.int64)
    u[u == 0x80000000] = 0
    key = np.where(u >> 31, 0xffffffff - u, u | 0x80000000)
    return np.argsort(-key, axis=1, kind="stable")[:, :k].astype(np.int32)


@pytest.mark.parametrize("T,E,k", [(3, 8, 2), (5, 64, 8), (5, 65, 8), (2, 256, 32), (40, 64, 6), (40, 200, 6), (300, 60, 4), (300, 128, 8)])
def test_nan_and_infinite_logits(T, E, k):
    rng = np.random.default_rng(T + E)
    lg = rng.standard_normal((T, E)).astype(np.float32)
    bits = lg.view(np.uint32)
    for t in range(T):
        at = rng.choice(E, min(E, 7), replace=False)
        kind = t % 5
        if kind == 1:
            bits[t, at[:3]] = [0x7fc00000, 0xffc00000, 0x7f800001]
        elif kind == 2:
            bits[t, at[:2]] = [0x7f800000, 0xff800000]
        elif kind == 3:
            bits[t, :] = 0x7fc00000
        elif kind == 4:
            bits[t, at] = 0xffffffff
    print("NaN logits T=%d E=%d k=%d" % (T, E, k), flush=True)
    got, want = gpu_route(lg, k), _chosen(lg, k)
    assert np.array_equal(got["idx"], want)
    count = np.bincount(want.ravel(), minlength=E)
    assert np.array_equal(got["count"], count) and np.array_equal(got["off"], np.concatenate([[0], np.cumsum(count)]))
    perm = np.argsort(want.ravel(), kind="stable")
    assert np.array_equal(got["perm"], perm) and np.array_equal(got["inv"][perm], np.arange(T * k))
    finite = np.all(np.isfinite(lg), axis=1)
    assert np.max(np.abs(got["w"][finite].sum(axis=1) - 1.0)) <= 1e-6
