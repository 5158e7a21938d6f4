"""The token assignment of at most 64 pairs (one wave) and around that line, against the oracle (what is an index bit for bit): 63 to 65 pairs, one
to 256 experts, one to all of them chosen, more slots than a wave has lanes, ties, both zeros and the lowest logits."""
import numpy as np
import pytest

from gpu_helpers import gpu_route

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,k", [(1, 2, 1), (1, 64, 64), (1, 65, 64), (1, 256, 63), (1, 200, 100), (2, 256, 256), (3, 129, 16), (4, 64, 16),
                                   (5, 64, 13), (7, 63, 9), (16, 64, 4), (17, 8, 4), (21, 3, 3), (64, 7, 1), (64, 256, 1), (63, 1, 1)])
def test_route_few_pairs(oracle, T, E, k):
    rng = np.random.default_rng(10 * T + E)
    lg = rng.standard_normal((T, E)).astype(np.float32)
    lg[::2] = np.round(lg[::2])  # ties, and zeros of both signs
    lg[1::3, :] = lg[1::3, :1]
    if E > k:
        lg[:, E // 2] = -3e38
    got, want = gpu_route(lg, k), oracle.route(lg, k)
    for key in ("idx", "count", "off", "perm", "inv"):
        assert np.array_equal(got[key], want[key]), key
    # fp32: the argument of the exponential is rounded once (up to 8 in size: 4 units of the last place of the result), a sum of k
    # terms, the exponential and the division 2 each
    assert np.all(np.abs(got["w"] - want["w"]) <= (k + 10) * 2.0 ** -24 * want["w"] + 1e-37)
