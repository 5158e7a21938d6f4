"""The token assignment on both sides of its dispatch lines, bit-exact against the oracle: one block / several (64 tokens,
1024 pairs a block, 64 blocks), one logit per lane / several (64 experts), a pair count that 4 does not divide, ties and
both zeros among the logits."""
import numpy as np
import pytest

from gpu_helpers import assert_routing_equal, gpu_route

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,k", [(64, 64, 8), (65, 64, 8), (128, 64, 8), (129, 65, 8), (341, 3, 3), (1023, 7, 1), (1025, 2, 1),
                                   (2011, 64, 8), (700, 256, 8), (33, 256, 16), (9001, 63, 8), (65537, 4, 2)])
def test_route_block_edges(oracle, T, E, k):
    rng = np.random.default_rng(T + E)
    lg = rng.standard_normal((T, E)).astype(np.float32)
    lg[::3] = np.round(lg[::3])  # ties, and zeros of both signs
    lg[1::7, :] = lg[1::7, :1]
    assert_routing_equal(gpu_route(lg, k), oracle.route(lg, k), T, k)
