"""A group's located workers and values do not depend on which other groups a call has: Algorithm 1's classes of a wave go round until the
slowest has settled."""
import numpy as np
import pytest

from oracle import approxifer_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K,A,S,N", [(4, 2, 0, 13), (8, 2, 4, 24), (9, 2, 0, 22), (12, 2, 0, 28)])
def test_settled_classes_are_not_moved_by_slower_ones(K, A, S, N):
    # Zeros but for the liars': a class that is settled at once, and whose locator is one of many, so that every bit of it shows in who
    # is picked next to the liars of fewer than A.  Noise beside them takes 12 to 50 rounds.
    import torch

    from paper_2109_09868_amd import binding
    G = 512
    rng = np.random.default_rng(K + N)
    alpha, beta = orc.chebyshev_nodes(K, N)
    mask = np.zeros((G, N), np.uint8)
    Y = np.zeros((G, N, 1), np.float32)
    for g in range(G):
        here = rng.permutation(N)[S:]
        mask[g, here] = 1
        Y[g, here[:1 + g % A], 0] = 1.0
    def located(Y, mask):
        return binding.approxifer_decode_byzantine_homogeneous(torch.from_numpy(Y).cuda(), torch.from_numpy(mask).cuda(), alpha, beta, S, A,
                                                               1)[1].cpu().numpy()
    alone = located(Y, mask)
    beside = located(np.concatenate([np.stack([Y, rng.standard_normal(Y.shape).astype(np.float32)], 1).reshape(2 * G, N, 1)] * 4),
                     np.tile(np.repeat(mask, 2, axis=0), (4, 1)))[0:2 * G:2]
    assert np.array_equal(alone, beside)
