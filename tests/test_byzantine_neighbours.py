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


@pytest.mark.parametrize("K,A,N,C", [(8, 2, 20, 10), (12, 2, 28, 10), (4, 1, 11, 3), (10, 3, 28, 20)])
def test_values_do_not_hang_on_how_many_groups_a_workgroup_has(K, A, N, C):
    # Answers whose decoded value at the first query cancels to some 1e-14 of them: float32 does not hide in which order they are added.  The
    # sum is balanced by one answer, what that one's rounding leaves by a second, and so on.
    import torch

    from paper_2109_09868_amd import binding
    G = 2600
    rng = np.random.default_rng(3 * K + N)
    alpha, beta = orc.chebyshev_nodes(K, N)
    liars = np.sort(rng.permutation([w for w in range(N) if abs(beta[w]) > 1e-9])[:A])
    Y = (orc.encode(rng.standard_normal((G, K, C)), alpha, beta)).astype(np.float32)
    Y[:, liars] += (30 * rng.standard_normal((G, A, C))).astype(np.float32)
    left = np.setdiff1d(np.arange(N), liars)
    w = (1.0 - 2.0 * (np.arange(left.size) % 2)) / (alpha[0] - beta[left])
    fix = left[np.argsort(-np.abs(w))]                       # the last class: balanced by three of the answers, each of the rest's rounding
    weight = dict(zip(left, w))
    rest = lambda: sum(weight[i] * Y[:, i, C - 1].astype(np.float64) for i in left)
    Y[:, fix[-3:], C - 1] = 0.0
    for i in fix[-3:]:
        Y[:, i, C - 1] = (-rest() / weight[i]).astype(np.float32)
    Yd, md = torch.from_numpy(Y).cuda(), torch.ones((G, N), dtype=torch.uint8).cuda()
    out, adv, _ = (t.cpu().numpy() for t in binding.approxifer_decode_byzantine(Yd, md, alpha, beta, 0, A, 1))
    small = np.abs(out[:, 0, C - 1]) < 1e-9
    assert small.mean() > 0.5
    for n in (1, 2, 6, 300, 700):                            # one, two and more groups to a workgroup
        part, adv_n, _ = (t.cpu().numpy() for t in binding.approxifer_decode_byzantine(Yd[:n], md[:n], alpha, beta, 0, A, 1))
        assert np.array_equal(adv_n, adv[:n]) and np.array_equal(part, out[:n]), n
