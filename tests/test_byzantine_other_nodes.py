"""The kernels for any nodes, and for groups that differ in how many workers answered, where the library's own nodes with a fixed number go
to a kernel of their own: picks that hang on rounding, the same in calls with and without a workspace and of every size."""
import numpy as np
import pytest

from oracle import approxifer_oracle as orc

pytestmark = pytest.mark.gpu

ENTRIES = ["approxifer_decode_byzantine", "approxifer_decode_byzantine_homogeneous"]


def _nodes(K, N, moved):
    alpha, beta = orc.chebyshev_nodes(K, N)
    return alpha, (beta + 1e-4 * np.cos(3.0 * np.arange(N)) if moved else beta)


def _answers(rng, alpha, beta, G, C):
    """Honest ones, one liar of A, softmax, noise: which innocent workers go is decided by the last bits of the fits."""
    Y = orc.encode(rng.uniform(0, 1, (G, alpha.size, 32)), alpha, beta) @ (rng.standard_normal((32, C)) / 6)
    one = Y.copy()
    one[:, 0] += 5 * rng.standard_normal((G, C))
    soft = np.exp(3 * Y) / np.exp(3 * Y).sum(-1, keepdims=True)
    return [d.astype(np.float32) for d in (Y, one, soft, rng.standard_normal(Y.shape))]


@pytest.mark.parametrize("entry", ENTRIES)
@pytest.mark.parametrize("moved", [True, False])             # False: the library's nodes, S read off the masks
@pytest.mark.parametrize("K,A,N,C", [(12, 2, 28, 10), (8, 2, 20, 10), (6, 2, 18, 3), (8, 2, 20, 16), (12, 2, 28, 40), (12, 3, 32, 15),
                                     (4, 1, 12, 200)])
def test_same_bits_with_and_without_workspace(entry, moved, K, A, N, C):
    import torch

    from paper_2109_09868_amd import binding
    decode = getattr(binding, entry)
    G = 60 if entry == ENTRIES[1] or C > 100 else 300
    rng = np.random.default_rng(K + C)
    alpha, beta = _nodes(K, N, moved)
    mask = np.ones((G, N), np.uint8)
    S = 0
    if not moved:
        S = binding.S_FROM_MASK
        mask[::3, N // 3] = 0 if N > 2 * (K + A) else 1
    md = torch.from_numpy(mask).cuda()
    for Y in _answers(rng, alpha, beta, G, C):
        Yd = torch.from_numpy(Y).cuda()
        for a, b in zip(decode(Yd, md, alpha, beta, S, A, 1), decode(Yd, md, alpha, beta, S, A, 1, workspace=binding.NO_WORKSPACE)):
            assert np.array_equal(a.cpu().numpy(), b.cpu().numpy())


@pytest.mark.parametrize("entry", ENTRIES)
@pytest.mark.parametrize("K,A,S,N,C", [(8, 2, 4, 24, 10), (6, 2, 4, 21, 7), (12, 2, 0, 28, 10), (8, 2, 0, 20, 15), (4, 1, 2, 12, 3)])
def test_groups_packed_into_workgroups(entry, K, A, S, N, C):
    # four, two or one group(s) to a workgroup, by the number of groups
    import torch

    from paper_2109_09868_amd import binding
    decode = getattr(binding, entry)
    rng = np.random.default_rng(77 * K + N)
    alpha, beta = _nodes(K, N, True)
    G = 2700
    Y = rng.standard_normal((G, N, C)).astype(np.float32)
    mask = np.zeros((G, N), np.uint8)
    for g in range(G):
        mask[g, rng.permutation(N)[S:]] = 1
    mask[5] = 0
    Yd, md = torch.from_numpy(Y).cuda(), torch.from_numpy(mask).cuda()
    res = {}
    for n in (2700, 1500, 40):
        out, adv = torch.full((n, K, C), -3.0, device="cuda:0"), torch.full((n, A), -7, dtype=torch.int32, device="cuda:0")
        res[n] = [t.cpu().numpy() for t in decode(Yd[:n], md[:n], alpha, beta, S, A, 1, out=out, adv=adv)]
    for n in (1500, 40):
        assert all(np.array_equal(whole[:n], part) for whole, part in zip(res[2700], res[n]))
    out, adv, st = res[2700]
    assert st[5] == 1 and st.sum() == 1 and np.all(out[5] == -3.0) and np.all(adv[5] == -7)
