"""Algorithms 2 and 1 on the library's own worker nodes with at most four workers missing (csrc/byzantine_pairs.h), at the edges of its
tiles: K + A odd and even, the fewest workers of eq. (3) and up to two more, none to four missing, a node in the middle and a
query node on a worker's, one class to several workgroups of them, and group counts that fill workgroups in part."""
import numpy as np
import pytest

from oracle import approxifer_oracle as orc
from parity_cases import TOL, assert_rounding_ties, group_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch

    from paper_2109_09868_amd import binding
    return torch, binding, torch.device("cuda:0")


def _inputs(K, A, S, N, C, G, seed):
    rng = np.random.default_rng(seed)
    alpha, beta = orc.chebyshev_nodes(K, N)
    Y = (orc.encode(rng.uniform(0, 1, (G, K, 32)), alpha, beta) @ (rng.standard_normal((32, C)) / 6)).astype(np.float32)
    sd = max(float(Y.std()), 1e-3)
    mask = np.zeros((G, N), np.uint8)
    adv = np.zeros((G, A), np.int32)
    for g in range(G):
        here = rng.permutation(N)[S:]
        mask[g, here] = 1
        adv[g] = np.sort([w for w in here if abs(beta[w]) > 1e-9][:A])
        Y[g, adv[g]] += (sd * rng.choice([-1, 1], (A, C)) * rng.uniform(3, 30, (A, C))).astype(np.float32)
        Y[g, mask[g] == 0] = np.nan                          # an answer that did not come is not looked at
    return alpha, beta, Y, mask, adv


# (K + A, missing, workers beyond eq. (3)): every column tile, both row tiles, odd and even numbers of rows before and after
# the missing workers are taken out; classes and groups vary along with them
SHAPES = [(K, A, S, ex) for K, A in ((1, 2), (2, 1), (3, 1), (2, 3), (4, 2), (6, 1), (6, 2), (7, 2), (8, 2), (9, 2), (10, 2), (12, 1),
                                     (12, 2), (12, 3)) for S in range(5) for ex in ((0, 1, 2) if K in (2, 8, 12) else (S % 3,))]


@pytest.mark.parametrize("K,A,S,ex", SHAPES)
def test_located_and_decoded_as_by_the_oracle(gpu, K, A, S, ex):
    torch, binding, dev = gpu
    N = 2 * (K + A) + S + ex
    mode = 1 if K < 6 else S % 2                             # the printed signs can have a pole at a query node there
    C = (10, 1, 16, 33, 7)[(K + A + S + ex) % 5]
    G = 9 if C == 33 else 261
    alpha, beta, Y, mask, planted = _inputs(K, A, S, N, C, G, 1000 * K + 10 * N + S)
    mask[3] = 0
    Yd, md = torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev)
    out = torch.full((G, K, C), -3.0, dtype=torch.float32, device=dev)
    adv = torch.full((G, A), -7, dtype=torch.int32, device=dev)
    got = binding.approxifer_decode_byzantine(Yd, md, alpha, beta, S, A, mode, out=out, adv=adv)
    out, adv, st = (t.cpu().numpy() for t in got)
    assert st[3] == 1 and st.sum() == 1 and np.all(out[3] == -3.0) and np.all(adv[3] == -7)
    few = slice(0, 8)
    Yz = np.where(mask[few, :, None] != 0, Y[few], 0.0).astype(np.float32)
    ref, adv_ref, _ = orc.decode_byzantine(Yz, mask[few], alpha, beta, S, A, mode)
    # one class may hold a lie that a rational function explains: then the oracle's own votes may miss the planted set
    sure = (st[few] == 0) & np.all(adv_ref == planted[few], axis=1)
    assert sure.sum() >= (7 if C >= 7 else 1)
    assert np.array_equal(adv[few][sure], adv_ref[sure])
    assert group_err(out[few][sure], ref[sure]).max() <= TOL
    # the other groups: the planted liars, and the decoder over the rest
    good = (st == 0) & np.all(adv == planted, axis=1)
    assert good.sum() >= (0.95 if C >= 7 else 0.5) * (G - 1)
    left = mask[good].copy()
    np.put_along_axis(left, adv[good].astype(np.int64), 0, axis=1)
    ref, _ = orc.decode(np.where(left[:, :, None] != 0, Y[good], 0.0).astype(np.float32), left, alpha, beta, S + A, mode)
    ok = np.abs(ref).max(axis=(1, 2)) < 1e6                    # printed signs can meet a pole
    assert group_err(out[good][ok], ref[ok]).max() <= TOL


@pytest.mark.parametrize("K,A,S,ex", SHAPES)
def test_fits_of_predictions_that_are_not_rational(gpu, K, A, S, ex):
    # Noise, one class to a group: every equation of the fits counts, where rational predictions satisfy them all.  The located
    # workers are the oracle's but where its two closest candidates agree to rounding.
    torch, binding, dev = gpu
    N, G = 2 * (K + A) + S + ex, 40
    rng = np.random.default_rng(10 * N + K)
    alpha, beta = orc.chebyshev_nodes(K, N)
    Y = rng.standard_normal((G, N, 1)).astype(np.float32)
    mask = np.zeros((G, N), np.uint8)
    for g in range(G):
        mask[g, rng.permutation(N)[S:]] = 1
    Yd, md = torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev)
    for locator, entry in ((orc.LOCATOR_ALGORITHM_2, binding.approxifer_decode_byzantine),
                           (orc.LOCATOR_ALGORITHM_1, binding.approxifer_decode_byzantine_homogeneous)):
        adv = entry(Yd, md, alpha, beta, S, A, 1)[1].cpu().numpy()
        _, adv_ref, _ = orc.decode_byzantine(Y, mask, alpha, beta, S, A, 1, locator)
        assert np.all(adv == adv_ref, axis=1).sum() >= (0.95 if K + A <= 12 else 0.8) * G
        assert_rounding_ties(Y, mask, beta, K, A, adv, adv_ref, locator)


@pytest.mark.parametrize("entry", ["approxifer_decode_byzantine", "approxifer_decode_byzantine_homogeneous"])
@pytest.mark.parametrize("K,A,S,N,C", [(8, 2, 4, 24, 10), (4, 1, 1, 12, 2), (2, 1, 0, 7, 1), (6, 2, 0, 16, 40), (8, 2, 2, 22, 128),
                                       (3, 1, 0, 9, 129), (8, 2, 1, 23, 260)])
def test_a_group_has_the_same_bits_in_calls_of_every_size(gpu, K, A, S, N, C, entry):
    # groups to a workgroup, and rows of lanes to a group, by the number of groups; with and without a workspace
    torch, binding, dev = gpu
    G = 1100 if C <= 40 else 270
    alpha, beta, Y, mask, _ = _inputs(K, A, S, N, C, G, 7 * K + N + C)
    decode = getattr(binding, entry)
    Yd, md = torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev)
    whole = [t.cpu().numpy() for t in decode(Yd, md, alpha, beta, S, A, 1)]
    for n in (1, 3, 255, 257, 700):
        if n > G:
            continue
        for ws in (None, binding.NO_WORKSPACE):
            part = decode(Yd[:n], md[:n], alpha, beta, S, A, 1, workspace=ws)
            for a, b in zip(whole, part):
                assert np.array_equal(a[:n], b.cpu().numpy())


def test_nodes_that_are_not_the_librarys_take_the_general_kernels(gpu):
    # the closed forms hold on cos(i pi / (N - 1)) only: nodes moved by 1e-4, and the same nodes in another order
    torch, binding, dev = gpu
    K, A, S, N, C, G = 6, 2, 2, 18, 10, 24
    alpha, beta, Y, mask, planted = _inputs(K, A, S, N, C, G, 5)
    for nodes in (beta + 1e-4 * np.cos(3.0 * np.arange(N)), beta[::-1].copy()):
        Yn = (Y if nodes[0] > 0 else Y[:, ::-1]).copy()
        mn = (mask if nodes[0] > 0 else mask[:, ::-1]).copy()
        out, adv, st = binding.approxifer_decode_byzantine(torch.from_numpy(Yn).to(dev), torch.from_numpy(mn).to(dev), alpha, nodes,
                                                           S, A, 1)
        out, adv, st = out.cpu().numpy(), adv.cpu().numpy(), st.cpu().numpy()
        Yz = np.where(mn[:, :, None] != 0, Yn, 0.0).astype(np.float32)
        ref, adv_ref, _ = orc.decode_byzantine(Yz, mn, alpha, nodes, S, A, 1)
        assert np.all(st == 0) and np.array_equal(adv, adv_ref)
        assert group_err(out, ref).max() <= TOL
