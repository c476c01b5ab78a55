"""Encoding rows that end in a partial vector on the matrix cores: one to three floats behind the last whole vector, rows of one vector
and a bit, whole rows at an address that is only 4-byte aligned, one group to several hundred, and memory behind the result."""
import numpy as np
import pytest

from oracle import approxifer_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch

    from paper_2109_09868_amd import binding
    return torch, binding, torch.device("cuda:0")


@pytest.mark.parametrize("K,N", [(9, 22), (16, 40), (17, 18), (17, 30), (20, 24), (31, 35), (40, 88), (64, 70)])
@pytest.mark.parametrize("D,G", [(5, 1), (6, 300), (7, 41), (17, 130), (63, 9), (127, 33), (129, 20), (151, 65), (152, 7)])
def test_rows_with_a_partial_last_vector(gpu, K, N, D, G):
    torch, binding, dev = gpu
    rng = np.random.default_rng(K + N + D)
    alpha, beta = orc.chebyshev_nodes(K, N)
    X = rng.standard_normal((G, K, D)).astype(np.float32)
    flat = torch.empty(G * K * D + 1, dtype=torch.float32, device=dev)
    q = flat[1:].view(G, K, D)                               # one float off: no row is aligned
    q.copy_(torch.from_numpy(X))
    room = torch.full((G * N * D + 64,), -5.0, dtype=torch.float32, device=dev)
    coded = room[:G * N * D].view(G, N, D)
    binding.approxifer_encode(q, alpha, beta, coded=coded)
    assert torch.all(room[G * N * D:] == -5.0)
    ref = orc.encode(X, alpha, beta)
    got = coded.cpu().numpy()
    # a sum of K products of float32 weights, |w| summed: (K + 2) half units each
    bound = (K + 2) * 6e-8 * np.abs(X).max() * np.abs(orc.encode(np.eye(K)[None], alpha, beta)).sum(axis=2).max()
    assert np.abs(got - ref).max() <= bound
    # an infinity in the last query reaches every worker's float of that column and no other column
    X[0, K - 1, D - 1] = np.inf
    q.copy_(torch.from_numpy(X))
    binding.approxifer_encode(q, alpha, beta, coded=coded)
    again = coded.cpu().numpy()
    assert np.array_equal(again[0, :, :D - 1], got[0, :, :D - 1]) and np.array_equal(again[1:], got[1:])
