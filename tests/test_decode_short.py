"""Decoding of rows of less than a hundred classes by more than sixteen queries (decode_short_kernel): one and several groups to a
wave, one to three stripes of sixteen vectors, last vectors of one to four classes, k-steps that the survivors fill in part, more
than one pass over the survivors, two and four rounds of sixteen queries, and groups that were not answered as the call says."""
import numpy as np
import pytest

from oracle import approxifer_oracle as orc
from parity_cases import TOL, group_err

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch

    from paper_2109_09868_amd import binding
    return torch, binding, torch.device("cuda:0")


@pytest.mark.parametrize("K,N,S,C,G", [(17, 18, 1, 20, 5003), (18, 23, 5, 50, 1201), (31, 34, 3, 36, 700), (32, 33, 1, 64, 450),
                                       (32, 64, 30, 65, 410), (21, 30, 9, 95, 430), (33, 44, 10, 18, 1000), (48, 60, 0, 33, 900),
                                       (64, 64, 0, 92, 500), (26, 59, 24, 19, 600), (27, 31, 2, 44, 900), (63, 63, 0, 70, 600),
                                       (45, 55, 7, 127, 520)])
@pytest.mark.parametrize("from_mask", [False, True])
@pytest.mark.parametrize("mode", [0, 1])
def test_short_rows_of_many_queries(gpu, K, N, S, C, G, from_mask, mode):
    torch, binding, dev = gpu
    rng = np.random.default_rng(K + 3 * N + C)
    alpha, beta = orc.chebyshev_nodes(K, N)
    Y = rng.standard_normal((G, N, C)).astype(np.float32)
    mask = np.zeros((G, N), np.uint8)
    for g in range(G):
        mask[g, rng.permutation(N)[:N - (rng.integers(0, S + 1) if from_mask else S)]] = 1
    mask[G // 2] = 0                                         # nobody answered
    Y[mask == 0] = np.nan
    out = torch.full((G, K, C), -3.0, dtype=torch.float32, device=dev)
    got, st = binding.approxifer_decode(torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev), alpha, beta,
                                        binding.S_FROM_MASK if from_mask else S, mode, out=out)
    got, st = got.cpu().numpy(), st.cpu().numpy()
    assert st[G // 2] == 1 and st.sum() == 1 and np.all(got[G // 2] == -3.0)
    for g in list(range(0, G, 41)) + [G - 1]:
        if g != G // 2:
            ref, _ = orc.decode(np.where(mask[g:g + 1, :, None] != 0, Y[g:g + 1], 0.0).astype(np.float32), mask[g:g + 1], alpha, beta,
                                N - int(mask[g].sum()), mode)
            if np.abs(ref).max() < 1e6:                        # alternating by worker index can meet a pole
                assert group_err(got[g:g + 1], ref).max() <= TOL
