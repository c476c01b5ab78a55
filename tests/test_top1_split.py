"""The class decision of few groups of thousands of classes (decode_top1_split_kernel): one chunk of rows and a last one in part,
one vector to more than a workgroup has lanes, last vectors of one to four classes, two and four queries to a workgroup, the last
of them alone, S read off the mask, and groups that were not answered as the call says."""
import numpy as np
import pytest

from oracle import approxifer_oracle as orc
from test_gpu_parity import _assert_top1

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch

    from paper_2109_09868_amd import binding
    return torch, binding, torch.device("cuda:0")


@pytest.mark.parametrize("K,N,S,C,G", [(1, 2, 1, 256, 1), (2, 9, 0, 260, 5), (3, 11, 3, 1025, 2), (5, 13, 4, 4098, 3), (7, 24, 1, 4099, 2),
                                       (9, 19, 3, 384, 30), (12, 28, 5, 4100, 2), (16, 33, 1, 8193, 1), (17, 20, 3, 1027, 3),
                                       (20, 100, 12, 1800, 2), (33, 40, 0, 300, 61), (64, 72, 8, 4097, 2), (64, 128, 0, 256, 32),
                                       (4, 6, 1, 5003, 500), (6, 12, 2, 400, 250), (18, 24, 3, 20, 7),
                                       (24, 31, 2, 66, 9), (40, 50, 5, 17, 12)])
@pytest.mark.parametrize("from_mask", [False, True])
def test_few_groups_of_many_classes(gpu, K, N, S, C, G, from_mask):
    torch, binding, dev = gpu
    rng = np.random.default_rng(K + 3 * N + C)
    alpha, beta = orc.chebyshev_nodes(K, N)
    Y = rng.standard_normal((G, N, C)).astype(np.float32)
    mask = np.zeros((G, N), np.uint8)
    for g in range(G):
        mask[g, rng.permutation(N)[:N - (rng.integers(0, S + 1) if from_mask else S)]] = 1
    mask[G // 2] = 0                                         # nobody answered
    Y[mask == 0] = np.nan
    Y[0, :, C - 1] = Y[0, :, 3]                              # the last class of a partial vector ties with an early one
    Yd, md = torch.from_numpy(Y).to(dev), torch.from_numpy(mask).to(dev)
    top1 = torch.full((G, K), -9, dtype=torch.int32, device=dev)
    score = torch.full((G, K), -9.0, dtype=torch.float32, device=dev)
    t, sc, st = binding.approxifer_decode_top1(Yd, md, alpha, beta, binding.S_FROM_MASK if from_mask else S, 1, top1=top1, score=score)
    t, sc, st = t.cpu().numpy(), sc.cpu().numpy(), st.cpu().numpy()
    assert st[G // 2] == 1 and st.sum() == 1 and np.all(t[G // 2] == -9) and np.all(sc[G // 2] == -9.0)
    for g in range(G):
        if g != G // 2 and (G < 40 or g % 37 == 0):
            n = int(mask[g].sum())
            Yg = Y[g:g + 1, :, :C - 1] if g == 0 else Y[g:g + 1]    # without the tie, which the smaller class has to win
            ref = orc.decode_top1(Yg, mask[g:g + 1], alpha, beta, N - n, 1)
            _assert_top1(Yg, mask[g:g + 1], alpha, beta, N - n, 1, t[g:g + 1], sc[g:g + 1], st[g:g + 1], *ref)
