"""Every instance of the kernel of two lanes to a class: columns, rows, missing workers, one workgroup to whole groups, to 128 classes of a
group or to all of them, either locator.  On the host: that the shapes below launch each of them.  On the GPU: their results."""
import numpy as np
import pytest

import launch_log
from oracle import approxifer_oracle as orc
from parity_cases import TOL, group_err

ENTRIES = ["approxifer_decode_byzantine", "approxifer_decode_byzantine_homogeneous"]
COLUMNS = range(2, 16)                                       # K + A
# few and many classes, without and with a workspace (its size asked for)
WAYS = ((11, 10, False), (2, 130, False), (2, 130, True))    # G, C, workspace


def _shapes(M, wide):
    """(K, A, S, N) of one row of tiles: K + A = M, as many workers as eq. (3) asks for or as many more as take the wider one."""
    for S in range(5):
        A = 1 if M == 2 else 1 + (M + S) % (3 if 4 <= M <= 12 else 2)
        yield M - A, A, S, 2 * M + S + (0 if not wide else (3 if M % 2 else 1 + S % 2))


def test_the_shapes_launch_every_instance(tmp_path):
    calls = [dict(entry=e, G=G, K=K, N=N, S=S, A=A, C=C, workspace=ws) for e in ENTRIES for M in COLUMNS for wide in (False, True)
             for K, A, S, N in _shapes(M, wide) for G, C, ws in WAYS]
    seen = set()
    for rc, names in launch_log.launches(tmp_path, calls):
        assert rc == 0
        seen |= {t for t in map(launch_log.pairs_tile, names) if t}
    built = {(mt, tq, S, mode, hom) for mt in range(4, 17, 2) for tq in (mt // 2, mt // 2 + 1) for S in range(5) for mode in range(3)
             for hom in (0, 1) if not (hom and (mt == 16 or mode == 1))}
    assert seen == built, built ^ seen


@pytest.mark.gpu
@pytest.mark.parametrize("entry", ENTRIES)
@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("M", COLUMNS)
def test_planted_liars_and_values(M, wide, entry):
    import torch

    from paper_2109_09868_amd import binding
    for K, A, S, N in _shapes(M, wide):
        for G, C, ws in WAYS:
            rng = np.random.default_rng(100 * M + 10 * S + C)
            alpha, beta = orc.chebyshev_nodes(K, N)
            Y = (orc.encode(rng.uniform(0, 1, (G, K, 32)), alpha, beta) @ (rng.standard_normal((32, C)) / 6)).astype(np.float32)
            sd = float(Y.std())
            mask, liars = np.zeros((G, N), np.uint8), np.zeros((G, A), np.int64)
            for g in range(G):
                here = rng.permutation(N)[S:]
                mask[g, here] = 1
                liars[g] = np.sort([w for w in here if abs(beta[w]) > 1e-9][:A])
                Y[g, liars[g]] += (sd * rng.choice([-1, 1], (A, C)) * rng.uniform(3, 30, (A, C))).astype(np.float32)
                Y[g, mask[g] == 0] = np.nan
            out, adv, st = (t.cpu().numpy() for t in getattr(binding, entry)(
                torch.from_numpy(Y).cuda(), torch.from_numpy(mask).cuda(), alpha, beta, S, A, 1,
                workspace=None if ws else binding.NO_WORKSPACE))
            found = np.all(adv == liars, axis=1)
            # ten classes' votes: one may hold a lie that a rational function explains
            assert np.all(st == 0) and found.sum() >= G - 1, (K, A, S, N, C, ws)
            left = mask[found].copy()
            np.put_along_axis(left, liars[found], 0, axis=1)
            ref, _ = orc.decode(np.where(left[:, :, None] != 0, Y[found], 0.0).astype(np.float32), left, alpha, beta, S + A, 1)
            assert group_err(out[found], ref).max() <= TOL, (K, A, S, N, C, ws)
