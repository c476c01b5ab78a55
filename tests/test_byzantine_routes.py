"""Which kernel a Byzantine call takes, read off its launches on the host: the shape decides, not the number of groups, since the kernels
round differently and a group's located workers may hang on the last bits."""
import pytest

import launch_log

ENTRIES = ["approxifer_decode_byzantine", "approxifer_decode_byzantine_homogeneous"]


@pytest.mark.parametrize("entry", ENTRIES)
def test_the_number_of_groups_does_not_choose_the_locator(tmp_path, entry):
    groups = (1, 7, 100, 199, 260, 401, 2100, 20000)
    shapes = [(K, A, S, ex, C) for K in range(1, 13) for A in (1, 2, 3) for S in range(6) for ex in range(4) for C in (1, 10, 20, 300)
              if (K + A + S + ex) % 2 == 0 or K + A > 9]
    calls = [dict(entry=entry, G=G, K=K, A=A, S=S, N=2 * (K + A) + S + ex, C=C, workspace=False) for K, A, S, ex, C in shapes for G in groups]
    got = launch_log.launches(tmp_path, calls)
    taken = 0
    for i, shape in enumerate(shapes):
        tiles = set()
        for rc, names in got[len(groups) * i:len(groups) * (i + 1)]:
            assert rc == 0 and names
            tiles.add(next((t for t in map(launch_log.pairs_tile, names) if t), None))
        assert len(tiles) == 1, (shape, tiles)
        taken += tiles != {None}
    assert taken > len(shapes) // 4
