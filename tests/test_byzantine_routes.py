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


@pytest.mark.parametrize("entry", ENTRIES)
def test_the_size_asked_for_is_the_size_that_is_used(tmp_path, entry):
    # more than 128 classes: a workgroup to every 128 of them, and the launches that clear and read their votes, or one workgroup to a group
    calls = [dict(entry=entry, G=G, K=K, A=A, S=S, N=2 * (K + A) + S, C=C, workspace=True)
             for G in (3, 512, 513, 5000) for K, A, S in ((8, 2, 4), (8, 2, 0), (12, 2, 0), (12, 1, 0), (12, 1, 1), (4, 1, 1)) for C in (257, 1000)]
    for c, (rc, names) in zip(calls, launch_log.launches(tmp_path, calls)):
        split = c["G"] <= 512 or (entry == ENTRIES[0] and c["S"] == 0 and c["K"] == 12)
        assert rc == 0 and [launch_log.pairs_tile(n) is not None for n in names] == ([False, True, False] if split else [True]), (c, names)


def test_the_built_in_workspace_refuses_what_it_refused(tmp_path):
    # votes that only the library's nodes have a use for are done without where they do not fit
    entry = "approxifer_decode_byzantine_static"
    refused = [dict(entry=entry, G=512, K=8, A=2, S=4, N=36, C=1000, workspace=False)]
    accepted = [dict(entry=entry, G=G, K=8, A=2, S=4, N=24, C=C, workspace=False) for G, C in ((1000, 300), (1024, 1000), (5000, 129), (2048, 10))]
    got = launch_log.launches(tmp_path, refused + accepted)
    assert [rc for rc, _ in got] == [-8, 0, 0, 0, 0]
    assert not got[0][1] and all(names for _, names in got[1:])
