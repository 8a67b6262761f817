"""The LDS rings of the tile bodies in a launch, cut to the k-tiles there are: a loop of the depth it is told never touches
more than the launch gives it and reads every tile from the stage it was copied to; launches of few workgroups and few
tiles request as many tiles before the first wait as with the whole planned ring."""
import pytest

import host_shim

AHEAD_MAX = 3                             # tiles that the lean loop keeps in flight beyond the one it works on


def walk(depth, tiles, lean):
    """(tiles requested before the first wait, stages touched) of a loop of `depth` over `tiles` k-tiles."""
    ahead = min(depth - 1, AHEAD_MAX) if lean else depth - 1
    ring = ahead + 1 if lean else depth
    stage = {}                            # stage -> tile it holds
    for t in range(min(ahead, tiles)):
        stage[t] = t
    first, touched = len(stage), len(stage)
    for t in range(tiles):
        if t + ahead < tiles:
            s = (t + ahead) % ring
            assert s not in stage or stage[s] < t, "a copy into a stage that is still to be read"
            stage[s] = t + ahead
            touched = max(touched, s + 1)
        assert stage[t % ring] == t
    return first, touched


def tiles_of(splitk, k_tiles):
    return [(k_tiles - w + 3) // 4 if k_tiles > w else 0 for w in range(4)] if splitk else [k_tiles]


# (split-k, planned stages, stage bytes) of a launch's bodies: alone, with a tail, a tail whose ring is the larger one
LAUNCHES = [[(0, s, 16384)] for s in range(2, 9)] + [[(1, s, 10240)] for s in range(2, 5)] + \
           [[(0, 2, 32768), (0, 8, 10240)], [(0, 5, 16384), (0, 8, 10240)], [(0, 3, 24576), (1, 4, 10240)], [(1, 5, 8192), (0, 4, 20480)]]


@pytest.mark.parametrize("workgroups", [48, 600, 100000])
@pytest.mark.parametrize("slots", LAUNCHES)
def test_rings(slots, workgroups):
    planned_lds = max((4 if sk else 1) * s * b for sk, s, b in slots)
    for k_tiles in range(1, 70):
        lds, depths = host_shim.ring_plan(slots, k_tiles, workgroups, 256, planned_lds)
        assert 0 < lds <= planned_lds
        for (splitk, planned, stage_bytes), depth in zip(slots, depths):
            assert 2 <= depth <= planned
            for tiles in tiles_of(splitk, k_tiles):
                most = max(tiles_of(splitk, k_tiles))
                room = depth if depth <= most else max(most, 2)                 # stages that a split-k body's rings lie apart
                for lean in ([False] if splitk else [False, True]):
                    first, touched = walk(depth, tiles, lean)
                    assert touched <= (room if splitk else lds // stage_bytes)
                    if most <= 2 and workgroups == 48:
                        assert first == walk(planned, tiles, lean)[0], "fewer tiles requested up front than with the whole ring"
            if splitk:
                assert 4 * room * stage_bytes <= lds


def test_crowded_launches_take_what_lets_more_workgroups_in():
    body = [(0, 3, 24576)]                # 128 x 64 tiles: two workgroups per CU with the planned ring, three with two stages
    assert host_shim.ring_plan(body, 2, 768, 256, 73728) == (49152, [2])
    assert host_shim.ring_plan(body, 2, 512, 256, 73728) == (49152, [3])
    assert host_shim.ring_plan([(0, 2, 32768), (0, 8, 10240)], 2, 768, 256, 81920) == (65536, [2, 3])
