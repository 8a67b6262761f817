"""Divisions by reciprocals that kernels and host share, against the integers: over the whole domain where that is small, else at the
multiples of the divisor and beside them, where a wrong quotient would show first."""
import random

import host_shim


def test_small_div():
    div = host_shim.load().shim_small_div
    assert all(div(x, d) == x // d for d in range(1, 513) for x in range(512))
    assert all(div(x, d) == x // d for d in range(4, 65) for x in range(4096))
    # whole rows divide chunks of 64 rows by a pitch, convolutions pixels of 384 by the width of a patch
    pitches = [host_shim.load().shim_run_pitch(n) for n in range(8, 321)]
    assert 4 <= min(pitches) and max(pitches) <= 64 and 64 * max(pitches) <= 4096


def test_grid_div():
    div, rng = host_shim.load().shim_grid_div, random.Random(3)
    for d in list(range(1, 300)) + [rng.randint(300, 32767) for _ in range(300)] + [32766, 32767]:
        near = {q * d + e for q in [rng.randint(0, 32767 // d) for _ in range(20)] + [1, 32767 // d] for e in (-1, 0, 1)}
        assert all(div(x, d) == x // d for x in near | {0, 32767} if 0 <= x <= 32767), d
