"""What the grid's plan takes a band's height by: rows and columns that the XCD with the most of them reads, against the walk itself."""
import random

import host_shim
import pytest


@pytest.mark.parametrize("nx", [1, 8, 5])
def test_reads_of_the_busiest_xcd(nx):
    reads, rng = host_shim.load().shim_grid_reads, random.Random(nx)
    grids = [(1, 1), (1, 9), (9, 1), (2, 3), (7, 16), (9, 24)] + [(rng.randint(1, 30), rng.randint(1, 40)) for _ in range(12)]
    for rows, cols in grids:
        for group in range(1, rows + 1):
            tiles = [host_shim.grid_tile(b, rows, cols, group, nx) for b in range(rows * cols)]
            most = max(16 * len({r for r, _ in tiles[x::nx]}) + 48 * len({c for _, c in tiles[x::nx]}) for x in range(nx))
            assert reads(rows, cols, group, nx, 16, 48) == most, (rows, cols, group)


def test_height_of_bands():
    """Never lower than the one an XCD's run would have at the top of a band, and another one only for a sixth less to read on the busiest
    XCD, the highest of equal ones."""
    lib, rng = host_shim.load(), random.Random(9)
    band, reads = lib.shim_grid_band, lib.shim_grid_reads
    assert band(8, 24, 8, 96, 128) == 8 and band(8, 24, 8, 48, 64) == 8                # (6, or 4 with as little to read as 8)
    assert band(1, 7, 8, 32, 32) == 1 and band(9, 24, 8, 32, 32) == 9 and band(31, 6, 8, 96, 128) == 6
    for _ in range(300):
        rows, cols, nx, tm, tn = rng.randint(1, 40), rng.randint(1, 50), rng.choice((1, 8, 8, 5)), rng.choice((16, 32, 48, 96, 128)), rng.choice((32, 64, 128, 192))
        run = -(-rows * cols // nx)
        first = min(range(1, rows + 1), key=lambda g: (g * -(--(-run // g) // cols) * tm + min(-(-run // g), cols) * tn, g))
        most = {g: reads(rows, cols, g, nx, tm, tn) for g in range(first, rows + 1)}
        higher = min((m, -g) for g, m in most.items())
        want = -higher[1] if higher[0] * 6 < most[first] * 5 else first
        assert band(rows, cols, nx, tm, tn) == want, (rows, cols, nx, tm, tn)
