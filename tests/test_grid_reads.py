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
