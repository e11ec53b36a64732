"""Layers per tile of the FP64 operator passes (host rule), seen in the slots that the
allocation-free entry point asks for; and that this entry point takes every grid whose
tiles of 8x8x4 elements, with a slot per node of their boxes, fit its scratch.  The node
mask's bytes and the rounding to 256 are the entry point's own."""
import random

import pytest

SLOT_PLANE = 9 * 9 * 5 * 8  # bytes of a tile's node plane


def up(n, d):
    return -(-n // d)


def slot_bytes(fe, nx, ny, nz):
    nn = (nx + 1) * (ny + 1) * (nz + 1)
    return fe.fe_jvp_noalloc_scratch_bytes(nx, ny, nz) - up(nn, 256) * 256


@pytest.fixture(scope="module")
def fe():
    from paper_1508_04596_amd import fe as fe_mod
    fe_mod.lib()
    return fe_mod


# 64^3: 64 columns of tiles, 8 layers; 129x129x3: 289 columns
@pytest.mark.parametrize("dims,want", [((8, 8, 8), 1), ((24, 24, 24), 1), ((32, 32, 16), 1),
                                       ((28, 28, 28), 2), ((32, 32, 32), 2), ((40, 40, 20), 2), ((9, 9, 65), 2),
                                       ((96, 64, 5), 1), ((40, 32, 25), 1), ((33, 33, 33), 2), ((40, 40, 40), 2),
                                       ((41, 33, 37), 3), ((64, 64, 64), 8), ((129, 129, 3), 3),
                                       ((96, 96, 96), 8), ((160, 160, 320), 16)])
def test_layers(fe, dims, want):
    nx, ny, nz = dims
    assert slot_bytes(fe, *dims) == up(nx, 8) * up(ny, 8) * up(nz, want) * (want + 1) * SLOT_PLANE


def test_no_grid_is_refused_that_fitted_as_boxes(fe):
    rng = random.Random(5)
    for _ in range(20000):
        nx, ny, nz = (round(2 ** rng.uniform(0, 12)) for _ in range(3))
        nn = (nx + 1) * (ny + 1) * (nz + 1)
        if up(nn, 256) * 256 + up(nx, 8) * up(ny, 8) * up(nz, 4) * 5 * SLOT_PLANE <= fe.FE_NOALLOC_SCRATCH_BYTES:
            assert fe.fe_jvp_noalloc_scratch_bytes(nx, ny, nz) <= fe.FE_NOALLOC_SCRATCH_BYTES, (nx, ny, nz)
