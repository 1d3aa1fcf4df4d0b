"""CPU checks of the choice between plane Couette's plane kernels (sps_couette_plane_kernels, no GPU): the sizes
below, which tests/test_gpu_kernel_edges.py compares with the oracle, run the row kernels of a known length, and every
padded x length that has them is among the sizes."""
import ctypes

import pytest

import paper_2506_14792_amd as sps

# nx, ny, nz: the padded x lengths with row kernels of their own (24, 36, 48, 72, 96, 108, 192), each with just as many
# blocks as they need or up to three more, of which every grid row's last one is not full (8 of 16, 6 of 16, 4 of
# 16, 3 of 8, 4 of 8, 2 of 8 and 2 of 4 row pairs).  The columns have kernels of their own too but at nz = 36.
ROW_SIZES = [(16, 32, 96), (24, 40, 72), (32, 54, 48), (48, 40, 36), (64, 32, 48), (72, 54, 24), (128, 32, 24)]
PAIRS = {24: 16, 36: 16, 48: 16, 72: 8, 96: 8, 108: 8, 192: 4}   # row pairs of a block
BLOCKS = 240


@pytest.mark.parametrize("nx,ny,nz", ROW_SIZES)
def test_row_sizes_run_the_known_length_kernels(nx, ny, nz):
    per, pairs = PAIRS[3 * nx // 2], 3 * nz // 4
    blocks = -(-pairs // per) * (3 * ny // 2)
    assert pairs % per != 0 and BLOCKS <= blocks <= BLOCKS + 3
    assert sps.couette_plane_kernels(nx, ny, nz) == (True, nz != 36)
    fewer = ny - 2 * ((blocks - BLOCKS) // (3 * -(-pairs // per)) + 1)
    assert sps.couette_plane_kernels(nx, fewer, nz) == (False, nz != 36)


def test_every_row_length_is_listed():
    """At 64 x 4096 the number of blocks is no bar: the x lengths with row kernels are those listed."""
    known = {3 * nx // 2 for nx in range(4, 260, 2) if sps.couette_plane_kernels(nx, 64, 4096)[0]}
    assert known == {3 * nx // 2 for nx, _, _ in ROW_SIZES} == set(PAIRS)


def test_bad_sizes_are_refused():
    L, r, c = sps.lib(), ctypes.c_int(), ctypes.c_int()
    for n in ((15, 8, 8), (16, 7, 8), (16, 8, 0), (-16, 8, 8), (1 << 30, 8, 8)):
        assert L.sps_couette_plane_kernels(*n, ctypes.byref(r), ctypes.byref(c)) == -1
    assert L.sps_couette_plane_kernels(16, 8, 8, None, ctypes.byref(c)) == -1
