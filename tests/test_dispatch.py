"""Which kernels the entry points launch (host code against tests/hip_double.c)."""
import pytest

from tests.host_driver import check

TILES = [(8, 32, 4), (8, 32, 8), (8, 16, 4), (8, 32, 2), (32, 8, 4), (16, 16, 4), (16, 16, 8)]


def tile_of(name):
    """The tile whose kernel this is."""
    if "fuse_block_kernel" in name or "fuse_bilinear_kernel" in name:
        return 6
    return [k for k, (x, y, z) in enumerate(TILES) if f"fuse_kernelILi{x}ELi{y}ELi{z}ELi" in name][0]


@pytest.mark.parametrize("sampling", [0, 1])
@pytest.mark.parametrize("grid,n,W,H", [((128, 128, 128), 8, 640, 480), ((40, 33, 20), 3, 320, 240), ((200, 200, 200), 12, 1280, 720)])
def test_a_set_tile_is_the_one_that_fuses(tmp_path_factory, sampling, grid, n, W, H):
    for tile, _, name, _, _ in check(tmp_path_factory, "fusion_kernels", dict(grid=grid, n=n, W=W, H=H, sampling=sampling)):
        assert tile == -1 or tile_of(name) == tile, name
