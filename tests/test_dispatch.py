"""Which kernels the entry points launch (host code against tests/hip_double.c)."""
import pytest

from tests.host_driver import check

TILES = [(8, 32, 4), (8, 32, 8), (8, 16, 4), (8, 32, 2), (32, 8, 4), (16, 16, 4), (16, 16, 8)]


def tile_of(name):
    """The tile whose kernel this is."""
    if any(part in name for part in ("fuse_block_kernel", "fuse_bilinear_kernel", "pipe_block_kernel")):
        return 6
    return [k for k, (x, y, z) in enumerate(TILES) if f"_kernelILi{x}ELi{y}ELi{z}ELi" in name][0]


@pytest.mark.parametrize("sampling", [0, 1])
@pytest.mark.parametrize("grid,n,W,H", [((128, 128, 128), 8, 640, 480), ((40, 33, 20), 3, 320, 240), ((200, 200, 200), 12, 1280, 720)])
def test_a_set_tile_is_the_one_that_fuses(tmp_path_factory, sampling, grid, n, W, H):
    for tile, _, name, _, _ in check(tmp_path_factory, "fusion_kernels", dict(grid=grid, n=n, W=W, H=H, sampling=sampling)):
        assert tile == -1 or tile_of(name) == tile, name


BATCH = [((160, 160, 160), 12, 640, 480), ((40, 40, 40), 4, 320, 240), ((128, 128, 128), 6, 640, 480), ((208, 200, 192), 8, 643, 477)]


@pytest.mark.parametrize("sampling", [0, 1])
def test_a_set_tile_is_the_one_that_every_frame_of_a_batch_runs(tmp_path_factory, sampling):
    runs = check(tmp_path_factory, "batch_kernels", dict(frames=BATCH, sampling=sampling))
    for tile, reported, first, again in runs:
        assert first == again
        if tile >= 0:
            fusions = [name for name, _, _ in first if "slm" not in name]
            assert {tile_of(name) for name in fusions} == {tile} and reported == tile
    # -1 gives the batch its own choice back, whatever was set in between
    assert runs[0][2:] == runs[-1][2:]
    if sampling == 0:
        assert len({tile_of(name) for name, _, _ in runs[0][2]}) == 3       # blocks, 2 voxels per lane, tile 0


@pytest.mark.parametrize("sampling", [0, 1])
@pytest.mark.parametrize("grid,n,W,H,nearest,bilinear", [
    ((40, 33, 20), 3, 320, 240, 3, 6), ((128, 128, 128), 8, 640, 480, 2, 6), ((200, 200, 200), 12, 1280, 720, 6, 6),
    ((64, 64, 64), 4, 1280, 720, 3, 0)])
def test_the_reported_tile_is_the_one_that_fuses(tmp_path_factory, sampling, grid, n, W, H, nearest, bilinear):
    for tile, reported, name, _, _ in check(tmp_path_factory, "fusion_kernels", dict(grid=grid, n=n, W=W, H=H, sampling=sampling)):
        assert reported == tile_of(name) == (tile if tile >= 0 else bilinear if sampling else nearest)


@pytest.mark.parametrize("frames", [BATCH, BATCH[:2], BATCH[1:2], BATCH[2:3], BATCH[1:3]])
def test_the_reported_tile_of_a_batch_is_that_of_its_largest_frame(tmp_path_factory, frames):
    largest = max(frames, key=lambda f: f[0][0] * f[0][1] * f[0][2] * f[1])
    args = [dict(frames=f, sampling=0, tiles=[-1]) for f in (frames, [largest])]
    (_, reported, _, _), = check(tmp_path_factory, "batch_kernels", args[0])
    (_, _, alone, _), = check(tmp_path_factory, "batch_kernels", args[1])
    assert {reported} == {tile_of(name) for name, _, _ in alone}


def _tile_kernel(tile):
    return "_kernelILi%dELi%dELi%dELi" % TILES[tile]


MIDDLE = dict(grid=(144, 144, 144), n=8, W=640, H=480)       # blocks for the fusion alone, columns for a step


@pytest.mark.parametrize("fusion,step", [(4, 1), (1, 6), (6, 6), (5, 5)])
def test_the_plan_tuner_times_what_it_sets(tmp_path_factory, fusion, step):
    """The fastest fusion and the fastest step, each for its own call."""
    name = lambda t, of: ("fuse" if of else "pipe") + ("_block_kernel" if t == 6 else _tile_kernel(t))
    got = check(tmp_path_factory, "tuned_plan", dict(MIDDLE, sampling=0, costs=[(name(fusion, True), 0.5), (name(step, False), 0.5)]))
    for k in ("timed", "cached"):
        assert got[k]["best"] == got[k]["reported"] == fusion
        assert [tile_of(x) for x in got[k]["kernels"]] == [fusion, step]
    assert got["timed"]["launched"] > 2 * 7 and got["cached"]["launched"] == 0


@pytest.mark.parametrize("sampling", [0, 1])
def test_a_tuned_plan_is_the_untuned_one_when_no_tile_is_clearly_faster(tmp_path_factory, sampling):
    """All launches take as long, but for one that is 1 % faster: noise."""
    got = check(tmp_path_factory, "tuned_plan", dict(MIDDLE, sampling=sampling, costs=[(_tile_kernel(4), 0.99)]))
    assert got["timed"]["kernels"] == got["cached"]["kernels"] == got["untuned"]["kernels"]


def test_the_bilinear_tuner_times_different_kernels(tmp_path_factory):
    got = check(tmp_path_factory, "tuned_plan", dict(MIDDLE, sampling=1, costs=[("fuse" + _tile_kernel(3), 0.5), ("pipe" + _tile_kernel(1), 0.5)]))
    assert got["timed"]["best"] == 3 and [tile_of(x) for x in got["timed"]["kernels"]] == [3, 1]


def test_choices_cached_for_other_kernels_are_not_applied(tmp_path_factory):
    """Entries under the keys that named neither the kernels nor the default tiles."""
    old = {f"gfx950/256cu/plan/s0/e8/n8/i{i}": 1 for i in range(24)}
    got = check(tmp_path_factory, "tuned_plan", dict(MIDDLE, sampling=0, cache=old, costs=[("fuse" + _tile_kernel(4), 0.5)]))
    assert got["timed"]["best"] == 4 and set(old.items()) <= set(got["cache"].items())


def test_the_smallest_workspace_tunes_the_fusion_alone(tmp_path_factory):
    """Maps, a posterior and an occupancy grid were enough before the step was timed."""
    got = check(tmp_path_factory, "tuned_plan", dict(MIDDLE, sampling=0, short=True, costs=[("fuse" + _tile_kernel(4), 0.5), ("pipe" + _tile_kernel(1), 0.5)]))
    assert got["timed"]["best"] == 4
    assert got["timed"]["kernels"][1] == got["untuned"]["kernels"][1]


def test_the_batch_tuner_knows_the_default(tmp_path_factory):
    """Where no tile is clearly faster than the tiles that suit the frames, the
    batch keeps these, also from the cache."""
    got = check(tmp_path_factory, "tuned_batch", dict(frames=BATCH, sampling=0, costs=[(_tile_kernel(4), 0.99)]))
    assert got["timed"]["kernels"] == got["cached"]["kernels"] == got["untuned"]["kernels"]
    assert got["timed"]["best"] == got["timed"]["reported"] == got["untuned"]["reported"] == 6
    assert got["timed"]["launched"] > 0 and got["cached"]["launched"] == 0


@pytest.mark.parametrize("sampling", [0, 1])
def test_the_batch_tuner_keeps_a_faster_tile(tmp_path_factory, sampling):
    for tile in (4, 6):
        part = "batch_pipe_block" if tile == 6 and sampling == 0 else _tile_kernel(tile)
        got = check(tmp_path_factory, "tuned_batch", dict(frames=BATCH, sampling=sampling, costs=[(part, 0.5)]))
        for k in ("timed", "cached"):
            assert got[k]["best"] == got[k]["reported"] == tile and {tile_of(x) for x in got[k]["kernels"]} == {tile}


def test_batch_choices_cached_for_other_kernels_are_not_applied(tmp_path_factory):
    first = check(tmp_path_factory, "tuned_batch", dict(frames=BATCH, sampling=0, costs=[(_tile_kernel(4), 0.5)]))
    (key, _), = first["cache"].items()
    old = {key.replace("/r2", ""): 1}
    got = check(tmp_path_factory, "tuned_batch", dict(frames=BATCH, sampling=0, costs=[(_tile_kernel(4), 0.5)], cache=old))
    assert list(old) != [key] and got["timed"]["best"] == 4


@pytest.mark.parametrize("grid", [(1, 1, 2 ** 25), (1, 1, 2 ** 31 - 1), (2, 32768, 32767), (4, 1, 2 ** 29 - 1), (3, 5, 10 ** 8), (1, 2 ** 30, 1), (60, 1, 2 ** 25)])
def test_no_axis_of_a_surface_launch_reaches_two_to_the_32(tmp_path_factory, grid):
    for name, groups, lanes in check(tmp_path_factory, "surface_launches", dict(grid=grid)):
        assert all(g * b < 2 ** 32 for g, b in zip(groups, lanes)), (name, groups, lanes)
        assert groups[1] <= 65535 and groups[2] <= 65535
        if "smooth" in name:                                # 16 voxels or more to a workgroup, few idle ones
            assert groups[0] * groups[1] <= grid[0] * grid[1] * grid[2] / 2 + 2 ** 20


@pytest.mark.parametrize("sampling", [0, 1])
@pytest.mark.parametrize("grid", [(1, 2 ** 28, 1), (2, 2 ** 28, 1), (8, 2 ** 28 - 1, 1), (1, 2 ** 28, 4), (2 ** 27 - 8, 1, 1), (1, 1, 2 ** 26 - 8)])
def test_the_default_fuses_what_tile_0_fuses(tmp_path_factory, sampling, grid):
    """Long rows of few columns, of which a tile of 8 x 32 columns holds twice as many as one of 16 x 16."""
    for tile, _, name, groups, lanes in check(tmp_path_factory, "fusion_kernels", dict(grid=grid, n=4, W=320, H=240, sampling=sampling)):
        if tile in (-1, 0):
            assert groups[0] * lanes[0] < 2 ** 32, (tile, name, groups, lanes)


@pytest.mark.parametrize("grid,n,W,H,side,kernel", [
    ((700, 700, 1), 6, 640, 480, 2.0, "fuse_bilinear_kernelILi2E"),      # no deeper than the grid
    ((700, 700, 2), 6, 640, 480, 2.0, "fuse_bilinear_kernelILi2E"),
    ((700, 700, 3), 6, 640, 480, 2.0, "fuse_bilinear_kernelILi4E"),
    ((700, 700, 5), 6, 640, 480, 2.0, "fuse_bilinear_kernelILi8E"),
    ((128, 128, 128), 8, 640, 480, 2.0, "fuse_bilinear_kernelILi8E"),
    ((5, 233, 233), 3, 320, 240, 2.0, _tile_kernel(0)),                  # blocks twice as wide as the grid: work
    ((2, 300, 300), 8, 320, 240, 2.0, _tile_kernel(0)),
    ((3, 100, 90), 12, 320, 240, 2.0, "fuse_bilinear_kernel"),           # latency
    ((67, 56, 55), 11, 114, 86, 4.9, _tile_kernel(0)),                   # hardly in view
    ((67, 56, 55), 11, 114, 86, 2.0, "fuse_bilinear_kernel"),
    ((71, 51, 69), 1, 255, 191, 2.0, _tile_kernel(0)),                   # one or two views
    ((69, 83, 67), 2, 102, 76, 3.5, _tile_kernel(0)),
    ((256, 256, 256), 1, 320, 240, 5.0, "fuse_bilinear_kernelILi8E"),
    ((128, 128, 128), 2, 320, 240, 2.0, "fuse_bilinear_kernelILi8E"),
])
def test_bilinear_boxes_where_they_pay(tmp_path_factory, grid, n, W, H, side, kernel):
    runs = check(tmp_path_factory, "fusion_kernels", dict(grid=[*grid, side], n=n, W=W, H=H, sampling=1))
    assert kernel in runs[0][2]


def test_the_views_that_hold_the_whole_grid(tmp_path_factory):
    """Of the grid itself, however far the tiles reach past its edge; never of a view
    that misses a voxel."""
    got = check(tmp_path_factory, "inside", dict(seed=3, count=400))
    assert not [missed for said, missed in got if said and missed]
    held = [said for said, missed in got if not missed]
    assert len(held) > 100 and sum(held) > 0.95 * len(held)


@pytest.mark.parametrize("grid,n,W,H,side,kernel", [
    ((144, 144, 144), 8, 640, 480, 2.0, "fuse_block_kernel"),
    ((144, 144, 144), 12, 1280, 720, 1.8, _tile_kernel(2)),              # few blocks of large boxes
    ((160, 160, 160), 12, 1280, 720, 2.0, "fuse_block_kernel"),
    ((128, 128, 128), 8, 640, 480, 2.0, _tile_kernel(2)),                # few blocks
    ((192, 192, 192), 7, 236, 177, 2.0, _tile_kernel(2)),                # small boxes
    ((256, 256, 256), 1, 643, 477, 2.0, "fuse_block_kernel"),
])
def test_blocks_where_they_pay(tmp_path_factory, grid, n, W, H, side, kernel):
    runs = check(tmp_path_factory, "fusion_kernels", dict(grid=[*grid, side], n=n, W=W, H=H, sampling=0))
    assert kernel in runs[0][2]
