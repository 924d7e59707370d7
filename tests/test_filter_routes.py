"""Which kernel takes a dense filter: the rules on sizes and values (planning only, no GPU)."""
import numpy as np
import pytest

import paper_1907_06154_amd as ssam


def route(kind, shape, filt, boundary="zero"):
    return ssam.ssam_describe(kind, shape, filt, boundary).split()[0]


def with_taps(shape, count):
    f = np.zeros(int(np.prod(shape)), dtype=np.float32)
    f[np.linspace(0, f.size - 1, count).astype(int)] = 0.5
    return f.reshape(shape)


@pytest.mark.parametrize("size", [9, 20, 25])
def test_filters_of_one_or_two_taps_keep_the_fp32_kernels(size):
    for taps, split in ((1, False), (2, False), (3, True), (9, True)):
        assert ("split3mx" in route("conv2d", (1000, 1000), with_taps((size, size), taps))) == split, taps


@pytest.mark.parametrize("M,N,K,split", [(1, 1, 9, False), (1, 1, 17, False), (2, 1, 5, False), (1, 2, 9, False), (1, 3, 5, True),
                                         (3, 1, 9, True), (5, 1, 1, True), (1, 9, 1, True), (5, 5, 5, True)])
def test_volume_filters_of_few_taps_per_plane_keep_the_fp32_kernels(M, N, K, split):
    f = np.full((K, N, M), 0.25, dtype=np.float32)
    assert ("split3mx" in route("conv3d", (300, 300, 300), f)) == split


@pytest.mark.parametrize("size", [5, 7, 9])
def test_sparse_volume_filters(size):
    shape = (size,) * 3
    for taps in (1, 2, 2 * size):
        assert "split3mx" not in route("conv3d", (200, 200, 200), with_taps(shape, taps)), taps
    assert "split3mx" in route("conv3d", (200, 200, 200), with_taps(shape, 3 * size))


def test_a_tap_far_below_the_largest():
    """A weight whose low parts would be subnormal once the largest is scaled to [1, 2)."""
    for kind, shape, size in (("conv2d", (1000, 1000), (9, 9)), ("conv3d", (100, 100, 100), (5, 5, 5))):
        f = np.full(size, 2.0 ** 40, dtype=np.float32)
        for e, split in ((-59, True), (-61, False), (-80, False)):
            f.flat[3] = 2.0 ** e
            assert ("split3mx" in route(kind, shape, f)) == split, (kind, e)


def plan(kind, shape, filt, boundary="zero"):
    name, *fields = ssam.ssam_describe(kind, shape, filt, boundary).split()
    return name, {k: v for k, v in (f.split("=") for f in fields)}


def test_the_description_is_of_the_launch_that_is_made():
    """Kernels that go by another's name: the register-tiled fp64 kernel instead of the direct one, the staged and the
    two-row forms of the block-cooperative 3D kernel."""
    for shape, filt in (((1500, 1600), np.ones((12, 12))), ((1500, 1600), np.ones((32, 32)))):
        name, g = plan("conv2d", shape, filt)
        assert name == "generic_direct" and g["form"] == "1" and int(g["lds"]) > 0
        assert int(g["strips_x"]) * int(g["tiles_y"]) * int(g["tiles_z"]) == int(g["tiles"]) <= int(g["blocks"]) < int(g["tiles"]) + 8
        assert int(g["strips_x"]) * 64 >= 1600 and int(g["tiles_y"]) * 64 >= 1500
    name, g = plan("conv2d", (1500, 1600), np.ones((12, 12), dtype=np.float32))
    assert "split3mx" in name and g["form"] == "0" and int(g["lds"]) > 0
    star = np.zeros((3, 3, 3))
    star[1, 1, :] = star[1, :, 1] = star[:, 1, 1] = 1.0
    for W, form in ((200, "0"), (201, "1")):
        name, g = plan("stencil3d", (200, 200, W), star)
        assert "p4w8star_ring3" in name and g["form"] == form, (W, g)
    assert plan("stencil3d", (512, 512, 512), star)[1]["P"] == "4"
    assert plan("stencil3d", (40, 40, 40), star)[1]["P"] == "2"


@pytest.mark.parametrize("shape", [(13200, 160), (65536, 40), (65536, 32), (22000, 90), (40000, 64)])
def test_fp64_filters_on_tall_narrow_pictures_fit_the_lds_of_a_block(shape):
    """Eight lanes side by side make a wave 32 rows tall; four of them and a large filter's halo pass 64 KB."""
    for M, N in ((20, 20), (21, 21), (25, 25), (32, 14), (32, 32), (12, 12)):
        name, g = plan("conv2d", shape, np.ones((N, M)))
        assert g["form"] == "1" and 0 < int(g["lds"]) <= 64 << 10, (shape, M, N, g)


@pytest.mark.parametrize("shape,size,tiled", [
    ((512, 515), (16, 16), 1), ((512, 515), (1, 16), 0), ((512, 515), (16, 1), 0), ((256, 259), (24, 24), 1), ((256, 259), (12, 3), 0),
    ((1024, 1027), (1, 12), 1), ((64, 64, 64), (3, 9, 13), 0), ((64, 64, 64), (9, 1, 1), 0), ((128, 128, 128), (9, 3, 3), 1),
    ((128, 128, 128), (9, 2, 2), 0), ((256, 256, 256), (9, 1, 1), 0), ((256, 256, 256), (9, 1, 7), 1)])
def test_fp64_filters_take_the_register_tiled_kernel_where_it_is_faster(shape, size, tiled):
    """Filters of a few taps per plane and grids too small to fill the machine stay on the direct kernel."""
    filt = np.ones(size)
    name, g = plan("conv2d" if len(shape) == 2 else "conv3d", shape, filt)
    assert name == "generic_direct" and int(g["form"]) == tiled
    for force, form in ((1, 0), (2, 1)):
        ssam.ssam_set_tuning("force_generic", force)
        try:
            assert int(plan("conv2d" if len(shape) == 2 else "conv3d", shape, filt)[1]["form"]) == form
        finally:
            ssam.ssam_set_tuning("force_generic", -1)


def test_embed_waste_asks_for_the_cube():
    filt = np.ones((4, 6, 5))
    assert route("conv3d", (64, 64, 64), filt) == "generic_direct"
    ssam.ssam_set_tuning("embed_waste", 4)
    try:
        assert route("conv3d", (64, 64, 64), filt).endswith("+embedded")
    finally:
        ssam.ssam_set_tuning("embed_waste", -1)


@pytest.mark.parametrize("M,N,H,W,split", [(1, 32, 512, 512, False), (1, 22, 130, 130, False), (1, 32, 1100, 1100, True), (2, 24, 256, 256, False),
                                           (2, 24, 512, 512, True), (3, 24, 256, 256, True), (32, 1, 512, 512, True), (1, 20, 512, 512, True)])
def test_tall_thin_fp32_filters_on_small_pictures(M, N, H, W, split):
    """One or two columns and more than 20 rows: the direct kernel, which is faster there."""
    name = route("conv2d", (H, W), np.ones((N, M), dtype=np.float32))
    assert ("split3mx" in name) == split and (split or name == "generic_direct"), name


def test_large_pictures_keep_the_wide_strips():
    """Tiles are at most 512 rows; a picture that would want taller ones keeps the strip width of the next smaller."""
    filt = np.ones((20, 20), dtype=np.float32)
    for n in (8192, 16384, 20000, 24000, 32768):
        _, g = plan("conv2d", (n, n), filt, "clamp")
        assert g["valid_lanes"] == "32" and int(g["rows_per_wave"]) <= 512, (n, g)
    ssam.ssam_set_tuning("rows_per_wave", 64)
    try:
        assert plan("conv2d", (24000, 24000), filt)[1]["rows_per_wave"] == "64"
    finally:
        ssam.ssam_set_tuning("rows_per_wave", -1)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_radius_3_stencils_on_small_ragged_grids(dtype):
    """Faces and edges (127 taps) and boxes inside the radius-3 box: the direct kernel until there is work for the box."""
    off = np.abs(np.indices((7, 7, 7)) - 3)
    edges = ((off != 0).sum(axis=0) <= 2).astype(dtype)
    box = np.ones((7, 5, 5), dtype=dtype)
    for shape, ring in (((11, 5, 11), False), ((101, 5, 41), False), ((40, 40, 33), False), ((200, 200, 301), True)):
        for coef in (edges, box):
            name = route("stencil3d", shape, coef)
            if ring:
                assert "ring" in name or "split3mx" in name, (shape, name)
            else:                                                      # (a box of 175 taps goes to the split kernel from W = 32 on)
                assert name == "generic_direct" or (coef is box and "split3mx" in name), (shape, name)
    assert "ring" in route("stencil3d", (40, 40, 9), np.ones((7, 7, 7), dtype=dtype))
    assert "ring" in route("stencil3d", (11, 5, 12), edges)            # whole 16-byte pieces: the unstaged form, as ever


@pytest.mark.parametrize("dtype,r,planes", [(np.float32, 4, 4), (np.float64, 4, 3), (np.float32, 2, 2), (np.float64, 2, 1), (np.float32, 1, 1)])
def test_stars_on_a_few_planes_of_ragged_rows(dtype, r, planes):
    """The staged form from `planes` planes on; below, the kernels with halo lanes."""
    coef = np.zeros((2 * r + 1,) * 3, dtype=dtype)
    coef[r, r, :] = coef[r, :, r] = coef[:, r, r] = 1.0
    for D in range(1, 6):
        _, g = plan("stencil3d", (D, 40, 131), coef)
        assert (g["form"] == "1") == (D >= planes), (D, g)
        assert (g["halo_lanes"] == "0+0") == (D >= planes), (D, g)
