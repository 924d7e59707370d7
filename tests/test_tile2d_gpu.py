"""Small 2D grids, many sweeps a launch on tiles held in registers: grids of exactly one tile, one point more, and tiles moved back
from the grid's end, in every vector width; buffers aligned to the element only; against the CPU oracle."""
import re
import time

import numpy as np
import pytest

import oracle
import workloads as wl
from parity_util import assert_parity

torch = pytest.importorskip("torch")

SHAPES = [("star", 1), ("star", 2), ("star", 5), ("box", 1), ("box", 2), ("box", 4)]
GRIDS = [(16, 64), (17, 65), (64, 128), (65, 129), (64, 256), (67, 257), (131, 449), (300, 190)]


def coefficients(kind, r, dtype):
    return wl.seeded_coefficients(wl.mask_box(r, r) if kind == "box" else wl.mask_star(r, r), 70 + r, dtype)[0]


def test_plans():
    """Which grids the kernel takes, and that the plans of the sweeps that remain add up."""
    import paper_1907_06154_amd as ssam

    def name(shape, coef, remaining):
        return ssam.ssam_describe("iterate2d", shape, coef, "zero", remaining=remaining).split()[0]

    star, box3 = coefficients("star", 1, np.float32), coefficients("box", 3, np.float32)
    assert "_tile_" in name((300, 400), star, 10) and "_tile_" not in name((8192, 8192), star, 10)
    assert "_tile_" not in name((300, 63), star, 10) and "_tile_" not in name((15, 300), star, 10)   # narrower than a wave, fewer rows than four waves
    assert "_tile_" not in name((300, 400), box3, 10)        # single sweeps on the split kernel, with less error
    for shape in GRIDS + [(1023, 1025), (2048, 64)]:
        left = 23
        while left:
            done = int((re.search(r"_fused(\d+)$", name(shape, star, left)) or [0, 1])[1])
            assert 1 <= done <= left
            left -= done


def test_planning_takes_no_longer_the_more_sweeps_remain():
    """Long iterations: the plan is found among depths, and with many sweeps left it is the same whatever their number."""
    import paper_1907_06154_amd as ssam
    coef = coefficients("star", 1, np.float32)

    def plan(shape, remaining):
        best, text = float("inf"), ""
        for _ in range(20):
            t = time.perf_counter()
            text = ssam.ssam_describe("iterate2d", shape, coef, "clamp", remaining=remaining)
            best = min(best, time.perf_counter() - t)
        return best, text

    for shape in ((512, 512), (1023, 1025), (4096, 4096)):
        short, long, longer = (plan(shape, n) for n in (24, 1000, 10 ** 6))
        assert "_tile_" in short[1] and long[1] == longer[1]
        assert longer[0] < 4 * short[0] + 5e-5, (shape, short[0], longer[0])     # 10^6 by numbers of launches: 40 ms and more


def test_plans_of_thin_grids():
    """An axis that one tile covers has no halo, so depth costs nothing there; with 17 to 31 rows tiles of 16 rows are mostly halo."""
    import paper_1907_06154_amd as ssam

    def depth(shape, coef, boundary, remaining):
        name = ssam.ssam_describe("iterate2d", shape, coef, boundary, remaining=remaining).split()[0]
        return "_tile_" in name, int((re.search(r"_fused(\d+)$", name) or [0, 1])[1])

    for dtype in (np.float32, np.float64):
        for r in (1, 3, 4, 6):
            coef = coefficients("star", r, dtype)
            for shape in ((16, 64), (16, 256), (16, 4096)):
                for boundary in ("zero", "clamp"):
                    tile, n = depth(shape, coef, boundary, 20)
                    assert tile and n >= (20 if shape[1] <= 256 and r < 4 else 5), (shape, r, n)
        for r in (3, 4) if dtype == np.float64 else (3,):
            for H in (17, 24, 31):
                assert depth((H, 2000), coefficients("star", r, dtype), "zero", 3) == (False, 3)
    assert not depth((20, 2000), coefficients("box", 4, np.float64), "zero", 20)[0]


@pytest.mark.parametrize("dtype,kind,r,shape,boundary,remaining,tile", [
    (np.float64, "star", 1, (3940, 980), "zero", 3, False), (np.float64, "star", 1, (980, 980), "zero", 3, True),
    (np.float64, "box", 1, (1312, 3054), "zero", 3, False), (np.float64, "star", 1, (1500, 2000), "clamp", 3, False),
    (np.float64, "star", 1, (1300, 1300), "zero", 4, False), (np.float64, "star", 1, (1300, 1300), "clamp", 4, True),
    (np.float64, "star", 1, (2000, 2000), "zero", 6, False), (np.float64, "star", 1, (2000, 2000), "zero", 7, True),
    (np.float64, "star", 1, (2048, 2048), "zero", 2, False), (np.float64, "star", 1, (2047, 2048), "zero", 2, True),
    (np.float32, "star", 1, (2000, 2000), "zero", 3, False), (np.float32, "star", 1, (1900, 1901), "zero", 3, True),
    (np.float64, "star", 3, (911, 2881), "zero", 3, False), (np.float64, "star", 3, (911, 2881), "zero", 9, False),
    (np.float64, "star", 3, (911, 2881), "zero", 10, True), (np.float64, "star", 3, (911, 2881), "clamp", 3, False),
    # rows of whole 16-byte pieces, where the marching kernels are faster: 1900x1900, three sweeps, 1.22 times there
    (np.float32, "star", 1, (1900, 1900), "zero", 3, False), (np.float32, "star", 1, (500, 500), "zero", 3, True),
    (np.float32, "box", 1, (2208, 2656), "zero", 2, False), (np.float32, "box", 1, (2208, 2657), "zero", 2, True),
    (np.float32, "box", 1, (2208, 2656), "clamp", 2, False), (np.float32, "box", 1, (2208, 2656), "clamp", 5, True),
    (np.float32, "star", 1, (1568, 5600), "zero", 4, False), (np.float32, "star", 1, (1568, 5601), "zero", 4, True),
    (np.float32, "star", 1, (1568, 5600), "clamp", 4, True), (np.float64, "box", 1, (2048, 2176), "clamp", 2, False),
    (np.float64, "box", 1, (2048, 2177), "clamp", 2, True), (np.float64, "box", 1, (3000, 3000), "zero", 8, False),
    (np.float64, "star", 3, (1200, 1200), "zero", 6, False), (np.float64, "star", 3, (1200, 1201), "zero", 6, True),
])
def test_few_sweeps_on_larger_grids(dtype, kind, r, shape, boundary, remaining, tile):
    """Where the marching kernels do all that remains in launches of their best depth."""
    import paper_1907_06154_amd as ssam
    name = ssam.ssam_describe("iterate2d", shape, coefficients(kind, r, dtype), boundary, remaining=remaining).split()[0]
    assert ("_tile_" in name) == tile


@pytest.mark.parametrize("shape,remaining,tile", [((860, 1954), 3, False), ((289, 5810), 9, False), ((774, 2240), 4, False), ((1510, 1120), 8, False),
                                                  ((900, 900), 4, True), ((1200, 1000), 4, True), ((1500, 1400), 4, True), ((2000, 2000), 3, True),
                                                  ((1500, 1400), 200, True), ((774, 2240), 200, False)])
def test_plans_of_the_fp64_box_of_radius_3(shape, remaining, tile):
    """Single sweeps where their waves fill the chip once."""
    import paper_1907_06154_amd as ssam
    name = ssam.ssam_describe("iterate2d", shape, coefficients("box", 3, np.float64), "zero", remaining=remaining).split()[0]
    assert ("_tile_" in name) == tile


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_one_tile_along_an_axis(dtype):
    import paper_1907_06154_amd as ssam
    for kind, r in (("star", 1), ("star", 3), ("star", 6), ("box", 2)):
        coef = coefficients(kind, r, dtype)
        for shape in ((16, 64), (16, 500), (32, 256), (48, 300), (64, 128), (300, 64), (200, 128), (150, 256)):
            fld = wl.uniform_field(shape, -1.0, 1.0, 710 + shape[1], dtype)
            for boundary in ("zero", "clamp"):
                for steps in (3, 17, 40):
                    print(f"one tile {np.dtype(dtype).name} {kind} r{r} {shape} {boundary} steps {steps}", flush=True)
                    a = torch.from_numpy(fld).cuda()
                    got = ssam.ssam_stencil_iterate(a, torch.full_like(a, float("nan")), coef, steps, boundary)
                    assert_parity(got.cpu().numpy(), oracle.iterate(fld, coef, steps, boundary), coef, 1.0,
                                  f"{kind} r{r} {shape} {boundary} steps {steps}")


@pytest.mark.gpu
def test_many_sweeps():
    """A plan kept for the launches of one iteration, and the plans of its rest."""
    import paper_1907_06154_amd as ssam
    for dtype, shape, steps in ((np.float32, (131, 449), 200), (np.float64, (70, 129), 131)):
        coef = coefficients("star", 1, dtype)
        fld = wl.uniform_field(shape, -1.0, 1.0, 77, dtype)
        for boundary in ("zero", "clamp"):
            print(f"many sweeps {np.dtype(dtype).name} {shape} {boundary} {steps}", flush=True)
            a = torch.from_numpy(fld).cuda()
            got = ssam.ssam_stencil_iterate(a, torch.empty_like(a), coef, steps, boundary)
            assert_parity(got.cpu().numpy(), oracle.iterate(fld, coef, steps, boundary), coef, 1.0, f"{shape} {boundary} {steps}")


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("kind,r", SHAPES)
def test_matches_oracle(dtype, kind, r):
    import paper_1907_06154_amd as ssam
    coef = coefficients(kind, r, dtype)
    for shape in GRIDS:
        fld = wl.uniform_field(shape, -1.0, 1.0, 700 + shape[1], dtype)
        n = fld.size
        for boundary in ("zero", "clamp"):
            for steps in (2, 3, 7, 20):
                print(f"tile {np.dtype(dtype).name} {kind} r{r} {shape} {boundary} steps {steps}", flush=True)
                buf = torch.full((2, n + 8), float("nan"), dtype=torch.from_numpy(fld).dtype, device="cuda")
                a, b = buf[0][1:n + 1].view(shape), buf[1][3:n + 3].view(shape)     # not aligned to a vector
                a.copy_(torch.from_numpy(fld))
                got = ssam.ssam_stencil_iterate(a, b, coef, steps, boundary)
                assert_parity(got.cpu().numpy(), oracle.iterate(fld, coef, steps, boundary), coef, 1.0,
                              f"{kind} r{r} {shape} {boundary} steps {steps}")
                guard = torch.cat([buf[0][:1], buf[0][n + 1:], buf[1][:3], buf[1][n + 3:]])
                assert torch.isnan(guard).all()


# grids of up to one and a half million points: blocks of twelve and sixteen waves, more than 64 KB of LDS
TALL = [(1437, 191), (903, 913), (145, 105), (2995, 371), (271, 1511), (390, 263), (1792, 751), (2219, 593), (2901, 505)]
ALL_SHAPES = [("star", r) for r in range(1, 7)] + [("box", r) for r in range(1, 5)]


def tall_blocks(kind, r, dtype):
    """(V, waves, boundary) of a launch -> the first of those grids, and the number of sweeps, that has it."""
    import paper_1907_06154_amd as ssam
    found = {}
    for shape in TALL:
        for steps, boundary in ((5, "zero"), (12, "clamp"), (5, "clamp"), (12, "zero")):
            text = ssam.ssam_describe("iterate2d", shape, coefficients(kind, r, dtype), boundary, remaining=steps)
            if "_tile_" in text:
                V, tiles, blocks = (int(re.search(rf" {name}=(\d+)", text).group(1)) for name in ("V", "tiles", "blocks"))
                found.setdefault((V, tiles // blocks, boundary), (shape, steps))
    return found


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("kind,r", ALL_SHAPES)
def test_tall_blocks_are_reached(dtype, kind, r):
    found = tall_blocks(kind, r, dtype)
    if kind == "box" and r > 2 and dtype == np.float32:      # single sweeps on the split kernel
        assert not found
        return
    widths = [1] if (kind, r) == ("box", 4) else [1, 2] if dtype == np.float64 else [1, 2, 4]
    assert set(found) >= {(V, waves, boundary) for V in widths for waves in (12, 16) for boundary in ("zero", "clamp")}


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("kind,r", ALL_SHAPES)
def test_tall_blocks(dtype, kind, r):
    import paper_1907_06154_amd as ssam
    coef = coefficients(kind, r, dtype)
    for (V, waves, boundary), (shape, steps) in tall_blocks(kind, r, dtype).items():
        print(f"tall {np.dtype(dtype).name} {kind} r{r} {shape} {boundary} steps {steps} V {V} waves {waves}", flush=True)
        fld = wl.uniform_field(shape, -1.0, 1.0, 750 + shape[1], dtype)
        a = torch.from_numpy(fld).cuda()
        got = ssam.ssam_stencil_iterate(a, torch.full_like(a, float("nan")), coef, steps, boundary)
        assert_parity(got.cpu().numpy(), oracle.iterate(fld, coef, steps, boundary), coef, 1.0, f"{kind} r{r} {shape} {boundary} steps {steps}")


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("kind,r", [("star", 1), ("star", 2), ("star", 4), ("star", 6), ("box", 1), ("box", 2)])
@pytest.mark.parametrize("boundary", ["zero", "clamp"])
def test_infinities_and_nan_stay_apart(dtype, kind, r, boundary):
    """They reach the points the sweeps carry them to and no others, at the grid's edges, which the clamp rule repeats, and beside a
    tile's rim, which every tile sees repeated."""
    import paper_1907_06154_amd as ssam
    coef, shape, steps = coefficients(kind, r, dtype), (150, 700), 6
    assert "_tile_" in ssam.ssam_describe("iterate2d", shape, coef, boundary, remaining=steps)
    ys, xs = np.mgrid[0:shape[0], 0:shape[1]]
    for value in (np.inf, np.nan):
        for at in ([(0, 0), (75, 350), (149, 699)], [(0, 300), (60, 0)], [(149, 128), (100, 699), (33, 64)]):
            fld = np.zeros(shape, dtype=dtype)
            near = np.zeros(shape, dtype=bool)
            for y, x in at:
                fld[y, x] = value
                dy, dx = (-(-np.abs(d) // r) for d in (ys - y, xs - x))      # sweeps to cover the distance along each axis
                near |= (dy + dx if kind == "star" else np.maximum(dy, dx)) <= steps
            a = torch.from_numpy(fld).cuda()
            got = ssam.ssam_stencil_iterate(a, torch.empty_like(a), coef, steps, boundary).cpu().numpy()
            assert np.array_equal(~np.isfinite(got), near) and not got[~near].any(), (value, at)


@pytest.mark.gpu
def test_zero_padding_keeps_infinities_apart():
    """An infinity reaches the points the sweeps carry it to and no others, at the grid's edge and beside a tile's rim."""
    import paper_1907_06154_amd as ssam
    coef = coefficients("star", 1, np.float32)
    fld = np.zeros((140, 300), dtype=np.float32)
    for y, x in ((0, 0), (70, 150), (139, 299)):
        fld[y, x] = np.inf
    a = torch.from_numpy(fld).cuda()
    got = ssam.ssam_stencil_iterate(a, torch.empty_like(a), coef, 6, "zero").cpu().numpy()
    ys, xs = np.mgrid[0:140, 0:300]
    near = np.zeros(fld.shape, dtype=bool)
    for y, x in ((0, 0), (70, 150), (139, 299)):
        near |= np.abs(ys - y) + np.abs(xs - x) <= 6
    assert np.array_equal(~np.isfinite(got), near) and not got[~near].any()
