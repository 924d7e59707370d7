"""How many sweeps of a 2D iteration one launch of the marching kernels does: the plan on the CPU, the deepest instances against the
CPU oracle on the GPU."""
import re

import numpy as np
import pytest

import oracle
import workloads as wl
from parity_util import assert_parity

torch = pytest.importorskip("torch")
import paper_1907_06154_amd.binding as ssam  # noqa: E402


def coefficients(kind, r, dtype, seed=1100):
    mask = wl.mask_box(r, r) if kind == "box" else wl.mask_star(r, r)
    return wl.seeded_coefficients(mask, seed + r, dtype)[0]


def depth(shape, coef, boundary, remaining):
    m = re.search(r"_fused(\d+)$", ssam.ssam_describe("iterate2d", shape, coef, boundary, remaining=remaining).split()[0])
    return int(m.group(1)) if m else 1


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("kind,r", [("box", 1), ("star", 1), ("box", 2), ("star", 2), ("star", 3), ("star", 4), ("star", 5), ("star", 6)])
def test_depths_take_no_more_launches_than_the_deepest_first(dtype, kind, r):
    coef = coefficients(kind, r, dtype)
    for shape in ((8192, 8192), (8191, 8001), (6000, 4100)):
        for boundary in ("zero", "clamp"):
            depths = {s for s in range(2, 9) if depth(shape, coef, boundary, s) == s}
            for steps in list(range(1, 34)) + [50, 100]:
                got, t = [], 0
                while t < steps:
                    got.append(depth(shape, coef, boundary, steps - t))
                    t += got[-1]
                assert t == steps and all(d == 1 or d in depths for d in got)
                count, n = 0, steps
                while n:
                    n -= max([d for d in depths if d <= n], default=1)
                    count += 1
                assert len(got) == count, (kind, r, shape, boundary, steps, got)


@pytest.mark.parametrize("kind,r,dtype,boundary,steps,want", [("star", 1, np.float32, "zero", 7, [6, 1]), ("star", 1, np.float32, "zero", 13, [6, 6, 1]),
                                                               ("star", 1, np.float32, "clamp", 7, [4, 3]), ("star", 1, np.float64, "zero", 7, [6, 1]),
                                                               ("star", 2, np.float64, "clamp", 9, [4, 4, 1])])
def test_a_single_sweep_left_over(kind, r, dtype, boundary, steps, want):
    """Where launches are bound by memory one sweep left over is cheaper than a share of a launch."""
    coef, got = coefficients(kind, r, dtype), []
    while sum(got) < steps:
        got.append(depth((7168, 3239), coef, boundary, steps - sum(got)))
    assert got == want


@pytest.mark.parametrize("kind,r,dtype", [("box", 2, np.float64), ("star", 2, np.float32), ("star", 3, np.float32), ("box", 2, np.float32)])
def test_depths_without_pairs(kind, r, dtype):
    """Below 2^22 points pairs of sweeps have no launch of their own: the fewest launches are not always those of the deepest first."""
    coef = coefficients(kind, r, dtype)
    ssam.ssam_set_tuning("variant", 0)             # the marching kernels
    try:
        for steps, want in ((5, [4, 1]), (6, [3, 3]), (9, [3, 3, 3]), (10, [3, 4, 3]), (13, [4, 3, 3, 3])):
            got, t = [], 0
            while t < steps:
                got.append(depth((1500, 2500), coef, "zero", steps - t))
                t += got[-1]
            assert got == want, (steps, got)
    finally:
        ssam.ssam_set_tuning("variant", -1)


@pytest.mark.parametrize("kind,r,dtype,depths", [("box", 2, np.float64, (2, 3, 4)), ("star", 1, np.float64, (2, 3, 4, 6, 8)),
                                                 ("star", 3, np.float32, (2, 3, 4)), ("star", 4, np.float64, (2, 3))])
def test_a_cap_limits_the_depth_and_not_the_sweeps_that_remain(kind, r, dtype, depths):
    coef = coefficients(kind, r, dtype)
    try:
        for cap in range(2, 10):
            ssam.ssam_set_tuning("fuse_sweeps", cap)
            assert depth((8192, 8192), coef, "zero", 100) == max(d for d in depths if d <= cap), cap
            assert depth((300, 400), coef, "zero", 100) <= cap                      # tiles
            star = wl.seeded_coefficients(wl.mask_star(1, 1, 1), 1131, np.float64)
            m = re.search(r"_levels_fused(\d+)$", ssam.ssam_describe("iterate3d", (200, 200, 200), star, "zero", remaining=100).split()[0])
            assert int(m.group(1)) == min(cap, 3)
    finally:
        ssam.ssam_set_tuning("fuse_sweeps", -1)


def check(shape, coef, boundary, steps, rows):
    fld = wl.uniform_field(shape, -1.0, 1.0, 1110 + shape[0], np.float64)
    print(f"depth {coef.shape} {shape} {boundary} rows {rows} steps {steps}", flush=True)
    ssam.ssam_set_tuning("rows_per_wave", rows)
    try:
        a = torch.from_numpy(fld).cuda()
        res = ssam.ssam_stencil_iterate(a, torch.full_like(a, float("nan")), coef, steps, boundary)
    finally:
        ssam.ssam_set_tuning("rows_per_wave", -1)
    assert_parity(res.cpu().numpy(), oracle.iterate(fld, coef, steps, boundary), coef, 1.0, f"{coef.shape} {shape} {boundary} {rows} {steps}")


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("kind,r", [("box", 1), ("star", 1), ("box", 2), ("star", 2), ("star", 3), ("star", 4), ("star", 5), ("star", 6)])
def test_marching_kernels_on_small_grids(dtype, kind, r):
    """The tile kernel takes these grids by itself; variant 0 names the marching kernels' own default: every depth, several tiles,
    ragged tails, rows that are not whole vectors."""
    coef = coefficients(kind, r, dtype)
    for shape in ((33, 224), (37, 113), (37, 449), (70, 300), (131, 449), (150, 1000), (260, 96)):
        fld = wl.uniform_field(shape, -1.0, 1.0, 1120 + shape[0], dtype)
        for boundary in ("zero", "clamp"):
            for steps in (2, 3, 4, 6, 7, 9):
                want = oracle.iterate(fld, coef, steps, boundary)
                for fuse in (-1, 2, 3):
                    print(f"marching {np.dtype(dtype).name} {kind} r{r} {shape} {boundary} steps {steps} fuse {fuse}", flush=True)
                    ssam.ssam_set_tuning("variant", 0)
                    ssam.ssam_set_tuning("fuse_sweeps", fuse)
                    try:
                        left, depths = steps, []
                        while left:
                            name = ssam.ssam_describe("iterate2d", shape, coef, boundary, remaining=left).split()[0]
                            depths.append(int((re.search(r"_fused(\d+)$", name) or [0, 1])[1]))
                            assert "_tile_" not in name
                            left -= depths[-1]
                        a = torch.from_numpy(fld).cuda()
                        res = ssam.ssam_stencil_iterate(a, torch.full_like(a, float("nan")), coef, steps, boundary)
                    finally:
                        ssam.ssam_set_tuning("variant", -1)
                        ssam.ssam_set_tuning("fuse_sweeps", -1)
                    assert fuse < 0 and (steps == 2 or r > 4) or max(depths) > 1, (shape, boundary, steps, fuse, depths)
                    assert_parity(res.cpu().numpy(), want, coef, 1.0, f"{kind} r{r} {shape} {boundary} steps {steps} fuse {fuse}")


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(5, 9), (33, 112), (61, 257), (97, 450), (130, 301)])
def test_eight_sweeps_two_rows_a_group(shape):
    """Tiles of a few rows, tails, rows that are not whole vectors, grids smaller than the halo."""
    coef = coefficients("star", 1, np.float64)
    for boundary in ("zero", "clamp"):
        for rows in (2, 24, 64):
            for steps in (8, 9):
                check(shape, coef, boundary, steps, rows)


@pytest.mark.gpu
@pytest.mark.parametrize("r,S", [(2, 6), (3, 4), (5, 3)])
@pytest.mark.parametrize("shape,boundary", [((3001, 3007), "zero"), ((2999, 3202), "zero"), ((7001, 7203), "clamp"), ((7103, 7202), "clamp")])
def test_deepest_instances_on_the_smallest_grids_that_take_them(r, S, shape, boundary):
    coef = coefficients("star", r, np.float64)
    assert (depth(shape, coef, boundary, S) == S) == (boundary == "zero" or r != 2)
    for rows in (-1, 8):
        if boundary == "zero" or rows < 0:
            check(shape, coef, boundary, S, rows)


def test_smaller_grids_keep_the_shallower_instances():
    for r, S in ((2, 6), (3, 4), (5, 3)):
        coef = coefficients("star", r, np.float64)
        assert depth((2999, 2999), coef, "zero", S) < S and depth((7000, 7001), coef, "clamp", S) < S


@pytest.mark.parametrize("steps,want", [(1, [1]), (2, [2]), (3, [3]), (4, [2, 2]), (10, [3, 3, 2, 2])])
def test_plan_of_a_3d_iteration(steps, want):
    coef = wl.seeded_coefficients(wl.mask_star(1, 1, 1), 1130, np.float64)
    got, t = [], 0
    while t < steps:
        m = re.search(r"_fused(\d+)$", ssam.ssam_describe("iterate3d", (512, 512, 512), coef, "zero", remaining=steps - t).split()[0])
        got.append(int(m.group(1)) if m else 1)
        t += got[-1]
    assert got == want
