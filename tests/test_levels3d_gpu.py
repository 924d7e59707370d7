"""Sweeps as levels of one march along z: grids of exactly one tile, one row or column more, and tiles moved back from the grid's
end, in every vector width; few planes, many; buffers aligned to the element only; against the CPU oracle."""
import re

import numpy as np
import pytest

import oracle
import workloads as wl
from parity_util import assert_parity

torch = pytest.importorskip("torch")

# (D, H, W), all of more than 2^18 points
GRIDS = [(257, 16, 64), (251, 17, 65), (65, 32, 128), (34, 61, 129), (33, 64, 130), (11, 100, 257), (5, 230, 300), (2, 400, 400),
         (1, 600, 500), (70, 90, 96)]
MASKS = {"star": wl.mask_star(1, 1, 1), "faces_edges": wl.mask_faces_edges(), "box": wl.mask_box(1, 1, 1)}


def plan(ssam, shape, coef, boundary):
    return ssam.ssam_describe("iterate3d", shape, coef, boundary).split()[0]


def test_plans():
    import paper_1907_06154_amd as ssam
    for kind, mask in MASKS.items():
        for dtype in (np.float32, np.float64):
            coef = wl.seeded_coefficients(mask, 90, dtype)
            assert "_levels_" in plan(ssam, (64, 64, 128), coef, "clamp")
            assert "_levels_" not in plan(ssam, (64, 64, 64), coef, "zero")       # 2^18 points
            assert "_levels_" not in plan(ssam, (300, 15, 128), coef, "zero")     # fewer rows than four waves'
            assert "_levels_" not in plan(ssam, (128, 128, 63), coef, "zero")     # narrower than a wave


def test_plans_of_large_grids():
    """19 and 27 points: single sweeps are no faster on grids of many points, under either rule, where tiles are filled."""
    import paper_1907_06154_amd as ssam
    for kind in ("faces_edges", "box"):
        for shape in ((420, 410, 400), (509, 511, 510), (320, 640, 640), (384, 384, 768)):
            for boundary in ("zero", "clamp"):
                assert "_levels_fused2" in plan(ssam, shape, wl.seeded_coefficients(MASKS[kind], 95, np.float64), boundary), (kind, shape, boundary)
    box = wl.seeded_coefficients(MASKS["box"], 95, np.float32)
    assert "_levels_" in plan(ssam, (416, 450, 444), box, "clamp") and "_levels_" not in plan(ssam, (509, 511, 510), box, "clamp")


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,kind", [(np.float64, "box"), (np.float64, "faces_edges"), (np.float32, "faces_edges")])
def test_a_large_grid(dtype, kind):
    import paper_1907_06154_amd as ssam
    shape, coef = (410, 407, 403), wl.seeded_coefficients(MASKS[kind], 95, dtype)
    assert "_levels_fused2" in plan(ssam, shape, coef, "clamp")
    fld = wl.uniform_field(shape, -1.0, 1.0, 98, dtype)
    a = torch.from_numpy(fld).cuda()
    got = ssam.ssam_stencil_iterate(a, torch.empty_like(a), coef, 2, "clamp").cpu().numpy()
    assert_parity(got, oracle.iterate(fld, coef, 2, "clamp"), coef, 1.0, f"{kind} {shape}")


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("kind", list(MASKS))
def test_matches_oracle(dtype, kind):
    import paper_1907_06154_amd as ssam
    coef = wl.seeded_coefficients(MASKS[kind], 91, dtype)
    for shape in GRIDS:
        fld = wl.uniform_field(shape, -1.0, 1.0, 900 + shape[2], dtype)
        n = fld.size
        for boundary in ("zero", "clamp"):
            for steps, skew in ((2, 0), (3, 1), (4, 0), (7, 1)):
                print(f"levels {np.dtype(dtype).name} {kind} {shape} {boundary} steps {steps}", flush=True)
                buf = torch.full((2, n + 8), float("nan"), dtype=torch.from_numpy(fld).dtype, device="cuda")
                a, b = buf[0][skew:n + skew].view(shape), buf[1][3 * skew:n + 3 * skew].view(shape)
                a.copy_(torch.from_numpy(fld))
                got = ssam.ssam_stencil_iterate(a, b, coef, steps, boundary)
                assert_parity(got.cpu().numpy(), oracle.iterate(fld, coef, steps, boundary), coef, 1.0,
                              f"{kind} {shape} {boundary} steps {steps}")
                guard = torch.cat([buf[0][:skew], buf[0][n + skew:], buf[1][:3 * skew], buf[1][n + 3 * skew:]])
                assert torch.isnan(guard).all()


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
def test_every_tile_width_with_its_halo(dtype):
    """Three sweeps on grids whose last tiles end one column after the others: each width's tiles with the least overlap."""
    import paper_1907_06154_amd as ssam
    coef = wl.seeded_coefficients(MASKS["star"], 92, dtype)
    for shape in ((200, 150, 300), (60, 70, 361), (48, 130, 241), (90, 59, 177)):
        fld = wl.uniform_field(shape, -1.0, 1.0, 93, dtype)
        a = torch.from_numpy(fld).cuda()
        got = ssam.ssam_stencil_iterate(a, torch.empty_like(a), coef, 3, "zero").cpu().numpy()
        assert_parity(got, oracle.iterate(fld, coef, 3, "zero"), coef, 1.0, f"{shape}")


# Grids that reach every kernel the planner picks: pieces of 8 bytes and of 16, four waves a block and eight, streaming stores
# beyond the caches, two sweeps and three of the star.
EVERY = {np.float32: [(24, 79, 139), (8, 520, 267), (17, 474, 132), (150, 65, 257), (69, 85, 256), (115, 21, 372), (70, 25, 412), (100, 222, 384),
                      (77, 198, 484), (44, 622, 388), (481, 74, 256), (408, 138, 448), (291, 208, 417)],
         np.float64: [(33, 82, 97), (100, 37, 71), (11, 423, 69), (201, 203, 199), (6, 236, 370), (54, 22, 238), (35, 311, 430), (12, 575, 494),
                      (127, 54, 410), (15, 472, 386), (81, 519, 300), (206, 169, 363), (70, 415, 434), (127, 424, 234)]}


def every_kernel(kind, dtype):
    """(V, waves, sweeps, boundary, streaming) of a launch -> the first of those grids that has it."""
    import paper_1907_06154_amd as ssam
    coef, elem, found = wl.seeded_coefficients(MASKS[kind], 96, dtype), np.dtype(dtype).itemsize, {}
    for shape in EVERY[dtype]:
        for boundary in ("zero", "clamp"):
            for remaining in (2, 3) if kind == "star" else (2,):
                text = ssam.ssam_describe("iterate3d", shape, coef, boundary, remaining=remaining)
                if "_levels_" not in text:
                    continue
                V, lds = (int(re.search(rf" {name}=(\d+)", text).group(1)) for name in ("V", "lds"))
                sweeps = int(re.search(r"_levels_fused(\d)", text).group(1))
                waves = (lds // (2 * sweeps * 64 * V * elem) - 1) // 2
                stream = V * elem == 16 and waves == 8 and 2 * np.prod(shape) * elem > 192 << 20
                found.setdefault((V, waves, sweeps, boundary, bool(stream)), shape)
    return found


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("kind", list(MASKS))
def test_every_kernel_is_reached(dtype, kind):
    V16 = 16 // np.dtype(dtype).itemsize
    found = every_kernel(kind, dtype)
    assert set(found) >= {(V, waves, sweeps, boundary, stream) for V in (V16 // 2, V16) for waves in (4, 8) for sweeps in ((2, 3) if kind == "star" else (2,))
                          for boundary in ("zero", "clamp") for stream in ((False, True) if (V, waves) == (V16, 8) else (False,))}


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("kind", list(MASKS))
def test_every_kernel(dtype, kind):
    import paper_1907_06154_amd as ssam
    coef = wl.seeded_coefficients(MASKS[kind], 96, dtype)
    for (V, waves, sweeps, boundary, stream), shape in every_kernel(kind, dtype).items():
        print(f"kernel {np.dtype(dtype).name} {kind} {shape} {boundary} sweeps {sweeps} V {V} waves {waves} stream {stream}", flush=True)
        fld = wl.uniform_field(shape, -1.0, 1.0, 97, dtype)
        a = torch.from_numpy(fld).cuda()
        got = ssam.ssam_stencil_iterate(a, torch.full_like(a, float("nan")), coef, sweeps, boundary).cpu().numpy()
        assert_parity(got, oracle.iterate(fld, coef, sweeps, boundary), coef, 1.0, f"{kind} {shape} {boundary} sweeps {sweeps}")


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("kind", list(MASKS))
@pytest.mark.parametrize("boundary", ["zero", "clamp"])
def test_infinities_and_nan_stay_apart(dtype, kind, boundary):
    """They reach the points the sweeps carry them to and no others: at the grid's corners and edges, which the clamp rule repeats,
    beside a tile's rim, which every tile sees repeated, and beside the first and last planes of a chunk."""
    import paper_1907_06154_amd as ssam
    coef, steps = wl.seeded_coefficients(MASKS[kind], 94, dtype), 5
    for shape in ((40, 70, 140), (61, 130, 193)):
        assert "_levels_" in plan(ssam, shape, coef, boundary)
        grid = np.indices(shape)
        D, H, W = shape
        for value in (np.inf, np.nan):
            for at in (((0, 0, 0), (D - 1, H - 1, W - 1), (D // 2, H // 2, W // 2)), ((0, H // 2, 62), (20, 0, 124), (D - 1, 31, 0)),
                       ((10, 30, W - 1), (9, H - 1, 60), (30, 5, 64))):
                fld = np.zeros(shape, dtype=dtype)
                near = np.zeros(shape, dtype=bool)
                for p in at:
                    fld[p] = value
                    d = [np.abs(g - c) for g, c in zip(grid, p)]
                    far, total = np.maximum(np.maximum(d[0], d[1]), d[2]), d[0] + d[1] + d[2]
                    near |= (total <= steps) if kind == "star" else (far <= steps) & (total <= (2 if kind == "faces_edges" else 3) * steps)
                a = torch.from_numpy(fld).cuda()
                got = ssam.ssam_stencil_iterate(a, torch.empty_like(a), coef, steps, boundary).cpu().numpy()
                assert np.array_equal(~np.isfinite(got), near) and not got[~near].any(), (shape, value, at)


@pytest.mark.gpu
def test_zero_padding_keeps_infinities_apart():
    """An infinity reaches the points the sweeps carry it to and no others: at the grid's corners and beside a tile's rim."""
    import paper_1907_06154_amd as ssam
    coef = wl.seeded_coefficients(MASKS["star"], 94, np.float32)
    shape = (40, 70, 140)
    at = ((0, 0, 0), (39, 69, 139), (20, 30, 62), (0, 35, 124))
    fld = np.zeros(shape, dtype=np.float32)
    grid = np.indices(shape)
    near = np.zeros(shape, dtype=bool)
    for p in at:
        fld[p] = np.inf
        near |= sum(np.abs(g - c) for g, c in zip(grid, p)) <= 5
    a = torch.from_numpy(fld).cuda()
    got = ssam.ssam_stencil_iterate(a, torch.empty_like(a), coef, 5, "zero").cpu().numpy()
    assert np.array_equal(~np.isfinite(got), near) and not got[~near].any()
