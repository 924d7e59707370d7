"""Dense fp32 filters on the bf16 matrix cores (every value as the exact sum of three bf16 values) against the CPU
oracle, at the sizes where the kernel can go wrong: patch widths around whole pieces of eight columns and around the
four-column tail piece, every band count, filters evaluated in several launches, strips of one to three 64-column parts
with ragged right edges, tiles of one band, the smallest width, anchors at the corners.

Tolerance, in units of sum|w| * max|in|: one rounding of 2^-24 per table piece added to a sum (at most 30), the sums of 32
products inside an instruction (at most 32 more), and less than 2^-24 for the partial products left out."""
import numpy as np
import pytest

import oracle
import workloads as wl
from parity_util import normalised_error

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

TOL = (30 + 32 + 1) * 2.0 ** -24


@pytest.fixture(scope="module")
def ssam():
    import paper_1907_06154_amd as s
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    s.lib()
    yield s
    s.ssam_set_tuning("rows_per_wave", -1)


def run(ssam, img, filt, boundary, anchor=None):
    out = ssam.ssam_conv2d(torch.from_numpy(img).cuda(), filt, boundary, anchor)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def name_of(ssam, img, filt, boundary):
    return ssam.ssam_describe("conv2d", img.shape, filt, boundary).split()[0]


@pytest.mark.parametrize("M,N", [(8, 8), (9, 9), (8, 1), (1, 8), (13, 5), (14, 13), (17, 16), (18, 17), (20, 20), (21, 21),
                                 (5, 21), (22, 22), (30, 9), (29, 14), (32, 32)])
@pytest.mark.parametrize("boundary", ["clamp", "zero"])
def test_shapes_and_edges(ssam, M, N, boundary):
    filt = wl.seeded_filter(M, N, 900 + 32 * M + N, np.float32)
    for k, (H, W) in enumerate([(256, 64), (127, 131), (90, 193), (33, 515), (3, 6000)]):
        img = wl.uniform_field((H, W), -1.0, 1.0, 910 + k, np.float32)
        anchor = [None, (0, 0), (M - 1, N - 1)][k % 3]
        print(f"split {M}x{N} {boundary} {H}x{W} anchor {anchor}", flush=True)
        assert "split3mx" in name_of(ssam, img, filt, boundary)
        got = run(ssam, img, filt, boundary, anchor)
        err = normalised_error(got, oracle.conv2d(img, filt, boundary, anchor), filt, 1.0)
        assert err <= TOL, (M, N, boundary, H, W, err)


@pytest.mark.parametrize("rows", [4, 8, 20, 36])
def test_tile_heights(ssam, rows):
    """Tiles shorter and taller than the filter: the steps above, inside and below a tile."""
    img = wl.uniform_field((150, 260), -1.0, 1.0, 930, np.float32)
    ssam.ssam_set_tuning("rows_per_wave", rows)
    try:
        for M, N in ((9, 9), (8, 21), (12, 3)):
            filt = wl.seeded_filter(M, N, 931, np.float32)
            print(f"split rows {rows} {M}x{N}", flush=True)
            err = normalised_error(run(ssam, img, filt, "zero"), oracle.conv2d(img, filt, "zero"), filt, 1.0)
            assert err <= TOL, (rows, M, N, err)
    finally:
        ssam.ssam_set_tuning("rows_per_wave", -1)


@pytest.mark.parametrize("M", [9, 20, 25])
def test_values_the_split_does_not_carry(ssam, M):
    """Infinities, NaN and very large inputs: the outputs in their reach are those of plain multiply-adds, every other
    output is untouched.  Tiny inputs keep their precision."""
    filt = wl.seeded_filter(M, M, 940, np.float32)
    img = wl.uniform_field((140, 300), -1.0, 1.0, 941, np.float32)
    clean = run(ssam, img, filt, "clamp")
    for value in (np.inf, -np.inf, np.nan, 1e30, -3e38):
        for y, x in ((70, 150), (0, 0), (139, 299), (64, 191)):
            dirty = img.copy()
            dirty[y, x] = value
            print(f"split {M} value {value} at {y},{x}", flush=True)
            got, want = run(ssam, dirty, filt, "zero"), oracle.conv2d(dirty, filt, "zero")
            with np.errstate(invalid="ignore"):
                assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want))
                fine = np.isfinite(want)
                tol = M * M * 2.0 ** -24 * (np.abs(filt).sum() + (abs(value) * np.abs(filt).max() if np.isfinite(value) else 0.0) *
                                            (np.abs(want) > 1e3))
            assert np.all(np.abs(got[fine].astype(np.float64) - want[fine]) <= np.broadcast_to(tol, want.shape)[fine])
    assert np.array_equal(run(ssam, img, filt, "clamp"), clean)
    for scale in (2.0 ** -100, 2.0 ** -60, 2.0 ** 60):      # exact powers of two change nothing but the exponent
        got = run(ssam, img * np.float32(scale), filt, "clamp")
        assert np.array_equal(got, clean * np.float32(scale)), scale


def assert_footprint(got, want, filt, value, what):
    """Non-finite results exactly where the oracle has them; everything else to the rounding of the filter's sum,
    outputs that read `value` itself to that of `value` times a weight."""
    assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want)), what
    fine = np.isfinite(want)
    tol = filt.size * 2.0 ** -24 * np.abs(filt).sum() * np.where(np.abs(want) > 1e3, abs(value), 1.0) if np.isfinite(value) else \
        np.full(want.shape, filt.size * 2.0 ** -24 * np.abs(filt).sum())
    assert np.all(np.abs(got[fine].astype(np.float64) - want[fine]) <= tol[fine]), what


@pytest.mark.parametrize("M,anchor", [(8, None), (14, None), (16, (0, 0)), (17, None), (25, (24, 0)), (32, None), (9, (0, 0)), (15, (14, 0))])
def test_one_row_filters_and_the_band_above(ssam, M, anchor):
    """Filters of one row whose last columns form a tail piece (two bands to a piece): a value above an output that
    its filter does not read stays out of it, whatever it is (2.1e31 is infinite once it is scaled)."""
    filt = wl.seeded_filter(M, 1, 945 + M, np.float32)
    img = wl.uniform_field((130, 300), -1.0, 1.0, 946, np.float32)
    if anchor is None:
        assert "split3mx" in name_of(ssam, img, filt, "zero")
    ssam.ssam_set_tuning("rows_per_wave", 24)       # several bands to a wave
    try:
        for value in (np.inf, np.nan, 2.1e31, -3e38):
            for y, x in ((70, 150), (0, 0), (129, 299), (67, 191)):
                dirty = img.copy()
                dirty[y, x] = value
                print(f"split {M}x1 value {value} at {y},{x}", flush=True)
                with np.errstate(invalid="ignore", over="ignore"):
                    assert_footprint(run(ssam, dirty, filt, "zero", anchor), oracle.conv2d(dirty, filt, "zero", anchor), filt, value, (y, x))
    finally:
        ssam.ssam_set_tuning("rows_per_wave", -1)


def test_filters_of_any_scale(ssam):
    img = wl.uniform_field((140, 300), -1.0, 1.0, 951, np.float32)
    filt = wl.seeded_filter(10, 10, 952, np.float32)
    base = run(ssam, img, filt, "zero")
    for e in (-80, 80):
        assert np.array_equal(run(ssam, img, filt * np.float32(2.0 ** e), "zero"), base * np.float32(2.0 ** e))
    # beyond the kernel's range, not finite, or nothing but zeros: the other kernels take the filter
    for f in (filt * np.float32(2.0 ** 100), filt * np.float32(2.0 ** -100), np.zeros_like(filt)):
        assert "split3mx" not in name_of(ssam, img, f, "zero")
        want = oracle.conv2d(img, f, "zero")
        assert normalised_error(run(ssam, img, f, "zero"), want, f, 1.0) <= TOL


def test_capture_and_replay(ssam):
    """A filter evaluated in several launches, recorded in a graph: every replay gives the eager result."""
    filt = wl.seeded_filter(25, 25, 960, np.float32)
    a = torch.from_numpy(wl.uniform_field((300, 400), 0.0, 1.0, 961, np.float32)).cuda()
    out = torch.empty_like(a)
    eager = ssam.ssam_conv2d(a, filt, "clamp").cpu().numpy()
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
        ssam.ssam_conv2d(a, filt, "clamp", d_out=out)
    for replay in range(3):
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), eager), replay
        assert np.array_equal(ssam.ssam_conv2d(a, filt, "clamp").cpu().numpy(), eager)


# ---- three dimensions -------------------------------------------------------------------------------------------------
# One rounding per chain added to a sum (at most 28), up to 18 inside a chain, the sums of 32 products inside an
# instruction, the parts of a filter added up in the output (at most 8), the partial products left out.
TOL3 = (28 + 18 + 32 + 8 + 1) * 2.0 ** -24


def run3(ssam, vol, filt, boundary, anchor=None):
    out = ssam.ssam_conv3d(torch.from_numpy(vol).cuda(), filt, boundary, anchor)
    torch.cuda.synchronize()
    return out.cpu().numpy()


@pytest.mark.parametrize("M,N,K", [(5, 5, 5), (4, 4, 4), (7, 7, 7), (6, 5, 3), (2, 9, 6), (9, 2, 8), (10, 4, 4), (14, 3, 5),
                                   (17, 17, 2), (9, 9, 9), (5, 1, 1), (1, 6, 1), (4, 13, 2), (8, 8, 16)])
@pytest.mark.parametrize("boundary", ["clamp", "zero"])
def test_volumes(ssam, M, N, K, boundary):
    """Small grids, on whatever kernel they take: many of them stay on the direct one."""
    rng = np.random.default_rng(970 + M + 20 * N + 400 * K)
    filt = rng.uniform(-1.0, 1.0, (K, N, M)).astype(np.float32)
    for i, (D, H, W) in enumerate([(40, 41, 64), (17, 70, 67), (9, 60, 131), (70, 33, 36), (1, 40, 1700)]):
        vol = wl.uniform_field((D, H, W), -1.0, 1.0, 980 + i, np.float32)
        anchor = [None, (0, 0, 0), (M - 1, N - 1, K - 1)][i % 3]
        name = ssam.ssam_describe("conv3d", vol.shape, filt, boundary).split()[0]
        print(f"split {M}x{N}x{K} {boundary} {vol.shape} anchor {anchor} {name}", flush=True)
        err = normalised_error(run3(ssam, vol, filt, boundary, anchor), oracle.conv3d(vol, filt, boundary, anchor), filt, 1.0)
        assert err <= TOL3, (M, N, K, boundary, vol.shape, err)


@pytest.mark.parametrize("M,N,K", [
    (1, 6, 1), (5, 1, 1), (2, 9, 6), (3, 2, 7), (4, 4, 4), (4, 13, 2), (5, 5, 5),                      # one group of eight columns
    (6, 5, 3), (6, 13, 2), (7, 7, 7), (8, 8, 16), (9, 2, 8), (9, 9, 9),                                # ... and a tail piece
    (10, 4, 4), (10, 10, 1), (11, 5, 3), (12, 9, 2), (12, 2, 9), (13, 1, 6), (13, 12, 5),              # two groups
    (14, 3, 5), (14, 11, 6), (15, 6, 4), (16, 9, 3), (16, 5, 1), (17, 1, 8), (17, 17, 2), (17, 17, 17)])   # ... and a tail piece
def test_volumes_on_the_split_kernel(ssam, M, N, K):
    """Every kind of instance, filters of one part and of several (more than 7 planes, 4 with two groups; more than 9 rows), on
    grids large enough that the filter goes to the split kernel wherever it is anchored."""
    filt = np.random.default_rng(975 + M + 20 * N + 400 * K).uniform(-1.0, 1.0, (K, N, M)).astype(np.float32)
    H, W = 67, 131
    vol = wl.uniform_field((max(11, int(5.1e7 / filt.size / (H * W)) + 1), H, W), -1.0, 1.0, 976, np.float32)
    for i, anchor in enumerate([None, (0, 0, 0), (M - 1, N - 1, K - 1), (M - 1, 0, K // 2)]):
        boundary = ("clamp", "zero")[(i + M) % 2]
        assert "split3mx" in ssam.ssam_describe("conv3d", vol.shape, filt, boundary)
        print(f"split {M}x{N}x{K} {boundary} {vol.shape} anchor {anchor}", flush=True)
        err = normalised_error(run3(ssam, vol, filt, boundary, anchor), oracle.conv3d(vol, filt, boundary, anchor), filt, 1.0)
        assert err <= TOL3 + 2 * 2.0 ** -24, (M, N, K, boundary, anchor, err)      # 17x17x17: ten parts


@pytest.mark.parametrize("planes", [1, 3, 5, 16])
def test_volume_chunks(ssam, planes):
    """z-chunks shorter and taller than the filter."""
    vol = wl.uniform_field((66, 50, 70), -1.0, 1.0, 990, np.float32)
    ssam.ssam_set_tuning("planes_per_wave", planes)
    try:
        for shape in ((5, 5, 5), (7, 9, 4)):
            filt = np.random.default_rng(991).uniform(-1.0, 1.0, shape).astype(np.float32)
            assert "split3mx" in ssam.ssam_describe("conv3d", vol.shape, filt, "zero")
            for boundary in ("clamp", "zero"):
                print(f"split volume planes {planes} {shape} {boundary}", flush=True)
                err = normalised_error(run3(ssam, vol, filt, boundary), oracle.conv3d(vol, filt, boundary), filt, 1.0)
                assert err <= TOL3, (planes, shape, err)
    finally:
        ssam.ssam_set_tuning("planes_per_wave", -1)


@pytest.mark.parametrize("radii", [(2, 2, 2), (3, 3, 3), (2, 1, 1), (1, 3, 2)])
def test_dense_stencils(ssam, radii):
    coef = wl.seeded_coefficients(wl.mask_box(*radii), 995, np.float32)
    fld = wl.uniform_field((30, 45, 66), -1.0, 1.0, 996, np.float32)
    assert "split3mx" in ssam.ssam_describe("stencil3d", fld.shape, coef, "zero")
    for boundary in ("clamp", "zero"):
        got = ssam.ssam_stencil3d(torch.from_numpy(fld).cuda(), coef, boundary).cpu().numpy()
        assert normalised_error(got, oracle.stencil(fld, coef, boundary), coef, 1.0) <= TOL3
    a = torch.from_numpy(fld).cuda()
    res = ssam.ssam_stencil_iterate(a, torch.empty_like(a), coef, 3, "zero").cpu().numpy()
    assert normalised_error(res, oracle.iterate(fld, coef, 3, "zero"), coef, 1.0) <= 3 * TOL3


def test_volume_values_the_split_does_not_carry(ssam):
    filt = np.random.default_rng(997).uniform(-1.0, 1.0, (5, 5, 5)).astype(np.float32)
    vol = wl.uniform_field((30, 45, 66), -1.0, 1.0, 998, np.float32)
    clean = run3(ssam, vol, filt, "clamp")
    for value in (np.inf, np.nan, 1e30):
        for at in ((15, 20, 30), (0, 0, 0), (29, 44, 65)):
            dirty = vol.copy()
            dirty[at] = value
            print(f"split volume value {value} at {at}", flush=True)
            got, want = run3(ssam, dirty, filt, "zero"), oracle.conv3d(dirty, filt, "zero")
            assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want))
            fine = np.isfinite(want) & (np.abs(want) < 1e3)
            assert np.all(np.abs(got[fine].astype(np.float64) - want[fine]) <= 125 * 2.0 ** -24 * np.abs(filt).sum())
            big = np.isfinite(want) & (np.abs(want) >= 1e3)
            assert np.all(np.abs(got[big].astype(np.float64) - want[big]) <= 125 * 2.0 ** -24 * 1e30)
    for scale in (2.0 ** -100, 2.0 ** 60):
        assert np.array_equal(run3(ssam, vol * np.float32(scale), filt, "clamp"), clean * np.float32(scale))


@pytest.mark.parametrize("M,N,K", [(9, 9, 9), (10, 5, 5), (5, 11, 5), (13, 11, 5), (3, 10, 15)])
def test_volume_footprint_of_filters_in_parts(ssam, M, N, K):
    """Filters cut into parts of which the last has fewer rows or planes than the others: infinities and NaN stay inside
    the filter's own extents."""
    filt = np.random.default_rng(1000 + M).uniform(-1.0, 1.0, (K, N, M)).astype(np.float32)
    vol = wl.uniform_field((40, 70, 90), -1.0, 1.0, 1001, np.float32)
    assert "split3mx" in ssam.ssam_describe("conv3d", vol.shape, filt, "zero")
    for anchor in (None, (0, 0, 0), (M - 1, N - 1, K - 1)):
        for value in (np.inf, np.nan):
            for at in ((20, 35, 45), (0, 0, 0), (39, 69, 89)):
                dirty = vol.copy()
                dirty[at] = value
                print(f"split volume {M}x{N}x{K} anchor {anchor} value {value} at {at}", flush=True)
                with np.errstate(invalid="ignore"):
                    assert_footprint(run3(ssam, dirty, filt, "zero", anchor), oracle.conv3d(dirty, filt, "zero", anchor), filt, value, at)


def sums64(x, filt):
    """The filter in 64 bits on the GPU, clamp rule, centre anchor, a tap at a time."""
    pad = []
    for n in reversed(filt.shape):
        pad += [n // 2, n - 1 - n // 2]
    xp = torch.nn.functional.pad(x.double()[None, None], pad, mode="replicate")[0, 0]
    out = torch.zeros(x.shape, dtype=torch.float64, device="cuda")
    for at in np.argwhere(filt != 0):
        out.add_(xp[tuple(slice(int(o), int(o) + n) for o, n in zip(at, x.shape))], alpha=float(filt[tuple(at)]))
    return out


@pytest.mark.parametrize("M,N,K", [(1, 1, 9), (2, 1, 5), (1, 2, 6), (1, 3, 5), (1, 4, 3), (1, 5, 1), (1, 9, 1), (2, 9, 1), (3, 1, 5),
                                   (4, 1, 1), (5, 5, 5), (9, 1, 2)])
def test_thin_volume_filters_are_no_further_off_than_fp32_multiply_adds(ssam, M, N, K):
    """2-norm of the error against 64 bits, in the quadratic mean over four filters, against that of the direct kernel.
    The two differ in the order and number of their roundings only; over four filters the mean scatters by a tenth."""
    vol = torch.rand((150, 290, 300), device="cuda", generator=torch.Generator("cuda").manual_seed(11))
    ratios = []
    for k in range(4):
        filt = np.random.default_rng(1100 + k).uniform(-1.0, 1.0, (K, N, M)).astype(np.float32)
        x = vol if k % 2 == 0 else vol * 2 - 1
        want = sums64(x, filt)
        err = [float((ssam.ssam_conv3d(x, filt, "clamp").double() - want).norm())]
        ssam.ssam_set_tuning("force_generic", 1)
        try:
            err.append(float((ssam.ssam_conv3d(x, filt, "clamp").double() - want).norm()))
        finally:
            ssam.ssam_set_tuning("force_generic", -1)
        ratios.append(err[0] / err[1])
    assert np.sqrt(np.mean(np.square(ratios))) <= 1.1, ratios


@pytest.mark.parametrize("M,taps", [(9, 1), (20, 1), (25, 2), (13, 3)])
def test_filters_of_few_taps_are_no_further_off_than_fp32_multiply_adds(ssam, M, taps):
    img = torch.rand((700, 900), device="cuda", generator=torch.Generator("cuda").manual_seed(12))
    ratios = []
    for k in range(6):
        rng = np.random.default_rng(1110 + k)
        filt = np.zeros(M * M, dtype=np.float32)
        filt[rng.choice(M * M, taps, replace=False)] = rng.uniform(-1.0, 1.0, taps)
        filt = filt.reshape(M, M)
        want = sums64(img, filt)
        err = [float((ssam.ssam_conv2d(img, filt, "clamp").double() - want).norm())]
        ssam.ssam_set_tuning("force_generic", 1)
        try:
            err.append(float((ssam.ssam_conv2d(img, filt, "clamp").double() - want).norm()))
        finally:
            ssam.ssam_set_tuning("force_generic", -1)
        ratios.append(err[0] / err[1])
    assert np.sqrt(np.mean(np.square(ratios))) <= (1.005 if taps <= 2 else 1.1), ratios


def test_a_tap_far_below_the_largest_keeps_its_bits(ssam):
    """Where the large taps meet zeros, the output is one small product."""
    img = np.zeros((300, 300), dtype=np.float32)
    img[150, 150] = 1.2345678
    filt = np.full((9, 9), 2.0 ** 40, dtype=np.float32)
    filt[0, 0] = np.float32(1.7654321) * np.float32(2.0 ** -80)
    got = run(ssam, img, filt, "zero")[154, 154]
    assert abs(float(got) - float(img[150, 150]) * float(filt[0, 0])) <= 2.0 ** -23 * float(img[150, 150]) * float(filt[0, 0])


@pytest.mark.parametrize("shape", [(9, 9), (20, 20), (25, 25), (1, 14), (5, 5, 5), (9, 9, 9), (5, 11, 10)])
@pytest.mark.parametrize("boundary", ["clamp", "zero"])
def test_many_values_the_split_does_not_carry(ssam, shape, boundary):
    """A picture with a hole of NaN, and single infinities and large values beside it: bands that a block's waves share out
    among themselves, inside the grid and at its edges, in filters of one part and of several."""
    filt = np.random.default_rng(1200 + len(shape)).uniform(-1.0, 1.0, shape).astype(np.float32)
    three = len(shape) == 3
    size = (50, 61, 190) if three else (203, 521)
    field = wl.uniform_field(size, -1.0, 1.0, 1201, np.float32)
    field[..., 20:35, 60:95] = np.nan
    rng = np.random.default_rng(1202)
    for value in (np.inf, -np.inf, 1e31):
        at = tuple(rng.integers(0, n, 6) for n in size)
        field[at] = value
    kind = "conv3d" if three else "conv2d"
    assert "split3mx" in ssam.ssam_describe(kind, size, filt, boundary)
    with np.errstate(invalid="ignore", over="ignore"):
        want = (oracle.conv3d if three else oracle.conv2d)(field, filt, boundary)
    for knob, value in (("rows_per_wave", -1), ("planes_per_wave" if three else "rows_per_wave", 24)):
        ssam.ssam_set_tuning(knob, value)
        try:
            print(f"split {shape} {boundary} {knob} {value}", flush=True)
            got = (run3 if three else run)(ssam, field, filt, boundary)
        finally:
            ssam.ssam_set_tuning(knob, -1)
        assert_footprint(got, want, filt, 1e31, (shape, boundary, knob, value))
