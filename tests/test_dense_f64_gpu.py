"""fp64 filters without a compiled shape: the register-tiled kernel against the CPU oracle and, bit for bit, against the
one-point-per-thread kernel (same order of additions), at the remainders of its tiles (4 x 4 outputs per lane, 64 or 32
columns, one to four waves in y, two planes in z), of its four-tap steps and of the parts a long filter is cut into.
Tolerance: one rounding of 2^-53 per tap, in units of sum|w| * max|in|."""
import numpy as np
import pytest

import oracle
import workloads as wl
from parity_util import normalised_error

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ssam():
    import paper_1907_06154_amd as s
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    s.lib()
    yield s
    s.ssam_set_tuning("force_generic", -1)


def both(ssam, call):
    """The register-tiled kernel's result (also on grids too small for it to be the choice), and the direct kernel's."""
    res = []
    try:
        for force in (2, 1):
            ssam.ssam_set_tuning("force_generic", force)
            res.append(call().cpu().numpy())
    finally:
        ssam.ssam_set_tuning("force_generic", -1)
    return res


def check(got, plain, want, filt, what):
    tol = (filt.size + 2) * 2.0 ** -53
    assert normalised_error(got, want, filt, 1.0) <= tol, what
    if filt.size <= 298:        # one launch of either kernel
        assert np.array_equal(got, plain), what


@pytest.mark.parametrize("M,N", [(12, 12), (13, 1), (14, 2), (15, 3), (16, 4), (1, 13), (2, 14), (3, 17), (12, 5), (21, 21), (32, 32)])
@pytest.mark.parametrize("boundary", ["clamp", "zero"])
def test_filters(ssam, M, N, boundary):
    filt = wl.seeded_filter(M, N, 1000 + 40 * M + N, np.float64)
    for k, (H, W) in enumerate([(64, 64), (65, 63), (17, 130), (130, 33), (1, 200), (200, 1), (3, 5), (270, 257)]):
        img = wl.uniform_field((H, W), -1.0, 1.0, 1010 + k, np.float64)
        anchor = [None, (0, 0), (M - 1, N - 1)][k % 3]
        assert ssam.ssam_describe("conv2d", (H, W), filt, boundary).split()[0] == "generic_direct"
        print(f"dense f64 {M}x{N} {boundary} {H}x{W} anchor {anchor}", flush=True)
        d = torch.from_numpy(img).cuda()
        got, plain = both(ssam, lambda: ssam.ssam_conv2d(d, filt, boundary, anchor))
        check(got, plain, oracle.conv2d(img, filt, boundary, anchor), filt, (M, N, boundary, H, W))


@pytest.mark.parametrize("M,N,K", [(9, 2, 8), (5, 6, 4), (9, 9, 9), (1, 9, 1), (10, 1, 3), (7, 7, 7), (4, 9, 2)])
@pytest.mark.parametrize("boundary", ["clamp", "zero"])
def test_volumes(ssam, M, N, K, boundary):
    filt = np.random.default_rng(1020 + M + 20 * N + 400 * K).uniform(-1.0, 1.0, (K, N, M))
    for k, (D, H, W) in enumerate([(8, 16, 64), (5, 21, 67), (1, 40, 33), (13, 3, 130), (2, 70, 5)]):
        vol = wl.uniform_field((D, H, W), -1.0, 1.0, 1030 + k, np.float64)
        anchor = [None, (0, 0, 0), (M - 1, N - 1, K - 1)][k % 3]
        print(f"dense f64 {M}x{N}x{K} {boundary} {vol.shape} anchor {anchor}", flush=True)
        d = torch.from_numpy(vol).cuda()
        got, plain = both(ssam, lambda: ssam.ssam_conv3d(d, filt, boundary, anchor))
        check(got, plain, oracle.conv3d(vol, filt, boundary, anchor), filt, (M, N, K, boundary, vol.shape))


@pytest.mark.parametrize("H,W,M,N", [(13200, 160, 20, 20), (65536, 32, 21, 21), (65536, 40, 32, 14), (13200, 160, 12, 12)])
def test_tall_narrow_pictures(ssam, H, W, M, N):
    """Blocks of up to four waves of 32 rows: the largest staged tiles."""
    filt = wl.seeded_filter(M, N, 1045, np.float64)
    d = torch.from_numpy(wl.uniform_field((H, W), -1.0, 1.0, 1046, np.float64)).cuda()
    print(f"dense f64 {M}x{N} {H}x{W}", flush=True)
    got, plain = both(ssam, lambda: ssam.ssam_conv2d(d, filt, "clamp"))
    check(got, plain, plain, filt, (M, N, H, W))


def test_infinities_and_nan_reach_their_footprint_only(ssam):
    filt = wl.seeded_filter(13, 14, 1040, np.float64)
    img = wl.uniform_field((90, 140), -1.0, 1.0, 1041, np.float64)
    for value in (np.inf, np.nan):
        for y, x in ((40, 70), (0, 0), (89, 139)):
            dirty = img.copy()
            dirty[y, x] = value
            print(f"dense f64 value {value} at {y},{x}", flush=True)
            got, _ = both(ssam, lambda: ssam.ssam_conv2d(torch.from_numpy(dirty).cuda(), filt, "zero"))
            want = oracle.conv2d(dirty, filt, "zero")
            assert np.array_equal(np.isnan(got), np.isnan(want)) and np.array_equal(np.isinf(got), np.isinf(want))


@pytest.mark.parametrize("M,N,K", [(7, 4, 2), (8, 4, 3), (5, 5, 5), (6, 6, 2), (1, 5, 4), (2, 6, 3), (3, 4, 4)])
def test_rows_that_all_output_rows_and_planes_share(ssam, M, N, K):
    """One, two and more such rows, each remainder of four filter columns, an odd and an even number of planes."""
    filt = np.random.default_rng(1050 + M + 20 * N + 400 * K).uniform(-1.0, 1.0, (K, N, M))
    for D, H, W in ((6, 33, 66), (7, 16, 65)):
        vol = wl.uniform_field((D, H, W), -1.0, 1.0, 1051, np.float64)
        print(f"dense f64 {M}x{N}x{K} {vol.shape}", flush=True)
        d = torch.from_numpy(vol).cuda()
        got, plain = both(ssam, lambda: ssam.ssam_conv3d(d, filt, "clamp"))
        check(got, plain, oracle.conv3d(vol, filt, "clamp"), filt, (M, N, K, vol.shape))
