"""2D stencils, filters and multi-sweep launches on rows that are not whole vectors: widths around the vector length and the
strip width, where a lane's vector starts inside the row and ends beyond it; tiles from one group of rows on."""
import numpy as np
import pytest

import oracle
import workloads as wl
from parity_util import assert_parity

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def ssam():
    import paper_1907_06154_amd as s
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    s.lib()
    yield s
    s.ssam_set_tuning("rows_per_wave", -1)


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("W", [1, 2, 3, 4, 5, 6, 7, 111, 113, 223, 225, 226, 227, 449])
def test_widths(ssam, dtype, W):
    for H in (1, 5, 37):
        fld = wl.uniform_field((H, W), -1.0, 1.0, 1100 + W, dtype)
        for mask in (wl.mask_box(1, 1), wl.mask_star(4, 4), wl.mask_box(2, 2)):
            coef = wl.seeded_coefficients(mask, 1101, dtype)[0]
            for boundary in ("zero", "clamp"):
                print(f"ragged {np.dtype(dtype).name} {H}x{W} {coef.shape} {boundary}", flush=True)
                a = torch.from_numpy(fld).cuda()
                got = ssam.ssam_stencil2d(a, coef, boundary).cpu().numpy()
                assert_parity(got, oracle.stencil(fld, coef, boundary), coef, 1.0, f"{H}x{W}")
                res = ssam.ssam_stencil_iterate(a, torch.empty_like(a), coef, 9, boundary).cpu().numpy()
                assert_parity(res, oracle.iterate(fld, coef, 9, boundary), coef, 1.0, f"iterate {H}x{W}")


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("rows", [4, 8, 20])
def test_short_tiles(ssam, dtype, rows):
    """Tiles of one group up: most of a tile's groups are the ones above it."""
    fld = wl.uniform_field((90, 451), -1.0, 1.0, 1110, dtype)
    ssam.ssam_set_tuning("rows_per_wave", rows)
    try:
        for mask in (wl.mask_star(1, 1), wl.mask_box(1, 1), wl.mask_star(3, 3)):
            coef = wl.seeded_coefficients(mask, 1111, dtype)[0]
            for boundary in ("zero", "clamp"):
                print(f"short tiles {np.dtype(dtype).name} rows {rows} {coef.shape} {boundary}", flush=True)
                a = torch.from_numpy(fld).cuda()
                res = ssam.ssam_stencil_iterate(a, torch.empty_like(a), coef, 8, boundary).cpu().numpy()
                assert_parity(res, oracle.iterate(fld, coef, 8, boundary), coef, 1.0, f"rows {rows}")
    finally:
        ssam.ssam_set_tuning("rows_per_wave", -1)


def test_views_that_start_off_a_vector_boundary(ssam):
    """A picture in the middle of a buffer: aligned to its element only."""
    for dtype in (np.float32, np.float64):
        img = wl.uniform_field((40, 300), -1.0, 1.0, 1120, dtype)
        buf = torch.zeros(img.size + 3, dtype=torch.from_numpy(img).dtype, device="cuda")
        a = buf[1:1 + img.size].view(img.shape)
        a.copy_(torch.from_numpy(img))
        for M in (3, 9):
            filt = wl.seeded_filter(M, M, 1121, dtype)
            print(f"view {np.dtype(dtype).name} {M}x{M}", flush=True)
            assert_parity(ssam.ssam_conv2d(a, filt, "clamp").cpu().numpy(), oracle.conv2d(img, filt, "clamp"), filt, 1.0, "view")


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("W", [2, 3, 4, 5, 7, 127, 129, 131, 255, 257, 262])
def test_widths_3d(ssam, dtype, W):
    """3D: a strip is 64 vectors wide, and the staged plane is put right before it is read."""
    for D, H in ((1, 1), (3, 9), (9, 37)):
        fld = wl.uniform_field((D, H, W), -1.0, 1.0, 1130 + W, dtype)
        buf = torch.zeros(fld.size + 1, dtype=torch.from_numpy(fld).dtype, device="cuda")
        for first in (0, 1):                               # aligned to 16 bytes, and to the element only
            a = buf[first:first + fld.size].view(fld.shape)
            a.copy_(torch.from_numpy(fld))
            for mask in (wl.mask_star(1, 1, 1), wl.mask_star(4, 4, 4), wl.mask_box(1, 1, 1), wl.mask_box(3, 3, 3)):
                coef = wl.seeded_coefficients(mask, 1131, dtype)
                for boundary in ("zero", "clamp"):
                    print(f"ragged 3d {np.dtype(dtype).name} {D}x{H}x{W}+{first} {coef.shape} {boundary}", flush=True)
                    got = ssam.ssam_stencil3d(a, coef, boundary).cpu().numpy()
                    assert_parity(got, oracle.stencil(fld, coef, boundary), coef, 1.0, f"{D}x{H}x{W}+{first}")


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("shape", [(20, 41, 263), (5, 16, 63), (33, 34, 130)])
def test_sweeps_3d(ssam, dtype, shape):
    fld = wl.uniform_field(shape, -1.0, 1.0, 1140, dtype)
    for mask in (wl.mask_star(2, 2, 2), wl.mask_box(1, 1, 1)):
        coef = wl.seeded_coefficients(mask, 1141, dtype)
        for boundary in ("zero", "clamp"):
            print(f"sweeps 3d {np.dtype(dtype).name} {shape} {coef.shape} {boundary}", flush=True)
            a = torch.from_numpy(fld).cuda()
            res = ssam.ssam_stencil_iterate(a, torch.empty_like(a), coef, 5, boundary).cpu().numpy()
            assert_parity(res, oracle.iterate(fld, coef, 5, boundary), coef, 1.0, f"iterate {shape}")
