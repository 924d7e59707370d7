"""A launch that fails is reported by the call that made it and by no later one: whatever kernel the dispatcher picks, the runtime's
last error is clear afterwards.  Host only: a stand-in for the runtime's launch, which always fails, is loaded before the library."""
import subprocess
import sys

import numpy as np
import pytest

import paper_1907_06154_amd as ssam

STAND_IN = r"""
static int last;
int hipGetLastError(void) { int e = last; last = 0; return e; }
int stand_in_last(void) { return last; }
int stand_in_launches;
int hipGetDevice(int *dev) { *dev = 0; return 0; }
int hipFuncSetAttribute(const void *f, int attr, int value) { (void)f; (void)attr; (void)value; return 0; }
struct dim { unsigned x, y, z; };
int __hipPushCallConfiguration(struct dim grid, struct dim block, unsigned long lds, void *stream)
{
    (void)grid; (void)block; (void)lds; (void)stream;
    return 0;
}
int __hipPopCallConfiguration(struct dim *grid, struct dim *block, unsigned long *lds, void **stream)
{
    *grid = *block = (struct dim){1, 1, 1};
    *lds = 0;
    *stream = 0;
    return 0;
}
int hipLaunchKernel(const void *f, struct dim grid, struct dim block, void **args, unsigned long lds, void *stream)
{
    (void)f; (void)grid; (void)block; (void)args; (void)lds; (void)stream;
    ++stand_in_launches;
    return last = 1;
}
"""

PROGRAM = r"""
import ctypes, sys
import numpy as np
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
L = ctypes.CDLL(sys.argv[2])
vp, ci = ctypes.c_void_p, ctypes.c_int
L.ssam_stencil_iterate.argtypes = [vp, vp, ci, ci, ci, vp, ci, ci, ci, ci, ci, ci, vp, vp]
W, H, D, taps, rz, steps = map(int, sys.argv[3:9])
coef = np.ones((taps if rz else 1, taps, taps), np.float32)
r = taps // 2
status = L.ssam_stencil_iterate(0x10000000, 0x50000000, W, H, D, coef.ctypes.data, r, r, rz, 0, 0, steps, None, None)
print(status, ctypes.c_int.in_dll(fake, "stand_in_launches").value, fake.stand_in_last())
"""

CALLS = {"tiles": (300, 300, 1, 3, 0, 4, "_tile_"), "marching": (5000, 5000, 1, 3, 0, 4, "_fused"), "levels": (200, 200, 200, 3, 1, 4, "_levels_"),
         "single": (300, 300, 1, 3, 0, 1, "float_M")}


@pytest.mark.parametrize("call", CALLS)
def test_a_failed_launch_leaves_no_error_behind(call, tmp_path):
    W, H, D, taps, rz, steps, plan = CALLS[call]
    coef = np.ones((taps,) * (3 if rz else 2), np.float32)
    kind = ("iterate3d" if rz else "iterate2d") if steps > 1 else "stencil2d"
    shape = (D, H, W) if rz else (H, W)
    assert plan in ssam.ssam_describe(kind, shape, coef, "zero", remaining=steps).split()[0]
    lib = tmp_path / "stand_in.so"
    (tmp_path / "stand_in.c").write_text(STAND_IN)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(lib), str(tmp_path / "stand_in.c")], check=True)
    res = subprocess.run([sys.executable, "-c", PROGRAM, str(lib), ssam.binding.LIB_PATH, *map(str, (W, H, D, taps, rz, steps))],
                         capture_output=True, text=True, timeout=120)
    status, launches, left = map(int, res.stdout.split())
    assert launches == 1 and status != 0 and left == 0, (call, res.stdout, res.stderr)
