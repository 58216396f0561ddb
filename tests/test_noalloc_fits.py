"""biq_gemm_noalloc takes every call that one of its plans fits the fixed buffer for - the tables' only up to four times
the matrix cores' time.  Run in a process that sees no GPU, where an accepted call ends with BIQ_EHIP and nothing is
launched."""
import json
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import ctypes, json, sys
from paper_2005_09904_amd.build import LIB_PATH
lib = ctypes.CDLL(LIB_PATH)
count = ctypes.c_int(0)
assert ctypes.CDLL("libamdhip64.so").hipGetDeviceCount(ctypes.byref(count)) != 0 or count.value == 0
f = lib.biq_gemm_noalloc
f.argtypes = [ctypes.c_void_p] * 4 + [ctypes.c_int] * 5 + [ctypes.c_void_p]
buf = ctypes.create_string_buffer(64)
p = (ctypes.addressof(buf) + 15) // 16 * 16
print(json.dumps([f(p, p, p, p, *shape, None) for shape in json.loads(sys.argv[1])]))
"""


def _statuses(shapes):
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1", ROCR_VISIBLE_DEVICES="-1")
    out = subprocess.run([sys.executable, "-c", CHILD, json.dumps(shapes)], check=True, capture_output=True, text=True, cwd=ROOT, env=env)
    return json.loads(out.stdout)


def test_a_plan_that_fits_is_taken():
    shapes = [
        # the tables' plan fits, digits or three 16-bit terms do not
        (404547, 180743, 2, 14, 8), (874962, 206108, 4, 14, 8), (42, 70796, 1, 79, 6), (20, 62289, 4, 193, 8), (61, 186587, 1, 1, 9),
        # only digits, only three 16-bit terms
        (399803, 1477, 2, 7, 5), (292233, 1950, 1, 8, 5), (49252, 145771, 1, 4, 3), (724545, 69374, 2, 1, 4)]
    assert _statuses(shapes) == [-4] * len(shapes)


def test_none_fits():
    shapes = [(1 << 20, 200000, 5, 8, 9), (60000, 30000, 2, 700, 6), (30000, 200000, 5, 100, 9)]
    import paper_2005_09904_amd as biq

    for m, n, q, b, mu in shapes:
        plans = [biq.biq_plan_get(m, n, q, b, mu), biq.biq_plan_get_lut(m, n, q, b, mu)]
        plans += [biq.biq_plan_get_mfma(m, n, q, b, mu, 3)] if q <= 4 else []
        assert all(biq.biq_plan_workspace_bytes(p, m, b) > biq.biq_noalloc_scratch_bytes() for p in plans)
    # (the last one: its tables need nothing, and several times as long as digits in a workspace)
    shapes.append((16384, 16384, 2, 512, 8))
    assert _statuses(shapes) == [-3] * len(shapes)
