"""The host workers' escape-time rows, AVX-512 (where this CPU has it) and
AVX2 + FMA: counts equal the oracle's, on orbits that escape, that end in a
cycle found early and that run to the cap, at widths around a vector and a
block of four, caps around the eight steps between two cycle tests, |c| near
2, zero, denormal, huge and NaN coordinates."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

from oracle import oracle as O

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1805_02755_amd", "csrc")
SHIM = """
#include "host_payloads.cpp"
static const ce::HostPayloadFns* fns(int wide) { return wide ? ce::host_payloads() : &ce::kFma; }
extern "C" const char* pick(int wide) { return fns(wide)->isa; }
extern "C" void rows(int wide, const ce_escape_params* p, uint64_t r0, uint64_t r1, uint32_t* out) {
  fns(wide)->escape_rows(*p, r0, r1, out);
}
"""
REGIONS = {
    "set": (-2.0, -1.5, None, None),
    "tip": (-2.0, -2e-5, 1e-6, 1e-6),
    "circle": (1.3, 1.3, 0.002, 0.002),
    "seahorse": (-0.75, 0.1, 2e-4, 2e-4),
    "near_zero": (-2e-6, -2e-6, 4e-8, 4e-8),
    "zero_row": (-2.0, 0.0, 0.02, 0.0),
    "negative_zero": (-0.0, -0.0, -0.02, -0.0),
    "denormal_imaginary": (-1.9, 0.0, 0.01, 1e-40),
    "huge": (-1e30, -1e38, 1e28, 3e36),
    "nan": (float("nan"), -1.0, 0.01, 0.02),
}


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    d = tmp_path_factory.mktemp("host_escape")
    src, out = d / "shim.cpp", str(d / "libshim.so")
    src.write_text(SHIM)
    subprocess.run(["g++", "-O3", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off", "-fno-math-errno", "-I", CSRC,
                    "-o", out, str(src)], check=True, capture_output=True)
    lib = C.CDLL(out)
    lib.pick.restype = C.c_char_p
    lib.rows.restype = None
    lib.rows.argtypes = [C.c_int, C.c_void_p, C.c_uint64, C.c_uint64, C.c_void_p]
    return lib


@pytest.mark.parametrize("w", [1, 15, 16, 17, 63, 64, 65, 131])
@pytest.mark.parametrize("region", sorted(REGIONS))
def test_rows_equal_the_oracles(shim, region, w):
    import paper_1805_02755_amd as ce
    h = 41
    x0, y0, dx, dy = REGIONS[region]
    x0, y0, dx, dy = (float(np.float32(v)) for v in (x0, y0, 3.0 / w if dx is None else dx, 3.0 / h if dy is None else dy))
    for max_iter in (1, 7, 8, 9, 64, 500):
        p = ce.ce_escape_params(w, h, x0, y0, dx, dy, max_iter)
        ref = O.escape(w, h, x0, y0, dx, dy, max_iter)
        for wide in (0, 1):
            out = np.full((h + 1, w), 0xABCD, np.uint32)
            shim.rows(wide, C.byref(p), 0, h, out.ctypes.data)
            assert np.array_equal(out[:h], ref), (shim.pick(wide), max_iter)
            assert (out[h] == 0xABCD).all()
