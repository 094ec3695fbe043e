"""CPU test of the scales of the window bounds (csrc/tm_window.h, compiled for
the host): over every binary exponent of float32, a pattern either has bounds
whose scales are normal powers of 2 that undo each other, with its scaled
maximum inside float16, or is left to the exhaustive scan."""
import os
import re
import shutil
import subprocess

import pytest

from conftest import ROOT

PROGRAM = r"""
#include <cstdio>
#include <cstdlib>
#include "tm_window.h"
using namespace tmlib;
static void check(bool ok, const char* what, float A) {
    if (!ok) { std::printf("%s at A = %a\n", what, A); std::exit(1); }
}
int main() {
    int with = 0, without = 0;
    for (int e = -149; e <= 127; ++e)
        for (float m : {1.0f, 1.5f, 1.99999988f}) {
            const float A = ldexpf(m, e);
            const float inv = inverse_up(static_cast<double>(A) * 8.0);
            check(static_cast<double>(inv) * (static_cast<double>(A) * 8.0) >= 1.0, "inverse rounded down", A);
            if (no_window_bounds(A, inv)) {
                ++without;
                check(e < -90 || e >= 121, "no bounds for an ordinary pattern", A);
                continue;
            }
            ++with;
            const WindowScale s = window_scale(A);
            for (float v : {s.image, s.undo, s.image * ldexpf(1.0f, kWeightExp)})
                check(std::isnormal(v), "scale out of range", A);
            check(s.image * ldexpf(1.0f, kWeightExp) * s.undo == 1.0f, "scales do not undo each other", A);
            check(A * s.image <= ldexpf(1.0f, kImageExp) && A * s.image >= ldexpf(1.0f, kImageExp - 1),
                  "maximum outside the image's range", A);
            check(h2f(f16_up(A * s.image)) >= A * s.image, "float16 rounded down", A);
        }
    check(with > 0 && without > 0, "both kinds", 0.0f);
    for (float x = 1e-9f; x < 70000.0f; x *= 1.0009f) check(h2f(f16_up(x)) >= x, "float16 rounded down", x);
    check(no_window_bounds(1.0f, INFINITY), "1 / norm past the range", 1.0f);
    check(no_window_bounds(0x1p-90f, 0x1p-90f), "a norm far above the pattern's", 0x1p-90f);
    check(no_window_bounds(0x1p60f, 0x1p60f), "a norm far below the pattern's", 0x1p60f);
    check(!no_window_bounds(1.0f, 0.0f), "no norm", 1.0f);
    check(!no_window_bounds(0.0f, 0.0f), "a blank pattern needs no scan", 0.0f);
    check(inverse_up(0.0) == 0.0f && inverse_up(-1.0) == 0.0f, "no norm", 0.0f);
    std::puts("ok");
}
"""


def test_scales_over_all_exponents(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    src, exe = tmp_path / "scale.hip", tmp_path / "scale"
    src.write_text(PROGRAM)
    csrc = os.path.join(ROOT, "paper_2111_07347_amd", "csrc")
    r = subprocess.run([hipcc, "-std=c++17", "-O2", "--offload-host-only", f"-I{csrc}", str(src), "-o", str(exe)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout


def test_window_image_is_declared_in_whole_entries():
    """The kernel reads the image's entries (4 float16) in one 8-byte LDS read:
    the dynamic LDS array has to be one of 8-byte elements, which is what
    places it on an 8-byte boundary behind the kernel's static LDS."""
    src = open(os.path.join(ROOT, "paper_2111_07347_amd", "csrc", "tm_bound.hip")).read()
    assert re.findall(r"extern __shared__ (\w+) \w+\[\]", src) == ["u32x2"]
    assert re.search(r"typedef uint32_t u32x2 __attribute__\(\(ext_vector_type\(2\)\)\)", src)
    assert re.search(r"lds_u32x2\*\)entries", src)
