"""The allocation-free product refuses, before any device call, a vector whose partial
slots do not fit the static scratch (CPU only: a C++ driver hands the library an
operator that has tables and no matrix)."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include "bie.h"
#include "bie_internal.hpp"
int main(int, char **argv) {
    bie_op op;
    op.mesh.N = op.pk.N = atoll(argv[1]);
    op.pk.nT = (op.pk.N + bie::TB - 1) / bie::TB;
    op.pk.ntiles = op.pk.nT * (op.pk.nT + 1) / 2;
    std::vector<int32_t> units, uptr;
    std::vector<int64_t> seg;
    bie::build_units(op.pk.nT, atoi(argv[2]), units, uptr, seg);
    op.pk.nslots = seg[op.pk.nT];
    double v[4];   // never read: the operator holds no matrix
    const int rc = bie_apply_noalloc(&op, v, v + 2, 1, atoi(argv[3]), 0, nullptr);
    std::printf("%d %lld", rc, (long long)op.pk.nslots);
    return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("ROCm clang++ not available")
    d = tmp_path_factory.mktemp("noalloc")
    src, exe = d / "drv.cpp", d / "drv"
    src.write_text(DRIVER)
    pkg = os.path.join(ROOT, "paper_2606_13482_amd")
    subprocess.run([CLANG, "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(pkg, "csrc"), str(src), "-o", str(exe), "-L" + pkg, "-lbie",
                    "-Wl,-rpath," + pkg, "-L/opt/rocm/lib", "-lamdhip64", "-Wl,-rpath,/opt/rocm/lib"], check=True)
    return exe


# length of the units (BIE_SYM_UNIT) and the sizes where one vector's slots pass 128 MiB
@pytest.mark.parametrize("unit,N,fits", [(1, 23168, True), (1, 23169, False), (1, 30720, False), (2, 26700, True),
                                         (2, 26800, False), (4, 29250, False), (4, 30720, False), (8, 30720, True)])
def test_slots_beyond_the_scratch_are_refused(driver, unit, N, fits):
    out = subprocess.run([str(driver), str(N), str(unit), "0"], check=True, capture_output=True, text=True,
                         env=dict(os.environ, BIE_SYM_UNIT=str(unit))).stdout.split()
    rc, slots = int(out[0]), int(out[1])
    assert (slots * 64 * 16 <= 128 << 20) == fits
    if not fits:
        assert rc == -1   # BIE_EINVAL
    else:   # no device or no matrix: past the size check
        assert rc != 0
