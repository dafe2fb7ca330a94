"""How many vectors a call of the allocation-free product takes: as many as units of 16 tiles
leave room for in the static scratch, whatever units the operator has (CPU only: a C++
driver hands the library an operator that has tables and no matrix)."""
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
    const int rc = bie_apply_noalloc(&op, v, v + 2, atoi(argv[3]), 0, 0, nullptr);
    std::printf("%d %s", rc, bie_last_error());
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


@pytest.mark.parametrize("N,unit,R", [(5202, 8, 36), (7680, 8, 17), (7680, 4, 17), (7680, 16, 17), (15360, 8, 4)])
def test_vectors_accepted_by_units_of_sixteen(driver, N, unit, R):
    nT = (N + 63) // 64
    slots = nT * (nT - 1) // 2 + sum((nT - i + 15) // 16 for i in range(nT))
    assert R == (128 << 20) // (slots * 64 * 16)
    for r, refused in ((R, False), (R + 1, True)):
        out = subprocess.run([str(driver), str(N), str(unit), str(r)], check=True, capture_output=True, text=True,
                             env={k: v for k, v in os.environ.items() if k != "BIE_SYM_UNIT"}).stdout
        assert ("scratch" in out) == refused, out
