"""Flagged pairs found on the host (meshes too large for the device search): the same list,
in order, as by their definition, which is also the device search's."""
import os
import subprocess

import numpy as np
import pytest

from near_lists import CASES, expected, mesh

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CLANG = "/opt/rocm/llvm/bin/clang++"

DRIVER = r"""
#include <cstdio>
#include <cstdlib>
#include "bie_internal.hpp"
template <typename T> static std::vector<T> slurp(const std::string &p)
{
    std::vector<T> v;
    FILE *f = std::fopen(p.c_str(), "rb");
    T x;
    while (f && std::fread(&x, sizeof(T), 1, f) == 1) v.push_back(x);
    if (f) std::fclose(f);
    return v;
}
int main(int, char **argv)
{
    const std::string d = argv[1];
    const auto V = slurp<double>(d + "/V");
    const auto T = slurp<int32_t>(d + "/T");
    const bie::Mesh m = bie::build_mesh(V.data(), int64_t(V.size() / 3), T.data(), int64_t(T.size() / 3), atof(argv[2]));
    FILE *f = std::fopen((d + "/near").c_str(), "wb");
    std::fwrite(m.near.data(), sizeof(int32_t), m.near.size(), f);
    return std::fclose(f);
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    if not os.path.exists(CLANG):
        pytest.skip("ROCm clang++ not available")
    d = tmp_path_factory.mktemp("near")
    src, exe = d / "drv.cpp", d / "drv"
    src.write_text(DRIVER)
    csrc = os.path.join(ROOT, "paper_2606_13482_amd", "csrc")
    subprocess.run([CLANG, "-std=c++17", "-O2", "-ffp-contract=off", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + csrc, str(src), os.path.join(csrc, "mesh.cpp"), "-o",
                    str(exe)], check=True)
    return exe


@pytest.mark.parametrize("name,factor", CASES)
def test_host_list(driver, tmp_path, name, factor):
    V, T = mesh(name)
    np.ascontiguousarray(V, np.float64).tofile(tmp_path / "V")
    np.ascontiguousarray(T, np.int32).tofile(tmp_path / "T")
    subprocess.run([str(driver), str(tmp_path), repr(factor)], check=True)
    assert np.array_equal(np.fromfile(tmp_path / "near", np.int32).reshape(-1, 2), expected(V, T, factor))


def test_each_search_where_it_is_the_faster():
    """The line lies between the measured sizes: device at 480 000 triangles, host at 1 044 300
    (2.87 against 1.94 s for the lists of a fast operator)."""
    import ctypes

    from paper_2606_13482_amd import bie
    on_device = ctypes.CDLL(bie.LIB_PATH)["_ZN3bie14near_on_deviceEl"]
    on_device.restype, on_device.argtypes = ctypes.c_bool, [ctypes.c_int64]
    assert on_device(5120) and on_device(480_000) and not on_device(800_000) and not on_device(1_044_300)
