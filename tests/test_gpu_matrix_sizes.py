"""The full matrix from the packed tiles, a quarter of a tile or a whole one to a block: entry
by entry the product with unit vectors, symmetric, every entry written, FP64 and FP32."""
import pytest
import torch

from paper_2606_13482_amd.inputs import cube_sphere, icosphere

pytestmark = pytest.mark.gpu


# 6, 30, 72, 480, 1152, 1458 unknowns: 1, 1, 3, 36, 171 tiles (quarters) and 276 (whole)
@pytest.mark.parametrize("mesh", [("i", 0), ("c", 2), ("i", 2), ("c", 8), ("c", 9)])
@pytest.mark.parametrize("storage", ["c128", "c64"])
def test_matrix(bie, mesh, storage):
    V, T = icosphere(mesh[1]) if mesh[0] == "i" else cube_sphere(mesh[1], "ellipsoid", axes=(1.0, 1.2, 1.5))
    op = bie.Operator(V, T, 2.0, storage=storage)
    for dt in (torch.complex128, torch.complex64) if storage == "c64" else (torch.complex128,):
        Z = torch.full((op.N, op.N), float("nan"), dtype=dt, device="cuda")
        code = bie.BIE_C128 if dt == torch.complex128 else bie.BIE_C64
        bie._check(bie._lib.bie_op_matrix(op._h, bie._dev(Z, dt), code, bie._stream()))
        assert torch.equal(Z, Z.T) and bool(torch.isfinite(torch.view_as_real(Z)).all())
        E = torch.zeros((64, op.N), dtype=dt, device="cuda")
        for i in range(64):
            E[i, (i * 61) % op.N] = 1
        Y = op.apply(E)
        assert torch.equal(Y, Z[[(i * 61) % op.N for i in range(64)]])   # each sum has one term
    op.close()
