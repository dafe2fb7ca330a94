"""The Calderon preconditioner's dual matrix cell by cell, where its launch changes:
vertices with more edges than a block's functions (7: blocks of 8; 10: two blocks),
a cell with more children than a block (70 edges: two parts), refined pairs within
and beyond the narrow phase range; and the Gram solves over the column widths."""
import numpy as np
import pytest
import torch

from oracle import calderon as ocal
from paper_2606_13482_amd.inputs import cube_sphere, icosphere

pytestmark = pytest.mark.gpu


def bipyramid(n):
    """2 n triangles around two apexes of degree n."""
    a = 2 * np.pi * np.arange(n) / n
    V = np.concatenate([np.stack([np.cos(a), np.sin(a), 0 * a], 1), [[0, 0, 0.9], [0, 0, -0.7]]])
    i, j = np.arange(n), (np.arange(n) + 1) % n
    T = np.concatenate([np.stack([i, j, 0 * i + n], 1), np.stack([j, i, 0 * i + n + 1], 1)])
    return V, T.astype(np.int32)


# 1e-10 of the largest entry, as the other comparisons of M: the Gram solves stop at
# 1e-13 and G's condition number is below 10.
@pytest.mark.parametrize("name,k", [("tet", 1.0), ("bi7", 2.0), ("bi10", 2.0), ("bi70", 2.0), ("ico1", 2.0),
                                    ("ico1", 15.0), ("box3", 3.0)])
def test_dual_matrix_by_cells(bie, name, k):
    if name == "tet":
        V, T = np.array([[1, 1, 1], [1, -1, -1], [-1, 1, -1], [-1, -1, 1.0]]), np.array(
            [[0, 1, 2], [0, 3, 1], [0, 2, 3], [1, 3, 2]], np.int32)
    elif name.startswith("bi"):
        V, T = bipyramid(int(name[2:]))
    else:
        V, T = icosphere(1) if name == "ico1" else cube_sphere(3, "rounded_cube")
    M = ocal.build(V, T, k)["M"]
    op = bie.Operator(V, T, k)
    pc = bie.Calderon(op)
    got = pc.apply(torch.eye(op.N, dtype=torch.complex128, device="cuda")).cpu().numpy().T
    info = pc.info()
    print(f"  {name} k={k}: Gram {info['cg_iters']} {max(info['cg_relres']):.1e}, "
          f"M {np.abs(got - M).max() / np.abs(M).max():.1e}", flush=True)
    assert max(info["cg_relres"]) <= 1e-13
    assert np.abs(got - M).max() <= 1e-10 * np.abs(M).max()
    pc.close()
    op.close()


# Both solvers stop at a residual of 1e-13 per column, twice in a row, on matrices of
# condition below 10: 1e-10 of the largest entry, as above.
@pytest.mark.parametrize("n", [8, 11, 14, 17, 20, 23])   # 1152 .. 9522 unknowns: 2, 3, 4, 6, 8 and 10 rows a lane
def test_gram_solves_over_the_column_widths(bie, monkeypatch, n):
    """Chebyshev iteration in LDS against CG on the normal equations in memory."""
    op = bie.Operator(*cube_sphere(n, "ellipsoid", axes=(1.0, 1.2, 1.5)), 4.0)
    g = torch.Generator(device="cpu").manual_seed(n)
    X = torch.randn(3, op.N, dtype=torch.complex128, generator=g).cuda()
    Y, its = [], []
    for form in ("", "cgnr"):
        monkeypatch.setenv("BIE_CALDERON_GRAM", form)
        pc = bie.Calderon(op)
        info = pc.info()
        assert max(info["cg_relres"]) <= 1e-13
        Y.append(pc.apply(X))
        its.append(max(info["cg_iters"]))
        pc.close()
    assert its[0] < its[1]
    assert float((Y[0] - Y[1]).abs().max()) <= 1e-10 * float(Y[1].abs().max())
    op.close()
