"""Block GMRES at the edges of its small dense kernels (tiles of 8, 16 and 32
columns, the last group narrower): solutions against the oracle's LU solve, and
the least-squares estimate of the last step against the true residual, which
tests the reflectors, their triangular factor and the back substitution.  The
estimate follows the true residual to the rounding of some tens of FP64 steps
times the matrix's condition, below 1e-11 of the right-hand side here; a residual
of 1e-8 leaves the solutions within 1e-5 at conditions below 1e3."""
import numpy as np
import pytest
import torch

from oracle import cfill
from oracle.mesh import rwg_table
from paper_2606_13482_amd.inputs import icosphere, planewave_set, random_directions

pytestmark = pytest.mark.gpu

_CACHE = {}


def _case(level, k):
    if (level, k) not in _CACHE:
        V, T = icosphere(level)
        _CACHE[level, k] = (V, T, cfill.fill(rwg_table(V, T), k))
    return _CACHE[level, k]


@pytest.mark.parametrize("precision", ["plain", "mixed"])
@pytest.mark.parametrize("block", [1, 2, 7, 8, 9, 15, 16, 17, 24, 31, 32])
def test_widths(bie, block, precision):
    V, T, Zo = _case(2, 2.0)
    op = bie.Operator(V, T, 2.0, storage="split_bf16")
    d, e = planewave_set(random_directions(block + (block + 1) // 2, 9), "theta")
    B = op.rhs(d, e)
    X, st = op.solve(B, bie.Solve(method="bgmres", block=block, restart=20, tol=1e-8, precision=precision))
    Xo = np.linalg.solve(Zo, B.cpu().numpy().T).T
    fwd = np.linalg.norm(X.cpu().numpy() - Xo, axis=1) / np.linalg.norm(Xo, axis=1)
    gap = max(abs(s["relres_est"] - s["relres_true"]) for s in st)
    print(f"  block {block} {precision}: iterations {max(s['iters'] for s in st)}, vs LU {fwd.max():.1e}, estimate {gap:.1e}",
          flush=True)
    assert all(s["converged"] for s in st) and max(s["relres_true"] for s in st) <= 1e-8
    assert fwd.max() <= 1e-5
    if precision == "plain":
        assert gap <= 1e-11
    op.close()
