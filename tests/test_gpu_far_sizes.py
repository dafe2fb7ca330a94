"""The multilevel far field's kernels over the sizes they are built for: splines per
axis up to 18 (the three forms of the way back), 16 points, degrees 1, 3 and 5, one to
three levels, target groups with a remainder, and several vectors; against the
oracle's multilevel product."""
import numpy as np
import pytest
import torch

from oracle import bspline as bs
from oracle.mesh import rwg_table
from paper_2606_13482_amd.inputs import complex_gaussian, icosphere

pytestmark = pytest.mark.gpu


# FP64 throughout on both sides: 1e-12 relative, as the other comparisons with the oracle.
@pytest.mark.parametrize("level,k,box,levels,s,p", [
    (2, 1.5, 0.8, 1, 6, 1), (2, 1.5, 0.9, 1, 9, 1), (2, 1.5, 0.8, 1, 8, 3), (2, 1.5, 0.9, 1, 7, 3),
    (3, 2.0, 0.7, 1, 12, 3), (3, 2.0, 0.7, 1, 14, 3), (2, 1.5, 0.9, 1, 11, 5), (3, 2.0, 0.7, 1, 13, 5),
    (3, 1.0, 0.35, 2, 10, 3), (3, 1.0, 0.35, 3, 8, 3), (3, 6.0, 0.35, 2, 8, 3)])
def test_multilevel_over_its_sizes(bie, level, k, box, levels, s, p):
    V, T = icosphere(level)
    op = bie.Operator(V, T, k)
    far = bie.FarFieldML(op, box, levels, s, p)
    X = complex_gaussian(op.N, 41, cols=2)
    Y = far.apply(torch.from_numpy(X).cuda())
    Yo, info = bs.ml_far_product(rwg_table(V, T), k, X, box, levels, s, p)
    sizes = [(c["boxes"], c["splines"], c["points_per_axis"]) for c in (far.level_info(l) for l in range(levels))]
    err = np.linalg.norm(Y.cpu().numpy() - Yo) / np.linalg.norm(Yo)
    print(f"  {sizes}: {err:.1e}", flush=True)
    assert err <= 1e-12
    again = far.apply(torch.from_numpy(X[1:]).cuda())
    assert torch.equal(again, Y[1:])          # vectors are independent, sums in a fixed order
    far.close()
    op.close()
