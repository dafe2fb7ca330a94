"""Columns of at most 1024 unknowns: the whole Arnoldi step in one block, with the
product's partial sums added there, against the launches that larger columns take.
Both add in the same order, so a small operator solved beside a large one (whose
columns set the launches of the batch) is bitwise the small one solved alone.  And
the allocation-free product in several passes over its scratch."""
import pytest
import torch

from paper_2606_13482_amd.inputs import complex_gaussian, icosphere, planewave_set, random_directions

pytestmark = pytest.mark.gpu


def _rhs(op, count):
    return op.rhs(*planewave_set(random_directions(count, 5), "theta"))


@pytest.mark.parametrize("level,k,count,m", [(0, 1.0, 1, 5), (1, 2.0, 3, 30), (2, 2.0, 2, 30), (2, 5.0, 1, 64)])
def test_alone_equals_beside_a_large_one(bie, level, k, count, m):
    small, large = bie.Operator(*icosphere(level), k), bie.Operator(*icosphere(3), 2.0)
    Bs, Bl = _rhs(small, count), _rhs(large, 1)
    opts = bie.Solve(restart=m, tol=1e-8)
    bie.batch_config(-1)
    try:
        Xs, st = bie.batch_solve([small, large], [Bs, Bl], opts)
        Xo, so = bie.batch_solve([small], [Bs], opts)
    finally:
        bie.batch_config(0)
    X1, s1 = small.solve(Bs, opts)
    print("  ", small.N, [s["iters"] for s in s1], flush=True)
    assert torch.equal(Xs[0], Xo[0]) and torch.equal(Xs[0], X1)
    assert [s["iters"] for s in st[0]] == [s["iters"] for s in s1] == [s["iters"] for s in so[0]]
    assert all(s["converged"] for s in s1)
    small.close()
    large.close()


@pytest.mark.parametrize("R", [1, 2048, 2049, 3500])
def test_noalloc_in_passes(bie, R):
    op = bie.Operator(*icosphere(2), 2.0)
    X = torch.from_numpy(complex_gaussian(op.N, 3, cols=R)).cuda()
    Y = torch.empty_like(X)
    rc = bie._lib.bie_apply_noalloc(op._h, bie._dev(X, torch.complex128), bie._dev(Y, torch.complex128, X.shape), R,
                                    bie.BIE_C128, 0, bie._stream())
    torch.cuda.synchronize()
    assert rc == bie.BIE_OK and torch.equal(Y, op.apply(X))
    op.close()
