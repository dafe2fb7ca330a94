"""Work units of the packed product: the autotuner's choices lie in the sets that products
of several vectors bear, and on both sides of each line of the units and of the passes
several vectors are each on its own, bit for bit, and the product of the full matrix."""
import pytest
import torch

from paper_2606_13482_amd.inputs import cube_sphere

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,storage,units", [(5, "c128", (2, 4)), (8, "c128", (2, 4)), (10, "c128", (2, 4)),
                                             (7, "c64", (2, 4)), (8, "c64", (4, 8)), (12, "c128", (4, 8)),
                                             (17, "c128", (8, 4, 0, 16))])
def test_chosen_units(bie, n, storage, units):
    bie.autotune(True)
    op = bie.Operator(*cube_sphere(n, "ellipsoid", axes=(1.0, 1.1, 1.4)), 3.0, storage=storage)
    key = f"sym:{op.N}:{'f64' if storage == 'c128' else 'f32'}"
    chosen = bie.autotune_report()[key]
    op.close()
    assert chosen[0] in units


# unknowns 882, 1152 (FP32: units of 2 and 4 tiles; FP64: passes) | 1458, 1800 (FP32: passes) |
# 1800, 2178 (FP64: units of 2 and 4 tiles) | 4608, 5202 (4 and 8)
@pytest.mark.parametrize("n,storage", [(5, "c128"), (7, "c64"), (8, "c64"), (9, "c64"), (10, "c64"), (7, "c128"),
                                       (8, "c128"), (10, "c128"), (11, "c128"), (16, "c64"), (17, "c64")])
@pytest.mark.parametrize("tune", [False, True])
def test_columns_on_both_sides_of_the_lines(bie, n, storage, tune):
    bie.autotune(tune)
    op = bie.Operator(*cube_sphere(n, "ellipsoid", axes=(1.0, 1.1, 1.4)), 3.0, storage=storage)
    bie.autotune(True)
    g = torch.Generator(device="cpu").manual_seed(n)
    for dtype in (torch.complex128,) if storage == "c128" else (torch.complex128, torch.complex64):
        X = torch.randn(33, op.N, dtype=torch.complex128, generator=g).to("cuda", dtype)
        one = torch.cat([op.apply(X[r:r + 1]) for r in range(33)])
        for R in (2, 3, 5, 16, 32, 33):
            assert torch.equal(op.apply(X[:R].contiguous()), one[:R]), (dtype, R)
        if op.N == 450:   # many vectors: the line by tiles and vectors lies between 138 and 139
            Xm = torch.randn(140, op.N, dtype=torch.complex128, generator=g).to("cuda", dtype)
            assert torch.equal(op.apply(Xm), torch.cat([op.apply(Xm[:70].contiguous()), op.apply(Xm[70:].contiguous())]))
        if op.N <= 2178 and dtype == torch.complex128:
            Z = op.matrix(torch.complex128)
            want = (Z.cpu() @ X.T.cpu()).T
            err = (one.cpu() - want).abs().max() / want.abs().max()
            # N terms a sum, each product and addition rounded in 64 bits
            assert err <= 4 * op.N ** 0.5 * 2.0 ** -52, float(err)
    op.close()
