"""The split-BF16 block product with 64-, 128- and 256-column blocks: a column's
sums do not depend on the block's width nor on the columns beside it, so at equal
K slices every product is bitwise the first columns of a 256-column one."""
import pytest
import torch

from paper_2606_13482_amd.inputs import complex_gaussian, icosphere

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("level", [1, 3])
def test_widths_bitwise(bie, level):
    V, T = icosphere(level)
    bie.autotune(False)
    op = bie.Operator(V, T, 3.0, storage="split_bf16")
    X = torch.from_numpy(complex_gaussian(op.N, 5, cols=128)).cuda()
    Y = op.apply(X, block=True)
    for R in (1, 2, 31, 32, 33, 63, 64, 65, 96, 127):
        print("  ", op.N, R, flush=True)
        assert torch.equal(op.apply(X[:R].contiguous(), block=True), Y[:R])
    op.close()
    bie.autotune(True)
