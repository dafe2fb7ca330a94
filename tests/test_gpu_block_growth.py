"""Split-BF16 block products: the partial sums that a wide product allocated serve narrower
ones too, so that a graph captured with the wide one still owns its memory after eager calls
of other widths."""
import pytest
import torch

from paper_2606_13482_amd.inputs import complex_gaussian, icosphere

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tuned", [False, True])
def test_narrow_after_wide_keeps_the_buffer(bie, tuned):
    V, T = icosphere(4)
    X = torch.from_numpy(complex_gaussian(7680, 5, cols=512)).cuda()
    narrow = [X[:R].contiguous() for R in (1, 20, 33, 64, 65, 128)]
    bie.autotune(tuned)
    try:
        op = bie.Operator(V, T, 10.0, storage="split_bf16")
        y = torch.empty_like(X)
        want = op.apply(X, block=True)
        outs = [torch.empty_like(x) for x in narrow]
        torch.cuda.synchronize()
        free = torch.cuda.mem_get_info()[0]
        for x, o in zip(narrow, outs):
            op.apply(x, block=True, out=o)
        torch.cuda.synchronize()
        assert torch.cuda.mem_get_info()[0] == free
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g):
            op.apply(X, block=True, out=y)
        for _ in range(3):
            for x, o in zip(narrow, outs):
                op.apply(x, block=True, out=o)
            y.zero_()
            g.replay()
            torch.cuda.synchronize()
            assert torch.equal(y, want)
        del g
        op.close()
    finally:
        bie.autotune(True)
