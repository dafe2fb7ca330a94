"""The kept device blocks are given back on request, and operators made before and after
that are what they were."""
import pytest
import torch

from paper_2606_13482_amd.inputs import icosphere

pytestmark = pytest.mark.gpu


def test_closed_operators_memory_is_given_back(bie):
    V, T = icosphere(4)
    Vs, Ts = icosphere(2)
    alive = bie.Operator(Vs, Ts, 2.0)
    want = alive.matrix()
    bie.release_memory()
    torch.cuda.synchronize()
    base = torch.cuda.mem_get_info()[0]
    bie.Operator(V, T, 4.0).close()
    held = base - torch.cuda.mem_get_info()[0]
    assert held > 1 << 30            # 1.9 GB of pair blocks and 0.5 GB of matrix
    given = bie.release_memory()
    print(f"  held {held >> 20} MiB, given back {given >> 20} MiB", flush=True)
    assert given >= held - (64 << 20)
    assert base - torch.cuda.mem_get_info()[0] <= 64 << 20
    assert bie.release_memory() == 0
    assert torch.equal(alive.matrix(), want)
    op = bie.Operator(Vs, Ts, 2.0)
    assert torch.equal(op.matrix(), want)
    op.close()
    alive.close()
