"""Device blocks kept between operators: matrices built in memory that other
operators have used are bitwise those built first, also by several threads on
streams of their own; kept memory is bounded and goes back after a while."""
import threading
import time

import pytest
import torch

from paper_2606_13482_amd.inputs import icosphere

pytestmark = pytest.mark.gpu


def _matrix(bie, level, k, storage="c128"):
    V, T = icosphere(level)
    op = bie.Operator(V, T, k, storage=storage)
    Z = op.matrix(torch.complex64 if storage == "c64" else torch.complex128)
    op.close()
    return Z


def test_reused_blocks_bitwise(bie):
    cases = [(3, 2.0, "c128"), (2, 1.0, "c64"), (3, 4.0, "c64"), (2, 3.0, "c128")]
    want = [_matrix(bie, *c) for c in cases]
    bad = []

    def work(first):
        with torch.cuda.stream(torch.cuda.Stream()):
            for i in range(8):
                j = (first + i) % len(cases)
                Z = _matrix(bie, *cases[j])
                torch.cuda.current_stream().synchronize()
                if not torch.equal(Z, want[j]):
                    bad.append((first, i))

    threads = [threading.Thread(target=work, args=(t,)) for t in range(3)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad


def test_kept_memory_bounded_and_returned(bie):
    V, T = icosphere(0)
    bie.Operator(V, T, 1.0).close()
    time.sleep(2.2)
    bie.Operator(V, T, 1.0).close()      # releases what was idle
    torch.cuda.synchronize()
    base = torch.cuda.mem_get_info()[0]
    Vl, Tl = icosphere(4)
    for k in (2.0, 3.0):
        bie.Operator(Vl, Tl, k).close()
        kept = base - torch.cuda.mem_get_info()[0]
        print(f"  kept {kept / 2**20:.0f} MiB", flush=True)
        assert kept <= (4 << 30) + (64 << 20)
    time.sleep(2.2)
    bie.Operator(V, T, 1.0).close()
    assert base - torch.cuda.mem_get_info()[0] <= 64 << 20
