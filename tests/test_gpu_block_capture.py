"""The split-BF16 block product captured with one number of vectors after an eager call with
another of the same 256-column block: nothing has to grow, whatever K slices the autotuner
has for the narrow blocks."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RUN = r"""
import sys
import torch
from paper_2606_13482_amd import bie
from paper_2606_13482_amd.inputs import complex_gaussian, icosphere
V, T = icosphere(2)
X = torch.from_numpy(complex_gaussian(480, 5, cols=128)).cuda()
for warm, R in ((40, 100), (20, 128), (20, 64), (64, 20)):
    print(warm, R, flush=True)
    op = bie.Operator(V, T, 3.0, storage="split_bf16")
    x, y = X[:R].contiguous(), torch.empty((R, 480), dtype=torch.complex128, device="cuda")
    op.apply(X[:warm].contiguous(), block=True)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        op.apply(x, block=True, out=y)
    bie.autotune(R <= 64)   # 256 columns have no choice yet: the captured product took the defaults
    for _ in range(3):
        y.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, op.apply(x, block=True))
        torch.cuda.synchronize()
    bie.autotune(True)
    del g
    op.close()
print("ok")
"""


def test_captured_beyond_the_warm_up(tmp_path):
    cache = tmp_path / "tune"   # one slice for the narrow blocks of 480 unknowns, fewer than the default
    cache.write_text("gemm_split:512x960:64:t3 0 1\ngemm_split:512x960:128:t3 0 1\n")
    p = subprocess.run([sys.executable, "-u", "-c", RUN], cwd=ROOT, capture_output=True, text=True, timeout=100,
                       env=dict(os.environ, BIE_AUTOTUNE_CACHE=str(cache)))
    assert p.returncode == 0 and p.stdout.strip().endswith("ok"), p.stdout + p.stderr[-2000:]
