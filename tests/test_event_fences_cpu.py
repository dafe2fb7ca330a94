"""Events that order streams keep their memory fences: what they order includes copies
from the host (the block solver's tables), which a second stream's kernels read."""
import glob
import os
import re

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_no_event_is_created_without_its_fence():
    seen = 0
    for path in sorted(glob.glob(os.path.join(ROOT, "paper_2606_13482_amd", "csrc", "*.*"))):
        text = open(path).read()
        for call in re.findall(r"hipEventCreateWithFlags\(.*?\);", text, flags=re.S):
            seen += 1
            assert "DisableSystemFence" not in call and "ReleaseToDevice" not in call, (os.path.basename(path), call)
    assert seen
