"""The test helpers themselves (no GPU needed)."""
import os
import subprocess
import sys
import textwrap

import numpy as np

from gpu_util import dev

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_dev_accepts_a_reversed_length_one_axis():
    """Reversing an axis of length 1 leaves a negative stride that
    ascontiguousarray keeps (the array still counts as contiguous); the helper
    must still hand torch a positive-stride copy."""
    X = np.arange(3, dtype=np.int32).reshape(3, 1)
    t = dev(X[:, ::-1], device="cpu")
    assert t.tolist() == [[0], [1], [2]]
    t = dev(np.arange(6, dtype=np.int32).reshape(2, 3)[:, ::-1], device="cpu")
    assert t.tolist() == [[2, 1, 0], [5, 4, 3]]


def test_package_imports_without_torchs_gpu_functions():
    """A torch built without GPU support lacks torch._C's stream functions; the
    package and its host-only calls load there."""
    code = textwrap.dedent("""
        import torch
        for name in [n for n in dir(torch._C) if n.startswith("_cuda_getCurrent")]:
            delattr(torch._C, name)
        import paper_2502_01637_amd as S
        print(S.discover_workspace_bytes(1, 1000, 3))
    """)
    p = subprocess.run([sys.executable, "-c", code], cwd=ROOT, capture_output=True, text=True)
    assert p.returncode == 0 and int(p.stdout) > 0, p.stderr[-2000:]
