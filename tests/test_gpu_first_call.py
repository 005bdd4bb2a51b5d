"""The first solve of a process finds its kernels on the device: they are put
there with the first plan, so that neither solve() nor solve_refined_noalloc
takes device memory for code.  In a process of its own (this one has loaded
everything already), over lengths from every unit of the library: the
per-length transforms and eliminations, the staging forms of 256 and 512, the
direct elimination."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import numpy as np, torch
from paper_1802_10323_amd import Plan
shapes = [(24, 30, 33), (32, 36, 144), (40, 48, 250), (50, 54, 64), (256, 512, 20), (270, 480, 17)]
plans = [Plan(*s, 1.0, 1.0, np.ones(s[2]), ("P", "ND", "DD")) for s in shapes]
shapes.append((64, 60, 128))
plans.append(Plan(*shapes[-1], 1.0, 1.0, np.ones(128), ("DD", "NN", "P")))     # lines along x
fields = [torch.ones(s, dtype=torch.float64, device="cuda") for s in shapes]
torch.cuda.synchronize()
free = torch.cuda.mem_get_info()[0]
for s, p, f in zip(shapes, plans, fields):
    p.solve_refined_noalloc(f, 1e-10, 3)
    p.solve(f)
    torch.cuda.synchronize()
    print(s, "device memory taken", free - torch.cuda.mem_get_info()[0], flush=True)
assert torch.cuda.mem_get_info()[0] == free
"""


def test_first_calls_take_no_device_memory():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    out = subprocess.run([sys.executable, "-u", "-c", CHILD], cwd=ROOT, capture_output=True, text=True,
                         timeout=100)
    print(out.stdout, out.stderr[-2000:], flush=True)
    assert out.returncode == 0, out.stderr[-2000:]
