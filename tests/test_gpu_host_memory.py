"""The pinned memory that kernels report through: an error where it cannot be
had, never a null address left for the calls after."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

# In the child process, found before the runtime's own: the first request for a
# device address fails, later ones get the host address, which is the same.
STUB = """
int hipHostGetDevicePointer(void** d, void* p, unsigned flags) {
    static int calls = 0;
    *d = calls++ ? p : 0;
    return *d ? 0 : 1;
}
"""

USE = """
import ctypes, sys
ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)
import numpy as np, torch
from paper_2408_03036_amd import tpcf as T
torch.zeros(1, device='cuda')
try:
    T.Handle(100.0, np.linspace(5.0, 20.0, 4), 2)
    print('no error')
except T.TpcfError as e:
    print('refused', e)
h = T.Handle(100.0, np.linspace(5.0, 20.0, 4), 2)
h.build_grid(torch.rand((300, 3), dtype=torch.float64, device='cuda') * 100.0)
print('precision', h.precision(torch.eye(3, dtype=torch.float64, device='cuda') * 4.0, 10).cpu().numpy()[0, 0])
"""


def test_no_device_address(tmp_path):
    src, lib = tmp_path / "stub.c", tmp_path / "stub.so"
    src.write_text(STUB)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(lib), str(src)], check=True)
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", USE, str(lib)], cwd=root, env=dict(os.environ, PYTHONPATH=root),
                       capture_output=True, text=True, timeout=100)
    print(r.stdout, r.stderr[-2000:], flush=True)
    assert r.returncode == 0
    assert "refused" in r.stdout
    # Hartlap factor (10 - 3 - 2) / 9 over a variance of 4
    assert abs(float(r.stdout.split("precision")[1]) - 5.0 / 36.0) < 1e-15
