"""The binding's way to the current stream's handle: torch's internal call where there is one, its public one otherwise."""
import subprocess
import sys

import pytest

from test_abi import ROOT

CHILD = """
import sys, types
sys.path.insert(0, %r)
import torch
for name in %r:
    delattr(torch._C, name)
torch.cuda.current_stream = lambda: types.SimpleNamespace(cuda_stream=77)
if not %r:
    torch._C._cuda_getDevice = lambda: 3
    torch._C._cuda_getCurrentRawStream = lambda device: 1000 + device
import paper_2311_15806_amd.binding as b
print(b._stream())
"""


@pytest.mark.parametrize("missing,handle", [((), "1003"), (("_cuda_getCurrentRawStream",), "77"), (("_cuda_getDevice",), "77")])
def test_stream_handle(missing, handle):
    r = subprocess.run([sys.executable, "-c", CHILD % (ROOT, missing, missing)], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.split()[-1] == handle, r.stdout + r.stderr
