"""Which torch functions the device helpers need: a call with a stream of its own works on a torch without the private ones that
give the current stream as a plain handle; only a call without a stream asks for them."""
import json
import subprocess
import sys

CODE = r"""
import json, torch
for name in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
    if hasattr(torch._C, name):
        delattr(torch._C, name)
from paper_2507_12205_amd import device
class Tensor:
    dtype, is_cuda, shape = torch.float16, True, (4, 2)
    def is_contiguous(self): return True
    def dim(self): return 2
    def data_ptr(self): return 0x1000
class Matrix:
    value_bits = 16
    def ecspmv_run(self, *args): calls.append(args)
    def ecspmv_run_multi(self, *args): calls.append(args)
class Stream:
    cuda_stream = 0x55
calls, refused, t = [], [], Tensor()
for call in (device.run, device.run_multi):
    call(Matrix(), t, t, stream=Stream())
    try:
        call(Matrix(), t, t)
    except AttributeError as e:
        refused.append(type(e).__name__)
print(json.dumps([calls, refused]))
"""


def test_a_given_stream_needs_nothing_private():
    res = subprocess.run([sys.executable, "-c", CODE], capture_output=True, text=True, timeout=240)
    assert res.returncode == 0, res.stderr[-1500:]
    calls, refused = json.loads(res.stdout.strip().splitlines()[-1])
    assert calls == [[0x1000, 0x1000, 0x55], [0x1000, 0x1000, 2, 0x55]] and refused == ["AttributeError"] * 2
