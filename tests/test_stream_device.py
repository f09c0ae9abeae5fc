"""A launch goes to the device of its stream, also where another device is the current one: the library against a stand-in
for the few runtime calls it makes on that way (two devices, no GPU needed), in a process of its own."""
import json
import os
import subprocess
import sys

FAKE = r"""
#include <stddef.h>
static int current = 0;
static unsigned long launched_f, launched_stream; static int launched_current, lookups;
int fake_set(int d) { current = d; return 0; }
int fake_current(void) { return current; }
int fake_lookups(void) { return lookups; }
unsigned long fake_f(void) { return launched_f; }
unsigned long fake_stream(void) { return launched_stream; }
int hipGetDevice(int *d) { *d = current; return 0; }
int hipSetDevice(int d) { current = d; return d < 2 ? 0 : 101; }
int hipGetDeviceCount(int *n) { *n = 2; return 0; }
int hipStreamGetDevice(void *s, int *d) { if ((unsigned long)s >= 0x3000) return 400; *d = (unsigned long)s >= 0x2000; return 0; }
int hipDeviceGetAttribute(int *v, int attr, int d) { *v = 160 * 1024; return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) { return 0; }
int hipStreamSynchronize(void *s) { return 0; }
int hipGetLastError(void) { return 0; }
int hipFuncSetAttribute(const void *f, int a, int v) { return 0; }
int hipGetFuncBySymbol(void **f, const void *sym) { ++lookups; *f = (void *)(0x100ul * (current + 1)); return 0; }
int hipModuleLaunchKernel(void *f, unsigned gx, unsigned gy, unsigned gz, unsigned bx, unsigned by, unsigned bz, unsigned lds,
                          void *stream, void **params, void **extra)
{
    launched_f = (unsigned long)f, launched_stream = (unsigned long)stream;
    return 0;
}
"""

CHILD = r"""
import ctypes, json, sys
sys.modules["torch"] = None                              # the library alone, on the stand-in
fake = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)      # found before the runtime the library names
fake.fake_f.restype = fake.fake_stream.restype = ctypes.c_ulong
sys.path.insert(0, sys.argv[2])
import numpy as np
from paper_2507_12205_amd import binding as B
W = (np.arange(64 * 64).reshape(64, 64) % 3 == 0).astype(np.float16)
A = B.ecspmv_build_dense(W)
A.ecspmv_upload(0x100000, A.ecspmv_device_bytes(), 0)
out = []
def launch(stream, call):
    try:
        call(stream)
        out.append([stream, fake.fake_f(), fake.fake_stream(), fake.fake_current()])
    except B.EcspmvError as e:
        out.append([stream, "refused", e.status, fake.fake_current()])
one = lambda s: A.ecspmv_run(0x200000, 0x300000, s)
two = lambda s: A.ecspmv_run_multi(0x200000, 0x300000, 2, s)
for current in (0, 1):
    fake.fake_set(current)
    for call in (one, two):
        for s in (0x1000, 0x2000, 0, 0x2000):
            launch(s, call)
launch(0x3000, one)
print(json.dumps({"out": out, "lookups": fake.fake_lookups(), "hip": B.ERR_HIP}))
"""


def test_launch_on_the_streams_device(tmp_path):
    src, so = tmp_path / "fake.c", tmp_path / "libfake.so"
    src.write_text(FAKE)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(so), str(src)], check=True)
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    res = subprocess.run([sys.executable, "-c", CHILD, str(so), root], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, res.stderr[-2000:]
    got = json.loads(res.stdout.strip().splitlines()[-1])
    want = []
    for current in (0, 1):
        for _ in range(2):
            for stream, dev in ((0x1000, 0), (0x2000, 1), (0, current), (0x2000, 1)):
                want.append([stream, 0x100 * (dev + 1), stream, current])
    assert got["out"][:-1] == want
    assert got["out"][-1] == [0x3000, "refused", got["hip"], 1]          # a stream that is none
    assert got["lookups"] == 4                                           # one per kernel and device
