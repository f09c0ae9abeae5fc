"""A stand-in for the few runtime calls the library makes on its way to a launch (two devices, no GPU needed): it records what
is launched.  The library runs on it in a process of its own."""
import json
import os
import subprocess
import sys

FAKE = r"""
#include <stddef.h>
static int current = 0, lookups = 0, named = 0, registered = 0;
static struct { const void *stub; const char *name; } kernels[2048];     /* what the library registers when it is loaded */
static unsigned long launched[5];                        /* kernel, stream, workgroups, threads, LDS bytes */
int fake_set(int d) { current = d; return 0; }
int fake_current(void) { return current; }
int fake_lookups(void) { return lookups; }
unsigned long fake_launched(int i) { return launched[i]; }
void fake_name_kernels(void) { named = 1; }              /* handles that stand for the kernel's name, not for the device */
const char *fake_kernel(void) { return named ? (const char *)launched[0] : ""; }
void __hipRegisterFunction(void **modules, const void *stub, char *fn, const char *name, unsigned limit, void *t, void *b, void *bd,
                           void *gd, int *ws)
{
    if (registered < 2048) kernels[registered].stub = stub, kernels[registered++].name = name;
}
int hipGetDevice(int *d) { *d = current; return 0; }
int hipSetDevice(int d) { current = d; return d < 2 ? 0 : 101; }
int hipGetDeviceCount(int *n) { *n = 2; return 0; }
int hipStreamGetDevice(void *s, int *d) { if ((unsigned long)s >= 0x3000) return 400; *d = (unsigned long)s >= 0x2000; return 0; }
int hipDeviceGetAttribute(int *v, int attr, int d) { *v = 160 * 1024; return 0; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st) { return 0; }
int hipStreamSynchronize(void *s) { return 0; }
int hipGetLastError(void) { return 0; }
int hipFuncSetAttribute(const void *f, int a, int v) { return 0; }
int hipGetFuncBySymbol(void **f, const void *sym)
{
    ++lookups;
    *f = (void *)(0x100ul * (current + 1));
    for (int i = 0; named && i < registered; ++i)
        if (kernels[i].stub == sym) *f = (void *)kernels[i].name;
    return 0;
}
int hipModuleLaunchKernel(void *f, unsigned gx, unsigned gy, unsigned gz, unsigned bx, unsigned by, unsigned bz, unsigned lds,
                          void *stream, void **params, void **extra)
{
    launched[0] = (unsigned long)f, launched[1] = (unsigned long)stream, launched[2] = gx, launched[3] = bx, launched[4] = lds;
    return 0;
}
"""

HEAD = r"""
import ctypes, json, sys
sys.modules["torch"] = None                              # the library alone, on the stand-in
fake = ctypes.CDLL(sys.argv[1], ctypes.RTLD_GLOBAL)      # found before the runtime the library names
fake.fake_launched.restype = ctypes.c_ulong
fake.fake_kernel.restype = ctypes.c_char_p
sys.path[:0] = [sys.argv[2], sys.argv[2] + "/tests"]
import numpy as np
from paper_2507_12205_amd import binding as B
arg = json.loads(sys.argv[3])
KERNEL, STREAM, GRID, THREADS, LDS = range(5)
"""


def run(tmp_path, code, arg=None):
    """Runs `code` in a process of its own (HEAD before it, `arg` in hand); what it prints last comes back, from JSON."""
    src, so = tmp_path / "fake.c", tmp_path / "libfake.so"
    src.write_text(FAKE)
    subprocess.run(["gcc", "-shared", "-fPIC", "-o", str(so), str(src)], check=True)
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    res = subprocess.run([sys.executable, "-c", HEAD + code, str(so), root, json.dumps(arg)], capture_output=True, text=True,
                         timeout=300)
    assert res.returncode == 0, res.stderr[-2000:]
    return json.loads(res.stdout.strip().splitlines()[-1])
