"""The two ways into the encoder (dense rows and CSR) give the same image, a CSR matrix takes memory by its entries, and block
columns are cut into units as defined where runs end inside a word of 64 columns, at its edge, or at the largest delta."""
import os
import subprocess
import sys

import numpy as np
import pytest
import scipy.sparse as sp

import paper_2507_12205_amd as E
from paper_2507_12205_amd import binding


def _matrix(m, n, ld, dtype, seed):
    rng = np.random.default_rng(seed)
    keep = rng.random((m, n)) < 0.4
    if m >= 8 and n >= 200:
        keep[np.ix_(rng.choice(m, 8, replace=False), rng.choice(n, 160, replace=False))] = True
        keep[:, n // 3:n // 3 + 300] = False                              # gaps beyond 255 columns
    full = np.zeros((m, ld), dtype=dtype)
    W = full[:, :n]
    W[...] = np.where(keep, rng.standard_normal((m, n)), 0)
    W[rng.random((m, n)) < 0.05] = -0.0                                    # not stored
    return W


@pytest.mark.parametrize("delta_bits", [4, 8, 16])
@pytest.mark.parametrize("m,n,ld", [(1, 1, 1), (3, 63, 70), (17, 64, 64), (40, 65, 66), (64, 1029, 1031), (33, 700, 707)])
@pytest.mark.parametrize("dtype", [np.float16, np.float32])
def test_dense_and_csr_builds_agree(m, n, ld, dtype, delta_bits):
    if dtype == np.float32 and delta_bits == 16:
        pytest.skip("absolute columns exist for FP16 values only")
    W = _matrix(m, n, ld, dtype, seed=m * 7919 + n)
    opts = E.make_opts(delta_bits=delta_bits)
    S = sp.csr_matrix(W.astype(np.float64))
    S.sort_indices()
    if dtype == np.float16:
        a, b = E.ecspmv_build_dense(W, opts), E.ecspmv_build_csr(S.indptr, S.indices, S.data.astype(dtype), m, n, opts)
        r, c, v = a.ecspmv_decode()
    else:
        a, b = E.ecspmv_build_dense_f32(W, opts), E.ecspmv_build_csr_f32(S.indptr, S.indices, S.data.astype(dtype), m, n, opts)
        r, c, v = a.ecspmv_decode_f32()
    assert np.array_equal(a.ecspmv_export_image(), b.ecspmv_export_image())
    back = np.zeros((m, n), dtype=dtype)
    back[r, c] = v.view(dtype)
    assert np.array_equal(back, W) and r.size == np.count_nonzero(W)


def _both(W, opts):
    """the images of W built from its rows and from CSR"""
    S = sp.csr_matrix(W.astype(np.float64))
    S.sort_indices()
    f32 = W.dtype == np.float32
    a = (E.ecspmv_build_dense_f32 if f32 else E.ecspmv_build_dense)(W, opts)
    b = (E.ecspmv_build_csr_f32 if f32 else E.ecspmv_build_csr)(S.indptr, S.indices, S.data.astype(W.dtype), *W.shape, opts)
    return a, b


# the bits of a CSR matrix are kept where a row has an entry per word of 64 columns or more, else made panel by panel, and not at all
# in panels without units
@pytest.mark.parametrize("flags", [0, binding.FLAG_CLUSTER_ROWS, binding.FLAG_GLOBAL_MATCHING])
@pytest.mark.parametrize("background,blocks,kept", [(0, 0, False), (1, 0, False), (1, 1, False), (33, 0, False), (34, 0, True),
                                                    (14, 1, False), (20, 1, True), (60, 2, True)])
@pytest.mark.parametrize("dtype,delta_bits", [(np.float16, 4), (np.float16, 8), (np.float16, 16), (np.float32, 8)])
def test_sparse_csr_builds_agree(background, blocks, kept, flags, dtype, delta_bits):
    m, n, words = 60, 2150, 34                            # 34 words of 64 columns, the last one not full
    rng = np.random.default_rng(100 * background + blocks)
    W = np.zeros((m, n), dtype=dtype)
    for i in range(m):
        W[i, rng.choice(n, background, replace=False)] = rng.standard_normal(background)
    for k in range(blocks):                               # rows of one panel and of several
        rows = np.arange(8) + 16 * k if k % 2 == 0 else rng.choice(m, 8, replace=False)
        W[np.ix_(rows, 200 * k + np.arange(130))] = 1.0 + k
    dense, csr = _both(W, E.make_opts(delta_bits=delta_bits, num_panels=4, flags=flags))
    assert np.array_equal(dense.ecspmv_export_image(), csr.ecspmv_export_image())
    assert (sum(csr.ecspmv_stats().units_by_g[1:]) > 0) == (blocks > 0)
    assert (np.count_nonzero(W) >= m * words) == kept


CHILD = r"""
import sys
sys.modules["torch"] = None                               # the library alone
sys.path.insert(0, sys.argv[1])
import numpy as np
from paper_2507_12205_amd import binding as B
m, n = 400000, 10000
first = np.random.default_rng(1).integers(0, n - 1, m)
col = np.stack([first, first + 1], 1).astype(np.int32).ravel()
args = np.arange(m + 1, dtype=np.int64) * 2, col, np.ones(2 * m, np.float16), m, n, B.make_opts(num_threads=2)
peak = lambda: int(open("/proc/self/status").read().split("VmHWM:")[1].split()[0]) * 1024
before = peak()
A = B.ecspmv_build_csr(*args)
print(peak() - before, A.ecspmv_device_bytes())
"""


def test_memory_of_a_tall_sparse_csr_build():
    """Beyond the image: a copy of the entries (8 bytes each), and per row a few tables of 4 or 8 bytes and its share of the panels in
    work.  A bit for every column of every row would be 500 MB."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    res = subprocess.run([sys.executable, "-c", CHILD, root], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-2000:]
    grown, image = map(int, res.stdout.split())
    m, n, panels, threads = 400000, 10000, 256, 2
    in_work = threads * (m // panels + 1) * (n // 64 + 1) * 8 * 2          # bits of a panel, and as much again on top
    assert grown < image + 8 * 2 * m + 100 * m + in_work + (32 << 20), (grown, image)


def _units(cols, max_delta):
    """Units of 64 columns of every longest sequence of columns with gaps of at most max_delta, from its first column on."""
    out = []
    for run in np.split(cols, np.nonzero(np.diff(cols) > max_delta)[0] + 1):
        whole = len(run) // 64 * 64
        out += list(run[:whole].reshape(-1, 64))
    return out


@pytest.mark.parametrize("delta_bits,gaps", [(4, [15, 16]), (8, [255, 256])])
@pytest.mark.parametrize("first", [0, 1, 37, 63])
@pytest.mark.parametrize("lengths", [(64, 64), (63, 65), (70, 130, 64), (128, 1, 63, 64)])
def test_runs_are_cut_where_the_gap_exceeds_the_largest_delta(delta_bits, gaps, first, lengths):
    # runs of neighbouring columns, `gap` columns from the last of one to the first of the next
    for gap in gaps:
        cols, at = [], first
        for length in lengths:
            cols += range(at, at + length)
            at += length - 1 + gap
        cols = np.array(cols)
        W = np.zeros((2, int(cols[-1]) + 1), dtype=np.float16)
        W[:, cols] = 1.0
        A = E.ecspmv_build_dense(W, E.make_opts(delta_bits=delta_bits, max_granularity=2, num_panels=1, flags=binding.FLAG_KEEP_SMALL_SETS))
        g, _, unit_cols = A.ecspmv_block_sets()
        want = _units(cols, 2 ** delta_bits - 1)
        assert len(g) == len(want) and np.array_equal(unit_cols.reshape(-1, 64), np.array(want).reshape(-1, 64))


LEAK = r"""
import ctypes, resource, sys
sys.modules["torch"] = None
sys.path.insert(0, sys.argv[1])
import numpy as np
from paper_2507_12205_amd import binding as B
class Info(ctypes.Structure):
    _fields_ = [(k, ctypes.c_size_t) for k in ("arena", "ordblks", "smblks", "hblks", "hblkhd", "usmblks", "fsmblks", "uordblks", "fordblks",
                                               "keepcost")]
info = ctypes.CDLL(None).mallinfo2
info.restype = Info
lib, W, out = B.lib(), np.zeros((60000, 20000), np.uint16), ctypes.c_void_p(0)     # 150 MB of bits
build = lambda: lib.ecspmv_build_dense(W.ctypes.data, *W.shape, W.shape[1], None, ctypes.byref(out))
size = int(open("/proc/self/status").read().split("VmSize:")[1].split()[0]) * 1024
resource.setrlimit(resource.RLIMIT_AS, (size + (64 << 20), -1))
statuses = {build()}
before = info().uordblks
for _ in range(1000):
    statuses.add(build())
print(sorted(statuses) == [B.ERR_NOMEM], info().uordblks - before)
"""


def test_a_build_that_runs_out_of_memory_leaves_nothing_behind():
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    res = subprocess.run([sys.executable, "-c", LEAK, root], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr[-2000:]
    refused, left = res.stdout.split()
    assert refused == "True" and int(left) < 100 * 1000         # less than a hundred bytes a call


SCRATCH = r"""
#include <cstdlib>
#include <new>
#include <atomic>
static std::atomic<long long> asked{0};
static void *counted(size_t n) { asked += (long long)n; return (malloc)(n); }
void *operator new(size_t n) { return counted(n); }
void operator delete(void *p) noexcept { free(p); }
void operator delete(void *p, size_t) noexcept { free(p); }
namespace std { using ::counted; }
#define malloc counted                                    // std::malloc as well
#include "%s/paper_2507_12205_amd/csrc/encoder.cpp"
#include <cstdio>
int main()
{
    const int m = 2000, n = 60000;
    std::vector<int64_t> rowptr(m + 1);
    std::vector<int32_t> col(2 * m);
    std::vector<uint16_t> val(2 * m, 0x3C00);
    for (int i = 0; i < m; ++i) rowptr[i + 1] = 2 * (i + 1), col[2 * i] = i, col[2 * i + 1] = i + 1000;
    ecs::Csr A;
    ecs::csr_from_csr(rowptr.data(), col.data(), val.data(), m, n, A);
    ecs::BuildParams bp;
    bp.num_panels = m, bp.num_threads = 2;
    ecs::Image im;
    const long long before = asked;
    const int e = ecs::build_image({m, n, 16, nullptr, 0, &A}, bp, im);
    printf("%%d %%lld\n", e, (asked - before - (long long)im.bytes.size()) / m);
}
"""


def test_memory_asked_for_by_a_small_panel(tmp_path):
    """A panel of one row with two entries and 60000 columns: beside the bits of a row, 7.5 KB, held by the panel and twice more while it is cut
    into units, only what goes by its entries, no list as long as the matrix is wide (120 KB)."""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    src, exe = tmp_path / "scratch.cpp", tmp_path / "scratch"
    src.write_text(SCRATCH % root)
    subprocess.run(["g++", "-O1", "-std=c++17", "-mpopcnt", "-pthread", "-w", str(src), "-o", str(exe)], check=True)
    status, per_panel = map(int, subprocess.run([str(exe)], capture_output=True, text=True, check=True, timeout=300).stdout.split())
    assert status == 0 and per_panel < 4 * 7504 + 8192, per_panel


@pytest.mark.parametrize("delta_bits", [4, 8, 16])
@pytest.mark.parametrize("density", [0.002, 0.05, 0.5])
def test_histogram_of_deltas_counts_entries(delta_bits, density):
    """Every stored entry but a row's first, by the delta it has behind the zeros that fill its gap; rows with such zeros and without"""
    W = np.where(np.random.default_rng(3).random((40, 3000)) < density, np.float16(1), np.float16(0))
    W[::3, ::5] = 1                                        # gaps of five columns at most
    A, most = E.ecspmv_build_dense(W, E.make_opts(delta_bits=delta_bits, max_granularity=1)), 2 ** delta_bits - 1
    want = [0] * 9
    for row in W:
        for gap in np.diff(np.nonzero(row)[0]).tolist():
            want[min(8, (gap - (gap - 1) // most * most).bit_length())] += 1
    assert list(A.ecspmv_stats().delta_hist) == want
