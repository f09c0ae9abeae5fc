"""Which kernel a launch takes, on both sides of every line: the variants for several matrices, the staging variants (16-byte pieces of
tables and x per thread), phases, and the widths of deltas and values."""
import batch_cases
import pytest
import standin
import x_first_cases

HEAD = r"""
import re
fake.fake_name_kernels()
X, Y = 0x200000, 0x300000
def upload(W, **o):
    f32 = W.dtype == np.float32
    A = (B.ecspmv_build_dense_f32 if f32 else B.ecspmv_build_dense)(W, B.make_opts(**o))
    A.ecspmv_upload(0x100000, A.ecspmv_device_bytes(), 0)
    return A
def kernel():
    return [int(v) for v in re.findall(r"Li(\d+)E", re.search(r"ecspmv_kernelI((?:Li\d+E){6})E", fake.fake_kernel().decode()).group(1))]
"""

BATCH = HEAD + r"""
import batch_cases as C
out = []
for c in arg:
    mats = [upload(C.matrix(c, k), **C.options(c)) for k in range(c["count"])]
    B.ecspmv_run_batch(mats, [X + 2 * (k % 2) for k in range(c["count"])], [Y] * c["count"], 0)
    st = [A.ecspmv_stats() for A in mats]
    out.append(dict(kernel=kernel(), grid=fake.fake_launched(GRID), chunks=sum(C.chunks(s) for s in st) / sum(s.num_panels for s in st),
                    per_wave=64 * sum(C.block_chunks(s) for s in st) / fake.fake_launched(GRID) / fake.fake_launched(THREADS),
                    sets=[int(any(s.units_by_g[g] for s in st)) for g in range(1, 5)]))
print(json.dumps(out))
"""


@pytest.mark.parametrize("cases", [batch_cases.RESIDUAL, batch_cases.ONE_SET], ids=["residual", "one_set"])
def test_several_matrices(tmp_path, cases):
    for c, got in zip(cases, standin.run(tmp_path, BATCH, cases)):
        tm, mode, k = c["kernel"]
        assert c["chunks"][0] <= got["chunks"] <= c["chunks"][1], (c, got)           # the case is what it says
        assert got["grid"] == c["panels"] * c["count"] and got["sets"] == [tm, 0, 0, 0], (c, got)
        if tm:
            assert (got["per_wave"] < 0.7) if mode == 2 else (got["per_wave"] > 0.76), (c, got)
        assert got["kernel"] == [tm, c["bits"], mode, k, 1, 2], (c, got)


PIECES = HEAD + r"""
def build(c, n):
    rng = np.random.default_rng(n)
    W = np.where(rng.random((c["rows"], n)) < c["density"], np.float16(0.5), np.float16(0)).astype(np.float32 if c["fp32"] else np.float16)
    return upload(W, max_granularity=1, delta_bits=c["bits"], num_panels=1, threads_per_wg=c["threads"])
out = []
for c in arg:
    vw, nb = 4 if c["fp32"] else 2, c["nb"]
    def pieces(n, x=True):
        return build(c, n).ecspmv_stats().meta_stride // 16 + (n * nb * vw // 16 if x else 0)
    def run(n, x):
        A = build(c, n)
        A.ecspmv_run_multi(x, Y, nb, 0) if nb > 1 else A.ecspmv_run(x, Y, 0)
        return kernel()
    lo, hi = 1, 8 * c["pieces"]                          # the widest that needs no more than `pieces`, and one that needs more
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if pieces(mid) <= c["pieces"] else (lo, mid)
    widths = range(max(1, lo - 8), lo + 9)
    below, above = max((n for n in widths if pieces(n) <= c["pieces"]), key=pieces), min((n for n in widths if pieces(n) > c["pieces"]), key=pieces)
    out.append(dict(below=run(below, X), above=run(above, X), at=[pieces(below), pieces(above)], unaligned=run(above, X + vw),
                    tables=pieces(above, False)))
print(json.dumps(out))
"""


@pytest.mark.parametrize("nb,fp32", [(1, False), (1, True), (2, False), (4, False), (8, False), (2, True), (4, True)])
def test_pieces_per_thread(tmp_path, nb, fp32):
    threads = 128
    cases = [dict(nb=nb, fp32=fp32, bits=bits, threads=threads, rows=8, density=0.1, pieces=k * threads) for bits in (4, 8) for k in (1, 2, 3)]

    def variant(per_thread):
        if nb == 1 and fp32:
            return 2 if per_thread <= 2 else 4
        return min(per_thread, 4)
    for c, got in zip(cases, standin.run(tmp_path, PIECES, cases)):
        k = c["pieces"] // threads
        assert got["at"][0] <= c["pieces"] < got["at"][1] and c["pieces"] - got["at"][0] <= 1 and got["at"][1] - c["pieces"] <= 3, (c, got)
        tail = [nb, 4 if fp32 else 2]
        assert got["below"] == [0, c["bits"], 0, variant(k), *tail], (c, got)
        assert got["above"] == [0, c["bits"], 0, variant(k + 1), *tail], (c, got)
        assert got["unaligned"] == [0, c["bits"], 0, variant(-(-got["tables"] // threads)), *tail], (c, got)   # x comes value by value


PHASES = HEAD + r"""
out = []
for c in arg:
    rng = np.random.default_rng(1)
    W = np.where(rng.random((c["rows"], c["n"])) < c["density"], np.float16(0.5), np.float16(0))
    A = upload(W, max_granularity=1, delta_bits=4, num_panels=1)
    A.ecspmv_run_multi(X, Y, c["nb"], 0)
    out.append(dict(kernel=kernel(), grid=fake.fake_launched(GRID), lds=fake.fake_launched(LDS)))
print(json.dumps(out))
"""


def test_phases(tmp_path):
    """eight right-hand sides whose partial sums fit LDS beside X, do not, and whose X does not fit: half the columns a workgroup"""
    cases = [dict(rows=16, n=1000, density=0.5, nb=8), dict(rows=100, n=1000, density=0.9, nb=8), dict(rows=16, n=10300, density=0.2, nb=8)]
    one, phases, split = standin.run(tmp_path, PHASES, cases)
    assert one["kernel"][:3] == [0, 4, 0] and one["kernel"][4:] == [8, 2] and one["grid"] == 1
    assert phases["kernel"] == [0, 4, 3, 4, 8, 2] and phases["grid"] == 1
    assert split["kernel"][2] in (0, 3) and split["kernel"][4:] == [4, 2] and split["grid"] == 2
    assert all(g["lds"] <= 160 * 1024 for g in (one, phases, split))


def test_rest_directly_fp32(tmp_path):
    """FP32, one vector: up to four pieces per thread, and more"""
    threads = 128
    cases = [dict(nb=1, fp32=True, bits=bits, threads=threads, rows=8, density=0.1, pieces=4 * threads) for bits in (4, 8)]
    for c, got in zip(cases, standin.run(tmp_path, PIECES, cases)):
        assert got["at"][0] <= c["pieces"] < got["at"][1], (c, got)
        assert got["below"] == [0, c["bits"], 0, 4, 1, 4] and got["above"] == [0, c["bits"], 0, 5, 1, 4], (c, got)


X_FIRST = HEAD + r"""
out = []
for c in arg:
    rng = np.random.default_rng(1)
    W = np.where(rng.random((c["rows"], c["n"])) < c["density"], np.float16(0.5), np.float16(0)).astype(np.float32 if c["fp32"] else np.float16)
    if c["stride"]: W[:, ::c["stride"]] = 0.5
    A = upload(W, max_granularity=2 if c["stride"] else 1, delta_bits=c["bits"], num_panels=c["panels"])
    B.ecspmv_run_batch([A] * c["count"], [X] * c["count"], [Y] * c["count"], 0)
    st = A.ecspmv_stats()
    out.append(dict(kernel=kernel(), chunks=st.units_by_g[0] / 64 / c["panels"]))
print(json.dumps(out))
"""


def test_x_first(tmp_path):
    """residual set only, alone, FP16, more than 30 chunks a panel, and three pieces per thread or more, or two with 8-bit deltas or
    fewer than 256 panels; and each of these not so"""
    base = dict(rows=40, n=9000, density=0.2, bits=4, panels=2, count=1, fp32=False, stride=0)
    full = dict(base, rows=18 * 256, panels=256, density=0.21)
    cases = [base, dict(base, bits=8), dict(base, n=17000, density=0.11), dict(base, n=33000, density=0.06), dict(full, bits=8),
             dict(full, rows=18 * 255, panels=255), dict(full, n=17000, density=0.11),
             full, dict(base, density=0.15), dict(base, n=4000, density=0.5), dict(base, count=2), dict(base, fp32=True),
             dict(base, stride=10)]
    got = standin.run(tmp_path, X_FIRST, cases)
    assert [g["kernel"][2:4] for g in got] == [[4, 2], [4, 2], [4, 3], [4, 4], [4, 2], [4, 2], [4, 3], [0, 2], [0, 2], [0, 1], [1, 3], [0, 4],
                                               [0, 2]], got
    assert all(31 < g["chunks"] < 70 for g in got[:8]) and 20 < got[8]["chunks"] < 30, got


X_FIRST_CASES = HEAD + r"""
import x_first_cases as C
out = []
for m, n, density, panels, bits in arg:
    A = upload(C.matrix(m, n, density), **C.options(panels, bits))
    got = []
    for offset in (0, 2):
        A.ecspmv_run(X + offset, Y, 0)
        got.append(kernel())
    out.append(dict(kernels=got, tables=A.ecspmv_stats().meta_stride // 16 / fake.fake_launched(THREADS)))
print(json.dumps(out))
"""


def test_x_first_cases(tmp_path):
    """what test_gpu_x_first runs on the GPU takes the kernels it is there for, with an aligned x and with one that is not"""
    cases = list(x_first_cases.CASES)
    beyond = 0
    for c, got in zip(cases, standin.run(tmp_path, X_FIRST_CASES, cases)):
        want = [[4, k] if k else [0, 1] for k in x_first_cases.CASES[c]]
        assert got["kernels"] == [[0, c[4], *w, 1, 2] for w in want], (c, got)
        beyond += got["tables"] > 4
    assert beyond == 2                                    # tables that alone are more than the four pieces


MIXED = HEAD + r"""
import batch_cases as C
out = []
for g, bits in arg:
    mats = [upload(C.mixed_matrix(n, g), **C.mixed_options(g, bits)) for n, _ in C.MIXED_FP32]
    B.ecspmv_run_batch(mats, [X + 4 * off for _, off in C.MIXED_FP32], [Y] * len(mats), 0)
    out.append(dict(kernel=kernel(), pieces=[(A.ecspmv_stats().meta_stride // 16 + (n // 4 if not off else 0)) / fake.fake_launched(THREADS)
                                             for A, (n, off) in zip(mats, C.MIXED_FP32)]))
print(json.dumps(out))
"""


def test_wide_and_narrow_in_one_launch(tmp_path):
    """the launch of test_gpu_staging_direct with matrices of unequal width takes the kernel that stages more than four pieces per thread,
    and holds matrices with more, with a few and with one"""
    cases = [(g, bits) for g in (1, 2, 4) for bits in (4, 8)]
    for (g, bits), got in zip(cases, standin.run(tmp_path, MIXED, cases)):
        assert got["kernel"] == [{1: 0, 2: 1, 4: 3}[g], bits, 1, 5, 1, 4], (g, bits, got)
        p = got["pieces"]
        assert sum(v > 4 for v in p) >= 2 and sum(1 < v <= 4 for v in p) >= 1 and sum(v <= 1 for v in p) >= 2, (g, bits, got)
