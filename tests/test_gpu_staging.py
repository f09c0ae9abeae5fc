"""Tables and X on their way to LDS: one to four 16-byte pieces per thread and a loop beyond, at both sides of every line between
them, with X aligned for pieces and not, for images without and with block sets and for both widths of values.  Every column has the bits
of a product with one vector (test_gpu_multi.check, test_gpu_f32.check_multi) and stays in the oracle's band."""
import numpy as np
import pytest

from workloads import generators as gen
from test_gpu_f32 import check_multi, make_f32
from test_gpu_multi import E, check  # noqa: F401  -- the fixture and the comparison with the oracle

pytestmark = pytest.mark.gpu

THREADS, ROWS = 128, 24


def widths_around(E, pieces, nb, delta_bits):  # noqa: F811
    """The widths whose [tables | X] of one panel, in 16-byte pieces (X in whole ones), come closest to `pieces`: at most as many,
    and more."""
    def count(n):
        W, _ = gen.small_random(ROWS, n, 0.2, 11)
        st = E.ecspmv_build_dense(W, E.make_opts(delta_bits=delta_bits, num_panels=1, threads_per_wg=THREADS)).ecspmv_stats()
        return st.meta_stride // 16 + n * nb * 2 // 16
    lo, hi = 1, 8 * pieces                                     # (a wider matrix has more of both, but for a table entry now and then)
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if count(mid) <= pieces else (lo, mid)
    counts = {n: count(n) for n in range(max(1, lo - 8), lo + 9)}
    below = max((n for n in counts if counts[n] <= pieces), key=counts.get)
    above = min((n for n in counts if counts[n] > pieces), key=counts.get)
    assert pieces - counts[below] <= 1 and counts[above] - pieces <= 3
    return below, above


@pytest.mark.parametrize("x_offset", [0, 1])
@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("nb,delta_bits", [(2, 4), (4, 8), (8, 4)])
def test_pieces_per_thread(E, nb, delta_bits, k, over, x_offset):  # noqa: F811
    n = widths_around(E, k * THREADS, nb, delta_bits)[over]
    W, _ = gen.small_random(ROWS, n, 0.2, 11)
    check(E, W, nb, f"{k} pieces per thread{' and more' if over else ''}", x_offset=x_offset, delta_bits=delta_bits, num_panels=1, threads_per_wg=THREADS)


def shared_columns(n, g, fp32):
    """ROWS rows, every third column (every one of a narrow matrix) shared by all of them where blocks of g rows are asked for"""
    W, _ = gen.small_random(ROWS, n, 0.1, 17)
    if g > 1:
        W[:, ::3 if n >= 1000 else 1] = np.float16(0.01)
    return make_f32(W, 17) if fp32 else W


def widths_at(build, pieces, nb, vw):
    """The widths closest below and above a line: [tables | X] in no more than `pieces`, and in more.  (Tables grow by whole units, so
    a wider matrix can have fewer pieces now and then.)"""
    def count(n):
        return build(n).ecspmv_stats().meta_stride // 16 + n * nb * vw // 16
    lo, hi = 1, 8 * pieces
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if count(mid) <= pieces else (lo, mid)
    counts = {n: count(n) for n in range(max(1, lo - 8), lo + 9)}
    below, above = max((n for n in counts if counts[n] <= pieces), key=counts.get), min((n for n in counts if counts[n] > pieces), key=counts.get)
    assert pieces - counts[below] <= 32 and counts[above] - pieces <= 32          # lines are 512 apart
    return below, above


@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("k", [1, 2, 3, 4])
@pytest.mark.parametrize("nb", [2, 4, 8])
@pytest.mark.parametrize("g,fp32", [(2, False), (4, False), (8, False), (1, True), (2, True), (4, True)])
def test_pieces_per_thread_with_sets_and_fp32(E, g, fp32, nb, k, over):  # noqa: F811
    opts = dict(delta_bits=8 if nb == 4 else 4, num_panels=1, threads_per_wg=512, max_granularity=g, flags=E.binding.FLAG_KEEP_SMALL_SETS)
    build = E.ecspmv_build_dense_f32 if fp32 else E.ecspmv_build_dense
    n = widths_at(lambda n: build(shared_columns(n, g, fp32), E.make_opts(**opts)), k * 512, nb, 4 if fp32 else 2)[over]
    for x_offset in (0, 1):
        A = (check_multi if fp32 else check)(E, shared_columns(n, g, fp32), nb, f"g={g} {k} pieces per thread{' and more' if over else ''}",
                                             x_offset=x_offset, **opts)
        assert A.ecspmv_stats().nnz_by_g[{1: 0, 2: 1, 4: 2, 8: 3}[g]] > 0
