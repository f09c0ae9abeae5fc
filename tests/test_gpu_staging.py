"""Tables and X on their way to LDS: one to four 16-byte pieces per thread and a loop beyond, at both sides of every line between
them, with X aligned for pieces and not.  Every column has the bits of a product with one vector (test_gpu_multi.check) and stays
in the oracle's band."""
import numpy as np
import pytest

from workloads import generators as gen
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
