"""Launches of one vector alone whose x is in LDS before the first chunks are requested, and the pieces per thread that each is staged
with: wide ones, whose pieces are x for the most part, and tall ones, whose tables alone are two pieces per thread or more, so that an x that is
no list of pieces is copied value by value in the same kernels."""
from workloads import generators as gen

# (rows, columns, density, panels, bits): pieces per thread with x aligned, and with x two bytes on (None: x is most of the list, and
# without it one piece is enough, which leaves the chunks first)
CASES = {(33, 9000, 0.3, 2): (2, None), (40, 9003, 0.3, 2): (2, None), (24, 17001, 0.3, 1): (3, None), (20, 33007, 0.3, 1): (4, None),
         (12, 40000, 0.3, 1): (4, None)}
CASES = {(*shape, bits): k for shape, k in CASES.items() for bits in (4, 8)}
CASES |= {(1000, 3000, 0.05, 1, 4): (2, 2), (2000, 2000, 0.03, 1, 8): (3, 3), (1200, 2999, 0.05, 1, 4): (3, 2), (1500, 8999, 0.03, 1, 8): (4, 3),
          (2500, 999, 0.05, 1, 4): (4, 4), (5000, 333, 0.1, 1, 8): (4, 4), (5000, 333, 0.1, 1, 4): (4, 4)}


def matrix(m, n, density):
    return gen.small_random(m, n, density, 7)[0]


def options(panels, bits):
    return dict(delta_bits=bits, max_granularity=1, num_panels=panels)
