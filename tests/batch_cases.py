"""Launches of several matrices of unequal width at both sides of the lines between their kernel variants, and of those between the
staging variants of the second one.  Which kernel each takes is checked where it is chosen (test_kernel_choice.py), what it computes
on the GPU (test_gpu_batch_variants.py)."""
import numpy as np


def case(kernel, count, panels, rows, n, density, chunks, stride=0, bits=(4, 8), step=1):
    """kernel: (TM, MODE, K); every panel of `rows` rows; item k has n - k * step columns; stride: every so many columns are shared by
    all rows (block units of two rows); chunks: between which the chunks per panel lie"""
    return [dict(kernel=kernel, count=count, panels=panels, rows=rows, n=n, density=density, stride=stride, bits=b, step=step, chunks=chunks)
            for b in bits]


# residual only: two buffers from 513 workgroups on if a panel has more than 45 chunks; one to four pieces per thread
RESIDUAL = (case((0, 2, 1), 3, 176, 18, 2901, 0.95, (46, 60))
            + case((0, 2, 2), 3, 176, 9, 6003, 0.92, (46, 60), step=7)
            + case((0, 2, 3), 3, 176, 6, 10005, 0.85, (46, 60), step=7)
            + case((0, 2, 4), 3, 176, 3, 20001, 0.9, (46, 60), step=7)
            + case((0, 2, 2), 3, 171, 9, 6003, 0.92, (46, 60))               # 513 workgroups
            + case((0, 1, 2), 4, 128, 9, 6003, 0.92, (46, 60))               # 512
            + case((0, 1, 3), 3, 176, 6, 10005, 0.75, (41, 44.9)))           # fewer chunks
# one block set: every set requested before the first barrier up to three block chunks for four wavefronts
ONE_SET = (case((1, 2, 1), 5, 4, 8, 601, 0.3, (3, 8), stride=4)
           + case((1, 2, 2), 5, 4, 4, 6003, 0.05, (4, 8), stride=12, step=7)
           + case((1, 2, 3), 5, 4, 2, 10005, 0.05, (3, 8), stride=12, step=7)
           + case((1, 2, 4), 5, 4, 2, 14007, 0.05, (3, 8), stride=12, step=7)
           + case((1, 2, 2), 5, 4, 16, 6003, 0.4, (35, 60), stride=64, step=7, bits=(4,))     # many chunks, few of them of blocks
           + case((1, 1, 1), 5, 4, 24, 601, 0.3, (9, 16), stride=3)                # few, more of blocks
           + case((1, 1, 2), 5, 4, 8, 6003, 0.05, (9, 16), stride=12, step=7)
           + case((1, 1, 3), 5, 4, 4, 10005, 0.05, (8, 16), stride=12, step=7)
           + case((1, 2, 1), 16, 65, 6, 601, 0.3, (2, 5), stride=4)                # four wavefronts
           + case((1, 1, 1), 16, 65, 16, 601, 0.3, (6, 10), stride=4))
CASES = RESIDUAL + ONE_SET


def matrix(c, k):
    """the k-th matrix of a case"""
    m, n = c["rows"] * c["panels"], c["n"] - k * c["step"]
    rng = np.random.default_rng([k, m, n])
    W = np.where(rng.random((m, n), dtype=np.float32) < c["density"], rng.standard_normal((m, n), dtype=np.float32) * np.float32(0.02),
                 np.float32(0)).astype(np.float16)
    if c["stride"]:
        W[:, ::c["stride"]] = np.float16(0.01)
    return W


def options(c):
    return dict(max_granularity=2 if c["stride"] else 1, num_panels=c["panels"], delta_bits=c["bits"])


def block_chunks(stats):
    return sum(stats.units_by_g[1:]) / 4


def chunks(stats):
    """what a wavefront takes at a time, of one image: 64 lane units, 4 units (the rule counts the last one of a panel and set in full, up
    to one more for each)"""
    return stats.units_by_g[0] / 64 + block_chunks(stats)


# FP32, one launch, 128 threads: (columns, x so many values on from a 16-byte boundary) of its matrices.  The widest need more than four
# pieces per thread, which is what the launch's kernel follows; the others have one, a few, or none but their tables.
MIXED_FP32 = [(333, 0), (1200, 0), (64, 1), (8001, 0), (1021, 1), (9000, 1), (2048, 0), (16, 0)]
MIXED_THREADS = 128


def mixed_matrix(n, g):
    """24 rows; every third column (every one of a narrow matrix) in all of them where blocks of g rows are asked for"""
    rng = np.random.default_rng([n, g])
    W = np.where(rng.random((24, n)) < 0.1, rng.standard_normal((24, n)) * 0.02, 0).astype(np.float32)
    if g > 1:
        W[:, ::3 if n >= 1000 else 1] = np.float32(0.0103)
    return W


def mixed_options(g, bits):
    return dict(delta_bits=bits, max_granularity=g, num_panels=2, threads_per_wg=MIXED_THREADS, flags=4)          # small sets are kept
