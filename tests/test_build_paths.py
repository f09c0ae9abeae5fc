"""The two ways into the encoder (dense rows and CSR) give the same image, and block columns are cut into units as defined where
runs end inside a word of 64 columns, at its edge, or at the largest delta."""
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
