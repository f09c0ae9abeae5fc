"""What four pieces per thread leave of tables and x goes straight to LDS: lists that end at, before and behind a wavefront's 64
pieces and a round of the workgroup, tables that alone are more than the four pieces, x that is no list of pieces.  FP32 with one
vector (FP32 sums in another order than the oracle's: test_gpu_f32.check's bounds), alone and with matrices of other widths in the
launch, several vectors in both widths, column by column with the bits of one vector."""
import batch_cases
import numpy as np
import pytest

from workloads import generators as gen
from test_gpu_f32 import check as check_f32, check_multi, make_f32
from test_gpu_multi import E, check  # noqa: F401  -- the fixture and the comparison with the oracle
from test_gpu_staging import shared_columns, widths_at

pytestmark = pytest.mark.gpu

THREADS = 128


@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("pieces", [4 * THREADS, 4 * THREADS + 64, 5 * THREADS, 9 * THREADS - 64])
@pytest.mark.parametrize("g,bits", [(1, 4), (2, 8), (4, 4)])
def test_fp32_one_vector(E, g, bits, pieces, over):  # noqa: F811
    import torch
    opts = dict(delta_bits=bits, num_panels=1, threads_per_wg=THREADS, max_granularity=g, flags=E.binding.FLAG_KEEP_SMALL_SETS)
    n = widths_at(lambda n: E.ecspmv_build_dense_f32(shared_columns(n, g, True), E.make_opts(**opts)), pieces, 1, 4)[over]
    x = gen.make_vector(n, seed=n).astype(np.float32)
    A, y = check_f32(E, shared_columns(n, g, True), x, f"g={g} {pieces} pieces{' and more' if over else ''}", **opts)
    assert A.ecspmv_stats().nnz_by_g[{1: 0, 2: 1, 4: 2}[g]] > 0
    flat = torch.zeros(n + 1, dtype=torch.float32, device="cuda")
    flat[1:].copy_(torch.from_numpy(x))
    yd = torch.full((y.size,), float("nan"), dtype=torch.float32, device="cuda")
    E.device.run(A, flat[1:], yd)
    torch.cuda.synchronize()
    assert np.array_equal(yd.cpu().numpy(), y)
    ys = [torch.full((y.size,), float("nan"), dtype=torch.float32, device="cuda") for _ in range(3)]      # and three in a launch
    xd = torch.from_numpy(x).cuda()
    E.ecspmv_run_batch([A] * 3, [xd.data_ptr()] * 3, [t.data_ptr() for t in ys])
    torch.cuda.synchronize()
    assert all(np.array_equal(t.cpu().numpy(), y) for t in ys)


@pytest.mark.parametrize("g,bits", [(g, bits) for g in (1, 2, 4) for bits in (4, 8)])
def test_wide_and_narrow_in_one_launch(E, g, bits):  # noqa: F811
    """Every workgroup of the launch lays out LDS by its own matrix: each result in the bounds of its own, and with the bits of a launch
    that carries it alone.  (test_kernel_choice.py holds which kernel this is.)"""
    import torch
    opts = batch_cases.mixed_options(g, bits)
    mats, xs, lone = [], [], []
    for n, off in batch_cases.MIXED_FP32:
        W, x = batch_cases.mixed_matrix(n, g), gen.make_vector(n, seed=n).astype(np.float32)
        A, y = check_f32(E, W, x, f"g={g} bits={bits} {n} columns", **opts)
        flat = torch.zeros(n + 4, dtype=torch.float32, device="cuda")
        flat[off:off + n].copy_(torch.from_numpy(x))
        mats.append(A), xs.append(flat), lone.append(y)
    ys = [torch.full((y.size,), float("nan"), dtype=torch.float32, device="cuda") for y in lone]
    for order in (range(len(mats)), reversed(range(len(mats)))):
        order = list(order)
        for y in ys:
            y.fill_(float("nan"))
        E.ecspmv_run_batch([mats[k] for k in order], [xs[k].data_ptr() + 4 * batch_cases.MIXED_FP32[k][1] for k in order],
                           [ys[k].data_ptr() for k in order])
        torch.cuda.synchronize()
        assert all(np.array_equal(t.cpu().numpy().view(np.uint32), y.view(np.uint32)) for t, y in zip(ys, lone)), (g, bits, order)


@pytest.mark.parametrize("x_offset", [0, 1])
@pytest.mark.parametrize("nb,fp32", [(1, True), (2, False), (4, True), (8, False)])
def test_tables_beyond_four_pieces(E, nb, fp32, x_offset):  # noqa: F811
    W, _ = gen.small_random(2500, 333, 0.1, 5)
    W = make_f32(W, 3) if fp32 else W
    opts = dict(delta_bits=4, num_panels=1, threads_per_wg=64)
    build = E.ecspmv_build_dense_f32 if fp32 else E.ecspmv_build_dense
    assert build(W, E.make_opts(**opts)).ecspmv_stats().meta_stride // 16 > 5 * 64
    if nb == 1:
        check_f32(E, W, gen.make_vector(333, seed=2).astype(np.float32), "tables", **opts)
    else:
        (check_multi if fp32 else check)(E, W, nb, "tables", x_offset=x_offset, **opts)
