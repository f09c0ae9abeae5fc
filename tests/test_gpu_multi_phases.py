"""Several right-hand sides where the partial sums of a panel do not fit LDS beside X (the residual chunks are then taken
in phases) and where the columns of X are split over several workgroups of one launch: every column has the bits of the
single-vector launch, and the oracle's band holds."""
import numpy as np
import pytest

from workloads import generators as gen
from test_gpu_multi import E, check  # noqa: F401  -- the fixture and the comparison with the oracle

pytestmark = pytest.mark.gpu

LDS = 160 * 1024


def one_phase_bytes(st, nb, value_bytes):
    """LDS of a launch that keeps all nb columns and every partial sum of a panel."""
    x = (st.n * value_bytes + 15) // 16 * 16
    slots = (st.lds_bytes - x - st.meta_stride) // 4
    return st.n * value_bytes * nb + st.meta_stride + 4 * nb * slots


@pytest.mark.parametrize("m,n,density,nb,opts", [
    (28, 9000, 0.85, 8, dict(num_panels=1, threads_per_wg=64, max_granularity=1)),     # rows longer than a phase
    (37, 6001, 0.6, 8, dict(num_panels=1, max_granularity=1)),                    # chunks and rows that straddle phases
    (37, 6001, 0.6, 8, dict(num_panels=2, threads_per_wg=192, max_granularity=1)),     # wavefronts not a power of two
    (60, 5300, 0.6, 8, dict(num_panels=2, threads_per_wg=256, max_granularity=8, delta_bits=8)),    # with block sets
    (19, 13824, 0.5, 8, dict(num_panels=1, max_granularity=1, delta_bits=4)),     # two workgroups per panel, phases
    (27, 13824, 0.3, 8, dict(num_panels=9, delta_bits=4)),                        # panels no multiple of eight
    (60, 20000, 0.2, 4, dict(num_panels=3, max_granularity=1, delta_bits=8)),
])
def test_phases_and_splits(E, m, n, density, nb, opts):  # noqa: F811
    W, _ = gen.small_random(m, n, density, 3)
    if opts.get("max_granularity") == 8:
        W[:, ::5] = W[0, ::5]
        W[:, ::5][:, W[0, ::5] == 0] = np.float16(0.01)                           # columns that all rows share: block units
    W[m // 2] = 0                                                                 # an empty row in the middle
    A = check(E, W, nb, f"{m}x{n} {opts}", **opts)
    assert one_phase_bytes(A.ecspmv_stats(), nb, 2) > LDS
    if opts.get("max_granularity") == 8:
        assert sum(A.ecspmv_stats().nnz_by_g[1:]) > 0


@pytest.mark.parametrize("m,n,density,nb,opts", [
    (37, 4001, 0.6, 8, dict(num_panels=1, delta_bits=4, max_granularity=1)),
    (21, 9000, 0.4, 8, dict(num_panels=3, delta_bits=8, max_granularity=1)),                         # X split and phases
    (40, 6500, 0.5, 4, dict(num_panels=1, threads_per_wg=256, delta_bits=8, max_granularity=2)),
])
def test_phases_fp32(E, m, n, density, nb, opts):  # noqa: F811
    import torch
    print(f"[case] fp32 {m}x{n} nb={nb} {opts}", flush=True)
    W = gen.small_random(m, n, density, 4)[0].astype(np.float32)
    A = E.ecspmv_build_dense_f32(W, E.make_opts(**opts))
    assert one_phase_bytes(A.ecspmv_stats(), nb, 4) > LDS
    E.device.upload(A)
    X = torch.from_numpy(np.random.default_rng(5).standard_normal((n, nb)).astype(np.float32)).cuda()
    Y = torch.full((m, nb), float("nan"), device="cuda")
    y = torch.empty(m, device="cuda")
    E.device.run_multi(A, X, Y)
    for b in range(nb):
        E.device.run(A, X[:, b].contiguous(), y)
        torch.cuda.synchronize()
        assert torch.equal(y.view(torch.int32), Y[:, b].contiguous().view(torch.int32)), b
    ref = W.astype(np.float64) @ X.cpu().numpy().astype(np.float64)
    S = np.abs(W).astype(np.float64) @ np.abs(X.cpu().numpy()).astype(np.float64)
    assert (np.abs(Y.cpu().numpy() - ref) <= 2.0 ** -17 * S + 1e-12).all()
