"""The workgroup size a launch chooses from the work in its panels, and the staging of an x too wide for the first four
pieces per thread: y does not depend on either, so every launch has the bits of one whose size the caller fixed."""
import numpy as np
import pytest

from workloads import generators as gen
from test_gpu_multi import E  # noqa: F401  -- the fixture

pytestmark = pytest.mark.gpu


def bits(t):
    import torch
    return t.view(torch.int16 if t.dtype == torch.float16 else torch.int32)


def in_band(y, W, x):
    """y against the 64-bit product, as far as the values' own width lets it be"""
    x = x.cpu().numpy().astype(np.float64)
    ref, S = W.astype(np.float64) @ x, np.abs(W).astype(np.float64) @ np.abs(x)
    rel, floor = (2.0 ** -17, 1e-12) if W.dtype == np.float32 else (2e-3, 1e-6)
    return (np.abs(y.cpu().numpy() - ref) <= rel * S + floor).all()


def upload(E, W, **opts):  # noqa: F811
    A = (E.ecspmv_build_dense_f32 if W.dtype == np.float32 else E.ecspmv_build_dense)(W, E.make_opts(**opts))
    E.device.upload(A)
    return A


# chunks per panel (64 lane units of 16 entries, or 4 units of 64 columns) on both sides of 16, 24 and 48, with and without
# block sets; more than 4096 pieces of x for the widest (which size each line gives: test_launch_shape.py)
@pytest.mark.parametrize("m,n,density,panels,opts", [
    (32, 640, 0.5, 2, dict(max_granularity=1)),                     # 5 chunks: 512 threads
    (48, 4000, 0.25, 2, dict(max_granularity=1, delta_bits=4)),     # 24: 768 (FP32: 512)
    (52, 4000, 0.25, 2, dict(max_granularity=1, delta_bits=4)),     # 26: 1024, no block sets
    (18, 4000, 0.4, 2, dict(max_granularity=2)),                    # one block set: 768
    (48, 4000, 0.48, 2, dict(max_granularity=1)),                   # 45: 1024
    (20, 4001, 0.4, 2, dict(max_granularity=4)),                    # two block sets: 1024
    (64, 4000, 0.5, 2, dict(max_granularity=1, delta_bits=4)),      # 63: 1024
    (8, 40001, 0.02, 2, dict(max_granularity=1, delta_bits=4)),     # few chunks, 5000 pieces of x
])
@pytest.mark.parametrize("fp32", [False, True])
def test_alone_and_several_vectors(E, m, n, density, panels, opts, fp32):  # noqa: F811
    import torch
    if fp32 and n > 20000:
        n = 20001
    print(f"[case] {m}x{n} {opts} fp32={fp32}", flush=True)
    W, x = gen.small_random(m, n, density, 7)
    if opts["max_granularity"] > 1:
        W[:, ::3] = np.float16(0.01)                                # columns that all rows share: block units
    W = W.astype(np.float32) if fp32 else W
    dt = torch.float32 if fp32 else torch.float16
    A, B = upload(E, W, num_panels=panels, **opts), upload(E, W, num_panels=panels, threads_per_wg=1024, **opts)
    xd = torch.from_numpy(x.astype(np.float32)).cuda().to(dt)
    y, z = torch.full((m,), float("nan"), dtype=dt, device="cuda"), torch.empty(m, dtype=dt, device="cuda")
    E.device.run(A, xd, y)
    E.device.run(B, xd, z)
    assert torch.equal(bits(y), bits(z))
    assert in_band(y, W, xd)
    assert all((A.ecspmv_stats().nnz_by_g[i] > 0) == (1 << i <= opts["max_granularity"]) for i in (1, 2))
    if n < 5000:
        X = torch.randn((n, 2), device="cuda").to(dt)
        Y, Z = torch.full((m, 2), float("nan"), dtype=dt, device="cuda"), torch.empty((m, 2), dtype=dt, device="cuda")
        E.device.run_multi(A, X, Y)
        E.device.run_multi(B, X, Z)
        assert torch.equal(bits(Y), bits(Z)) and in_band(Y, W, X)


# 256 threads from 257 panels on (small x, up to 16 chunks a panel), or from 1024 panels with an 8-grained set whatever the
# chunks; otherwise 512; with 512, x of 20001 or 9001 entries takes up to six pieces per thread
@pytest.mark.parametrize("count,m,n,density,panels,opts,fp32", [
    (5, 128, 700, 0.3, 51, dict(max_granularity=1, delta_bits=4), False),
    (7, 128, 700, 0.3, 64, dict(max_granularity=1, delta_bits=4), False),
    (7, 768, 700, 0.2, 48, dict(max_granularity=2), False),                   # 256, one block set
    (7, 768, 700, 0.2, 48, dict(max_granularity=4), True),                    # 256, two, FP32
    (8, 128, 701, 0.3, 128, dict(max_granularity=8, flags=4), False),         # one row a panel: no blocks
    (16, 1024, 2400, 0.4, 64, dict(max_granularity=8, flags=4, delta_bits=4), False),     # 1024 panels, 8-grained, 20 chunks: 256
    (15, 1024, 2400, 0.4, 64, dict(max_granularity=8, flags=4, delta_bits=4), False),     # 960: 512
    (3, 30, 20001, 0.1, 5, dict(max_granularity=1, delta_bits=4), False),
    (3, 30, 9001, 0.1, 5, dict(max_granularity=2), True),
])
def test_several_matrices(E, count, m, n, density, panels, opts, fp32):  # noqa: F811
    import torch
    print(f"[case] {count} x {m}x{n} panels={panels} {opts} fp32={fp32}", flush=True)
    dt = torch.float32 if fp32 else torch.float16
    mats, fixed, xs, ys, Ws = [], [], [], [], []
    for k in range(count):
        W, x = gen.small_random(m, n - k, density, 20 + k)
        if opts["max_granularity"] > 1 and panels < m:
            W[:, ::3] = np.float16(0.01)                            # columns that all rows share: block units
        W = W.astype(np.float32) if fp32 else W
        Ws.append(W)
        mats.append(upload(E, W, num_panels=panels, **opts))
        fixed.append(upload(E, W, num_panels=panels, threads_per_wg=512, **opts))
        top = {1: 0, 2: 1, 4: 2, 8: 3}[opts["max_granularity"]] if panels < m else 0
        assert all((mats[-1].ecspmv_stats().nnz_by_g[i] > 0) == (i <= top) for i in (1, 2, 3))
        buf = torch.zeros(n + 1, dtype=dt, device="cuda")
        buf[k % 2:k % 2 + n - k].copy_(torch.from_numpy(x.astype(np.float32)).cuda())
        xs.append(buf[k % 2:k % 2 + n - k])                         # every second x is off a 16-byte boundary
        ys.append(torch.full((m,), float("nan"), dtype=dt, device="cuda"))
    stream = torch.cuda.current_stream().cuda_stream
    E.ecspmv_run_batch(mats, [x.data_ptr() for x in xs], [y.data_ptr() for y in ys], stream)
    z = torch.empty(m, dtype=dt, device="cuda")
    for A, x, y, W in zip(fixed, xs, ys, Ws):
        A.ecspmv_run(x.data_ptr(), z.data_ptr(), stream)
        torch.cuda.synchronize()
        assert torch.equal(bits(y), bits(z)) and in_band(y, W, x)
