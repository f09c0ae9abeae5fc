"""Launches of several matrices at both sides of the lines between their two kernel variants (two residual buffers; every set
requested before the first barrier): y has the bits of lone launches and stays in the oracle's band, with x that ends in a whole
16-byte piece and not, one image for all items, and items with a matrix of their own."""
import numpy as np
import pytest

import batch_cases
from workloads import generators as gen
from test_gpu_multi import E  # noqa: F401  -- the fixture
from test_gpu_workgroup_size import bits, in_band, upload

pytestmark = pytest.mark.gpu


def chunks_per_panel(A):
    st = A.ecspmv_stats()
    return (st.units_by_g[0] / 64 + sum(st.units_by_g[1:]) / 4) / st.num_panels


@pytest.mark.parametrize("m,n,density,panels,count,g,chunks", [
    (528, 20001, 0.9, 176, 3, 1, (46, 60)),            # residual only: 528 workgroups of more than 45 chunks
    (510, 20001, 0.9, 170, 3, 1, (46, 60)),            # 510 workgroups
    (704, 12000, 0.9, 176, 3, 1, (39, 44.5)),          # fewer chunks
    (32, 601, 0.5, 4, 5, 2, (3, 8)),                   # one block set: few chunks
    (32, 1600, 0.5, 4, 5, 2, (9.5, 20)),
])
@pytest.mark.parametrize("delta_bits", [4, 8])
def test_both_variants(E, m, n, density, panels, count, g, chunks, delta_bits):  # noqa: F811
    import torch
    print(f"[case] {count} x {m}x{n} g={g} bits={delta_bits}", flush=True)
    W, _ = gen.small_random(m, n, density, 13)
    if g > 1:
        W[:, ::3] = np.float16(0.01)                   # columns that all rows share: block units
    A = upload(E, W, max_granularity=g, num_panels=panels, delta_bits=delta_bits)
    assert chunks[0] < chunks_per_panel(A) < chunks[1] and (sum(A.ecspmv_stats().nnz_by_g[1:]) > 0) == (g > 1)
    xs = [torch.from_numpy(np.random.default_rng(k).standard_normal(n).astype(np.float16)).cuda() for k in range(count)]
    ys = [torch.full((m,), float("nan"), dtype=torch.float16, device="cuda") for _ in range(count)]
    z = torch.empty(m, dtype=torch.float16, device="cuda")
    E.ecspmv_run_batch([A] * count, [x.data_ptr() for x in xs], [y.data_ptr() for y in ys], E.device._stream_handle())
    for k in range(count):
        E.device.run(A, xs[k], z)
        assert torch.equal(bits(ys[k]), bits(z)), k
    assert in_band(ys[0], W, xs[0])


# every item narrower than the one before it, every second x off a 16-byte boundary, with the two kernel variants and all four
# staging variants of the second one
@pytest.mark.parametrize("c", batch_cases.CASES, ids=lambda c: "{kernel}-{count}x{panels}x{rows}x{n}-d{bits}".format(**c).replace(" ", ""))
def test_unequal_matrices(E, c):  # noqa: F811
    import torch
    print(f"[case] {c}", flush=True)
    count, m = c["count"], c["rows"] * c["panels"]
    Ws = [batch_cases.matrix(c, k) for k in range(count)]
    mats = [upload(E, W, **batch_cases.options(c)) for W in Ws]
    st = [A.ecspmv_stats() for A in mats]
    assert c["chunks"][0] < sum(map(batch_cases.chunks, st)) / sum(s.num_panels for s in st) < c["chunks"][1]
    xs, ys = [], [torch.full((m,), float("nan"), dtype=torch.float16, device="cuda") for _ in range(count)]
    for k, W in enumerate(Ws):
        buf = torch.zeros(W.shape[1] + 1, dtype=torch.float16, device="cuda")
        x = buf[k % 2:k % 2 + W.shape[1]]
        x.copy_(torch.from_numpy(np.random.default_rng(k).standard_normal(W.shape[1]).astype(np.float32)).cuda())
        xs.append(x)
    E.ecspmv_run_batch(mats, [x.data_ptr() for x in xs], [y.data_ptr() for y in ys], E.device._stream_handle())
    z = torch.empty(m, dtype=torch.float16, device="cuda")
    for A, W, x, y in zip(mats, Ws, xs, ys):
        E.device.run(A, x, z)
        assert torch.equal(bits(y), bits(z)) and in_band(y, W, x)
