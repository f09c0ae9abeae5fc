"""One vector alone whose x is in LDS before the first chunks are requested: two, three, four and more pieces per thread, widths that
leave values behind the last piece, x that is no list of pieces (in tall matrices, whose tables keep the kernel the same; in wide ones
it is then another kernel's), both delta widths.  In the oracle's band, and with the bits of a launch of several matrices, which requests
its chunks first.  Which kernel each case takes is held by test_kernel_choice.py."""
import numpy as np
import pytest
import x_first_cases

from oracle import oracle as orc
from workloads import generators as gen
from test_gpu_multi import ABS, E, REL  # noqa: F401  -- the fixture

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("x_offset", [0, 1])
@pytest.mark.parametrize("m,n,density,panels,bits", list(x_first_cases.CASES))
def test_x_first(E, m, n, density, panels, bits, x_offset):  # noqa: F811
    import torch
    print(f"[case] x first {m}x{n} bits={bits} x_offset={x_offset}", flush=True)
    W = x_first_cases.matrix(m, n, density)
    A = E.ecspmv_build_dense(W, E.make_opts(**x_first_cases.options(panels, bits)))
    assert A.ecspmv_stats().units_by_g[0] > 64 * 30 * panels + 64 * panels
    E.device.upload(A)
    x = gen.make_vector(n, seed=n)
    flat = torch.zeros(n + 16, dtype=torch.float16, device="cuda")
    xd = flat[x_offset:x_offset + n]
    xd.copy_(torch.from_numpy(x.view(np.int16)).cuda().view(torch.float16))
    ys = [torch.full((m,), float("nan"), dtype=torch.float16, device="cuda") for _ in range(3)]
    E.device.run(A, xd, ys[0])
    E.ecspmv_run_batch([A, A], [xd.data_ptr()] * 2, [y.data_ptr() for y in ys[1:]])
    torch.cuda.synchronize()
    y = ys[0].cpu().numpy()
    assert all(np.array_equal(t.cpu().numpy().view(np.uint16), y.view(np.uint16)) for t in ys[1:])
    y_ref, S = orc.spmv_oracle(W, x)
    assert np.all(np.abs(y.astype(np.float64) - y_ref) <= REL * S + ABS)
