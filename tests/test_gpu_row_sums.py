"""Sums over the 16 lanes that share a block unit, and over those that share a row of Y: every granularity, delta width, value
width and number of right-hand sides that a launch takes.  Weights and x are small integers, so every sum is exact in FP32 in any
order and, at most 5 * 3 * 128 < 2048, as an FP16 result: Y equals the integer product, and a sum that went to the wrong lane
shows."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def E():
    import torch
    assert torch.cuda.is_available()
    import paper_2507_12205_amd as pkg
    from paper_2507_12205_amd import device
    pkg.binding.lib()
    pkg.device = device
    return pkg


CASES = [(g, bits, fp32, nb) for g in (1, 2, 4, 8, 16) for bits in (4, 8, 16) for fp32 in (False, True) for nb in (1, 2, 4, 8)
         if not (nb > 1 and (g == 16 or bits == 16 or (fp32 and g == 8))) and not (fp32 and bits == 16)]


@pytest.mark.parametrize("g,bits,fp32,nb", CASES)
def test_exact_sums(E, g, bits, fp32, nb):
    import torch
    print(f"[case] row sums g={g} bits={bits} fp32={fp32} nb={nb}", flush=True)
    n = 128
    rng = np.random.default_rng([g, bits, nb])
    rows = np.arange(g + 3)[:, None]
    w = (7 * rows + 3 * np.arange(n)) % 11 - 5
    w[w == 0] = 1
    w[g:] *= rng.random((3, n)) < 0.2                     # rows that share no unit with the others
    if g > 1:
        w[:g, 64:] *= np.arange(64) % 2                   # a unit, and 32 columns each that stay residual
    x = rng.integers(-3, 4, (n, nb))
    dt = np.float32 if fp32 else np.float16
    opts = E.make_opts(delta_bits=bits, max_granularity=g, flags=E.binding.FLAG_KEEP_SMALL_SETS)
    A = (E.ecspmv_build_dense_f32 if fp32 else E.ecspmv_build_dense)(w.astype(dt), opts)
    assert A.ecspmv_stats().units_by_g[{1: 0, 2: 1, 4: 2, 8: 3, 16: 4}[g]] > 0
    E.device.upload(A)
    X = torch.from_numpy(x.astype(dt)).cuda()
    Y = torch.full((g + 3, nb), float("nan"), dtype=X.dtype, device="cuda")
    if nb == 1:
        E.device.run(A, X.view(n), Y.view(g + 3))
    else:
        E.device.run_multi(A, X, Y)
    torch.cuda.synchronize()
    assert np.array_equal(Y.cpu().numpy().astype(np.int64), w @ x)
