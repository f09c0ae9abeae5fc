"""The workgroup size a launch chooses from its chunks per panel, its block sets, the rows of a panel, its x and the number
of workgroups, on both sides of every line of the rule."""
import pytest

import standin

CHILD = r"""
def build(c, k):
    rng = np.random.default_rng(k)
    m, n = c["rows"] * c["panels"], c["n"]
    W = np.where(rng.random((m, n)) < c["density"], np.float16(0.5), np.float16(0)).astype(np.float32 if c["fp32"] else np.float16)
    if c["g"] > 1:
        W[:, ::3] = 0.25                                 # columns that all rows share: block units
    o = B.make_opts(max_granularity=c["g"], num_panels=c["panels"], delta_bits=c["bits"], threads_per_wg=c["fixed"], flags=c["flags"])
    A = (B.ecspmv_build_dense_f32 if c["fp32"] else B.ecspmv_build_dense)(W, o)
    A.ecspmv_upload(0x100000, A.ecspmv_device_bytes(), 0)
    return A
out = []
for c in arg:
    A = build(c, 1)
    st = A.ecspmv_stats()
    if c["nb"] > 1:
        A.ecspmv_run_multi(0x200000, 0x300000, c["nb"], 0)
    elif c["count"] == 1:
        A.ecspmv_run(0x200000, 0x300000, 0)
    else:
        B.ecspmv_run_batch([A] * c["count"], [0x200000] * c["count"], [0x300000] * c["count"], 0)
    units = list(st.units_by_g)
    out.append(dict(threads=fake.fake_launched(THREADS), grid=fake.fake_launched(GRID), sets=[int(u > 0) for u in units[1:]],
                    chunks=(units[0] / 64 + sum(units[1:]) / 4) / st.num_panels,
                    pieces=(st.meta_stride + c["n"] * (4 if c["fp32"] else 2)) // 16))
print(json.dumps(out))
"""


def case(threads, rows, n, density, chunks, g=1, panels=2, count=1, nb=1, fp32=False, bits=4, fixed=0, pieces=None, flags=0):
    """`chunks`, `pieces`: between which the case has to lie"""
    return dict(threads=threads, rows=rows, n=n, density=density, chunks=chunks, g=g, panels=panels, count=count, nb=nb, fp32=fp32,
                bits=bits, fixed=fixed, pieces=pieces, flags=flags)


ALONE = [
    case(512, 16, 4000, 0.2, (8, 15.5)),
    case(512, 68, 1000, 0.2, (8, 15.5)),                         # tall panels too
    case(768, 16, 4000, 0.3, (16.5, 23.5)),
    case(768, 68, 1000, 0.28, (16.5, 23.5)),
    case(512, 16, 4000, 0.3, (16.5, 23.5), fp32=True),
    case(768, 68, 1000, 0.28, (16.5, 23.5), fp32=True),
    case(1024, 16, 4000, 0.5, (26, 47)),
    case(512, 16, 1800, 0.05, (16.5, 23.5), g=2),                 # one block set
    case(512, 28, 1000, 0.05, (16.5, 23.5), g=2),
    case(768, 32, 900, 0.05, (16.5, 23.5), g=2),
    case(768, 16, 2800, 0.1, (26, 47), g=2),
    case(768, 40, 1200, 0.1, (26, 47), g=2),
    case(1024, 48, 1000, 0.1, (26, 47), g=2),
    case(512, 64, 800, 0.05, (16.5, 23.5), g=4),                # two
    case(1024, 16, 5000, 0.3, (26, 47), g=4),
    case(768, 16, 5000, 0.3, (26, 47), g=8, flags=4),            # three: 8-grained
    case(1024, 64, 2000, 0.15, (26, 47), g=8, flags=4),
    case(1024, 16, 4000, 0.9, (49, 90)),
    case(768, 4, 20480, 0.02, (1, 15.5), pieces=(2049, 3072)),   # more than four pieces for each of 512 threads
    case(1024, 4, 40000, 0.02, (1, 15.5), pieces=(3073, 9999)),
    case(448, 16, 4000, 0.2, (8, 15.5), fixed=448),              # the caller's choice stands
]
SEVERAL = [
    case(512, 16, 900, 0.3, (2, 15.5), panels=50, count=5, pieces=(1, 256)),                       # 250 workgroups
    case(256, 16, 900, 0.3, (2, 15.5), panels=54, count=5, pieces=(1, 256)),                       # 270
    case(512, 24, 900, 0.3, (2, 15.5), panels=54, count=5, pieces=(1, 256)),                       # taller panels
    case(512, 16, 2400, 0.1, (2, 15.5), panels=54, count=5, pieces=(257, 512)),                    # a wider x
    case(256, 16, 1200, 0.2, (2, 15.5), panels=54, count=5, fp32=True, pieces=(257, 512)),
    case(512, 16, 2400, 0.1, (2, 15.5), panels=54, count=5, fp32=True, pieces=(513, 1024)),
    case(512, 16, 2400, 0.1, (2, 15.5), panels=128, count=8, pieces=(257, 512)),                   # 1024
    case(256, 24, 2400, 0.1, (2, 15.5), panels=129, count=8, pieces=(257, 512)),                   # 1032
    case(512, 24, 2400, 0.1, (2, 15.5), panels=96, count=7, fp32=True, pieces=(513, 1024)),        # 672
    case(256, 24, 2400, 0.1, (2, 15.5), panels=96, count=8, fp32=True, pieces=(513, 1024)),        # 768
    case(512, 16, 2400, 0.5, (17, 40), panels=129, count=8, pieces=(257, 1024)),
    case(256, 16, 2400, 0.4, (17, 40), g=8, flags=4, panels=64, count=16, pieces=(257, 1024)),     # 1024, 8-grained
    case(512, 16, 2400, 0.4, (17, 40), g=8, flags=4, panels=63, count=16, pieces=(257, 1024)),     # 1008
    case(512, 16, 2400, 0.4, (17, 40), g=4, panels=64, count=16, pieces=(257, 1024)),
    case(512, 4, 20480, 0.02, (1, 15.5), panels=65, count=16, pieces=(2049, 3072)),                # 512 at most
]
MULTI = [
    case(512, 16, 2000, 0.2, (4, 11.5), nb=8),
    case(1024, 16, 2000, 0.4, (12.5, 19.5), nb=4),
    case(512, 16, 2000, 0.4, (12.5, 19.5), nb=2),
    case(1024, 16, 2000, 0.8, (21, 30), nb=2),
    case(512, 16, 4096, 0.1, (4, 11.5), nb=8),                                                     # 64 KB of X
    case(1024, 16, 4097, 0.1, (4, 11.5), nb=8),
    case(1024, 16, 2400, 0.1, (4, 11.5), nb=8, fp32=True),
    case(512, 16, 4096, 0.2, (12.5, 19.5), nb=2, fp32=True),                                       # 32 KB
    case(1024, 16, 4097, 0.2, (12.5, 19.5), nb=2, fp32=True),
]


@pytest.mark.parametrize("cases", [ALONE, SEVERAL, MULTI], ids=["alone", "several", "multi"])
def test_workgroup_size(tmp_path, cases):
    for c, got in zip(cases, standin.run(tmp_path, CHILD, cases)):
        assert c["chunks"][0] <= got["chunks"] <= c["chunks"][1], (c, got)           # the case is what it says
        if c["pieces"]:
            assert c["pieces"][0] <= got["pieces"] <= c["pieces"][1], (c, got)
        top = {1: 0, 2: 1, 4: 2, 8: 3}[c["g"]]
        assert max([i + 1 for i, s in enumerate(got["sets"]) if s], default=0) == top, (c, got)
        if c["nb"] == 1:
            assert got["grid"] == c["panels"] * c["count"]
        assert got["threads"] == c["threads"], (c, got)
