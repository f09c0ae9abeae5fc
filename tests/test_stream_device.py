"""A launch goes to the device of its stream, also where another device is the current one."""
import standin

CHILD = r"""
W = (np.arange(64 * 64).reshape(64, 64) % 3 == 0).astype(np.float16)
A = B.ecspmv_build_dense(W)
A.ecspmv_upload(0x100000, A.ecspmv_device_bytes(), 0)
out = []
def launch(stream, call):
    try:
        call(stream)
        out.append([stream, fake.fake_launched(KERNEL), fake.fake_launched(STREAM), fake.fake_current()])
    except B.EcspmvError as e:
        out.append([stream, "refused", e.status, fake.fake_current()])
one = lambda s: A.ecspmv_run(0x200000, 0x300000, s)
two = lambda s: A.ecspmv_run_multi(0x200000, 0x300000, 2, s)
for current in (0, 1):
    fake.fake_set(current)
    for call in (one, two):
        for s in (0x1000, 0x2000, 0, 0x2000):
            launch(s, call)
launch(0x3000, one)
print(json.dumps({"out": out, "lookups": fake.fake_lookups(), "hip": B.ERR_HIP}))
"""


def test_launch_on_the_streams_device(tmp_path):
    got = standin.run(tmp_path, CHILD)
    want = []
    for current in (0, 1):
        for _ in range(2):
            for stream, dev in ((0x1000, 0), (0x2000, 1), (0, current), (0x2000, 1)):
                want.append([stream, 0x100 * (dev + 1), stream, current])
    assert got["out"][:-1] == want
    assert got["out"][-1] == [0x3000, "refused", got["hip"], 1]          # a stream that is none
    assert got["lookups"] == 4                                           # one per kernel and device
