"""What the launching calls of the binding take as an address or a stream: what ctypes.c_void_p(value) takes, and nothing else that
ctypes would turn into an address by itself (a bytes object's own memory is host memory)."""
import standin

CODE = r"""
import ctypes
A = B.ecspmv_build_dense(np.ones((16, 128), np.float16), B.make_opts())
A.ecspmv_upload(0x100000, A.ecspmv_device_bytes(), 0)
one = B.Batch([A], [0x200000], [0x300000])
class Passes:
    _as_parameter_ = 0x200000
def outcome(f):
    try:
        f()
        return "ok"
    except B.EcspmvError as e:
        return e.status
    except Exception as e:
        return type(e).__name__
def taken(f):
    got = outcome(f)
    return [got, fake.fake_launched(STREAM) if got == "ok" else 0]
values = [0x1000, True, None, 0, np.int64(0x1000), 1.0, b"stream", "stream", bytearray(8), ctypes.c_void_p(0x1000), ctypes.c_char_p(b"x"),
          (ctypes.c_int * 2)(), ctypes.byref(ctypes.c_int()), Passes(), 2**64 + 0x1000, -2**64 + 0x1000]
rows = []
for v in values:
    try:
        want = ctypes.c_void_p(v).value or 0
    except Exception as e:
        want = type(e).__name__
    rows.append(dict(value=repr(v)[:40], want=want,
                     streams=[taken(lambda: A.ecspmv_run(0x200000, 0x300000, v)), taken(lambda: A.ecspmv_run_multi(0x200000, 0x300000, 2, v)),
                              taken(lambda: one.ecspmv_run_batch(v))],
                     pointers=[outcome(lambda: A.ecspmv_run(v, 0x300000, 0)), outcome(lambda: A.ecspmv_run(0x200000, v, 0)),
                               outcome(lambda: A.ecspmv_run_multi(v, 0x300000, 2, 0)), outcome(lambda: A.ecspmv_run_multi(0x200000, v, 2, 0))]))
counts = []
for v in [2, np.int32(2), 2**32 + 2, 3, None, 2.0, "2", ctypes.c_int32(2), Passes()]:
    try:
        want = ctypes.c_int32(v).value
    except Exception as e:
        want = type(e).__name__
    counts.append([repr(v)[:40], want, outcome(lambda: A.ecspmv_run_multi(0x200000, 0x300000, v, 0))])
print(json.dumps([rows, counts]))
"""


def test_addresses_and_streams(tmp_path):
    rows, counts = standin.run(tmp_path, CODE)
    assert [r["want"] for r in rows] == [0x1000, 1, 0, 0] + ["TypeError"] * 10 + [0x1000, 0x1000]
    for r in rows:
        if r["want"] == "TypeError":
            assert r["streams"] == [["TypeError", 0]] * 3 and r["pointers"] == ["TypeError"] * 4, r
        else:
            assert r["streams"] == [["ok", r["want"]]] * 3 and r["pointers"] == [-1 if r["want"] == 0 or r["want"] % 2 else "ok"] * 4, r
    for value, want, got in counts:
        assert got == (want if want == "TypeError" else "ok" if want == 2 else -1), (value, want, got)
