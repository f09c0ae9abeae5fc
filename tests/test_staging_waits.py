"""What goes from memory straight to LDS carries no register that a later instruction would wait for, and a workgroup's barrier does not wait
for it either: every kernel that stages this way waits for all of its loads by itself between the last such load and the first barrier.
Read from the code the compiler makes of the source before it orders instructions, so that it holds whatever order they get."""
import re
import shutil
import subprocess

import pytest

from paper_2507_12205_amd import build

# (TM, DB, MODE, K, NB, VW): FP32 and one vector, alone and several matrices; several vectors, in one phase and in several
KERNELS = [(0, 8, 0, 5, 1, 4), (3, 4, 1, 5, 1, 4), (0, 4, 0, 4, 2, 2), (0, 4, 3, 4, 8, 2)]
ARGS = ("const uint32_t, const uint32_t, const uint8_t *, const uint16_t *, uint16_t *, const uint32_t, const uint32_t, const uint32_t, "
        "const uint32_t, const uint32_t, const uint32_t, const uint64_t, const std::conditional_t<alone(%d), NoTable, ecs::EcsBatch>")


def compiled(folder, kernels, *flags):
    """{kernel: its code} of some kernels, compiled alone"""
    csrc = folder / "package" / "csrc"
    shutil.copytree(build.CSRC, csrc)
    text = (csrc / "kernels.hip").read_text()
    text = text[:text.index("// ---- plain CSR")].replace("namespace {\n", "namespace kernels {\n", 1)
    text += "".join(f"template __global__ void ecspmv_kernel<{', '.join(map(str, k))}>({ARGS % k[2]});\n" for k in kernels) + "}\n"
    (csrc / "some.hip").write_text(text)
    out = csrc / "some.ll"
    res = subprocess.run(["hipcc", "-O3", "-std=c++17", "--offload-arch=gfx950", "-w", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                          "-x", "hip", *flags, "--cuda-device-only", "-S", "-emit-llvm", str(csrc / "some.hip"), "-o", str(out)],
                         capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    found = {}
    for part in out.read_text().split("\ndefine ")[1:]:
        name = re.search(r"ecspmv_kernelI((?:Li\d+E){6})E", part.split("{")[0])
        if name:
            found[tuple(int(v) for v in re.findall(r"Li(\d+)E", name.group(1)))] = part[:part.index("\n}")]
    return found


@pytest.fixture(scope="module")
def bodies(tmp_path_factory):
    return compiled(tmp_path_factory.mktemp("kernels"), KERNELS)


def first_barriers(body):
    """From every load that goes straight to LDS along every path to the next barrier: whether a wait for all loads (vmcnt(0)) lies on it"""
    blocks = {}
    for part in re.split(r"\n(?=[\w.]+:)", body[body.index("{") + 1:]):
        label = re.match(r"([\w.]+):", part)
        events = re.findall(r"call void @llvm\.amdgcn\.(global\.load\.lds|s\.waitcnt\(i32 3952\)|s\.barrier\(\))", part)
        blocks[label.group(1) if label else "entry"] = (events, re.findall(r"label %([\w.]+)", part))
    waited = []

    def follow(name, at, seen):
        for event in blocks[name][0][at:]:
            if event.startswith("s."):
                waited.append(event.startswith("s.waitcnt"))
                return
        for target in blocks[name][1]:
            if target not in seen:
                seen.add(target)
                follow(target, 0, seen)
    for name, (events, _) in blocks.items():
        for k, event in enumerate(events):
            if event == "global.load.lds":
                follow(name, k + 1, set())
    return waited


@pytest.mark.skipif(not shutil.which("hipcc"), reason="needs the compiler")
@pytest.mark.parametrize("kernel", KERNELS)
def test_loads_to_lds_are_waited_for(bodies, kernel):
    waited = first_barriers(bodies[kernel])
    assert waited and all(waited), waited


@pytest.mark.skipif(not shutil.which("hipcc"), reason="needs the compiler")
def test_the_stamp_behind_the_pieces(tmp_path):
    """Clock stamps, the point where a wavefront's pieces are here: all loads have returned but those of the first chunks, where they were
    requested before: x first, chunks first (indices and two loads of values), the same with two chunks, FP32 (four)."""
    kernels = {(0, 8, 4, 2, 1, 2): 0, (0, 4, 0, 2, 1, 2): 3, (0, 4, 2, 2, 1, 2): 6, (0, 4, 0, 2, 1, 4): 5, (0, 4, 0, 2, 2, 2): 0}
    found = {k: [int(v) for v in re.findall(r'asm sideeffect "s_waitcnt vmcnt\(\$0\)".*?\(i32 (\d+)\)', body)]
             for k, body in compiled(tmp_path, kernels, "-DECS_TRACE=1").items()}
    assert found == {k: [v] for k, v in kernels.items()}
