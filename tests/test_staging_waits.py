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


@pytest.fixture(scope="module")
def bodies(tmp_path_factory):
    """{kernel: its code} of the kernels above, compiled alone"""
    csrc = tmp_path_factory.mktemp("kernels") / "package" / "csrc"
    shutil.copytree(build.CSRC, csrc)
    text = (csrc / "kernels.hip").read_text()
    text = text[:text.index("// ---- plain CSR")].replace("namespace {\n", "namespace kernels {\n", 1)
    text += "".join(f"template __global__ void ecspmv_kernel<{', '.join(map(str, k))}>({ARGS % k[2]});\n" for k in KERNELS) + "}\n"
    (csrc / "some.hip").write_text(text)
    out = csrc / "some.ll"
    res = subprocess.run(["hipcc", "-O3", "-std=c++17", "--offload-arch=gfx950", "-w", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                          "-x", "hip", "--cuda-device-only", "-S", "-emit-llvm", str(csrc / "some.hip"), "-o", str(out)], capture_output=True, text=True)
    assert res.returncode == 0, res.stderr[-2000:]
    found = {}
    for part in out.read_text().split("\ndefine ")[1:]:
        name = re.search(r"ecspmv_kernelI((?:Li\d+E){6})E", part.split("{")[0])
        if name:
            found[tuple(int(v) for v in re.findall(r"Li(\d+)E", name.group(1)))] = part[:part.index("\n}")]
    return found


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
