"""The encoder's two ways through bits and values, 64 columns at a time where the processor has AVX-512 and one by one anywhere, write
the same images, from dense rows and from CSR, whatever the memory they are written to held before: widths around words and vectors,
dense rows, rows with empty words and gaps beyond the largest delta, both value widths, every delta width and granularity, several
threads and one."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HARNESS = r"""
#include "%s/paper_2507_12205_amd/csrc/encoder.cpp"
#include <cstdio>
#include <cmath>
#include <malloc.h>
static int from_csr(const std::vector<int64_t> &p, const std::vector<int32_t> &c, const std::vector<uint16_t> &v, int m, int n, ecs::Csr &out)
{
    return ecs::csr_from_csr(p.data(), c.data(), v.data(), m, n, out);
}
static int from_csr(const std::vector<int64_t> &p, const std::vector<int32_t> &c, const std::vector<uint32_t> &v, int m, int n, ecs::Csr &out)
{
    return ecs::csr_from_csr_f32(p.data(), c.data(), v.data(), m, n, out);
}
// a matrix of m x n: entries kept with probability `density`, `shared` columns in %% kept by all rows, columns from n / 3 on empty
// for `hole` columns
template <typename T> static void one(int m, int n, double density, int shared, int hole, int bits, int g, int threads)
{
    const int ld = n + (n & 1);
    uint64_t s = 88172645463325252ull + (uint64_t)m * 1000003u + (uint64_t)n;
    auto rnd = [&]() { s ^= s << 13, s ^= s >> 7, s ^= s << 17; return s; };
    std::vector<T> W((size_t)m * ld, 0);
    std::vector<char> all(n);
    for (auto &a : all) a = (int)(rnd() %% 100) < shared;
    for (int i = 0; i < m; ++i)
        for (int j = 0; j < n; ++j) {
            if (j >= n / 3 && j < n / 3 + hole) continue;
            if (all[j] || (double)(rnd() >> 11) * 0x1p-53 < density) W[(size_t)i * ld + j] = (T)(rnd() | 1u);
            else if (rnd() %% 50 == 0) W[(size_t)i * ld + j] = (T)((T)1 << (8 * sizeof(T) - 1));          // a negative zero: not stored
        }
    ecs::BuildParams bp;
    bp.delta_bits = bits, bp.max_granularity = g, bp.num_threads = threads, bp.keep_small_sets = true;
    std::vector<int64_t> rowptr{0};                       // the same as CSR
    std::vector<int32_t> col;
    std::vector<T> val;
    for (int i = 0; i < m; ++i, rowptr.push_back((int64_t)col.size()))
        for (int j = 0; j < n; ++j)
            if (W[(size_t)i * ld + j]) col.push_back(j), val.push_back(W[(size_t)i * ld + j]);
    ecs::Csr csr;
    if (from_csr(rowptr, col, val, m, n, csr)) printf("refused\n");
    for (const ecs::Csr *from : {(const ecs::Csr *)nullptr, (const ecs::Csr *)&csr}) {
        ecs::Image im;
        const int e = ecs::build_image({m, n, (int)(8 * sizeof(T)), from ? nullptr : W.data(), from ? 0 : ld, from}, bp, im);
        uint64_t h = 1469598103934665603ull;
        if (!e)
            for (uint8_t b : im.bytes) h = (h ^ b) * 1099511628211ull;
        printf("%%d %%d %%d %%d %%d %%d: %%d %%zu %%016llx", (int)sizeof(T), m, n, bits, g, threads, e, im.bytes.size(), (unsigned long long)h);
        if (!e)
            for (auto d : im.stats.delta_hist) printf(" %%lld", (long long)d);
        printf("\n");
    }
}
int main(int, char **argv)
{
    mallopt(M_PERTURB, atoi(argv[1]));                    // what fresh memory holds
#ifdef ECS_AVX512
    fprintf(stderr, "%%d\n", (int)ecs::kWide);
#endif
    const int widths[] = {1, 31, 32, 33, 63, 64, 65, 127, 129, 511, 1024, 1029, 4997};
    for (int n : widths)
        for (int bits : {4, 8, 16})
            for (int g : {1, 2, 16}) {
                one<uint16_t>(37, n, 0.4, 30, 0, bits, g, 3), one<uint16_t>(16, n, 0.03, 10, n / 4, bits, g, 1);
                if (bits < 16) one<uint32_t>(37, n, 0.4, 30, 0, bits, g, 3), one<uint32_t>(16, n, 0.03, 10, n / 4, bits, g, 1);
            }
    one<uint16_t>(64, 700, 1.0, 0, 0, 8, 8, 4), one<uint16_t>(64, 700, 0.0, 0, 0, 8, 8, 4), one<uint32_t>(64, 1500, 0.5, 60, 300, 4, 4, 16);
}
"""


def test_same_images(tmp_path):
    src = tmp_path / "harness.cpp"
    src.write_text(HARNESS % ROOT)
    builds = {}
    for name, flags in (("wide", []), ("plain", ["-DECS_NO_AVX512"])):
        exe = tmp_path / name
        builds[name] = (exe, subprocess.Popen(["g++", "-O1", "-std=c++17", "-mpopcnt", "-pthread", "-w", *flags, str(src), "-o", str(exe)]))
    assert all(p.wait() == 0 for _, p in builds.values())
    got = {(name, fill): subprocess.run([str(exe), str(fill)], capture_output=True, text=True, check=True, timeout=300)
           for name, (exe, _) in builds.items() for fill in (0x55, 0xAA)}
    lines = {k: v.stdout.splitlines() for k, v in got.items()}
    first = lines["plain", 0x55]
    assert len(first) == 2 * (13 * 3 * 3 * 2 + 13 * 2 * 3 * 2 + 3) and first[::2] == first[1::2]         # dense, CSR
    assert sum(line.split(": ")[1].startswith("0 ") for line in first) == len(first)
    assert all(v == first for v in lines.values())
    if got["wide", 0x55].stderr.strip() != "1":
        pytest.skip("this processor has no AVX-512: the plain way only")
