// Offline phase of EC-SpMV on the host: row panels, hierarchical block extraction (paper Section 4,
// Algorithms 1 and 2), clipping into fixed-size units and ordering (Section 5), EC-CSR encoding with 8-bit
// delta indices, padding and the load permutation (Section 6), plus the decoder used for round-trip checks.
#include "encoder.h"

#include <algorithm>
#include <atomic>
#include <chrono>
#include <condition_variable>
#include <cstring>
#include <exception>
#include <functional>
#include <mutex>
#include <system_error>
#include <thread>

#if defined(__x86_64__) && !defined(ECS_NO_AVX512) && !defined(__HIP_DEVICE_COMPILE__)
#include <immintrin.h>
#define ECS_AVX512 __attribute__((target("avx512f,avx512bw,avx512vl,avx512vpopcntdq,avx512vbmi2,bmi2,popcnt")))
#endif

namespace ecs {

// ------------------------------------------------------------------------------------------------------
// small helpers
// ------------------------------------------------------------------------------------------------------

// The threads of a build: started once, at the first loop that has work for them, and taken through every loop after it (a build has three to
// five; starting 15 threads takes some 0.12 ms, as long as a loop of a 1024 x 1024 matrix: us of a build with threads for each loop /
// once 730 / 590).  Between loops a thread looks for the next one for some 20 us before it sleeps.
class Team {
public:
    explicit Team(int threads) : size_(std::max(1, threads)) {}
    Team(const Team &) = delete;
    Team &operator=(const Team &) = delete;
    ~Team()
    {
        {
            std::lock_guard<std::mutex> g(lock_);
            stop_ = true;
            loop_.fetch_add(1);
        }
        start_.notify_all();
        for (auto &th : pool_) th.join();
    }

    // body(0) ... body(count - 1), in any order and side by side.  An exception in a worker (out of memory) must not end the process: the
    // first one is kept, the other workers stop taking items, and it is thrown again here once every worker is done.  If a thread
    // cannot be started the ones already running do all the work.
    template <class F>
    void run(int64_t count, F &&body)
    {
        if (count <= 0) return;
        if (size_ == 1 || count == 1) {
            for (int64_t i = 0; i < count; ++i) body(i);
            return;
        }
        std::atomic<int64_t> next(0);
        std::atomic<bool> failed(false);
        std::exception_ptr first;
        std::mutex first_lock;
        const std::function<void()> work = [&]() {
            try {
                for (;;) {
                    const int64_t i = next.fetch_add(1);
                    if (i >= count || failed.load(std::memory_order_relaxed)) break;
                    body(i);
                }
            } catch (...) {
                std::lock_guard<std::mutex> g(first_lock);
                if (!first) first = std::current_exception();
                failed.store(true);
            }
        };
        for (int64_t want = std::min<int64_t>(size_, count) - 1; (int64_t)pool_.size() < want;) {
            try {
                pool_.emplace_back([this]() { serve(); });
            } catch (const std::system_error &) {
                break;
            }
        }
        {
            std::lock_guard<std::mutex> g(lock_);
            work_ = &work;
            loop_.fetch_add(1);
        }
        start_.notify_all();
        work();                                       // the calling thread is the last worker
        {
            std::unique_lock<std::mutex> g(lock_);
            done_.wait(g, [&]() { return active_ == 0; });
            work_ = nullptr;                          // a thread that wakes up later finds nothing to do
        }
        if (first) std::rethrow_exception(first);
    }

private:
    void serve()
    {
        uint64_t seen = 0;
        for (;;) {
            for (int k = 0; k < 1000 && loop_.load(std::memory_order_relaxed) == seen; ++k) pause();
            std::unique_lock<std::mutex> g(lock_);
            start_.wait(g, [&]() { return loop_.load() != seen; });
            seen = loop_.load();
            if (stop_) return;
            if (!work_) continue;
            const std::function<void()> &work = *work_;
            ++active_;
            g.unlock();
            work();
            g.lock();
            if (--active_ == 0) done_.notify_one();
        }
    }
    static void pause()
    {
#if defined(__x86_64__)
        __builtin_ia32_pause();
#endif
    }
    const int size_;
    std::vector<std::thread> pool_;
    std::mutex lock_;
    std::condition_variable start_, done_;
    std::atomic<uint64_t> loop_{0};                   // counts the loops; written under the lock
    const std::function<void()> *work_ = nullptr;
    int active_ = 0;
    bool stop_ = false;
};

static inline uint32_t align_up(uint32_t v, uint32_t a) { return (v + a - 1) / a * a; }

static int resolve_threads(int req)
{
    if (req > 0) return std::min(req, 64);
    unsigned hc = std::thread::hardware_concurrency();
    if (hc == 0) hc = 1;
    return (int)std::min<unsigned>(hc, 16);
}

// ------------------------------------------------------------------------------------------------------
// CSR input
// ------------------------------------------------------------------------------------------------------

namespace {

// an entry is stored iff it is neither +0 nor -0
inline bool stored16(uint16_t v) { return (v & 0x7FFFu) != 0; }
inline bool stored32(uint32_t v) { return (v & 0x7FFFFFFFu) != 0; }

template <typename T, typename Stored>
int csr_from_dense_t(const T *W, int64_t m, int64_t n, int64_t ld, int threads, int value_bits, Stored stored, Csr &out)
{
    out.m = m;
    out.n = n;
    out.value_bits = value_bits;
    out.rowptr.assign((size_t)m + 1, 0);
    std::vector<int64_t> cnt((size_t)m, 0);
    Team team(resolve_threads(threads));
    team.run(m, [&](int64_t i) {
        const T *row = W + i * ld;
        int64_t c = 0;
        for (int64_t j = 0; j < n; ++j) c += stored(row[j]);
        cnt[(size_t)i] = c;
    });
    for (int64_t i = 0; i < m; ++i) out.rowptr[(size_t)i + 1] = out.rowptr[(size_t)i] + cnt[(size_t)i];
    out.col.resize((size_t)out.rowptr[(size_t)m]);
    out.val.resize((size_t)out.rowptr[(size_t)m]);
    team.run(m, [&](int64_t i) {
        const T *row = W + i * ld;
        int64_t p = out.rowptr[(size_t)i];
        for (int64_t j = 0; j < n; ++j)
            if (stored(row[j])) {
                out.col[(size_t)p] = (int32_t)j;
                out.val[(size_t)p] = row[j];
                ++p;
            }
    });
    return 0;
}

template <typename T, typename Stored>
int csr_from_csr_t(const int64_t *rowptr, const int32_t *col, const T *val, int64_t m, int64_t n, int value_bits,
                   Stored stored, Csr &out)
{
    if (rowptr[0] != 0) return -1;
    out.m = m;
    out.n = n;
    out.value_bits = value_bits;
    out.rowptr.assign((size_t)m + 1, 0);
    out.col.clear();
    out.val.clear();
    out.col.reserve((size_t)rowptr[m]);
    out.val.reserve((size_t)rowptr[m]);
    for (int64_t i = 0; i < m; ++i) {
        if (rowptr[i + 1] < rowptr[i]) return -1;
        int64_t prev = -1;
        for (int64_t p = rowptr[i]; p < rowptr[i + 1]; ++p) {
            int64_t c = col[p];
            if (c < 0 || c >= n || c <= prev) return -1;
            prev = c;
            if (stored(val[p])) {
                out.col.push_back((int32_t)c);
                out.val.push_back(val[p]);
            }
        }
        out.rowptr[(size_t)i + 1] = (int64_t)out.col.size();
    }
    return 0;
}

}  // namespace

int csr_from_dense(const uint16_t *W, int64_t m, int64_t n, int64_t ld, int threads, Csr &out)
{
    return csr_from_dense_t(W, m, n, ld, threads, 16, stored16, out);
}
int csr_from_csr(const int64_t *rowptr, const int32_t *col, const uint16_t *val, int64_t m, int64_t n, Csr &out)
{
    return csr_from_csr_t(rowptr, col, val, m, n, 16, stored16, out);
}
int csr_from_csr_f32(const int64_t *rowptr, const int32_t *col, const uint32_t *val, int64_t m, int64_t n, Csr &out)
{
    return csr_from_csr_t(rowptr, col, val, m, n, 32, stored32, out);
}

// ------------------------------------------------------------------------------------------------------
// which entries are stored: one bit per column and row
// ------------------------------------------------------------------------------------------------------

// Everything below works on these bits, and a value is fetched from where the caller has it once its place in the image is known:
// no CSR copy of a dense matrix is made (two passes over it, 8 bytes per entry of fresh memory filled twice), no entry is
// searched for.  4096 x 4096 at 50 %, default options, 16 threads, from the dense matrix to the image: 37.9 ms (19.2 of them CSR,
// 11 encoding, the rest extraction and the copy into the image) -> 2.6 (0.35 bits, 1.1 extraction, 0.9 encoding, a third of that for
// fresh pages).

namespace {

// bit k of the result: the k-th of `count` <= 64 values is stored
inline uint64_t stored_bits(const uint16_t *v, int count)
{
    uint64_t out = 0;
    int k = 0;
    for (; k + 4 <= count; k += 4) {                      // four values at a time: the sum of 15 bits and 0x7FFF carries unless they are 0
        uint64_t t;
        std::memcpy(&t, v + k, 8);
        t = ((t & 0x7FFF7FFF7FFF7FFFull) + 0x7FFF7FFF7FFF7FFFull) & 0x8000800080008000ull;
        out |= (((t >> 15) * 0x0001000200040008ull) >> 48) << k;
    }
    for (; k < count; ++k) out |= (uint64_t)stored16(v[k]) << k;
    return out;
}
inline uint64_t stored_bits(const uint32_t *v, int count)
{
    uint64_t out = 0;
    for (int k = 0; k < count; ++k) out |= (uint64_t)stored32(v[k]) << k;
    return out;
}

#ifdef ECS_AVX512
// What follows is done 64 columns at a time where the processor has AVX-512 with its bit counts and compressions; the plain functions
// beside it do the same anywhere.  4096 x 4096 at 50 %, default options, 16
// threads, ms of a build plain / so: 3.31 / 2.58, 4-bit at 30 % 2.07 / 1.79, FP32 3.79 / 3.07.
bool have_avx512()
{
    __builtin_cpu_init();
    return __builtin_cpu_supports("avx512f") && __builtin_cpu_supports("avx512bw") && __builtin_cpu_supports("avx512vl") &&
           __builtin_cpu_supports("avx512vpopcntdq") && __builtin_cpu_supports("avx512vbmi2") && __builtin_cpu_supports("bmi2") &&
           __builtin_cpu_supports("popcnt");
}
const bool kWide = have_avx512();

// the lowest `count` bits, count <= 64
inline uint64_t low_mask(int64_t count) { return count >= 64 ? ~0ull : (1ull << count) - 1ull; }

// bits of a row of n values; returns how many are set
ECS_AVX512 int64_t stored_row_wide(const uint16_t *row, int64_t n, uint64_t *bits)
{
    const __m512i magnitude = _mm512_set1_epi16(0x7FFF);
    int64_t count = 0;
    for (int64_t k = 0; k < n; k += 64) {
        const uint64_t in = low_mask(n - k);
        const __m512i lo = _mm512_maskz_loadu_epi16((__mmask32)in, row + k), hi = _mm512_maskz_loadu_epi16((__mmask32)(in >> 32), row + k + 32);
        const uint64_t b = (uint64_t)_mm512_test_epi16_mask(lo, magnitude) | (uint64_t)_mm512_test_epi16_mask(hi, magnitude) << 32;
        bits[k / 64] = b;
        count += __builtin_popcountll(b);
    }
    return count;
}
ECS_AVX512 int64_t stored_row_wide(const uint32_t *row, int64_t n, uint64_t *bits)
{
    const __m512i magnitude = _mm512_set1_epi32(0x7FFFFFFF);
    int64_t count = 0;
    for (int64_t k = 0; k < n; k += 64) {
        const uint64_t in = low_mask(n - k);
        uint64_t b = 0;
        for (int q = 0; q < 4; ++q) {
            const __m512i v = _mm512_maskz_loadu_epi32((__mmask16)(in >> (16 * q)), row + k + 16 * q);
            b |= (uint64_t)_mm512_test_epi32_mask(v, magnitude) << (16 * q);
        }
        bits[k / 64] = b;
        count += __builtin_popcountll(b);
    }
    return count;
}

ECS_AVX512 int popcount_and_wide(const uint64_t *a, const uint64_t *b, int nw)
{
    __m512i s = _mm512_setzero_si512(), s2 = s;
    int w = 0;
    for (; w + 16 <= nw; w += 16) {
        s = _mm512_add_epi64(s, _mm512_popcnt_epi64(_mm512_and_si512(_mm512_loadu_si512(a + w), _mm512_loadu_si512(b + w))));
        s2 = _mm512_add_epi64(s2, _mm512_popcnt_epi64(_mm512_and_si512(_mm512_loadu_si512(a + w + 8), _mm512_loadu_si512(b + w + 8))));
    }
    for (; w < nw; w += 8) {
        const __mmask8 in = (__mmask8)low_mask(std::min(8, nw - w));
        s = _mm512_add_epi64(s, _mm512_popcnt_epi64(_mm512_and_si512(_mm512_maskz_loadu_epi64(in, a + w), _mm512_maskz_loadu_epi64(in, b + w))));
    }
    return (int)_mm512_reduce_add_epi64(_mm512_add_epi64(s, s2));
}

// bits set, the first and the last word that has some, and how many have
ECS_AVX512 int count_columns_wide(const uint64_t *bits, int nw, int &first, int &last, int &words)
{
    __m512i s = _mm512_setzero_si512();
    for (int w = 0; w < nw; w += 8) {
        const __m512i v = _mm512_maskz_loadu_epi64((__mmask8)low_mask(std::min(8, nw - w)), bits + w);
        s = _mm512_add_epi64(s, _mm512_popcnt_epi64(v));
        const unsigned some = _mm512_test_epi64_mask(v, v);
        if (!some) continue;
        if (last < 0) first = w + __builtin_ctz(some);
        last = w + 31 - __builtin_clz(some);
        words += __builtin_popcount(some);
    }
    return (int)_mm512_reduce_add_epi64(s);
}

// columns and values of the set bits of a row, one after the other; up to 64 of each are written behind the last
ECS_AVX512 inline __m512i iota_bytes()
{
    alignas(64) static const struct Iota {
        uint8_t b[64];
        constexpr Iota() : b()
        {
            for (int k = 0; k < 64; ++k) b[k] = (uint8_t)k;
        }
    } iota;
    return _mm512_load_si512(&iota);
}
ECS_AVX512 inline void put_columns(uint64_t m, int w, int count, uint16_t *cols)
{
    const __m512i at = _mm512_maskz_compress_epi8(m, iota_bytes()), base = _mm512_set1_epi16((short)(64 * w));
    _mm512_storeu_si512(cols, _mm512_add_epi16(_mm512_cvtepu8_epi16(_mm512_castsi512_si256(at)), base));
    if (count > 32) _mm512_storeu_si512(cols + 32, _mm512_add_epi16(_mm512_cvtepu8_epi16(_mm512_extracti64x4_epi64(at, 1)), base));
}
ECS_AVX512 void list_columns_wide(const uint64_t *bits, int nw, uint16_t *cols)
{
    for (int w = 0; w < nw; ++w) {
        const int count = __builtin_popcountll(bits[w]);
        put_columns(bits[w], w, count, cols);
        cols += count;
    }
}
ECS_AVX512 int64_t entries_wide(const uint64_t *bits, int nw, const uint16_t *row, uint16_t *cols, uint16_t *vals)
{
    int64_t n = 0;
    for (int w = 0; w < nw; ++w) {
        const uint64_t m = bits[w];
        if (!m) continue;
        const int count = __builtin_popcountll(m), low = __builtin_popcountll(m & 0xFFFFFFFFull);
        put_columns(m, w, count, cols + n);
        _mm512_storeu_si512(vals + n, _mm512_maskz_compress_epi16((__mmask32)m, _mm512_maskz_loadu_epi16((__mmask32)m, row + 64 * w)));
        const __mmask32 up = (__mmask32)(m >> 32);
        if (up) _mm512_storeu_si512(vals + n + low, _mm512_maskz_compress_epi16(up, _mm512_maskz_loadu_epi16(up, row + 64 * w + 32)));
        n += count;
    }
    return n;
}
ECS_AVX512 int64_t entries_wide(const uint64_t *bits, int nw, const uint32_t *row, uint16_t *cols, uint32_t *vals)
{
    int64_t n = 0;
    for (int w = 0; w < nw; ++w) {
        const uint64_t m = bits[w];
        if (!m) continue;
        const int count = __builtin_popcountll(m);
        put_columns(m, w, count, cols + n);
        uint32_t *to = vals + n;
        for (int q = 0; q < 4; ++q) {
            const __mmask16 in = (__mmask16)(m >> (16 * q));
            if (!in) continue;
            _mm512_storeu_si512(to, _mm512_maskz_compress_epi32(in, _mm512_maskz_loadu_epi32(in, row + 64 * w + 16 * q)));
            to += __builtin_popcount(in);
        }
        n += count;
    }
    return n;
}
#endif

// The rows as the encoder reads them: nw words of bits each, and how many are set.  The bits of a dense matrix are made once (a
// sixteenth of its size at most), and so are those of a CSR matrix where they take no more than its entries do (8 bytes each).
// Otherwise, tall and very sparse, they are made of one panel at a time, whenever they are read: 1 000 000 x 60 000 with two
// entries per row would be 7.5 GB of bits beside 16 MB of entries.
struct Rows {
    int nw = 0;
    const Csr *csr = nullptr;
    RawVector<uint64_t> bits;             // empty: made when they are read
    std::vector<int64_t> count;
    const uint64_t *row(int64_t i) const { return bits.data() + (size_t)i * nw; }
    void from_csr(int64_t i, uint64_t *to) const
    {
        std::memset(to, 0, 8 * (size_t)nw);
        for (int64_t p = csr->rowptr[(size_t)i]; p < csr->rowptr[(size_t)i + 1]; ++p) {
            const int32_t c = csr->col[(size_t)p];
            to[c >> 6] |= 1ull << (c & 63);
        }
    }
    void read(int64_t i, uint64_t *to) const
    {
        if (bits.empty()) from_csr(i, to);
        else std::memcpy(to, row(i), 8 * (size_t)nw);
    }
};

template <typename T>
void read_dense(const Source &A, Team &team, Rows &out)
{
    constexpr int64_t kRows = 16;                         // rows a worker takes at a time
    const int nw = out.nw;
    const T *W = static_cast<const T *>(A.dense);
    team.run((A.m + kRows - 1) / kRows, [&](int64_t blk) {
        for (int64_t i = blk * kRows; i < std::min(A.m, (blk + 1) * kRows); ++i) {
            const T *row = W + i * A.ld;
            uint64_t *b = out.bits.data() + (size_t)i * nw;
            int64_t c = 0;
#ifdef ECS_AVX512
            if (kWide) {
                out.count[(size_t)i] = stored_row_wide(row, A.n, b);
                continue;
            }
#endif
            for (int w = 0; w < nw; ++w) {
                b[w] = stored_bits(row + 64 * w, (int)std::min<int64_t>(64, A.n - 64 * w));
                c += __builtin_popcountll(b[w]);
            }
            out.count[(size_t)i] = c;
        }
    });
}

void read_rows(const Source &A, Team &team, Rows &out)
{
    out.nw = (int)((A.n + 63) / 64);
    out.csr = A.csr;
    out.count.resize((size_t)A.m);
    if (A.csr) {
        for (int64_t i = 0; i < A.m; ++i) out.count[(size_t)i] = A.csr->rowptr[(size_t)i + 1] - A.csr->rowptr[(size_t)i];
        if (A.m * out.nw > A.csr->rowptr[(size_t)A.m]) return;
    }
    out.bits.resize((size_t)A.m * out.nw);
    if (A.csr) team.run(A.m, [&](int64_t i) { out.from_csr(i, out.bits.data() + (size_t)i * out.nw); });
    else if (A.value_bits == 16) read_dense<uint16_t>(A, team, out);
    else read_dense<uint32_t>(A, team, out);
}

// ------------------------------------------------------------------------------------------------------
// hierarchical block extraction inside one panel
// ------------------------------------------------------------------------------------------------------

// The rows of a level matrix (Algorithm 1's A_E / A_R).  At level l a row stands for 2^l original rows
// (`members`) and a set bit at column c means all of them hold a stored entry at c (Section 4.2).
struct Level {
    int nw, width;                        // words per row; 2^l
    std::vector<uint64_t> bits;
    std::vector<int> cnt;
    std::vector<int> child_a, child_b;    // the two rows of the level below a block was extracted from
    std::vector<int> members;             // panel-local original rows, `width` of each row
    int rows() const { return (int)cnt.size(); }
    uint64_t *row(int i) { return bits.data() + (size_t)i * nw; }
};

// What extraction leaves of a panel
struct PanelUnits {
    // extracted units per block type t (g = 2 << t): g member rows (panel-local) and 64 sorted columns each, and how many units
    // the unit's block has
    struct Set {
        std::vector<int> rows, block_len;
        std::vector<uint16_t> cols;
        uint32_t size() const { return (uint32_t)block_len.size(); }
    } units[ECS_NUM_BTYPES];
    std::vector<uint64_t> resid;          // bits of the residual entries, row by row (empty where they are found again when the panel is written)
};

inline int popcount_and(const uint64_t *a, const uint64_t *b, int nw)
{
#ifdef ECS_AVX512
    if (kWide) return popcount_and_wide(a, b, nw);
#endif
    int s = 0;
    for (int w = 0; w < nw; ++w) s += __builtin_popcountll(a[w] & b[w]);
    return s;
}

// the lowest `keep` set bits of v
inline uint64_t lowest_bits(uint64_t v, int keep)
{
    uint64_t rest = v;
    for (int k = 0; k < keep; ++k) rest &= rest - 1;
    return v ^ rest;
}

// the columns set, one after the other (up to 64 more are written behind the last)
inline void list_columns(const uint64_t *bits, int nw, uint16_t *to)
{
#ifdef ECS_AVX512
    if (kWide) return list_columns_wide(bits, nw, to);
#endif
    for (int w = 0; w < nw; ++w)
        for (uint64_t v = bits[w]; v; v &= v - 1) *to++ = (uint16_t)(64 * w + __builtin_ctzll(v));
}

// How many columns are set, and whether a word between two that have some has none
inline int count_columns(const uint64_t *bits, int nw, bool &gaps)
{
    int total = 0, first = nw, last = -1, words = 0;
#ifdef ECS_AVX512
    if (kWide) {
        total = count_columns_wide(bits, nw, first, last, words);
        gaps = total && words != last - first + 1;
        return total;
    }
#endif
    for (int w = 0; w < nw; ++w) {
        if (!bits[w]) continue;
        total += __builtin_popcountll(bits[w]);
        first = std::min(first, w), last = w, ++words;
    }
    gaps = total && words != last - first + 1;
    return total;
}

// Cut the columns set in `bits` into units of 64 columns whose successive gaps fit a delta index (Section 6.2: a
// block takes only columns that lie within the delta range of their neighbour; Section 6.3.1: block widths are
// whole multiples of the load quantum, here one unit).  A run is a longest sequence of columns with such gaps; its units are its
// first 64, 128, ... columns, and what is left of it is in no unit.  Leaves the columns of units in `bits`, the others in `rest`
// (if it is not null); returns the number of units.
int form_units(uint64_t *bits, uint64_t *rest, int nw, int32_t max_delta)
{
    int units = 0, run = 0;               // columns of the current run
    int64_t last = -1;                    // its last column
    // the last `n` columns set at or before word w belong to no unit
    auto drop = [&](int w, int n) {
        for (; n > 0; --w) {
            const int here = __builtin_popcountll(bits[w]), take = std::min(n, here);
            const uint64_t stay = lowest_bits(bits[w], here - take);
            if (rest) rest[w] |= bits[w] ^ stay;
            bits[w] = stay;
            n -= take;
        }
    };
    auto end_run = [&](int w) {
        units += run / (int)ECS_UNIT_COLS;
        drop(w, run % (int)ECS_UNIT_COLS);
        run = 0;
    };
    if (rest) std::memset(rest, 0, 8 * (size_t)nw);
    // Too few columns for a unit, or, as mostly, one run: where no word between two columns is empty there are at most 126 zeros side by side
    bool gaps;
    const int total = count_columns(bits, nw, gaps);
    if (total < (int)ECS_UNIT_COLS || (!gaps && max_delta > 126)) {
        run = total;
        end_run(nw - 1);
        return units;
    }
    for (int w = 0; w < nw; ++w) {
        if (max_delta >= 63) {            // no run ends inside a word
            const uint64_t v = bits[w];
            if (!v) continue;
            if (run && 64 * (int64_t)w + __builtin_ctzll(v) - last > max_delta) end_run(w - 1);
            run += __builtin_popcountll(v);
            last = 64 * (int64_t)w + 63 - __builtin_clzll(v);
        } else {
            for (uint64_t v = bits[w], done = 0; v;) {
                const uint64_t low = v & (0 - v);
                const int64_t col = 64 * (int64_t)w + __builtin_ctzll(v);
                if (run && col - last > max_delta) {      // the run ends inside this word, or with one before it
                    const uint64_t later = bits[w] & ~done;
                    bits[w] &= done;
                    end_run(w);
                    bits[w] |= later;
                }
                ++run;
                last = col;
                done |= low;
                v ^= low;
            }
        }
    }
    if (run) end_run(nw - 1);
    return units;
}

// Greedy row matching (Algorithm 2).  Rows are popped in order of decreasing column count (ties: lower
// index first); the popped row takes the still unselected row with which it shares the most columns
// (ties: lower index).  A pair is kept only if the shared count reaches one unit, otherwise the popped
// row stays single this round.
// `seen`: for every two rows how many columns they shared when that was last counted in this level, or more.  Rows only lose
// columns from one round to the next, so two rows that cannot beat the current best by it need not be counted again
// (4096 x 4096 at 50 %, blocks of up to 8 rows: 585 000 counts in the place
// of 918 000, 1.7 ms of 16 threads in the place of 2.2 with words counted one by one, 0.4 eight at a time).  Empty for levels too large to keep it.
void row_matching(Level &L, std::vector<int> &seen, std::vector<int> &order, std::vector<char> &unselected,
                  std::vector<std::pair<int, int>> &pairs)
{
    pairs.clear();
    order.clear();
    const int R = L.rows();
    unselected.assign((size_t)R, 0);
    for (int i = 0; i < R; ++i)
        if (L.cnt[i] >= (int)ECS_UNIT_COLS) order.push_back(i), unselected[i] = 1;
    std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return L.cnt[a] > L.cnt[b]; });
    for (int a : order) {
        if (!unselected[a]) continue;
        unselected[a] = 0;
        int best = -1, best_sim = (int)ECS_UNIT_COLS - 1;
        for (int b = 0; b < R; ++b) {
            if (!unselected[b]) continue;
            if (L.cnt[b] <= best_sim) continue;             // cannot beat the current best
            int *last = seen.empty() ? nullptr : &seen[(size_t)std::min(a, b) * R + std::max(a, b)];
            if (last && *last <= best_sim) continue;
            const int sim = popcount_and(L.row(a), L.row(b), L.nw);
            if (last) *last = sim;
            if (sim > best_sim) {
                best_sim = sim;
                best = b;
            }
        }
        if (best >= 0) {
            pairs.emplace_back(a, best);
            unselected[best] = 0;
        }
    }
}

void extract_panel(const Rows &A, const int32_t *prow, int nrows, int max_g, int max_rounds, int delta_bits, PanelUnits &out)
{
    const int32_t max_delta = (int32_t)ECS_MAX_DELTA(delta_bits);
    const int nw = A.nw;
    std::vector<Level> levels(1);
    {
        Level &L = levels[0];
        L.nw = nw, L.width = 1;
        L.bits.resize((size_t)nrows * nw);
        for (int r = 0; r < nrows; ++r) {
            A.read(prow[r], L.row(r));
            L.members.push_back(r);
            L.cnt.push_back((int)A.count[(size_t)prow[r]]);
        }
    }

    std::vector<std::pair<int, int>> pairs;
    std::vector<int> order, seen;
    std::vector<char> unselected;
    std::vector<uint64_t> common(nw), rest(nw);

    // Algorithm 1: multi-level aggregation (outer), multi-round extraction (inner).
    for (int level = 0; (2 << level) <= max_g; ++level) {
        Level next;                                 // blocks extracted at this level = rows of the next A_E
        next.nw = nw, next.width = 2 << level;
        Level &AR = levels[level];
        seen.assign(AR.rows() <= 1024 ? (size_t)AR.rows() * AR.rows() : 0, nw * 64);
        for (int round = 0; round < max_rounds; ++round) {
            row_matching(AR, seen, order, unselected, pairs);
            bool any = false;
            for (auto &pr : pairs) {
                uint64_t *__restrict__ a = AR.row(pr.first), *__restrict__ b = AR.row(pr.second);
                for (int w = 0; w < nw; ++w) common[w] = a[w] & b[w];
                const int nu = form_units(common.data(), nullptr, nw, max_delta);
                if (!nu) continue;
                any = true;
                for (int w = 0; w < nw; ++w) a[w] &= ~common[w], b[w] &= ~common[w];      // extracted entries leave A_R
                const int cnt = nu * (int)ECS_UNIT_COLS;
                AR.cnt[pr.first] -= cnt;
                AR.cnt[pr.second] -= cnt;
                next.bits.insert(next.bits.end(), common.begin(), common.end());
                next.cnt.push_back(cnt);
                next.child_a.push_back(pr.first);
                next.child_b.push_back(pr.second);
                for (int side : {pr.first, pr.second})
                    next.members.insert(next.members.end(), AR.members.begin() + (size_t)side * AR.width,
                                        AR.members.begin() + (size_t)(side + 1) * AR.width);
            }
            if (!any) break;
        }
        if (!next.rows()) break;
        levels.push_back(std::move(next));
    }

    // Decode what is left at every level into blocks of that level's granularity, coarsest first.  Columns
    // of a level >= 1 row that no longer form a valid unit (a neighbour was lifted to a coarser block and the
    // gap now exceeds the delta range) fall back to the two rows of the level below.
    std::vector<uint16_t> columns(levels.size() > 1 ? 64 * (size_t)nw + 64 : 0);
    for (int level = (int)levels.size() - 1; level >= 1; --level) {
        Level &L = levels[level], &below = levels[level - 1];
        PanelUnits::Set &set = out.units[level - 1];
        for (int i = 0; i < L.rows(); ++i) {
            const int nu = form_units(L.row(i), rest.data(), nw, max_delta);
            uint64_t *__restrict__ ca = below.row(L.child_a[i]), *__restrict__ cb = below.row(L.child_b[i]);
            for (int w = 0; w < nw; ++w) ca[w] |= rest[w], cb[w] |= rest[w];
            if (!nu) continue;
            list_columns(L.row(i), nw, columns.data());
            set.cols.insert(set.cols.end(), columns.begin(), columns.begin() + (size_t)ECS_UNIT_COLS * nu);
            for (int u = 0; u < nu; ++u) {
                set.rows.insert(set.rows.end(), L.members.begin() + (size_t)i * L.width, L.members.begin() + (size_t)(i + 1) * L.width);
                set.block_len.push_back(nu);
            }
        }
    }
    out.resid = std::move(levels[0].bits);
}

inline int hist_bin(unsigned d)
{
    return d == 0 ? 0 : std::min(8, 32 - __builtin_clz(d));
}

// index k of an array of `bits`-wide indices: a delta with 8 or 4 bits (with 4 bits the earlier delta of a byte
// sits in its low nibble), the column itself with 16 bits (index compression switched off)
inline uint32_t get_delta(const uint8_t *d, size_t k, int bits)
{
    if (bits == 16) return reinterpret_cast<const uint16_t *>(d)[k];
    return bits == 8 ? d[k] : ((d[k >> 1] >> (4 * (k & 1))) & 0xF);
}

// Where everything of a panel goes, known before any of it is written
struct PanelLayout {
    uint32_t hdr[ECS_PANEL_HEADER / 4];
    std::vector<uint32_t> rowlu, rowslot;                 // first lane unit, first slot of every row
    uint64_t bytes = 0;
    uint32_t meta_bytes = 0, nslots = 0, nchunks = 0;
    int64_t value_bytes = 0, delta_bytes = 0, pad_elements = 0, gap_pads = 0;
    int64_t nnz_by_g[5] = {0, 0, 0, 0, 0};
    int64_t units_by_g[5] = {0, 0, 0, 0, 0};
    int64_t delta_hist[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    int err = 0;
};

// Whether there are `width` zeros in a row between the lowest and the highest bit set (width 15: the only one asked for)
inline bool has_gap(uint64_t v, int width)
{
    uint64_t z = ~v & (((1ull << (63 - __builtin_clzll(v))) - 1ull) & ~(((v & (0 - v)) << 1) - 1ull));       // zeros between the two
    for (int run = 1; run < width && z; run *= 2) z &= z >> std::min(run, width - run);
    return z != 0;
}

// How many residual entries a row has, and how many zeros fill its gaps beyond the largest delta (one every R_P - 1 columns,
// Section 6.2).  Where the largest delta covers a word no gap inside one is too wide.
inline void count_residual(const uint64_t *bits, int nw, int32_t max_delta, int64_t &entries, int64_t &fillers)
{
    int64_t last = -1;
    entries = fillers = 0;
    for (int w = 0; w < nw; ++w) {
        uint64_t v = bits[w];
        if (!v) continue;
        entries += __builtin_popcountll(v);
        const int64_t first = 64 * (int64_t)w + __builtin_ctzll(v);
        if (last >= 0) fillers += (first - last - 1) / max_delta;
        last = 64 * (int64_t)w + 63 - __builtin_clzll(v);
        if (max_delta < 63 && has_gap(v, max_delta))
            for (int64_t prev = first; v &= v - 1;) {
                const int64_t col = 64 * (int64_t)w + __builtin_ctzll(v);
                fillers += (col - prev - 1) / max_delta;
                prev = col;
            }
    }
}

void lay_out_panel(const Rows &A, const int32_t *prow, int nrows, const PanelUnits &pu, int delta_bits, int value_bits, PanelLayout &out)
{
    const int32_t max_delta = (int32_t)ECS_MAX_DELTA(delta_bits);
    const uint32_t unit_db = ECS_UNIT_DBYTES(delta_bits), lane_db = ECS_LANE_DBYTES(delta_bits);
    const uint32_t vw = (uint32_t)value_bits / 8u;        // bytes per value
    // ---- slots: one per (unit, member row), a row's slots are consecutive; the residual set needs no table for
    // its partial sums (one per lane unit, in stream order) beyond the first lane unit of every row
    out.rowslot.assign((size_t)nrows + 1, 0);
    for (int t = 0; t < ECS_NUM_BTYPES; ++t)
        for (int r : pu.units[t].rows) ++out.rowslot[(size_t)r + 1];
    for (int r = 0; r < nrows; ++r) out.rowslot[(size_t)r + 1] += out.rowslot[(size_t)r];
    out.nslots = out.rowslot[(size_t)nrows];
    // ---- residual rows: entries, gap fillers and tail padding -> lane units, and the row segments of the chunks
    out.rowlu.assign((size_t)nrows + 1, 0);
    uint32_t nentries = 0;
    for (int r = 0; r < nrows; ++r) {
        int64_t entries, fillers;
        count_residual(pu.resid.data() + (size_t)r * A.nw, A.nw, max_delta, entries, fillers);
        const int64_t lanes = (entries + fillers + ECS_LANE_ELEMS - 1) / ECS_LANE_ELEMS;
        const uint32_t l0 = out.rowlu[(size_t)r], l1 = l0 + (uint32_t)lanes;
        out.rowlu[(size_t)r + 1] = l1;
        if (lanes) nentries += (l1 - 1) / ECS_CHUNK_LANES - l0 / ECS_CHUNK_LANES + 1;
        out.nnz_by_g[0] += entries;
        out.gap_pads += fillers;
        out.pad_elements += lanes * ECS_LANE_ELEMS - entries;
    }
    const uint32_t nlanes = out.rowlu[(size_t)nrows];
    const uint32_t nchunks = out.nchunks = (nlanes + ECS_CHUNK_LANES - 1) / ECS_CHUNK_LANES;
    out.units_by_g[0] = nlanes;
    if (out.nslots > 65535u || nrows > 65535) {
        out.err = -2;
        return;
    }

    uint32_t *hdr = out.hdr;
    std::memset(hdr, 0, sizeof(out.hdr));
    uint64_t off = ECS_PANEL_HEADER;
    auto up = [](uint64_t v, uint64_t a) { return (v + a - 1) / a * a; };
    hdr[PH_ROW0] = (uint32_t)prow[0];
    hdr[PH_NROWS] = (uint32_t)nrows;
    hdr[PH_NSLOTS] = out.nslots;
    hdr[PH_NRLANES] = nlanes;
    hdr[PH_NRENTRIES] = nentries;
    hdr[PH_ROWSLOT_OFF] = (uint32_t)off;
    off = up(off + 2u * (uint32_t)(nrows + 1), 16);
    hdr[PH_ROWLU_OFF] = (uint32_t)off;
    off = up(off + 4u * (uint32_t)(nrows + 1), 16);
    hdr[PH_ROWIDX_OFF] = (uint32_t)off;
    off = up(off + 4u * (uint32_t)nrows, 16);
    for (int t = ECS_NUM_BTYPES - 1; t >= 0; --t) {
        const uint32_t g = 2u << t;
        hdr[PH_NUNITS + t] = pu.units[t].size();
        hdr[PH_UTAB_OFF + t] = (uint32_t)off;
        off = up(off + 2ull * (1 + g) * pu.units[t].size(), 16);
    }
    hdr[PH_RCHUNK_OFF] = (uint32_t)off;
    off += sizeof(EcsRChunk) * (uint64_t)nchunks;
    hdr[PH_RENTRY_OFF] = (uint32_t)off;
    off = up(off + sizeof(EcsREntry) * (uint64_t)nentries, 16);
    hdr[PH_ZERO_OFF] = (uint32_t)off;
    off += 16;
    out.meta_bytes = (uint32_t)off;
    hdr[PH_META_BYTES] = (uint32_t)off;
    // Residual chunks first: a chunk = the deltas of its 64 lane units, then their values, the k-th 128-bit load of
    // lane l at k * 1024 + 16 * l; a last chunk of nl < 64 lane units is stored tightly (nl delta runs padded to 16
    // bytes, then the k-th load of lane l at 16 * nl * k + 16 * l).
    const uint64_t res_off = off;                                       // a multiple of 16
    const uint32_t chunk_bytes = ECS_CHUNK_DBYTES(delta_bits) + 1024u * vw;
    hdr[PH_RD_OFF] = (uint32_t)res_off;
    hdr[PH_RV_OFF] = chunk_bytes;
    off = res_off + (uint64_t)chunk_bytes * nchunks;
    if (nchunks) {
        const uint32_t nl_last = nlanes - (nchunks - 1) * ECS_CHUNK_LANES;
        if (nl_last < ECS_CHUNK_LANES)
            off = res_off + (uint64_t)chunk_bytes * (nchunks - 1) + align_up(lane_db * nl_last, 16) + 16u * vw * nl_last;
    }
    out.delta_bytes += (int64_t)lane_db * nlanes;
    out.value_bytes += 16ll * vw * nlanes;
    for (int t = ECS_NUM_BTYPES - 1; t >= 0; --t) {
        const uint32_t g = 2u << t;
        const uint64_t nu = pu.units[t].size();
        hdr[PH_BD_OFF + t] = (uint32_t)off;
        off += unit_db * nu;              // multiple of 16
        hdr[PH_BV_OFF + t] = (uint32_t)off;
        off += 64u * vw * g * nu;
        out.delta_bytes += (int64_t)(unit_db * nu);
        out.value_bytes += (int64_t)(64ull * vw * g * nu);
        out.units_by_g[t + 1] = (int64_t)nu;
        out.nnz_by_g[t + 1] = (int64_t)(nu * ECS_UNIT_COLS * g);
    }
    out.bytes = up(off, 256);
    hdr[PH_PANEL_BYTES] = (uint32_t)out.bytes;
}

// f(column, value) for every set bit of a row in turn
template <class Row, class F>
inline void for_each_entry(const uint64_t *bits, int nw, const Row &row, F &&f)
{
    for (int w = 0; w < nw; ++w)
        for (uint64_t m = bits[w]; m; m &= m - 1) {
            const int32_t col = 64 * w + __builtin_ctzll(m);
            f(col, row[(uint32_t)col]);
        }
}

// f(column, value) put one after the other; returns how many
template <typename T, class Each>
inline int64_t list_entries(uint16_t *cols, T *vals, Each &&each)
{
    int64_t n = 0;
    each([&](int32_t col, uint32_t value) { cols[n] = (uint16_t)col, vals[n] = (T)value, ++n; });
    return n;
}

// Where the values of a panel's stored entries come from: row(r)[column], and the residual entries of row r, columns and values
// (up to 64 of each may be written behind the last).
template <typename T>
struct DensePanel {
    const T *W;
    int64_t ld;
    const int32_t *prow;
    const uint64_t *resid;
    int nw;
    struct Row {
        const T *v;
        uint32_t operator[](uint32_t col) const { return v[col]; }
    };
    Row row(int r) const { return {W + (int64_t)prow[r] * ld}; }
    // Units read their rows here and there, a miss at a time: the rows are asked for one after the other first.
    void expect(int nrows, int64_t n) const
    {
        for (int r = 0; r < nrows; ++r) {
            const char *v = reinterpret_cast<const char *>(row(r).v);
            for (int64_t k = 0; k < n * (int64_t)sizeof(T); k += 64) __builtin_prefetch(v + k);
        }
    }
    void blocks_written() {}
    int64_t entries(int r, uint16_t *cols, T *vals) const
    {
        const uint64_t *b = resid + (size_t)r * nw;
#ifdef ECS_AVX512
        if (kWide) return entries_wide(b, nw, row(r).v, cols, vals);
#endif
        return list_entries(cols, vals, [&](auto &&f) { for_each_entry(b, nw, row(r), f); });
    }
};

// An entry's place in its row is how many bits are set before its column: `rank` holds how many before each word (a row has fewer
// than 65536 columns).
struct CsrRow {
    const uint32_t *v;
    const uint16_t *rank;
    const uint64_t *bits;
    uint32_t operator[](uint32_t col) const
    {
        const uint32_t w = col >> 6;
        return v[rank[w] + (uint32_t)__builtin_popcountll(bits[w] & ((1ull << (col & 63)) - 1ull))];
    }
};
inline void rank_words(const uint64_t *bits, int nw, uint16_t *rank)
{
    uint32_t before = 0;
    for (int w = 0; w < nw; ++w) {
        rank[w] = (uint16_t)before;
        before += (uint32_t)__builtin_popcountll(bits[w]);
    }
}

// a CSR matrix whose bits were kept
struct CsrPanel {
    const Rows &rows;
    const int32_t *prow;
    const uint64_t *resid;
    std::vector<uint16_t> rank;
    CsrPanel(const Rows &all, const int32_t *panel_rows, int nrows, const PanelUnits &pu)
        : rows(all), prow(panel_rows), resid(pu.resid.data()), rank((size_t)nrows * all.nw)
    {
        for (int r = 0; r < nrows; ++r) rank_words(rows.row(prow[r]), rows.nw, rank.data() + (size_t)r * rows.nw);
    }
    CsrRow row(int r) const
    {
        return {rows.csr->val.data() + rows.csr->rowptr[(size_t)prow[r]], rank.data() + (size_t)r * rows.nw, rows.row(prow[r])};
    }
    void expect(int, int64_t) const {}
    void blocks_written() {}
    template <typename T>
    int64_t entries(int r, uint16_t *cols, T *vals) const
    {
        return list_entries(cols, vals, [&](auto &&f) { for_each_entry(resid + (size_t)r * rows.nw, rows.nw, row(r), f); });
    }
};

// A CSR matrix whose bits were not: a panel with units makes its own, and takes the units' columns out of them once the blocks are
// written.  Without units every entry is a residual one.
struct SparseCsrPanel {
    const Rows &rows;
    const int32_t *prow;
    const PanelUnits &pu;
    std::vector<uint64_t> bits;
    std::vector<uint16_t> rank;
    SparseCsrPanel(const Rows &all, const int32_t *panel_rows, int nrows, const PanelUnits &units)
        : rows(all), prow(panel_rows), pu(units)
    {
        bool any = false;
        for (auto &set : pu.units) any |= set.size() != 0;
        if (!any) return;
        bits.resize((size_t)nrows * rows.nw);
        rank.resize((size_t)nrows * rows.nw);
        for (int r = 0; r < nrows; ++r) {
            rows.read(prow[r], bits.data() + (size_t)r * rows.nw);
            rank_words(bits.data() + (size_t)r * rows.nw, rows.nw, rank.data() + (size_t)r * rows.nw);
        }
    }
    CsrRow row(int r) const
    {
        return {rows.csr->val.data() + rows.csr->rowptr[(size_t)prow[r]], rank.data() + (size_t)r * rows.nw, bits.data() + (size_t)r * rows.nw};
    }
    void expect(int, int64_t) const {}
    void blocks_written()
    {
        for (int t = 0; t < ECS_NUM_BTYPES; ++t) {
            const PanelUnits::Set &set = pu.units[t];
            const uint32_t g = 2u << t;
            for (uint32_t u = 0; u < set.size(); ++u)
                for (uint32_t r = 0; r < g; ++r) {
                    uint64_t *b = bits.data() + (size_t)set.rows[(size_t)g * u + r] * rows.nw;
                    for (uint32_t k = 0; k < ECS_UNIT_COLS; ++k) {
                        const uint32_t col = set.cols[(size_t)ECS_UNIT_COLS * u + k];
                        b[col >> 6] &= ~(1ull << (col & 63));
                    }
                }
        }
    }
    template <typename T>
    int64_t entries(int r, uint16_t *cols, T *vals) const
    {
        const Csr &A = *rows.csr;
        const uint64_t *b = bits.empty() ? nullptr : bits.data() + (size_t)r * rows.nw;
        return list_entries(cols, vals, [&](auto &&f) {
            for (int64_t p = A.rowptr[(size_t)prow[r]]; p < A.rowptr[(size_t)prow[r] + 1]; ++p) {
                const int32_t col = A.col[(size_t)p];
                if (!b || (b[col >> 6] >> (col & 63) & 1)) f(col, A.val[(size_t)p]);
            }
        });
    }
};

// The values of a unit of G rows (`cols`: its 64 columns).  Permutation: lane j owns the values f = column * G + row of its columns 4 j ...
// 4 j + 3; its k-th 128-bit group (8 halfs or 4 floats) goes to byte k * 256 + 16 * j of the unit.
template <uint32_t G, typename T, class Values>
void write_unit(const Values &values, const int *rows, const uint16_t *cols, T *v)
{
    constexpr uint32_t ep = 16u / sizeof(T);
    decltype(values.row(0)) row[G];
    for (uint32_t r = 0; r < G; ++r) row[r] = values.row(rows[r]);
    for (uint32_t j = 0; j < 16; ++j)
        for (uint32_t f = 0; f < 4 * G; ++f) v[f / ep * 16 * ep + ep * j + f % ep] = (T)row[f % G][cols[4 * j + f / G]];
}

// 16 indices, `col` being their columns and col[-1] the one before: deltas, or the columns themselves with 16 bits.  Whole bytes are put
// together and written once: what was there before is not read.
template <int BITS>
void write_indices(const uint16_t *col, uint8_t *d)
{
    if constexpr (BITS == 16) {
        std::memcpy(d, col, 32);
        return;
    }
    uint8_t b[16];
    for (int i = 0; i < 16; ++i) b[i] = (uint8_t)(col[i] - col[i - 1]);
    if constexpr (BITS == 4)
        for (int i = 0; i < 8; ++i) b[i] = (uint8_t)(b[2 * i] | b[2 * i + 1] << 4);
    std::memcpy(d, b, 2 * BITS);
}
inline void write_indices(int bits, const uint16_t *col, uint8_t *d)
{
    if (bits == 8) write_indices<8>(col, d);
    else if (bits == 4) write_indices<4>(col, d);
    else write_indices<16>(col, d);
}

// Writes a panel of `bytes` bytes to P.
template <typename T, class Values>
void encode_panel(Values &&values, int64_t n, const int32_t *prow, int nrows, const PanelUnits &pu, bool reorder, int delta_bits,
                  PanelLayout &lay, uint8_t *P, size_t bytes)
{
    const uint32_t *hdr = lay.hdr;
    const int32_t max_delta = (int32_t)ECS_MAX_DELTA(delta_bits);
    const uint32_t unit_db = ECS_UNIT_DBYTES(delta_bits), lane_db = ECS_LANE_DBYTES(delta_bits);
    constexpr uint32_t vw = sizeof(T), ep = 16u / vw;     // bytes per value, values per 128-bit load

    // zeros where nothing is written below: in the tables, after the indices of a last chunk, and behind the values of the last set
    const uint32_t last_chunk = hdr[PH_RD_OFF] + hdr[PH_RV_OFF] * (lay.nchunks ? lay.nchunks - 1 : 0);
    const size_t end = hdr[PH_BV_OFF] + 64ull * vw * 2 * hdr[PH_NUNITS];
    std::memset(P, 0, hdr[PH_META_BYTES]);
    if (lay.nchunks) std::memset(P + last_chunk, 0, align_up(lane_db * (hdr[PH_NRLANES] - ECS_CHUNK_LANES * (lay.nchunks - 1)), 16));
    std::memset(P + end, 0, bytes - end);
    values.expect(nrows, n);
    std::memcpy(P, hdr, sizeof(lay.hdr));
    uint16_t *rs = (uint16_t *)(P + hdr[PH_ROWSLOT_OFF]);
    for (int r = 0; r <= nrows; ++r) rs[r] = (uint16_t)lay.rowslot[(size_t)r];
    std::memcpy(P + hdr[PH_ROWLU_OFF], lay.rowlu.data(), 4u * (size_t)(nrows + 1));
    std::memcpy(P + hdr[PH_ROWIDX_OFF], prow, 4u * (size_t)nrows);

    // ---- block sets.  Ordering (Section 5): sets by decreasing granularity (fixed by the layout); inside a set the
    // units of longer blocks first.
    std::vector<uint32_t> cursor(lay.rowslot.begin(), lay.rowslot.end() - 1), order;
    for (int t = ECS_NUM_BTYPES - 1; t >= 0; --t) {
        const uint32_t g = 2u << t;
        const PanelUnits::Set &set = pu.units[t];
        order.resize(set.size());
        for (uint32_t u = 0; u < set.size(); ++u) order[u] = u;
        if (reorder)
            std::stable_sort(order.begin(), order.end(), [&](uint32_t a, uint32_t b) { return set.block_len[a] > set.block_len[b]; });
        uint16_t *utab = (uint16_t *)(P + hdr[PH_UTAB_OFF + t]);
        for (uint32_t u = 0; u < set.size(); ++u) {
            const uint16_t *cols = set.cols.data() + (size_t)ECS_UNIT_COLS * order[u];
            const int *rows = set.rows.data() + (size_t)g * order[u];
            uint16_t *ue = utab + u * (1 + g);
            ue[0] = cols[0];
            uint8_t *d = P + hdr[PH_BD_OFF + t] + (size_t)unit_db * u;
            uint16_t with_first[1 + ECS_UNIT_COLS] = {cols[0]};                     // the first column's delta is 0
            std::memcpy(with_first + 1, cols, sizeof(uint16_t) * ECS_UNIT_COLS);
            for (unsigned k = 0; k < ECS_UNIT_COLS; k += ECS_LANE_ELEMS) write_indices(delta_bits, with_first + 1 + k, d + lane_db * (k / ECS_LANE_ELEMS));
            T *v = (T *)(P + hdr[PH_BV_OFF + t] + 64ull * vw * g * u);
            for (uint32_t r = 0; r < g; ++r) ue[1 + r] = (uint16_t)cursor[rows[r]]++;
            if (g == 2) write_unit<2>(values, rows, cols, v);
            else if (g == 4) write_unit<4>(values, rows, cols, v);
            else if (g == 8) write_unit<8>(values, rows, cols, v);
            else write_unit<16>(values, rows, cols, v);
        }
    }
    for (int r = 0; r < nrows; ++r)
        if (cursor[r] != lay.rowslot[(size_t)r + 1]) lay.err = -100;

    // ---- residual set: the row's elements (delta, value) with gap fillers and tail padding, 16 to a lane unit
    const uint32_t nlanes = hdr[PH_NRLANES];
    EcsRChunk *rchunks = (EcsRChunk *)(P + hdr[PH_RCHUNK_OFF]);
    EcsREntry *rentries = (EcsREntry *)(P + hdr[PH_RENTRY_OFF]);
    uint32_t lane = 0, nentries = 0;
    int64_t scan = 0;                                     // sum of the deltas of earlier lanes in this chunk
    values.blocks_written();
    // a row's elements: columns (from `col` on; col[-1]: the column "before" the first one, whose delta counts from there: that column
    // itself, the delta is 0) and values, and once more with the zeros that fill gaps; by the longest row, not by the width
    uint32_t longest = 0;
    for (int r = 0; r < nrows; ++r) longest = std::max(longest, lay.rowlu[(size_t)r + 1] - lay.rowlu[(size_t)r]);
    const size_t most = (size_t)ECS_LANE_ELEMS * longest + 256;
    RawVector<uint16_t> columns(most), filled_columns;
    RawVector<T> row_values(most), filled_values;
    uint32_t by_delta[4][256] = {};
    for (int r = 0; r < nrows; ++r) {
        const uint32_t l0 = lay.rowlu[(size_t)r], l1 = lay.rowlu[(size_t)r + 1];
        if (l0 == l1) continue;
        uint16_t *col = columns.data() + 1;
        T *val = row_values.data();
        int64_t count = values.entries(r, col, val);
        int widest = 0;
        for (int64_t i = 1; i < count; ++i) widest = std::max(widest, (int)col[i] - (int)col[i - 1]);
        if (widest > max_delta) {                         // explicit zero every R_P - 1 columns (Section 6.2)
            filled_columns.resize(most), filled_values.resize(most);
            uint16_t *fc = filled_columns.data() + 1;
            T *fv = filled_values.data();
            int64_t k = 0;
            for (int64_t i = 0; i < count; ++i) {
                if (i) {
                    int at = col[i - 1];
                    for (const int left = (int)col[i] - max_delta; at < left;) at += max_delta, fc[k] = (uint16_t)at, fv[k++] = 0;
                    ++by_delta[i & 3][(int)col[i] - at];
                }
                fc[k] = col[i], fv[k++] = val[i];
            }
            col = fc, val = fv, count = k;
        } else if (max_delta < 256) {                     // four counters for a delta, so that the same one again does not wait for itself
            for (int64_t i = 1; i < count; ++i) ++by_delta[i & 3][(col[i] - col[i - 1]) & 0xFF];
        } else {
            for (int64_t i = 1; i < count; ++i) ++lay.delta_hist[hist_bin((unsigned)(col[i] - col[i - 1]))];
        }
        col[-1] = col[0];
        if ((count + ECS_LANE_ELEMS - 1) / ECS_LANE_ELEMS != l1 - l0 || lane != l0 || l1 > nlanes) {
            lay.err = -100;
            return;
        }
        for (; count % ECS_LANE_ELEMS; ++count) col[count] = col[count - 1], val[count] = 0;      // tail alignment: zeros on the last column
        for (; lane < l1; ++lane, col += ECS_LANE_ELEMS, val += ECS_LANE_ELEMS) {
            const uint32_t c = lane / ECS_CHUNK_LANES, l = lane % ECS_CHUNK_LANES;
            const uint32_t nl = std::min<uint32_t>(ECS_CHUNK_LANES, nlanes - c * ECS_CHUNK_LANES);
            if (l == 0) {
                rchunks[c].head_mask = 0;
                rchunks[c].entry0 = nentries;
                rchunks[c].nlanes = nl;
                scan = 0;
            }
            if (l == 0 || lane == l0) {
                rchunks[c].head_mask |= 1ull << l;
                rentries[nentries].c = (int32_t)((int64_t)col[-1] - scan);
                rentries[nentries].reserved_ = 0;
                rentries[nentries].row_local = (uint16_t)r;
                ++nentries;
            }
            const bool tight = nl < ECS_CHUNK_LANES;                             // only ever the last chunk
            const uint32_t step = ep * (tight ? nl : ECS_CHUNK_LANES);           // values from one load of a lane to the next
            uint8_t *chunk = P + hdr[PH_RD_OFF] + (size_t)hdr[PH_RV_OFF] * c;
            uint8_t *d = chunk + lane_db * l;
            T *v = (T *)(chunk + (tight ? align_up(lane_db * nl, 16) : ECS_CHUNK_DBYTES(delta_bits))) + ep * l;
            write_indices(delta_bits, col, d);
            for (uint32_t k = 0; k < ECS_LANE_ELEMS / ep; ++k) std::memcpy(v + step * k, val + ep * k, 16);
            scan += (int64_t)col[ECS_LANE_ELEMS - 1] - (int64_t)col[-1];
        }
    }
    for (int bin = 0; bin <= 8; ++bin) {                   // hist_bin: 0, 1, 2-3, 4-7, ... 128-255
        uint32_t sum = 0;
        for (int k = 0; k < 4; ++k)
            for (unsigned d = bin ? 1u << (bin - 1) : 0u; d < 1u << bin; ++d) sum += by_delta[k][d];
        lay.delta_hist[bin] += sum;
    }
    if (lane != nlanes || nentries != hdr[PH_NRENTRIES]) lay.err = -100;
}

}  // namespace

// ------------------------------------------------------------------------------------------------------
// row clustering: Algorithm 2 over ALL rows, level by level, to decide which rows share a panel
// ------------------------------------------------------------------------------------------------------

// The paper matches rows over the whole matrix (Section 4: the rows of a block need not be neighbours).  Here a
// panel owns its rows, so rows that belong together must first be brought into the same panel: the multi-level
// aggregation of Algorithm 1 is run once over all rows with one matching round per level (greedy row matching,
// Algorithm 2; a group stands for the columns all its members share), groups of up to `group` rows result, and the
// rows are listed group by group.  Panels are then cut from that list and extraction proper runs inside each panel.
// Returns the row order.
static void cluster_rows(const Rows &A, int group, Team &team, std::vector<int32_t> &order)
{
    const int64_t m = (int64_t)A.count.size();
    const int nw = A.nw;
    struct Grp {
        std::vector<uint64_t> bits;
        int cnt;
        std::vector<int32_t> members;
    };
    std::vector<Grp> cur((size_t)m);
    team.run(m, [&](int64_t i) {
        Grp &g = cur[(size_t)i];
        g.bits.resize(nw);
        A.read(i, g.bits.data());
        g.cnt = (int)A.count[(size_t)i];
        g.members.assign(1, (int32_t)i);
    });
    for (int size = 1; size < group && cur.size() > 1; size *= 2) {
        const int R = (int)cur.size();
        // every group's best partner over all others (ties: lower index), in parallel; the greedy pass below takes it
        // if it is still free and searches again among the free ones if not
        std::vector<int> best(R, -1), best_sim(R, 0);
        team.run(R, [&](int64_t a) {
            int b_best = -1, s_best = 0;
            for (int b = 0; b < R; ++b) {
                if (b == a || cur[b].cnt <= s_best) continue;
                const int sim = popcount_and(cur[a].bits.data(), cur[b].bits.data(), nw);
                if (sim > s_best) s_best = sim, b_best = b;
            }
            best[a] = b_best, best_sim[a] = s_best;
        });
        std::vector<int> pop(R);
        for (int i = 0; i < R; ++i) pop[i] = i;
        std::stable_sort(pop.begin(), pop.end(), [&](int a, int b) { return cur[a].cnt > cur[b].cnt; });
        std::vector<char> free_(R, 1);
        std::vector<Grp> next;
        next.reserve((size_t)R / 2 + 1);
        std::vector<int> single;
        for (int a : pop) {
            if (!free_[a]) continue;
            free_[a] = 0;
            int b = best[a];
            if (b < 0 || !free_[b]) {
                b = -1;
                int s_best = 0;
                for (int c = 0; c < R; ++c) {
                    if (!free_[c] || cur[c].cnt <= s_best) continue;
                    const int sim = popcount_and(cur[a].bits.data(), cur[c].bits.data(), nw);
                    if (sim > s_best) s_best = sim, b = c;
                }
            }
            if (b < 0) {
                single.push_back(a);
                continue;
            }
            free_[b] = 0;
            Grp g;
            g.bits.resize(nw);
            int cnt = 0;
            for (int w = 0; w < nw; ++w) {
                g.bits[w] = cur[a].bits[w] & cur[b].bits[w];
                cnt += __builtin_popcountll(g.bits[w]);
            }
            g.cnt = cnt;
            g.members = cur[a].members;
            g.members.insert(g.members.end(), cur[b].members.begin(), cur[b].members.end());
            next.push_back(std::move(g));
        }
        for (int a : single) next.push_back(std::move(cur[a]));
        cur.swap(next);
    }
    order.clear();
    order.reserve((size_t)m);
    for (const Grp &g : cur) order.insert(order.end(), g.members.begin(), g.members.end());
}

// ------------------------------------------------------------------------------------------------------
// build
// ------------------------------------------------------------------------------------------------------

int build_image(const Source &A, const BuildParams &bp, Image &out)
{
    auto t0 = std::chrono::steady_clock::now();
    const int64_t m = A.m, n = A.n;
    if (n > 65535 || m > 0x7fffffff) return -2;
    Team team(resolve_threads(bp.num_threads));
    Rows rows;
    read_rows(A, team, rows);
    int64_t nnz = 0;
    for (int64_t i = 0; i < m; ++i) nnz += rows.count[(size_t)i];
    int P = bp.num_panels;
    if (P <= 0) {
        P = (int)std::min<int64_t>(256, std::max<int64_t>(1, m / 16));
        // x and one FP32 partial sum per residual lane unit (16 entries) of a panel must fit the LDS of a compute
        // unit: where a panel of this size could not (few, long rows), more panels are made, down to one row each
        int64_t longest = 0;
        for (int64_t i = 0; i < m; ++i) longest = std::max(longest, rows.count[(size_t)i]);
        const int64_t x_bytes = n * (A.value_bits / 8), budget = 150 * 1024;
        while (P < m && x_bytes + 4 * ((nnz / P + longest) / 16 + m / P + 64) + 4096 > budget)
            P = (int)std::min<int64_t>(m, 2 * (int64_t)P);
    }
    if (bp.global_matching) P = 1;
    P = (int)std::min<int64_t>(P, m);

    // the order in which rows are dealt to panels: as they come, or brought together by similarity first
    std::vector<int32_t> order;
    if (bp.cluster_rows && P > 1 && bp.max_granularity > 1) {
        cluster_rows(rows, std::max(2, bp.max_granularity), team, order);
    } else {
        order.resize((size_t)m);
        for (int64_t i = 0; i < m; ++i) order[(size_t)i] = (int32_t)i;
    }
    std::vector<int64_t> pre((size_t)m + 1, 0);                                // stored entries before the k-th row dealt
    for (int64_t k = 0; k < m; ++k) pre[(size_t)k + 1] = pre[(size_t)k] + rows.count[(size_t)order[(size_t)k]];

    // nnz-balanced panels of consecutive rows of that order (Section 5: even work per processing unit): panel p ends
    // at the first row where the running nnz reaches (p + 1) / P of the total; ties in rows for empty matrices.
    std::vector<int64_t> bound(P + 1, 0);
    {
        int64_t r = 0;
        for (int p = 0; p < P; ++p) {
            bound[p] = r;
            const int64_t rows_left = m - r, panels_left = P - p;
            int64_t take;
            if (nnz == 0) {
                take = (rows_left + panels_left - 1) / panels_left;
            } else {
                const double target = (double)nnz * (p + 1) / P;
                int64_t e = r;
                while (e < m && (double)pre[(size_t)e + 1] <= target) ++e;
                // also take the row that crosses the target if that lands closer to it
                if (e < m && (double)pre[(size_t)e + 1] - target < target - (double)pre[(size_t)e]) ++e;
                take = e - r;
            }
            take = std::max<int64_t>(take, 1);                               // every panel owns at least one row
            take = std::min<int64_t>(take, rows_left - (panels_left - 1));   // and leaves one for each later panel
            r += take;
        }
        bound[P] = m;                                                        // the last panel ends at m
    }
    // Every panel is extracted and laid out first: the size of the image, and so where each panel lies in it, follows from the
    // largest one.
    // Every block set the image holds costs the SpMV launch a pipeline stage of its own, so a coarsest set that holds
    // next to nothing (under 1 % of the stored entries over the whole matrix) is not worth having: the granularity
    // cap is lowered and the matrix extracted again, until the coarsest set carries weight or no extraction is left.
    std::vector<PanelUnits> units;
    std::vector<PanelLayout> lays;
    for (int max_g = bp.max_granularity;; max_g >>= 1) {
        units.assign(P, PanelUnits());
        lays.assign(P, PanelLayout());
        team.run(P, [&](int64_t p) {
            const int32_t *prow = order.data() + bound[p];
            const int nrows = (int)(bound[p + 1] - bound[p]);
            extract_panel(rows, prow, nrows, max_g, bp.max_rounds, bp.delta_bits, units[p]);
            lay_out_panel(rows, prow, nrows, units[p], bp.delta_bits, A.value_bits, lays[p]);
            if (rows.bits.empty()) std::vector<uint64_t>().swap(units[p].resid);
        });
        if (bp.keep_small_sets || max_g == 1) break;
        int top = 0;                                                         // coarsest set present
        int64_t by_t[ECS_NUM_BTYPES + 1] = {0, 0, 0, 0, 0};
        for (auto &lay : lays)
            for (int t = 1; t <= ECS_NUM_BTYPES; ++t) by_t[t] += lay.nnz_by_g[t];
        for (int t = 1; t <= ECS_NUM_BTYPES; ++t)
            if (by_t[t] > 0) top = t;
        if (top == 0 || by_t[top] * 100 >= nnz) break;
        max_g = 1 << top;                                                    // halved by the loop: drops set `top`
    }
    uint32_t stride = 256, meta = 16, slots = 1;
    out.max_block_slots = out.max_chunks = 0;
    out.total_chunks = out.block_chunks = 0;
    for (auto &lay : lays) {
        if (lay.err) return lay.err;
        if (lay.bytes > 0xFFFFF000ull) return -2;                            // offsets inside a panel are 32-bit
        stride = std::max<uint32_t>(stride, (uint32_t)lay.bytes);
        meta = std::max(meta, lay.meta_bytes);
        slots = std::max(slots, lay.nslots + ECS_CHUNK_LANES * lay.nchunks);
        out.max_block_slots = std::max(out.max_block_slots, lay.nslots);
        out.max_chunks = std::max(out.max_chunks, lay.nchunks);
        out.total_chunks += lay.nchunks;
        for (int t = 1; t <= ECS_NUM_BTYPES; ++t) out.block_chunks += (uint64_t)(lay.units_by_g[t] + 3) / 4;
    }
    out.total_chunks += out.block_chunks;
    meta = align_up(meta, 16);
    // 4 KB of zeros after the last panel: loads that stand in for missing chunks may run past a short last panel
    const uint64_t total = ECS_IMAGE_HEADER + (uint64_t)stride * (uint64_t)P + 4096u;
    if (total > 0xFFFFFFFF00ull) return -2;
    out.bytes.resize((size_t)total);                                         // not filled: every byte is written below
    auto encode = [&](auto zero) {
        typedef decltype(zero) T;
        team.run(P, [&](int64_t p) {
            uint8_t *to = out.bytes.data() + ECS_IMAGE_HEADER + (size_t)stride * (size_t)p;
            const int32_t *prow = order.data() + bound[p];
            const int nrows = (int)(bound[p + 1] - bound[p]);
            const size_t bytes = stride + (p + 1 == P ? 4096u : 0u);
            auto from = [&](auto &&values) { encode_panel<T>(values, n, prow, nrows, units[p], bp.reorder, bp.delta_bits, lays[p], to, bytes); };
            if (!A.csr) from(DensePanel<T>{static_cast<const T *>(A.dense), A.ld, prow, units[p].resid.data(), rows.nw});
            else if (rows.bits.empty()) from(SparseCsrPanel(rows, prow, nrows, units[p]));
            else from(CsrPanel(rows, prow, nrows, units[p]));
            units[p] = PanelUnits();
        });
    };
    if (A.value_bits == 16) encode(uint16_t(0));
    else encode(uint32_t(0));
    for (auto &lay : lays)
        if (lay.err) return lay.err;
    out.m = m;
    out.n = n;
    out.nnz = nnz;
    out.num_panels = P;
    out.threads_per_wg = bp.threads_per_wg;
    out.delta_bits = bp.delta_bits;
    out.value_bits = A.value_bits;
    out.panel_stride = stride;
    out.meta_stride = meta;
    out.max_slots = slots;
    const uint32_t x_bytes = align_up((uint32_t)n * (uint32_t)(A.value_bits / 8), 16);
    out.lds_bytes = x_bytes + meta + align_up(slots * 4u, 16);

    ecspmv_stats_t &st = out.stats;
    std::memset(&st, 0, sizeof(st));
    st.struct_size = sizeof(st);
    st.m = m;
    st.n = n;
    st.nnz = nnz;
    st.image_bytes = (int64_t)total;
    st.csr32_bytes = (4 + A.value_bits / 8) * nnz + 4 * (m + 1);
    st.csr16_bytes = (2 + A.value_bits / 8) * nnz + 4 * (m + 1);
    st.value_bits = A.value_bits;
    st.num_panels = P;
    st.threads_per_wg = bp.threads_per_wg;
    st.delta_bits = bp.delta_bits;
    st.panel_stride = stride;
    st.meta_stride = meta;
    st.lds_bytes = out.lds_bytes;
    st.min_panel_bytes = INT64_MAX;
    for (int p = 0; p < P; ++p) {
        PanelLayout &im = lays[p];
        st.value_bytes += im.value_bytes;
        st.delta_bytes += im.delta_bytes;
        st.meta_bytes += im.meta_bytes;
        st.pad_elements += im.pad_elements;
        st.gap_pad_elements += im.gap_pads;
        st.max_panel_bytes = std::max<int64_t>(st.max_panel_bytes, (int64_t)im.bytes);
        st.min_panel_bytes = std::min<int64_t>(st.min_panel_bytes, (int64_t)im.bytes);
        for (int k = 0; k < 5; ++k) {
            st.nnz_by_g[k] += im.nnz_by_g[k];
            st.units_by_g[k] += im.units_by_g[k];
        }
        for (int k = 0; k < 9; ++k) st.delta_hist[k] += im.delta_hist[k];
    }
    out.type_mask = 0;
    for (int t = 0; t < ECS_NUM_BTYPES; ++t)
        if (st.units_by_g[t + 1] > 0) out.type_mask |= 1u << t;
    st.meta_bytes += ECS_IMAGE_HEADER;
    st.slack_bytes = st.image_bytes - st.value_bytes - st.delta_bytes - st.meta_bytes;
    for (int k = 0; k < 5; ++k) st.x_access_cost += (double)st.nnz_by_g[k] / (double)(1 << k);

    EcsImageHeader ih;
    std::memset(&ih, 0, sizeof(ih));
    ih.magic = ECS_MAGIC;
    ih.version = ECS_VERSION;
    ih.m = (uint32_t)m;
    ih.n = (uint32_t)n;
    ih.num_panels = (uint32_t)P;
    ih.threads_per_wg = (uint32_t)bp.threads_per_wg;
    ih.panel_stride = stride;
    ih.meta_stride = meta;
    ih.max_slots = slots;
    ih.lds_bytes = out.lds_bytes;
    ih.image_bytes = total;
    ih.nnz = (uint64_t)nnz;
    ih.delta_bits = (uint32_t)bp.delta_bits;
    ih.value_bits = (uint32_t)A.value_bits;
    std::memset(out.bytes.data(), 0, ECS_IMAGE_HEADER);
    std::memcpy(out.bytes.data(), &ih, sizeof(ih));
    st.build_seconds = std::chrono::duration<double>(std::chrono::steady_clock::now() - t0).count();
    return 0;
}

// ------------------------------------------------------------------------------------------------------
// decode: walk the image as the kernel does
// ------------------------------------------------------------------------------------------------------

namespace {

struct PanelView {
    const uint8_t *P;
    const uint32_t *hdr;
    const uint16_t *rowslot;
    uint32_t nrows;
    int row_of_slot(uint32_t s) const
    {
        // rowslot is non-decreasing; the owner of slot s is the last row whose first slot is <= s
        const uint16_t *e = std::upper_bound(rowslot, rowslot + nrows + 1, (uint16_t)s);
        return (int)(e - rowslot) - 1;
    }
};

}  // namespace

int walk_image(const Image &im, Triples *tri, BlockSets *bs)
{
    const uint8_t *base = im.bytes.data() + ECS_IMAGE_HEADER;
    const int bits = im.delta_bits;
    const uint32_t vw = (uint32_t)im.value_bits / 8u, ep = 16u / vw;
    auto get_val = [vw](const uint8_t *base, size_t idx) -> uint32_t {
        return vw == 2 ? (uint32_t)reinterpret_cast<const uint16_t *>(base)[idx]
                       : reinterpret_cast<const uint32_t *>(base)[idx];
    };
    const uint32_t absmask = vw == 2 ? 0x7FFFu : 0x7FFFFFFFu;
    for (int p = 0; p < im.num_panels; ++p) {
        PanelView pv;
        pv.P = base + (size_t)im.panel_stride * p;
        pv.hdr = (const uint32_t *)pv.P;
        pv.nrows = pv.hdr[PH_NROWS];
        pv.rowslot = (const uint16_t *)(pv.P + pv.hdr[PH_ROWSLOT_OFF]);
        const uint32_t *rowidx = (const uint32_t *)(pv.P + pv.hdr[PH_ROWIDX_OFF]);
        for (int t = ECS_NUM_BTYPES - 1; t >= 0; --t) {
            const uint32_t g = 2u << t, nu = pv.hdr[PH_NUNITS + t];
            const uint16_t *utab = (const uint16_t *)(pv.P + pv.hdr[PH_UTAB_OFF + t]);
            for (uint32_t u = 0; u < nu; ++u) {
                const uint16_t *ue = utab + u * (1 + g);
                const uint8_t *d = pv.P + pv.hdr[PH_BD_OFF + t] + ECS_UNIT_DBYTES(bits) * u;
                const uint8_t *v = pv.P + pv.hdr[PH_BV_OFF + t] + 64u * vw * g * u;
                int32_t cols[ECS_UNIT_COLS];
                // 16 lanes x 4 columns: local prefix inside a lane, exclusive scan over lanes, plus base
                uint32_t lane_excl = 0;
                for (uint32_t j = 0; j < 16; ++j) {
                    uint32_t rel = 0;
                    for (uint32_t c = 0; c < 4; ++c) {
                        rel += get_delta(d, 4 * j + c, bits);
                        cols[4 * j + c] = bits == 16 ? (int32_t)get_delta(d, 4 * j + c, bits) : (int32_t)(ue[0] + lane_excl + rel);
                    }
                    lane_excl += rel;
                }
                int rows[16];
                for (uint32_t r = 0; r < g; ++r) {
                    rows[r] = pv.row_of_slot(ue[1 + r]);
                    if (rows[r] < 0 || rows[r] >= (int)pv.nrows) return -100;
                }
                if (bs) {
                    bs->g.push_back((int32_t)g);
                    for (uint32_t r = 0; r < g; ++r) bs->rows.push_back((int32_t)rowidx[rows[r]]);
                    for (uint32_t k = 0; k < ECS_UNIT_COLS; ++k) bs->cols.push_back(cols[k]);
                }
                if (tri)
                    for (uint32_t j = 0; j < 16; ++j)
                        for (uint32_t k = 0; k < 4 * g / ep; ++k)
                            for (uint32_t i = 0; i < ep; ++i) {
                                const uint32_t f = ep * k + i;         // index in lane j's run
                                const uint32_t c = f / g, r = f % g;
                                const uint32_t val = get_val(v, k * 16 * ep + ep * j + i);
                                if ((val & absmask) == 0) continue;
                                tri->rows.push_back((int32_t)rowidx[rows[r]]);
                                tri->cols.push_back(cols[4 * j + c]);
                                tri->vals.push_back(val);
                            }
            }
        }
        if (!tri) continue;
        const uint32_t nlanes = pv.hdr[PH_NRLANES];
        const uint32_t nchunks = (nlanes + ECS_CHUNK_LANES - 1) / ECS_CHUNK_LANES;
        const EcsRChunk *rch = (const EcsRChunk *)(pv.P + pv.hdr[PH_RCHUNK_OFF]);
        const EcsREntry *ren = (const EcsREntry *)(pv.P + pv.hdr[PH_RENTRY_OFF]);
        for (uint32_t c = 0; c < nchunks; ++c) {
            const uint32_t nl = std::min<uint32_t>(ECS_CHUNK_LANES, nlanes - c * ECS_CHUNK_LANES);
            if (rch[c].nlanes != nl || !(rch[c].head_mask & 1)) return -101;
            const bool tight = nl < ECS_CHUNK_LANES;
            const uint32_t stride = tight ? nl : ECS_CHUNK_LANES;
            const uint8_t *d = pv.P + pv.hdr[PH_RD_OFF] + pv.hdr[PH_RV_OFF] * c;            // chunk c: deltas, then values
            const uint8_t *v = d + (tight ? align_up(ECS_LANE_DBYTES(bits) * nl, 16) : ECS_CHUNK_DBYTES(bits));
            int64_t excl = 0;
            for (uint32_t l = 0; l < nl; ++l) {
                const uint64_t below = rch[c].head_mask & ((l == 63) ? ~0ull : ((2ull << l) - 1));
                const EcsREntry &e = ren[rch[c].entry0 + (uint32_t)__builtin_popcountll(below) - 1];
                const int row = (int)e.row_local;
                const uint32_t *rowlu = (const uint32_t *)(pv.P + pv.hdr[PH_ROWLU_OFF]);
                const uint32_t L = c * ECS_CHUNK_LANES + l;
                if (row >= (int)pv.nrows || L < rowlu[row] || L >= rowlu[row + 1]) return -102;
                int64_t rel = 0;
                for (uint32_t k = 0; k < ECS_LANE_ELEMS; ++k) {
                    rel += get_delta(d + ECS_LANE_DBYTES(bits) * l, k, bits);
                    const uint32_t val = get_val(v, ep * stride * (k / ep) + ep * l + (k % ep));
                    if ((val & absmask) == 0) continue;
                    tri->rows.push_back((int32_t)rowidx[row]);
                    tri->cols.push_back(bits == 16 ? (int32_t)get_delta(d + ECS_LANE_DBYTES(bits) * l, k, bits)
                                                   : (int32_t)(e.c + excl + rel));
                    tri->vals.push_back(val);
                }
                excl += rel;
            }
        }
    }
    return 0;
}

}  // namespace ecs
