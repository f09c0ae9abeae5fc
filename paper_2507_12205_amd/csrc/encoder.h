// Host-side data structures of the offline phase (see encoder.cpp).
#ifndef ECSPMV_ENCODER_H
#define ECSPMV_ENCODER_H

#include <cstdint>
#include <cstdlib>
#include <new>
#include <vector>

#include <sys/mman.h>

#include "../../include/ecspmv.h"
#include "ecspmv_format.h"

namespace ecs {

struct Csr {
    int64_t m = 0, n = 0;
    int value_bits = 16;                // 16: FP16 bit patterns, 32: FP32 bit patterns (both held in 32-bit containers)
    std::vector<int64_t> rowptr;
    std::vector<int32_t> col;
    std::vector<uint32_t> val;
};

// What an image is built from: a dense matrix (rows of n values, `ld` apart, 16 or 32 bits each), or a CSR matrix.
struct Source {
    int64_t m = 0, n = 0;
    int value_bits = 16;
    const void *dense = nullptr;
    int64_t ld = 0;
    const Csr *csr = nullptr;
};

// Memory that is written in full before it is read: not filled beforehand (by one thread, with every page touched twice), and
// in huge pages where it is large (4096 x 4096 at 50 %: 22 MB of image, 5400 page faults against 11).
template <class T>
struct RawAllocator {
    typedef T value_type;
    RawAllocator() = default;
    template <class U>
    RawAllocator(const RawAllocator<U> &) {}
    T *allocate(size_t n)
    {
        constexpr size_t kHuge = 2u << 20;
        if (n > (size_t)-1 / 2 / sizeof(T)) throw std::bad_alloc();
        const size_t bytes = n * sizeof(T);
        void *p = nullptr;
        if (bytes >= 2 * kHuge) {
            p = std::aligned_alloc(kHuge, (bytes + kHuge - 1) / kHuge * kHuge);
            if (p) (void)madvise(p, bytes, MADV_HUGEPAGE);                   // no more than advice
        } else {
            p = std::malloc(bytes);
        }
        if (!p) throw std::bad_alloc();
        return static_cast<T *>(p);
    }
    void deallocate(T *p, size_t) { std::free(p); }
    template <class U>
    void construct(U *p)
    {
        ::new ((void *)p) U;                                                 // leaves the bytes as they are
    }
    template <class U, class... Args>
    void construct(U *p, Args &&...args)
    {
        ::new ((void *)p) U(static_cast<Args &&>(args)...);
    }
    template <class U>
    bool operator==(const RawAllocator<U> &) const { return true; }
    template <class U>
    bool operator!=(const RawAllocator<U> &) const { return false; }
};
template <class T>
using RawVector = std::vector<T, RawAllocator<T>>;

struct BuildParams {
    int delta_bits = 8;
    int max_granularity = 8;
    int max_rounds = 64;
    int num_panels = 0;
    int num_threads = 0;
    int threads_per_wg = 0;
    bool global_matching = false;
    bool reorder = true;
    bool keep_small_sets = false;
    bool cluster_rows = false;          // bring similar rows into the same panel before the panels are cut
};

struct Image {
    RawVector<uint8_t> bytes;
    int64_t m = 0, n = 0, nnz = 0;
    int num_panels = 0, threads_per_wg = 1024, delta_bits = 8, value_bits = 16;
    uint32_t panel_stride = 0, meta_stride = 0, max_slots = 0, lds_bytes = 0;
    uint32_t max_block_slots = 0, max_chunks = 0;      // over the panels: slots of the block sets, residual chunks
    uint64_t total_chunks = 0, block_chunks = 0;       // what a wavefront takes at a time (64 lane units, 4 units), all panels; those of units
    uint32_t type_mask = 0;   // bit t set: some panel holds units of granularity 2 << t
    ecspmv_stats_t stats;
};

struct Triples {
    std::vector<int32_t> rows, cols;
    std::vector<uint32_t> vals;         // FP16 or FP32 bit patterns
};

struct BlockSets {
    std::vector<int32_t> g, rows, cols;
};

int csr_from_dense(const uint16_t *W, int64_t m, int64_t n, int64_t ld, int threads, Csr &out);
int csr_from_csr(const int64_t *rowptr, const int32_t *col, const uint16_t *val, int64_t m, int64_t n, Csr &out);
int csr_from_csr_f32(const int64_t *rowptr, const int32_t *col, const uint32_t *val, int64_t m, int64_t n, Csr &out);
int build_image(const Source &A, const BuildParams &bp, Image &out);
int walk_image(const Image &im, Triples *tri, BlockSets *bs);

}  // namespace ecs
#endif
