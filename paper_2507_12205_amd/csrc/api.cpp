// C ABI of the library (see include/ecspmv.h): argument checks, option defaults, handle bookkeeping.
#include <algorithm>
#include <atomic>
#include <cstddef>
#include <cstring>
#include <memory>
#include <new>
#include <vector>

#include "../../include/ecspmv.h"
#include "encoder.h"
#include "launch.h"

struct ecspmv_matrix {
    ecs::Image image;
    void *d_image = nullptr;
};

struct ecspmv_csr {
    int64_t m = 0, n = 0, nnz = 0;
    std::vector<int32_t> rowptr, col;
    std::vector<uint16_t> val;
    size_t off_col = 0, off_val = 0, bytes = 0;
    uint8_t *d_buf = nullptr;
};

namespace {

thread_local int g_last_hip_error = 0;

int hip_status(int e)
{
    if (e == 0) return ECSPMV_OK;
    g_last_hip_error = e;
    return ECSPMV_ERR_HIP;
}

// LDS a workgroup may use on the current device, asked once per device and kept (the hot calls must not query the
// runtime on every launch)
int lds_limit(int *bytes)
{
    constexpr int kMaxDev = 64;
    static std::atomic<int> cached[kMaxDev];
    int dev = 0;
    int e = ecs::current_device(&dev);
    if (e) return e;
    if (dev >= 0 && dev < kMaxDev) {
        const int v = cached[dev].load(std::memory_order_relaxed);
        if (v > 0) {
            *bytes = v;
            return 0;
        }
    }
    e = ecs::device_lds_limit(bytes);
    if (e) return e;
    if (dev >= 0 && dev < kMaxDev) cached[dev].store(*bytes, std::memory_order_relaxed);
    return 0;
}

// Workgroup size of a launch of `grid` workgroups in all that have `chunks` chunks between them (a wavefront takes one at
// a time); `pieces`: 16-byte pieces of tables and x the widest of them brings to LDS; `rows`: rows of a panel
// on average, the most of all matrices (16 threads add up one); `sets`: the coarsest block set is the `sets`-th.  Measured, us
// with 512 / 768 / 1024 threads, 256 panels of 16 to 20 rows unless said otherwise, launches inside a graph over three matrices
// in turn:
//   alone, up to 16 chunks: eight wavefronts are up and past the first barrier sooner, and two rounds are enough, also for tall
//     panels: 4096 x 4096 at 20 %, 4-bit (13 chunks) 4.11 / 4.08 / 4.38, 16384 x 512 at 20 % (7, 64 rows) 3.43 / 3.53 / 3.88,
//     768 x 768 (8, 48 panels) 2.76 / 3.19 / 3.07;
//   up to 24, without block sets twelve: 4096 x 4096 at 35 % (23) 4.79 / 4.54 / 4.81, 1984 x 6558 at 18 % (20, 124 panels) 4.62 / 4.24 /
//     4.37, 8192 x 2048 at 30 % (20, 32 rows) 4.63 / 4.32 / 4.58, 17216 x 1186 at 20 % (17, 67 rows) 5.05 / 4.54 / 4.62; FP32 values
//     eight but for the tallest, 1216 x 6080 at 18 % (18, 76 panels) 3.76 / 4.07 / 4.09, 10240 x 2048 at 25 % (21, 40 rows) 5.58 / 5.58 /
//     5.83, 17216 x 1186 5.62 / 4.94 / 5.59;
//   up to 24, with block sets eight: 7168 x 2048 at 22 %, 8-bit (17, 28 rows) 4.01 / 4.39 / 4.68, 3776 x 3776 at 25 %, 8-bit (23) 4.12 /
//     4.32 / 4.47; taller with one set twelve: 8192 x 2048 at 22 % (20, 32 rows) 4.52 / 4.36 / 4.68; with two sets eight all the
//     same: 16384 x 512 at 50 % (21, 64 rows) 4.47 / 4.83 / 4.85;
//   up to 48, one block set or an 8-grained one: twelve, 4096 x 4096 at 50 %, 4-bit (44) 6.43 / 5.96 / 6.27, 3072 x 3072 at 50 %,
//     8-bit, 8-grained (33) 5.48 / 5.43 / 6.22, 10240 x 2048 at 25 %, 8-bit (30, 40 rows) 5.46 / 5.03 / 5.30; sixteen where more
//     than 40 rows keep all of them in the sums: 10304 x 1858 at 35 % (26, 41 rows) 6.11 / 5.76 / 5.67, 17216 x 1186 at 30 %, 8-bit (33,
//     67 rows) 5.82 / 5.77 / 5.32 (but 18240 x 3584 at 11 %, 29 chunks, 72 rows, 6.66 / 6.12 / 6.37); and sixteen with two sets
//     (2- and 4-grained), where a wavefront requests up to four chunks before it computes, and sixteen have all of them on
//     the way at once: 5120 x 5120 at 30 %, 8-bit (45) 6.54 / 6.30 / 5.85;
//   up to 48 without block sets: sixteen.  Twelve are faster in a launch over and over, 5120 x 5120 at 30 %, 4-bit (30) 5.96 / 5.52 /
//     5.84 (cold 6.05 / 5.71 / 5.90), but among the seven products of a decoder layer, launched from the host, four such
//     took 52.03 us in all with twelve and 51.83 with sixteen;
//   beyond, sixteen: 11008 x 4096 at 40 %, 4-bit (72) 10.27 / 10.06 / 9.48.
//   Several matrices, 256 / 512 threads: with up to 16 chunks a panel 256, where the launch is more than a compute unit holds
//     at 512 threads (2048 threads each: 1024 workgroups), 5 x 4096 x 4096 at 15 % (11 chunks, 1280 workgroups) 8.65 / 8.97, 5 x
//     16384 x 512 (7, 1280, 64 rows) 7.29 / 8.62, FP32 values from 768 on, 3 x 4096 x 4096 at 15 % (768) 8.26 / 8.72; or where
//     there is more than one workgroup for a compute unit, a thread brings one piece (FP32: two) and 16 lanes a row or little
//     more: 16 x 512 x 512 (3, 512) 3.94 / 4.44, 6 x 768 x 768 (8, 288) 4.24 / 4.50, FP32 4.80 / 5.73, 5 x 1024 x 1024 (5, 320)
//     3.80 / 3.93, 3 x 5120 x 1024 (4, 768, 20 rows) 4.62 / 4.70; one for each: 8 x 512 x 512 (3, 256) 3.68 / 3.67, 3 x 1024 x 1024
//     (5, 192) 3.67 / 3.43.  Larger panels, wider x or taller panels want more wavefronts: 16 x 512 x 5120 (24, 512) 8.05 / 7.23,
//     2 x 4096 x 4096 at 20 % (13, 512) 6.10 / 5.59, 3 x 3562 x 3562 (8, 666) 5.96 / 5.68, 3 x 6144 x 1024 (5, 768, 24 rows) 4.85 /
//     4.80, 3 x 16384 x 512, 8-bit (11, 768, 64 rows) 7.72 / 7.02.  With an 8-grained set a kernel takes 80 registers, and a compute
//     unit holds three workgroups of 512 but seven of 256: 16 x 1024 x 4096 at 50 %, 8-bit, 128 panels each (22, 2048) 17.94 / 21.55,
//     5 x 4096 x 4096 (44, 1280) 20.56 / 21.27; 6 x 8192 x 2048 at 60 % (47, 1536, 32 rows) 27.73 / 27.59.
// The size then grows, up to 1024 alone and 512 among several, until the four pieces per thread that travel together bring
//   all of x: 512 x 20480 (17 chunks, 2630 pieces) 5.12 / 4.66 / 5.15.
uint32_t choose_threads(uint32_t grid, uint64_t chunks, uint32_t pieces, uint32_t rows, bool fp32, bool alone, uint32_t sets)
{
    auto up_to = [&](uint64_t per_panel) { return chunks <= per_panel * grid; };
    uint32_t t;
    if (alone) {
        t = 1024u;
        if (sets == 0u ? up_to(24) : sets != 2u && up_to(48) && rows <= 40u) t = 768u;
        const bool short_panels = sets == 0u ? fp32 && rows <= 48u : sets == 2u || rows <= 28u;
        if (up_to(16) || (up_to(24) && short_panels)) t = 512u;
    } else {
        const bool crowded = grid > (fp32 ? 767u : 1024u), light = grid > 256u && pieces <= (fp32 ? 512u : 256u) && rows <= 20u;
        t = (up_to(16) && (crowded || light)) || (sets >= 3u && grid >= 1024u) ? 256u : 512u;
    }
    while (pieces > 4u * t && t < (alone ? 1024u : 512u)) t += 256u;
    return t;
}

int map_build_error(int e)
{
    if (e == 0) return ECSPMV_OK;
    if (e == -2) return ECSPMV_ERR_UNSUPPORTED;
    return ECSPMV_ERR_INVALID;
}

int parse_opts(const ecspmv_build_opts *o, ecs::BuildParams &bp, int value_bits = 16)
{
    ecspmv_build_opts opts;
    std::memset(&opts, 0, sizeof(opts));
    if (o) {
        if (o->struct_size < sizeof(uint32_t)) return ECSPMV_ERR_INVALID;
        std::memcpy(&opts, o, o->struct_size < sizeof(opts) ? o->struct_size : sizeof(opts));
    }
    if (opts.delta_bits != 0 && opts.delta_bits != 8 && opts.delta_bits != 4 && opts.delta_bits != 16)
        return ECSPMV_ERR_UNSUPPORTED;
    if (opts.delta_bits == 16 && value_bits != 16) return ECSPMV_ERR_UNSUPPORTED;      // the ablation point exists for FP16 only
    bp.delta_bits = opts.delta_bits ? opts.delta_bits : 8;
    // default cap on g: 8, and 4 for FP32 values (an 8-grained FP32 unit holds 32 value registers per lane and the
    // kernel starts to spill; larger caps can still be asked for)
    const int g = opts.max_granularity ? opts.max_granularity : (value_bits == 32 ? 4 : 8);
    if (g != 1 && g != 2 && g != 4 && g != 8 && g != 16) return ECSPMV_ERR_UNSUPPORTED;
    bp.max_granularity = g;
    if (opts.max_rounds < 0 || opts.num_panels < 0 || opts.num_threads < 0) return ECSPMV_ERR_INVALID;
    bp.max_rounds = opts.max_rounds ? opts.max_rounds : 64;
    bp.num_panels = opts.num_panels;
    bp.num_threads = opts.num_threads;
    const int t = opts.threads_per_wg;
    if (t != 0 && (t < 64 || t > 1024 || t % 64)) return ECSPMV_ERR_INVALID;
    bp.threads_per_wg = t;
    bp.global_matching = (opts.flags & ECSPMV_FLAG_GLOBAL_MATCHING) != 0;
    bp.reorder = (opts.flags & ECSPMV_FLAG_NO_REORDER) == 0;
    bp.keep_small_sets = (opts.flags & ECSPMV_FLAG_KEEP_SMALL_SETS) != 0;
    bp.cluster_rows = (opts.flags & ECSPMV_FLAG_CLUSTER_ROWS) != 0;
    return ECSPMV_OK;
}

int finish_build(const ecs::Source &A, const ecs::BuildParams &bp, ecspmv_matrix **out)
{
    std::unique_ptr<ecspmv_matrix> h(new (std::nothrow) ecspmv_matrix);       // released on every way out but the last
    if (!h) return ECSPMV_ERR_NOMEM;
    const int e = ecs::build_image(A, bp, h->image);
    if (e) return map_build_error(e);
    if (h->image.lds_bytes > 160u * 1024u) return ECSPMV_ERR_UNSUPPORTED;
    *out = h.release();
    return ECSPMV_OK;
}

// shared by ecspmv_decode (FP16 images, 16-bit values out) and ecspmv_decode_f32 (FP32 images, 32-bit values out)
template <typename T>
int decode_t(const ecspmv_matrix *A, int value_bits, int64_t *nnz, int32_t *rows, int32_t *cols, T *vals)
{
    if (!A || !nnz) return ECSPMV_ERR_INVALID;
    if (A->image.value_bits != value_bits) return ECSPMV_ERR_INVALID;
    try {
        ecs::Triples t;
        if (ecs::walk_image(A->image, &t, nullptr)) return ECSPMV_ERR_INVALID;
        const int64_t count = (int64_t)t.rows.size();
        if (!rows && !cols && !vals) {
            *nnz = count;
            return ECSPMV_OK;
        }
        if (!rows || !cols || !vals) return ECSPMV_ERR_INVALID;
        if (*nnz < count) return ECSPMV_ERR_TOO_SMALL;
        if (count) {
            std::memcpy(rows, t.rows.data(), sizeof(int32_t) * (size_t)count);
            std::memcpy(cols, t.cols.data(), sizeof(int32_t) * (size_t)count);
            for (int64_t i = 0; i < count; ++i) vals[i] = (T)t.vals[(size_t)i];
        }
        *nnz = count;
        return ECSPMV_OK;
    } catch (const std::bad_alloc &) {
        return ECSPMV_ERR_NOMEM;
    } catch (...) {                                  // nothing may leave through the C ABI (a worker thread that could
        return ECSPMV_ERR_INTERNAL;                  // not be started, for instance)
    }
}

}  // namespace

extern "C" {

int ecspmv_build_dense(const uint16_t *W, int64_t m, int64_t n, int64_t ld, const ecspmv_build_opts *opts,
                       ecspmv_matrix **out)
{
    if (!W || !out || m <= 0 || n <= 0 || ld < n) return ECSPMV_ERR_INVALID;
    if (n > 65535 || m > 0x7fffffff) return ECSPMV_ERR_UNSUPPORTED;
    ecs::BuildParams bp;
    int s = parse_opts(opts, bp);
    if (s) return s;
    try {
        return finish_build({m, n, 16, W, ld, nullptr}, bp, out);
    } catch (const std::bad_alloc &) {
        return ECSPMV_ERR_NOMEM;
    } catch (...) {                                  // nothing may leave through the C ABI (a worker thread that could
        return ECSPMV_ERR_INTERNAL;                  // not be started, for instance)
    }
}

int ecspmv_build_csr(const int64_t *rowptr, const int32_t *col, const uint16_t *val, int64_t m, int64_t n,
                     const ecspmv_build_opts *opts, ecspmv_matrix **out)
{
    if (!rowptr || !out || m <= 0 || n <= 0) return ECSPMV_ERR_INVALID;
    if (rowptr[m] < 0 || (rowptr[m] > 0 && (!col || !val))) return ECSPMV_ERR_INVALID;
    if (n > 65535 || m > 0x7fffffff) return ECSPMV_ERR_UNSUPPORTED;
    ecs::BuildParams bp;
    int s = parse_opts(opts, bp);
    if (s) return s;
    try {
        ecs::Csr A;
        if (ecs::csr_from_csr(rowptr, col, val, m, n, A)) return ECSPMV_ERR_INVALID;
        return finish_build({m, n, 16, nullptr, 0, &A}, bp, out);
    } catch (const std::bad_alloc &) {
        return ECSPMV_ERR_NOMEM;
    } catch (...) {                                  // nothing may leave through the C ABI (a worker thread that could
        return ECSPMV_ERR_INTERNAL;                  // not be started, for instance)
    }
}

int ecspmv_build_dense_f32(const float *W, int64_t m, int64_t n, int64_t ld, const ecspmv_build_opts *opts,
                           ecspmv_matrix **out)
{
    if (!W || !out || m <= 0 || n <= 0 || ld < n) return ECSPMV_ERR_INVALID;
    if (n > 65535 || m > 0x7fffffff) return ECSPMV_ERR_UNSUPPORTED;
    ecs::BuildParams bp;
    int s = parse_opts(opts, bp, 32);
    if (s) return s;
    try {
        return finish_build({m, n, 32, W, ld, nullptr}, bp, out);
    } catch (const std::bad_alloc &) {
        return ECSPMV_ERR_NOMEM;
    } catch (...) {                                  // nothing may leave through the C ABI (a worker thread that could
        return ECSPMV_ERR_INTERNAL;                  // not be started, for instance)
    }
}

int ecspmv_build_csr_f32(const int64_t *rowptr, const int32_t *col, const float *val, int64_t m, int64_t n,
                         const ecspmv_build_opts *opts, ecspmv_matrix **out)
{
    if (!rowptr || !out || m <= 0 || n <= 0) return ECSPMV_ERR_INVALID;
    if (rowptr[m] < 0 || (rowptr[m] > 0 && (!col || !val))) return ECSPMV_ERR_INVALID;
    if (n > 65535 || m > 0x7fffffff) return ECSPMV_ERR_UNSUPPORTED;
    ecs::BuildParams bp;
    int s = parse_opts(opts, bp, 32);
    if (s) return s;
    try {
        ecs::Csr A;
        if (ecs::csr_from_csr_f32(rowptr, col, reinterpret_cast<const uint32_t *>(val), m, n, A)) return ECSPMV_ERR_INVALID;
        return finish_build({m, n, 32, nullptr, 0, &A}, bp, out);
    } catch (const std::bad_alloc &) {
        return ECSPMV_ERR_NOMEM;
    } catch (...) {                                  // nothing may leave through the C ABI (a worker thread that could
        return ECSPMV_ERR_INTERNAL;                  // not be started, for instance)
    }
}

void ecspmv_destroy(ecspmv_matrix *A) { delete A; }

int ecspmv_stats(const ecspmv_matrix *A, ecspmv_stats_t *st)
{
    if (!A || !st || st->struct_size < sizeof(uint32_t)) return ECSPMV_ERR_INVALID;
    const uint32_t want = st->struct_size < sizeof(ecspmv_stats_t) ? st->struct_size : (uint32_t)sizeof(ecspmv_stats_t);
    ecspmv_stats_t tmp = A->image.stats;
    tmp.struct_size = want;
    std::memcpy(st, &tmp, want);
    return ECSPMV_OK;
}

int ecspmv_decode(const ecspmv_matrix *A, int64_t *nnz, int32_t *rows, int32_t *cols, uint16_t *vals)
{
    return decode_t<uint16_t>(A, 16, nnz, rows, cols, vals);
}

int ecspmv_decode_f32(const ecspmv_matrix *A, int64_t *nnz, int32_t *rows, int32_t *cols, float *vals)
{
    return decode_t<uint32_t>(A, 32, nnz, rows, cols, reinterpret_cast<uint32_t *>(vals));
}

int ecspmv_block_sets(const ecspmv_matrix *A, int64_t *n_units, int64_t *n_rows, int32_t *g, int32_t *unit_rows,
                      int32_t *unit_cols)
{
    if (!A || !n_units || !n_rows) return ECSPMV_ERR_INVALID;
    try {
        ecs::BlockSets b;
        if (ecs::walk_image(A->image, nullptr, &b)) return ECSPMV_ERR_INVALID;
        const int64_t nu = (int64_t)b.g.size(), nr = (int64_t)b.rows.size();
        if (!g && !unit_rows && !unit_cols) {
            *n_units = nu;
            *n_rows = nr;
            return ECSPMV_OK;
        }
        if (!g || !unit_rows || !unit_cols) return ECSPMV_ERR_INVALID;
        if (*n_units < nu || *n_rows < nr) return ECSPMV_ERR_TOO_SMALL;
        if (nu) {
            std::memcpy(g, b.g.data(), sizeof(int32_t) * (size_t)nu);
            std::memcpy(unit_rows, b.rows.data(), sizeof(int32_t) * (size_t)nr);
            std::memcpy(unit_cols, b.cols.data(), sizeof(int32_t) * (size_t)nu * ECS_UNIT_COLS);
        }
        *n_units = nu;
        *n_rows = nr;
        return ECSPMV_OK;
    } catch (const std::bad_alloc &) {
        return ECSPMV_ERR_NOMEM;
    } catch (...) {                                  // nothing may leave through the C ABI (a worker thread that could
        return ECSPMV_ERR_INTERNAL;                  // not be started, for instance)
    }
}

int ecspmv_device_bytes(const ecspmv_matrix *A, size_t *bytes)
{
    if (!A || !bytes) return ECSPMV_ERR_INVALID;
    *bytes = A->image.bytes.size();
    return ECSPMV_OK;
}

int ecspmv_export_image(const ecspmv_matrix *A, void *host_dst, size_t bytes)
{
    if (!A || !host_dst) return ECSPMV_ERR_INVALID;
    if (bytes < A->image.bytes.size()) return ECSPMV_ERR_TOO_SMALL;
    std::memcpy(host_dst, A->image.bytes.data(), A->image.bytes.size());
    return ECSPMV_OK;
}

int ecspmv_upload(ecspmv_matrix *A, void *d_buf, size_t bytes, void *stream)
{
    if (!A || !d_buf || (reinterpret_cast<uintptr_t>(d_buf) & 255)) return ECSPMV_ERR_INVALID;
    if (bytes < A->image.bytes.size()) return ECSPMV_ERR_TOO_SMALL;
    int lim = 0;
    int e = lds_limit(&lim);
    if (e) return hip_status(e);
    if ((int64_t)A->image.lds_bytes > (int64_t)lim) return ECSPMV_ERR_UNSUPPORTED;
    e = ecs::copy_to_device(d_buf, A->image.bytes.data(), A->image.bytes.size(), stream);
    if (e) return hip_status(e);
    A->d_image = d_buf;
    return ECSPMV_OK;
}

int ecspmv_run_batch(const ecspmv_matrix *const *As, const void *const *d_xs, void *const *d_ys, int32_t count,
                     void *stream)
{
    if (!As || !d_xs || !d_ys || count <= 0) return ECSPMV_ERR_INVALID;
    for (int32_t i = 0; i < count; ++i) {
        if (!As[i] || !d_xs[i] || !d_ys[i]) return ECSPMV_ERR_INVALID;
        const uintptr_t align = (uintptr_t)(As[i]->image.value_bits / 8 - 1);       // x, y: 2- or 4-byte aligned
        if ((reinterpret_cast<uintptr_t>(d_xs[i]) & align) || (reinterpret_cast<uintptr_t>(d_ys[i]) & align))
            return ECSPMV_ERR_INVALID;
        if (!As[i]->d_image) return ECSPMV_ERR_NOT_UPLOADED;
    }
    // one launch per run of up to ECS_MAX_BATCH matrices with the same delta width and value width; nothing on
    // this path allocates or can throw
    for (int32_t base = 0, nb = 0; base < count; base += nb) {
        const int bits = As[base]->image.delta_bits;
        const int vbits = As[base]->image.value_bits;
        for (nb = 1; base + nb < count && nb < ECS_MAX_BATCH; ++nb) {
            const ecs::Image &nx = As[base + nb]->image;
            if (nx.delta_bits != bits || nx.value_bits != vbits) break;
        }
        ecs::EcsBatch b;
        std::memset(&b, 0, offsetof(ecs::EcsBatch, item) + sizeof(ecs::EcsBatchItem) * (size_t)(nb == 1 ? 1 : ECS_MAX_BATCH));
        b.count = (uint32_t)nb;
        uint32_t blocks = 0, lds = 0, mask = 0, pieces = 0, rows = 0;
        uint64_t chunks = 0, block_chunks = 0;
        for (int32_t i = 0; i < nb; ++i) {
            const int32_t src = base + i;
            const ecs::Image &im = As[src]->image;
            ecs::EcsBatchItem &it = b.item[i];
            it.image = static_cast<const uint8_t *>(As[src]->d_image);
            it.x = static_cast<const uint16_t *>(d_xs[src]);
            it.y = static_cast<uint16_t *>(d_ys[src]);
            it.n = (uint32_t)im.n;
            it.panel_stride = im.panel_stride;
            it.meta_stride = im.meta_stride;
            it.x_bytes = ((uint32_t)im.n * (uint32_t)(vbits / 8) + 15u) / 16u * 16u;
            blocks += (uint32_t)im.num_panels;
            it.block_end = blocks;
            lds = im.lds_bytes > lds ? im.lds_bytes : lds;
            mask |= im.type_mask;
            chunks += im.total_chunks;
            block_chunks += im.block_chunks;
            pieces = std::max(pieces, (im.meta_stride + it.x_bytes) / 16u);
            rows = std::max(rows, (uint32_t)((im.m + im.num_panels - 1) / im.num_panels));
        }
        uint32_t threads = choose_threads(blocks, chunks, pieces, rows, vbits == 32, nb == 1,
                                          mask >= 8u ? 4u : mask >= 4u ? 3u : mask >= 2u ? 2u : mask);
        for (int32_t i = 0; i < nb; ++i) {
            const int t = As[base + i]->image.threads_per_wg;
            if (t) threads = (uint32_t)t;                      // a build-time choice overrides
        }
        int s = hip_status(ecs::launch_ecspmv(b, threads, lds, mask, (uint32_t)bits, (uint32_t)vbits, chunks, block_chunks, stream));
        if (s) return s;
    }
    return ECSPMV_OK;
}

int ecspmv_run(const ecspmv_matrix *A, const void *d_x, void *d_y, void *stream)
{
    return ecspmv_run_batch(&A, &d_x, &d_y, 1, stream);
}

int ecspmv_run_multi(const ecspmv_matrix *A, const void *d_X, void *d_Y, int32_t nb, void *stream)
{
    if (!A || !d_X || !d_Y) return ECSPMV_ERR_INVALID;
    if (nb == 1) return ecspmv_run(A, d_X, d_Y, stream);
    if (nb != 2 && nb != 4 && nb != 8) return ECSPMV_ERR_INVALID;
    const ecs::Image &im = A->image;
    const uint32_t vw = (uint32_t)im.value_bits / 8u;                 // bytes per value of W, X and Y
    if ((reinterpret_cast<uintptr_t>(d_X) & (vw - 1u)) || (reinterpret_cast<uintptr_t>(d_Y) & (vw - 1u)))
        return ECSPMV_ERR_INVALID;
    if (!A->d_image) return ECSPMV_ERR_NOT_UPLOADED;
    // registers run out with a 16-grained set, and with an 8-grained one if the values are FP32; absolute 16-bit
    // columns (index compression off) exist for one vector only
    if (im.type_mask & (vw == 4 ? ~3u : ~7u)) return ECSPMV_ERR_UNSUPPORTED;
    if (im.delta_bits == 16) return ECSPMV_ERR_UNSUPPORTED;
    int lim = 0;
    int e = lds_limit(&lim);
    if (e) return hip_status(e);
    // Small panels: eight wavefronts, as with one vector, us with 512 / 1024 threads: up to 12 chunks a panel (768 x 768, eight
    // right-hand sides, 8 chunks: 4.04 / 4.50; 16384 x 512, 7 chunks, four: 3.98 / 4.52), with two right-hand sides up to 20
    // (FP32 2048 x 2048 at 30 %, 8-bit, 15 chunks: 4.22 / 5.26; 2048 x 8192 at 12 %, 18: 4.20 / 4.46; 16384 x 1024 at 25 %, 17:
    // 5.12 / 5.24; four, 2048 x 4096 at 25 %, 16: 5.29 / 5.11); but not with more X than they bring well (up to 12 chunks 64 KB:
    // FP32, eight, 1024 x 4096 at 15 %, 11 chunks, 128 KB: 7.89 / 7.39; up to 20 chunks 32 KB: FP32, two, 1408 x 6144 at 17 %, 17
    // chunks, 48 KB: 5.69 / 5.53).  Larger ones sixteen (5120 x 5120, two, 30 chunks: 6.96 / 6.55).
    const uint64_t all_x = (uint64_t)im.n * vw * (uint32_t)nb;
    auto up_to = [&](uint64_t per_panel) { return im.total_chunks <= per_panel * (uint64_t)im.num_panels; };
    const bool small = (up_to(12) && all_x <= 65536u) || (nb == 2 && up_to(20) && all_x <= 32768u);
    const uint32_t threads = im.threads_per_wg ? (uint32_t)im.threads_per_wg : small ? 512u : 1024u, waves = threads / 64u;
    // `per` columns of X and their partial sums sit in the LDS of a workgroup, so a panel takes nb / per workgroups, all
    // of one launch.  Where the partial sums of a whole panel do not fit beside X, the residual chunks are taken in
    // phases of k chunks per wavefront, and the partial sums of a phase are added up before the next one.
    auto x_bytes_of = [&](uint32_t per) -> uint64_t { return ((uint64_t)im.n * vw * per + 15u) / 16u * 16u; };
    auto lds_of = [&](uint32_t per, uint32_t k) -> uint64_t {           // k = 0: one phase
        const uint64_t fixed = x_bytes_of(per) + im.meta_stride;
        if (k == 0) return fixed + ((uint64_t)im.max_slots * 4u * per + 15u) / 16u * 16u;
        return fixed + 2u * 16u * 4u * per + ((uint64_t)im.max_block_slots + 64u * waves * k) * 4u * per;
    };
    if (lds_of(2, 0) > (uint64_t)lim) return ECSPMV_ERR_UNSUPPORTED;    // not even two right-hand sides fit
    uint32_t per = (uint32_t)nb, k = 0;
    for (;; per /= 2) {
        k = 0;
        if (lds_of(per, 0) <= (uint64_t)lim) break;
        if (lds_of(per, 1) > (uint64_t)lim) continue;                  // (with per = 2 one phase always fits)
        const uint32_t want = (im.max_chunks + waves - 1u) / waves;    // chunks of a wavefront
        for (k = 1; k < want && lds_of(per, k + 1u) <= (uint64_t)lim; ++k) {}
        break;
    }
    ecs::EcsBatch b;
    std::memset(&b, 0, offsetof(ecs::EcsBatch, item) + sizeof(ecs::EcsBatchItem));       // the only item
    b.count = 1;
    b.per_phase = k;
    ecs::EcsBatchItem &it = b.item[0];
    it.image = static_cast<const uint8_t *>(A->d_image);
    it.x = static_cast<const uint16_t *>(d_X);
    it.y = static_cast<uint16_t *>(d_Y);
    it.n = (uint32_t)im.n;
    it.panel_stride = im.panel_stride;
    it.meta_stride = im.meta_stride;
    it.x_bytes = (uint32_t)x_bytes_of(per);
    it.block_end = (uint32_t)im.num_panels;
    it.row_stride = (uint32_t)nb;                                       // of X and Y, in elements
    return hip_status(ecs::launch_ecspmv_multi(b, threads, (uint32_t)lds_of(per, k), im.type_mask, (uint32_t)im.delta_bits,
                                               (uint32_t)im.value_bits, per, stream));
}

int ecspmv_csr_build_dense(const uint16_t *W, int64_t m, int64_t n, int64_t ld, ecspmv_csr **out)
{
    if (!W || !out || m <= 0 || n <= 0 || ld < n) return ECSPMV_ERR_INVALID;
    try {
        ecs::Csr A;
        ecs::csr_from_dense(W, m, n, ld, 0, A);
        if (A.rowptr[(size_t)m] > 0x7fffffff || m > 0x7ffffffe) return ECSPMV_ERR_UNSUPPORTED;
        std::unique_ptr<ecspmv_csr> c(new (std::nothrow) ecspmv_csr);
        if (!c) return ECSPMV_ERR_NOMEM;
        c->m = m;
        c->n = n;
        c->nnz = A.rowptr[(size_t)m];
        c->rowptr.resize((size_t)m + 1);
        for (int64_t i = 0; i <= m; ++i) c->rowptr[(size_t)i] = (int32_t)A.rowptr[(size_t)i];
        c->col.swap(A.col);
        c->val.assign(A.val.begin(), A.val.end());                 // FP16 bit patterns out of their 32-bit containers
        auto up = [](size_t v) { return (v + 255) / 256 * 256; };
        c->off_col = up(4 * ((size_t)m + 1));
        c->off_val = c->off_col + up(4 * (size_t)c->nnz);
        c->bytes = c->off_val + up(2 * (size_t)c->nnz) + 256;
        *out = c.release();
        return ECSPMV_OK;
    } catch (const std::bad_alloc &) {
        return ECSPMV_ERR_NOMEM;
    } catch (...) {                                  // nothing may leave through the C ABI (a worker thread that could
        return ECSPMV_ERR_INTERNAL;                  // not be started, for instance)
    }
}

void ecspmv_csr_destroy(ecspmv_csr *C) { delete C; }

int ecspmv_csr_device_bytes(const ecspmv_csr *C, size_t *bytes)
{
    if (!C || !bytes) return ECSPMV_ERR_INVALID;
    *bytes = C->bytes;
    return ECSPMV_OK;
}

int ecspmv_csr_upload(ecspmv_csr *C, void *d_buf, size_t bytes, void *stream)
{
    if (!C || !d_buf || (reinterpret_cast<uintptr_t>(d_buf) & 255)) return ECSPMV_ERR_INVALID;
    if (bytes < C->bytes) return ECSPMV_ERR_TOO_SMALL;
    uint8_t *d = static_cast<uint8_t *>(d_buf);
    int e = ecs::copy_to_device(d, C->rowptr.data(), 4 * C->rowptr.size(), stream);
    if (!e && C->nnz) e = ecs::copy_to_device(d + C->off_col, C->col.data(), 4 * C->col.size(), stream);
    if (!e && C->nnz) e = ecs::copy_to_device(d + C->off_val, C->val.data(), 2 * C->val.size(), stream);
    if (e) return hip_status(e);
    C->d_buf = d;
    return ECSPMV_OK;
}

int ecspmv_csr_run(const ecspmv_csr *C, const void *d_x, void *d_y, void *stream)
{
    if (!C || !d_x || !d_y) return ECSPMV_ERR_INVALID;
    if (!C->d_buf) return ECSPMV_ERR_NOT_UPLOADED;
    return hip_status(ecs::launch_csr(C->d_buf, C->d_buf + C->off_col, C->d_buf + C->off_val, d_x, d_y, (uint32_t)C->m,
                                      stream));
}

int ecspmv_stream_read(const void *d_buf, size_t bytes, void *d_out, int32_t num_wg, void *stream)
{
    if (!d_buf || !d_out || num_wg <= 0 || (bytes & 15) || (reinterpret_cast<uintptr_t>(d_buf) & 15))
        return ECSPMV_ERR_INVALID;
    return hip_status(ecs::launch_stream_read(d_buf, bytes, d_out, (uint32_t)num_wg, 1024u, false, stream));
}

int ecspmv_stream_read_sliced(const void *d_buf, size_t bytes, void *d_out, int32_t num_wg, int32_t threads_per_wg,
                              void *stream)
{
    if (!d_buf || !d_out || num_wg <= 0 || (bytes & 15) || (reinterpret_cast<uintptr_t>(d_buf) & 15))
        return ECSPMV_ERR_INVALID;
    if (threads_per_wg != 256 && threads_per_wg != 512 && threads_per_wg != 1024) return ECSPMV_ERR_INVALID;
    return hip_status(ecs::launch_stream_read(d_buf, bytes, d_out, (uint32_t)num_wg, (uint32_t)threads_per_wg, true,
                                              stream));
}

int ecspmv_empty_launch(void *d_out, int32_t num_wg, int32_t threads_per_wg, int32_t count, void *stream)
{
    if (!d_out || num_wg <= 0 || count <= 0 || threads_per_wg < 64 || threads_per_wg > 1024 || (threads_per_wg & 63))
        return ECSPMV_ERR_INVALID;
    for (int32_t i = 0; i < count; ++i) {
        int s = hip_status(ecs::launch_empty(d_out, (uint32_t)num_wg, (uint32_t)threads_per_wg, stream));
        if (s) return s;
    }
    return ECSPMV_OK;
}

#ifdef ECS_TRACE
// Only in the library built with -DECS_TRACE (libecspmv_trace.so, which the timeline script loads; the product library
// has no stamps compiled in).  Each of the next `regions` launches leaves, per wavefront, the clock at its first
// instruction, at point `sel` of the kernel and at its last instruction in its own region of d_words (device,
// regions x wgs_per_region x 128 uint64).  NULL switches the stamps off.
int ecspmv_trace_buffer(void *d_words, uint32_t regions, uint32_t wgs_per_region, uint32_t sel)
{
    return hip_status(ecs::set_trace_buffer(d_words, regions, wgs_per_region, sel));
}
#endif

const char *ecspmv_strerror(int status)
{
    switch (status) {
    case ECSPMV_OK: return "ok";
    case ECSPMV_ERR_INVALID: return "invalid argument";
    case ECSPMV_ERR_UNSUPPORTED: return "unsupported size or option";
    case ECSPMV_ERR_NOMEM: return "out of host memory";
    case ECSPMV_ERR_HIP: return "HIP call failed (see ecspmv_last_hip_error)";
    case ECSPMV_ERR_NOT_UPLOADED: return "matrix has no device image yet";
    case ECSPMV_ERR_TOO_SMALL: return "buffer too small";
    case ECSPMV_ERR_INTERNAL: return "unexpected failure inside the library";
    default: return "unknown status";
    }
}

int ecspmv_last_hip_error(void) { return g_last_hip_error; }

}  // extern "C"
