// Common definitions of the amghess library (gfx950): error handling, device
// allocations, CSR containers and launch geometry.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <mutex>
#include <string>
#include <utility>
#include <vector>

#include "amghess.h"

namespace amg {

struct Error {
    int code;
    std::string msg;
};

[[noreturn]] inline void fail(int code, const std::string &msg) { throw Error{code, msg}; }

#define AMG_HIP(call)                                                                      \
    do {                                                                                   \
        hipError_t e_ = (call);                                                            \
        if (e_ != hipSuccess)                                                              \
            ::amg::fail(e_ == hipErrorOutOfMemory ? AMG_ERR_OOM : AMG_ERR_HIP,             \
                        std::string(#call) + ": " + hipGetErrorString(e_));                \
    } while (0)

// Device blocks that ended contexts give back, kept per device for later
// contexts of the process (what a framework's caching allocator does): a
// context then starts and ends without hipMalloc / hipFree calls, each of
// which waits for the device.  A request takes the smallest cached block of
// its device that is at least as large and at most a third larger;
// amg_release_memory hands every cached block back to the driver.
struct DevPool {
    struct Blk {
        int dev;
        size_t bytes;
        void *p;
    };
    std::mutex m;
    std::vector<Blk> blks;
    size_t held = 0;
    static constexpr size_t kMaxHeld = size_t(32) << 30;
    // never destroyed: no hipFree may run after the runtime has shut down
    static DevPool &get() {
        static DevPool *pool = new DevPool();
        return *pool;
    }
    // a cached block (and its size) or {nullptr, 0}
    std::pair<void *, size_t> take(int dev, size_t bytes) {
        std::lock_guard<std::mutex> g(m);
        int best = -1;
        for (size_t i = 0; i < blks.size(); ++i)
            if (blks[i].dev == dev && blks[i].bytes >= bytes && blks[i].bytes <= bytes + bytes / 3 &&
                (best < 0 || blks[i].bytes < blks[best].bytes))
                best = (int)i;
        if (best < 0) return {nullptr, 0};
        const Blk b = blks[best];
        blks.erase(blks.begin() + best);
        held -= b.bytes;
        return {b.p, b.bytes};
    }
    // false: not kept (the cache is full), the caller frees it
    bool give(int dev, void *p, size_t bytes) {
        std::lock_guard<std::mutex> g(m);
        if (held + bytes > kMaxHeld) return false;
        blks.push_back({dev, bytes, p});
        held += bytes;
        return true;
    }
    // every cached block of device dev (all devices when dev < 0) to the driver
    void release(int dev) {
        std::vector<Blk> out;
        {
            std::lock_guard<std::mutex> g(m);
            std::vector<Blk> keep;
            for (const Blk &b : blks) (dev < 0 || b.dev == dev ? out : keep).push_back(b);
            blks.swap(keep);
            for (const Blk &b : out) held -= b.bytes;
        }
        for (const Blk &b : out) (void)hipFree(b.p);
    }
};

// Every device allocation of a context goes through one arena so that a
// failure anywhere in setup releases everything.  Requests up to a quarter of a
// chunk are carved from large chunks (few hipMalloc calls, and few hipFree
// calls when the context ends: each waits for the device); larger ones get
// their own allocation.  A released block is kept and handed out again to a
// later request of at most its size (and at least half of it): all work of a
// context runs in order on its one stream, so the kernels that used the block
// are ahead of any that reuse it.
struct Arena {
    struct Blk {
        void *p;
        size_t bytes;
        bool live;
    };
    std::vector<Blk> blks;                         // every block handed out
    std::vector<std::pair<void *, size_t>> chunks; // device allocations (cached or new) and sizes
    int dev = -1;                                  // device of the allocations
    char *cur = nullptr;
    size_t cur_left = 0, next_chunk = size_t(8) << 20;
    size_t bytes = 0;
    static constexpr size_t kMaxChunk = size_t(128) << 20;

    void *dev_malloc(size_t b) {
        if (dev < 0 && hipGetDevice(&dev) != hipSuccess) fail(AMG_ERR_HIP, "hipGetDevice failed");
        auto got = DevPool::get().take(dev, b);
        if (!got.first) {
            void *p = nullptr;
            hipError_t e = hipMalloc(&p, b);
            if (e != hipSuccess) {  // once more without the cache's blocks of this device
                (void)hipGetLastError();
                DevPool::get().release(dev);
                e = hipMalloc(&p, b);
            }
            if (e != hipSuccess) {
                (void)hipGetLastError();
                fail(AMG_ERR_OOM, "hipMalloc of " + std::to_string(b) + " bytes failed");
            }
            got = {p, b};
        }
        chunks.push_back(got);
        bytes += got.second;
        return got.first;
    }
    template <class T> T *alloc(size_t n) {
        if (n == 0) n = 1;
        const size_t want = (n * sizeof(T) + 255) & ~(size_t)255;
        Blk *best = nullptr;
        for (auto &b : blks)
            if (!b.live && b.bytes >= want && b.bytes <= 2 * want && (!best || b.bytes < best->bytes)) best = &b;
        if (best) {
            best->live = true;
            return static_cast<T *>(best->p);
        }
        void *p;
        if (want > kMaxChunk / 4) {
            p = dev_malloc(want);
        } else {
            if (want > cur_left) {
                const size_t c = std::max(next_chunk, want);
                cur = static_cast<char *>(dev_malloc(c));
                cur_left = c;
                next_chunk = std::min(kMaxChunk, 2 * next_chunk);
            }
            p = cur;
            cur += want;
            cur_left -= want;
        }
        blks.push_back({p, want, true});
        return static_cast<T *>(p);
    }
    void release(void *p) {
        for (auto &b : blks)
            if (b.p == p) b.live = false;
    }
    // back to the process's cache (the context's streams have drained)
    void free_all() {
        for (auto &ch : chunks)
            if (!DevPool::get().give(dev, ch.first, ch.second)) (void)hipFree(ch.first);
        chunks.clear();
        blks.clear();
        cur = nullptr;
        cur_left = 0;
        bytes = 0;
    }
};

// CSR matrix in device memory: int32 indices, FP64 values and an optional
// float32 copy of the values for the mixed-precision path.
struct DCsr {
    int n = 0, m = 0, nnz = 0;
    int *rp = nullptr;
    int *ci = nullptr;
    double *v = nullptr;
    float *v32 = nullptr;
    // optional sliced-ELL copy (finest level): slices of 64 rows stored column
    // by column, entry k of row 64 s + l at sl_off[s] + 64 k + l; a column is
    // kept as a 16-bit offset from the slice's smallest column sl_base[s] (the
    // copy exists only when every slice spans fewer than 65536 columns), and the
    // rows of a slice are padded to its longest with (the row's last offset, value 0)
    int nsl = 0;
    long sl_tot = 0;        // stored entries, padding included
    bool sl_over8 = true;   // some slice is wider than 8 entries per row
    int *sl_off = nullptr;  // [nsl + 1]
    int *sl_base = nullptr; // [nsl]
    uint16_t *sl_cd = nullptr;
    double *sl_v = nullptr;
    float *sl_v32 = nullptr;
    // whether products on nb columns run on the copy: always for one column.  A batch
    // pays for a padded entry's gathers and multiplications as for a stored one's: only
    // up to half as many again (3D P1 rows pad by 12 %).  And it needs rows enough: a
    // lane takes a whole row (of up to four columns), in rounds of eight entries, while
    // the CSR product spreads a small matrix over 2^17 lanes.  Rows of up to eight
    // entries take the copy from 2^15 lanes on (the three level-0 passes of a FP64
    // Chebyshev cycle on 7-point rows, copy / CSR in us: 29791 rows x 4 11.2 / 10.0,
    // 39304 x 4 11.3 / 12.2, 12167 x 8 10.9 / 10.0, 29791 x 8 11.6 / 12.6, 6859 x 16
    // 11.3 / 10.1, 12167 x 16 11.2 / 12.2), longer ones, two rounds, from 2^16 rows on
    // (15-point mass rows: 1728 x 8 6.3 / 4.0, 39304 x 2 5.4 / 4.4, 39304 x 8 8.8 / 7.7,
    // 91125 x 4 9.0 / 10.9, 91125 x 8 12.2 / 13.2).
    bool sell_for(int nb) const {
        if (!sl_off || nb == 1) return sl_off != nullptr;
        const bool rows_enough = nnz <= 8L * n ? (long)n * (nb > 4 ? nb / 4 : 1) >= 1L << 15 : n >= 1 << 16;
        return rows_enough && 2 * sl_tot <= 3L * nnz;
    }
    // optional 16-bit columns of a large coarse matrix for products on one column:
    // entry p of row i is column row_base(i, c16_scale) + c16[p] (present only when
    // every offset fits)
    int16_t *c16 = nullptr;
    uint32_t c16_scale = 0;
    // lanes-per-row choice set by the autotuner: log2 G for batch width
    // 2^k (k = 0..4) and values FP64 (0) / float32 (1); -1 = the default rule
    int8_t tuned_lg[5][2] = {{-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}, {-1, -1}};
};

// The column about which row i of an n x m hierarchy matrix is centred: the levels
// are numbered alike (an aggregate's number follows its root's), so a row's columns
// lie around i m / n; the row itself when n = m.  scale = m 2^24 / n, m < 256 n.
__host__ __device__ inline int row_base(int i, uint32_t scale) { return (int)(((uint64_t)(uint32_t)i * scale) >> 24); }

constexpr int kBlock = 256;      // threads per workgroup (4 wavefronts of 64)
constexpr int kMaxGrid = 16384;        // workgroups times columns at most for kernels with reductions
constexpr int kMaxGridPlain = 1 << 20; // workgroups at most for kernels without
// Workgroups of a reducing launch on NB columns at most, each sweeping its share.
// One or two columns take 1024, about what is resident at once (four per CU at the
// registers of the FP64 products): few partials keep the finalize folded into the
// next product (with up to 16384 workgroups for one column, a CG iteration on 184344
// rows took two finalize launches more, 4.7 + 4.2 us, one on 2.1e6 rows too).  More
// columns take kMaxGrid / NB, 16, 8 and 4 per CU for 4, 8 and 16: at most kMaxGrid
// partials per quantity, which finalize launches sum.  Fewer for 4 and 8 columns have
// not been measured.
template <int NB> constexpr int red_grid_max() { return NB <= 2 ? 1024 : kMaxGrid / NB; }
constexpr int kMaxPart = 2 * kMaxGrid;  // partials of a reducing launch at most: two quantities
constexpr int kFinBlock = 1024;        // threads of a finalize kernel
constexpr int kXcd = 8;          // XCDs of an MI355X

__host__ __device__ inline int ceil_div(long a, long b) { return (int)((a + b - 1) / b); }

// Grid for a row-blocked kernel: a multiple of 8 so that the XCD-aware remap
// (see xcd_share) is a permutation.
inline int grid_rows(long rows, int rows_per_block, int maxg) {
    int g = ceil_div(rows, rows_per_block);
    if (g > maxg) g = maxg;
    if (g < 1) g = 1;
    return ceil_div(g, kXcd) * kXcd;
}

}  // namespace amg
