// P1 finite-element assembly on the GPU (paper, Section 2: [A]_ij =
// a(phi_j, phi_i), [M]_ij = (phi_j, phi_i)), bit-identical to the host
// assembler: every entry adds its elements' contributions in ascending element
// index, formed with the shared element arithmetic (p1_element.hpp, no fused
// multiply-add), exactly the order in which the host adds them.
//
// Steps: vertex -> element lists (k_vertex_lists counts, scan, k_vertex_lists
// places); row lengths (k_row_count) and their scan; then columns and values
// of a row together (k_row_fill).  The row kernels give a row 16 lanes and
// keep it in LDS; rows with too many elements or entries for that take the
// general kernels (k_vertex_sort, k_row_pattern, k_row_values).
#include <climits>
#include <cstdint>
#include <mutex>
#include <new>

#include "common.hpp"
#include "p1_element.hpp"

#pragma clang fp contract(off)

namespace amg {
namespace {

constexpr int kAsmBlock = 256;

int blocks_for(long n) {
    long b = (n + kAsmBlock - 1) / kAsmBlock;
    if (b < 1) b = 1;
    if (b > 65536) b = 65536;
    return (int)b;
}

// Orders the LDS accesses of one wavefront around a point all its lanes reach.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Words of AsmScratch::flags.
enum Flag { kBadId = 0, kOver = 1, kMaxDeg = 2, kMaxLen = 3, kTotal = 4, kFlags = 8 };

// The slot of key in an open-addressing table of SLOTS words (-1: empty) in
// LDS, entered if it is not there yet; *fresh: this call entered it.
template <int SLOTS> __device__ __forceinline__ int hash_slot(int32_t *tab, int32_t key, bool *fresh) {
    constexpr int kShift = 32 - __builtin_ctz(SLOTS);
    int h = (int)((uint32_t)key * 2654435761u >> kShift);  // Fibonacci hashing: 2^32 / golden ratio
    *fresh = false;
    for (;;) {
        const int32_t was = atomicCAS(&tab[h], -1, key);
        if (was == -1) *fresh = true;
        if (was == -1 || was == key) return h;
        h = (h + 1) & (SLOTS - 1);
    }
}

// Vertex counts (PLACE false: cur[v] += occurrences of v, ids outside
// 0..nv-1 raise flags[kBadId] and are left out) or the placement of every
// element in its vertices' lists (PLACE true: cur starts as the lists' first
// positions; the order within a list is arbitrary).  Elements that are near
// each other share vertices, so a workgroup first counts its 2048 ids per
// distinct vertex in LDS and then sends one atomic per distinct vertex (a
// Kuhn cube's ids: about 250 instead of 2048): contended global atomics were
// the whole cost of a pass of one atomic per id (64^3 cube, 6.3 million ids:
// 114 us counting, 152 us placing).  kSlots is twice the ids, so the probing
// ends whatever the ids are.
constexpr int kListIds = 2048, kListSlots = 2 * kListIds;
template <int NL, bool PLACE>
__global__ __launch_bounds__(kAsmBlock) void k_vertex_lists(int32_t n, const int32_t *__restrict__ ids, int32_t nv,
                                                            int32_t *cur, int32_t *ve, int32_t *flags) {
    constexpr int PT = kListIds / kAsmBlock;
    __shared__ int32_t key[kListSlots], cnt[kListSlots];
    const int t = threadIdx.x;
    const long base = (long)blockIdx.x * kListIds;
    for (int i = t; i < kListSlots; i += kAsmBlock) {
        key[i] = -1;
        cnt[i] = 0;
    }
    int32_t id[PT];
#pragma unroll
    for (int k = 0; k < PT; ++k) {
        const long i = base + k * kAsmBlock + t;
        const int32_t x = ids[i < n ? i : n - 1];
        const bool ok = x >= 0 && x < nv;
        if (!PLACE && !ok) flags[kBadId] = 1;
        id[k] = i < n && ok ? x : -1;
    }
    __syncthreads();
    int slot[PT], rank[PT];
#pragma unroll
    for (int k = 0; k < PT; ++k) {
        if (id[k] < 0) continue;
        bool fresh;
        slot[k] = hash_slot<kListSlots>(key, id[k], &fresh);
        rank[k] = atomicAdd(&cnt[slot[k]], 1);
    }
    __syncthreads();
    for (int i = t; i < kListSlots; i += kAsmBlock) {
        if (key[i] < 0) continue;
        if constexpr (PLACE) cnt[i] = atomicAdd(&cur[key[i]], cnt[i]);
        else atomicAdd(&cur[key[i]], cnt[i]);
    }
    if constexpr (PLACE) {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < PT; ++k)
            if (id[k] >= 0) ve[cnt[slot[k]] + rank[k]] = (int32_t)((base + k * kAsmBlock + t) / NL);
    }
}

// out[0..n]: exclusive sums of in[0..n-1], out[n] the total, in two launches
// over chunks of kScanChunk entries: chunk sums, then each workgroup adds the
// sums before its chunk and scans it.  out2 (or null, may be in) gets a copy
// of out[0..n-1]; flags get the largest entry (word `most`), the total and,
// beyond int32, kOver.
constexpr int kScanPer = 8, kScanChunk = kAsmBlock * kScanPer;

// the sum over the workgroup, in every thread; w: kAsmBlock / 64 words of LDS
__device__ __forceinline__ long long block_sum(long long v, long long *w) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = v;
    __syncthreads();
    long long r = 0;
    for (int k = 0; k < kAsmBlock / 64; ++k) r += w[k];
    return r;
}

__global__ __launch_bounds__(kAsmBlock) void k_scan_chunks(int32_t n, const int32_t *in, long long *csum,
                                                           int32_t *most) {
    __shared__ long long w[kAsmBlock / 64];
    const long c0 = (long)blockIdx.x * kScanChunk;
    long long s = 0;
    int32_t m = 0;
    for (int i = 0; i < kScanPer; ++i) {
        const long j = c0 + (long)i * kAsmBlock + threadIdx.x;
        const int32_t x = j < n ? in[j] : 0;
        s += x;
        m = max(m, x);
    }
    s = block_sum(s, w);
    if (threadIdx.x == 0) csum[blockIdx.x] = s;
    for (int o = 32; o > 0; o >>= 1) m = max(m, __shfl_xor(m, o));
    // the stored maximum only grows: a stale read never skips a needed update
    if ((threadIdx.x & 63) == 0 && m > __hip_atomic_load(most, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
        atomicMax(most, m);
}

__global__ __launch_bounds__(kAsmBlock) void k_scan_write(int32_t n, const int32_t *in, const long long *csum,
                                                          int32_t *out, int32_t *out2, int32_t *flags) {
    __shared__ long long w[kAsmBlock / 64];
    const int t = threadIdx.x, lane = t & 63;
    long long before = 0;
    for (int c = t; c < (int)blockIdx.x; c += kAsmBlock) before += csum[c];
    before = block_sum(before, w);
    const long base = (long)blockIdx.x * kScanChunk + (long)t * kScanPer;  // this thread's entries
    int32_t v[kScanPer];
    long long s = 0;
#pragma unroll
    for (int i = 0; i < kScanPer; ++i) {
        v[i] = base + i < n ? in[base + i] : 0;
        s += v[i];
    }
    long long inc = s;
    for (int d = 1; d < 64; d <<= 1) {
        const long long y = __shfl_up(inc, d);
        if (lane >= d) inc += y;
    }
    __syncthreads();
    if (lane == 63) w[t >> 6] = inc;
    __syncthreads();
    long long run = before + inc - s;
    for (int k = 0; k < (t >> 6); ++k) run += w[k];
#pragma unroll
    for (int i = 0; i < kScanPer; ++i) {
        const int32_t o = run > INT_MAX ? INT_MAX : (int32_t)run;
        if (base + i < n) {
            out[base + i] = o;
            if (out2) out2[base + i] = o;
        }
        run += v[i];
    }
    if (blockIdx.x == gridDim.x - 1 && t == kAsmBlock - 1) {
        out[n] = run > INT_MAX ? INT_MAX : (int32_t)run;
        flags[kTotal] = out[n];
        if (run > INT_MAX) flags[kOver] = 1;
    }
}

// ---- rows in LDS: 16 lanes per row, four rows per wavefront ----
constexpr int kRowLanes = 16, kRowsPerBlock = kAsmBlock / kRowLanes;
constexpr int kCountElems = 64;  // elements around a vertex at most for k_row_count
constexpr int kFillLen = 127;    // entries of a row at most for k_row_fill (7-bit positions)

// Row lengths of the mesh graph: the number of distinct vertices of the row
// vertex's elements, by entering them all in a small table (at most
// 1 + 64 * 3 of its 256 slots are taken).  Rows with more elements are left
// to k_row_pattern.  (Searching a row's candidates for the next larger column
// again and again took 276 us at 64^3.)
template <int NL>
__global__ __launch_bounds__(kAsmBlock) void k_row_count(int32_t nv, const int32_t *__restrict__ elems,
                                                         const int32_t *__restrict__ vp,
                                                         const int32_t *__restrict__ ve, int32_t *cnt) {
    constexpr int SLOTS = 4 * kCountElems;
    __shared__ int32_t tabs[kRowsPerBlock][SLOTS];
    const int g = threadIdx.x % kRowLanes, r = threadIdx.x / kRowLanes;
    int32_t *tab = tabs[r];
    for (long v0 = (long)blockIdx.x * kRowsPerBlock; v0 < nv; v0 += (long)gridDim.x * kRowsPerBlock) {
        const long v = v0 + r;
        const int32_t p0 = v < nv ? vp[v] : 0, deg = v < nv ? vp[v + 1] - p0 : 0;
        const bool on = v < nv && deg <= kCountElems;
        for (int i = g; i < SLOTS; i += kRowLanes) tab[i] = -1;
        wave_sync();
        int c = 0;
        if (on)
            for (int j = g; j < deg; j += kRowLanes) {
                const int32_t e = ve[p0 + j];
                int32_t k[NL];
#pragma unroll
                for (int b = 0; b < NL; ++b) k[b] = elems[(long)e * NL + b];
#pragma unroll
                for (int b = 0; b < NL; ++b) {
                    bool fresh;
                    hash_slot<SLOTS>(tab, k[b], &fresh);
                    c += fresh;
                }
            }
        for (int o = kRowLanes / 2; o > 0; o >>= 1) c += __shfl_xor(c, o);
        if (on && g == 0) cnt[v] = c;
        wave_sync();
    }
}

// One row of both matrices, columns and values (rows of at most E elements
// and kFillLen entries; rowptr is written for every row).  A row's elements
// are ranked by index, their vertices entered in a table whose distinct keys,
// ranked, are the row's columns; each lane then forms the row's contributions
// of its elements (the element arithmetic once per row and element) into LDS
// at the element's rank, with the positions of its vertices in the row as
// bytes (the row vertex's own place marked by the top bit), and the lanes turn
// to the row's entries: an entry walks the elements in order and adds the
// contributions whose position byte is its own, in registers.  Bound by
// instruction issue and LDS latency at four wavefronts per SIMD (FP64 divisions
// of the gradients, four times per element, the rankings and the walk): every
// loop over a row's lists therefore reads LDS in 16-byte words, four entries or
// elements at a time, and lists share storage where their uses end (2064 bytes
// per row).  64^3: 235 us, 318 us with one entry per LDS read and 2816 bytes;
// one thread per row that added into global memory behind a binary search took
// 2021 us for the values alone.
template <int DIM, int E>
__global__ __launch_bounds__(kAsmBlock) void k_row_fill(int32_t nv, const double *__restrict__ coords,
                                                        const int32_t *__restrict__ elems,
                                                        const double *__restrict__ kappa,
                                                        const int32_t *__restrict__ vp,
                                                        const int32_t *__restrict__ ve,
                                                        const int32_t *__restrict__ rp, int32_t *__restrict__ rowptr,
                                                        int32_t *__restrict__ col, double *__restrict__ valA,
                                                        double *__restrict__ valM) {
    constexpr int NL = DIM + 1, SLOTS = 4 * E, KP = E / kRowLanes;
    constexpr int KEYS = (1 + E * DIM < kFillLen ? 1 + E * DIM : kFillLen) / 4 * 4 + 4;  // entries, in fours
    struct Row {
        union {
            int32_t tab[SLOTS];  // the distinct vertices; its keys are read out before s is written
            double s[E][NL];     // stiffness contributions, by element rank and place in the element
        };
        double m[E];             // mass contribution off the diagonal (the diagonal's is twice it)
        union {
            int4 se4[E / 4];     // the elements, read out before key is written
            int32_t se[E];
            int4 key4[KEYS / 4]; // the distinct vertices in table order, then INT_MAX
            int32_t key[KEYS];
        };
        union {
            uint4 pos4[E / 4];
            uint32_t pos[E];
        };
        uint8_t at[KEYS];        // the keys' slots
        uint8_t rk[SLOTS];       // slot -> position in the row
        uint32_t pad[4];         // rows of a wavefront start in different banks
    };
    static_assert(SLOTS <= 256, "slots are kept in a byte");
    __shared__ Row rows[kRowsPerBlock];
    const int g = threadIdx.x % kRowLanes;
    Row &R = rows[threadIdx.x / kRowLanes];
    for (long v0 = (long)blockIdx.x * kRowsPerBlock; v0 < nv; v0 += (long)gridDim.x * kRowsPerBlock) {
        const long v = v0 + threadIdx.x / kRowLanes;
        int32_t p0 = 0, deg = 0, r0 = 0, len = 0;
        if (v < nv) {
            p0 = vp[v];
            deg = vp[v + 1] - p0;
            r0 = rp[v];
            len = rp[v + 1] - r0;
            if (g == 0) rowptr[v] = r0;
            if (g == 0 && v == nv - 1) rowptr[nv] = r0 + len;
        }
        if (deg > E || len > kFillLen) deg = len = 0;  // left to the general kernels
        for (int i = g; i < SLOTS; i += kRowLanes) R.tab[i] = -1;
        int32_t eid[KP], vid[KP][NL];
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            const int j = k * kRowLanes + g;
            eid[k] = j < deg ? ve[p0 + j] : INT_MAX;
            R.se[j] = eid[k];
#pragma unroll
            for (int b = 0; b < NL; ++b) vid[k][b] = j < deg ? elems[(long)eid[k] * NL + b] : 0;
        }
        wave_sync();
        int rank[KP], slot[KP][NL];
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            rank[k] = 0;
#pragma unroll
            for (int b = 0; b < NL; ++b) slot[k][b] = 0;
            const int j = k * kRowLanes + g;
            if (j >= deg) continue;
            // an element that holds the vertex twice is listed twice; the list ends in INT_MAX
#pragma unroll
            for (int i = 0; i < E / 4; ++i) {
                const int4 x = R.se4[i];
                rank[k] += (x.x < eid[k] || (x.x == eid[k] && 4 * i < j)) +
                           (x.y < eid[k] || (x.y == eid[k] && 4 * i + 1 < j)) +
                           (x.z < eid[k] || (x.z == eid[k] && 4 * i + 2 < j)) +
                           (x.w < eid[k] || (x.w == eid[k] && 4 * i + 3 < j));
            }
#pragma unroll
            for (int b = 0; b < NL; ++b) {
                bool fresh;
                slot[k][b] = hash_slot<SLOTS>(R.tab, vid[k][b], &fresh);
            }
        }
        wave_sync();
        // the table's keys, gathered (len of them), then each one's rank
        int mine = 0;
#pragma unroll
        for (int i = 0; i < SLOTS / kRowLanes; ++i) mine += deg > 0 && R.tab[i * kRowLanes + g] >= 0;
        int o = mine;
#pragma unroll
        for (int d = 1; d < kRowLanes; d <<= 1) {
            const int y = __shfl_up(o, d, kRowLanes);
            if (g >= d) o += y;
        }
        o -= mine;
        if (deg > 0)
#pragma unroll
            for (int i = 0; i < SLOTS / kRowLanes; ++i) {
                const int32_t x = R.tab[i * kRowLanes + g];
                if (x < 0 || o >= KEYS) continue;
                R.key[o] = x;
                R.at[o] = (uint8_t)(i * kRowLanes + g);
                ++o;
            }
        if (g < 4 && len + g < KEYS) R.key[len + g] = INT_MAX;  // the last four read may pass the row's end
        wave_sync();
        for (int i = g; i < len; i += kRowLanes) {
            const int32_t x = R.key[i];
            int q = 0;
#pragma unroll 4
            for (int k = 0; k < len; k += 4) {
                const int4 y = R.key4[k / 4];
                q += (y.x < x) + (y.y < x) + (y.z < x) + (y.w < x);
            }
            R.rk[R.at[i]] = (uint8_t)q;
            col[r0 + q] = x;
        }
        wave_sync();
#pragma unroll
        for (int k = 0; k < KP; ++k) {
            if (k * kRowLanes + g >= deg) continue;
            double X[NL * DIM];
#pragma unroll
            for (int a = 0; a < NL; ++a)
#pragma unroll
                for (int d = 0; d < DIM; ++d) X[a * DIM + d] = coords[(long)vid[k][a] * DIM + d];
            double gr[4][3], meas;
            p1_grads(DIM, X, gr, meas);
            const double w = kappa[eid[k]] * meas;
            int a = 0;  // the vertex's place in the element (its first, as on the host)
#pragma unroll
            for (int b = NL - 1; b >= 0; --b)
                if (vid[k][b] == v) a = b;
            double ga[3] = {0.0, 0.0, 0.0};
#pragma unroll
            for (int b = 0; b < NL; ++b)
                if (b == a) {
#pragma unroll
                    for (int d = 0; d < DIM; ++d) ga[d] = gr[b][d];
                }
            uint32_t pos = NL == 3 ? 0x7f000000u : 0u;  // no entry has position 127
#pragma unroll
            for (int b = 0; b < NL; ++b) {
                R.s[rank[k]][b] = p1_stiff_vec(DIM, ga, gr[b], w);
                pos |= (uint32_t)(R.rk[slot[k][b]] | (b == a ? 0x80u : 0u)) << (8 * b);
            }
            R.m[rank[k]] = p1_mass(DIM, meas, 0, 1);
            R.pos[rank[k]] = pos;
        }
        wave_sync();
        for (int q = g; q < len; q += kRowLanes) {
            double sA = 0.0, sM = 0.0;
            const uint32_t want = (uint32_t)q * 0x01010101u;
            for (int j0 = 0; j0 < deg; j0 += 4) {  // four elements' contributions in flight
                const uint4 p4 = R.pos4[j0 / 4];
                const uint32_t pp[4] = {p4.x, p4.y, p4.z, p4.w};
                uint32_t hit[4];
                double cs[4], cm[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    // the top bit of every byte whose position is q (7-bit values: the
                    // sum does not carry from byte to byte)
                    hit[i] = ~(((pp[i] & 0x7f7f7f7fu) ^ want) + 0x7f7f7f7fu) & 0x80808080u;
                    if (j0 + i >= deg) hit[i] = 0;
                    const int b = hit[i] ? (__ffs(hit[i]) - 1) >> 3 : 0;
                    cs[i] = R.s[j0 + i][b];
                    const double m = R.m[j0 + i];
                    cm[i] = (pp[i] >> (8 * b)) & 0x80u ? 2.0 * m : m;
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (!hit[i]) continue;
                    sA = sA + cs[i];
                    sM = sM + cm[i];
                    for (uint32_t h = hit[i] & (hit[i] - 1); h; h &= h - 1) {  // a vertex held twice
                        const int b = (__ffs(h) - 1) >> 3;
                        const double m = R.m[j0 + i];
                        sA = sA + R.s[j0 + i][b];
                        sM = sM + ((pp[i] >> (8 * b)) & 0x80u ? 2.0 * m : m);
                    }
                }
            }
            valA[r0 + q] = sA;
            valM[r0 + q] = sM;
        }
        wave_sync();
    }
}

// ---- the general kernels, for rows beyond the limits above: a row is theirs
// when it has more than max_deg elements or (rp not null) more than kFillLen
// entries ----
__device__ __forceinline__ bool general_row(int32_t v, const int32_t *vp, const int32_t *rp, int32_t max_deg) {
    return vp[v + 1] - vp[v] > max_deg || (rp && rp[v + 1] - rp[v] > kFillLen);
}

// each vertex's element list in ascending order (insertion sort: the lists
// are as long as the number of elements around a vertex)
__global__ void k_vertex_sort(int32_t nv, const int32_t *vp, int32_t *ve, const int32_t *rp, int32_t max_deg) {
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
        if (!general_row(v, vp, rp, max_deg)) continue;
        const int32_t p0 = vp[v], p1 = vp[v + 1];
        for (int32_t p = p0 + 1; p < p1; ++p) {
            const int32_t x = ve[p];
            int32_t q = p - 1;
            while (q >= p0 && ve[q] > x) {
                ve[q + 1] = ve[q];
                --q;
            }
            ve[q + 1] = x;
        }
    }
}

// Row lengths (count) or columns (fill) of the mesh graph, sorted and
// distinct: one wavefront per row.  The candidates are the vertices of the row
// vertex's elements (candidate c: vertex c % nl of its (c / nl)-th element);
// lane l holds candidates l and l + 64 in registers and reads any further ones
// from memory.  Each step takes the smallest candidate above the last one by a
// wavefront minimum (INT_MAX, never a vertex id, marks none).  The count runs
// before the host knows whether any row needs it: it returns when the largest
// element count (*most) is within k_row_count's.
template <bool FILL>
__global__ void k_row_pattern(int32_t nv, int nl, const int32_t *elems, const int32_t *vp, const int32_t *ve,
                              int32_t *cnt, const int32_t *rowptr, int32_t *col, int32_t max_deg,
                              const int32_t *most) {
    if (!FILL && *most <= max_deg) return;
    const int lane = threadIdx.x & 63;
    const long w0 = (blockIdx.x * (long)blockDim.x + threadIdx.x) >> 6;
    const long nw = ((long)gridDim.x * blockDim.x) >> 6;
    for (long v = w0; v < nv; v += nw) {
        if (!general_row((int32_t)v, vp, rowptr, max_deg)) continue;
        const int32_t p0 = vp[v];
        const int32_t nc = (vp[v + 1] - p0) * nl;
        auto cand = [&](int32_t c) { return elems[(long)ve[p0 + c / nl] * nl + c % nl]; };
        const int32_t c0 = lane < nc ? cand(lane) : INT_MAX;
        const int32_t c1 = lane + 64 < nc ? cand(lane + 64) : INT_MAX;
        const int32_t base = FILL ? rowptr[v] : 0;
        int32_t last = -1, m = 0;
        for (;;) {
            int32_t best = INT_MAX;
            if (c0 > last) best = c0;
            if (c1 > last && c1 < best) best = c1;
            for (int32_t c = lane + 128; c < nc; c += 64) {
                const int32_t k = cand(c);
                if (k > last && k < best) best = k;
            }
            for (int off = 32; off > 0; off >>= 1) best = min(best, __shfl_xor(best, off));
            if (best == INT_MAX) break;  // the same value in every lane: the loop ends for the wavefront
            if constexpr (FILL)
                if (lane == 0) col[base + m] = best;
            ++m;
            last = best;
        }
        if constexpr (!FILL)
            if (lane == 0) cnt[v] = m;
    }
}

// DIM is a template parameter so that the small coordinate and gradient arrays
// stay in registers (all their indices are compile-time after unrolling; the
// row's own gradient is picked by predication).
template <int DIM>
__global__ void k_row_values(int32_t nv, const double *coords, const int32_t *elems, const double *kappa,
                             const int32_t *vp, const int32_t *ve, const int32_t *rowptr, const int32_t *col,
                             double *valA, double *valM, int32_t max_deg) {
    constexpr int NL = DIM + 1;
    for (int32_t v = blockIdx.x * blockDim.x + threadIdx.x; v < nv; v += gridDim.x * blockDim.x) {
        if (!general_row(v, vp, rowptr, max_deg)) continue;
        const int32_t r0 = rowptr[v], r1 = rowptr[v + 1];
        for (int32_t q = r0; q < r1; ++q) {
            valA[q] = 0.0;
            valM[q] = 0.0;
        }
        for (int32_t p = vp[v]; p < vp[v + 1]; ++p) {  // elements in ascending order
            const int32_t e = ve[p];
            const int32_t *ev = elems + (long)e * NL;
            int32_t vid[NL];
            double X[NL * DIM];
#pragma unroll
            for (int a = 0; a < NL; ++a) {
                vid[a] = ev[a];
#pragma unroll
                for (int r = 0; r < DIM; ++r) X[a * DIM + r] = coords[(long)vid[a] * DIM + r];
            }
            // the row of the element matrices that belongs to v, formed by the
            // same helpers (hence the same operations) as the host's full matrices
            double g[4][3];
            double meas;
            p1_grads(DIM, X, g, meas);
            const double w = kappa[e] * meas;
            int a = 0;  // v's place in the element (its first, as on the host)
#pragma unroll
            for (int b = NL - 1; b >= 0; --b)
                if (vid[b] == v) a = b;
            double ga[3];
#pragma unroll
            for (int r = 0; r < 3; ++r) ga[r] = 0.0;
#pragma unroll
            for (int b = 0; b < NL; ++b)
                if (b == a) {
#pragma unroll
                    for (int r = 0; r < DIM; ++r) ga[r] = g[b][r];
                }
#pragma unroll
            for (int b = 0; b < NL; ++b) {
                const int32_t k = vid[b];
                int32_t lo = r0, hi = r1;  // first position with col >= k
                while (lo < hi) {
                    const int32_t mid = lo + (hi - lo) / 2;
                    if (col[mid] < k) lo = mid + 1;
                    else hi = mid;
                }
                valA[lo] = valA[lo] + p1_stiff_vec(DIM, ga, g[b], w);
                valM[lo] = valM[lo] + p1_mass(DIM, meas, a, b);
            }
        }
    }
}

#define ASM_HIP(x)                                                                   \
    do {                                                                             \
        const hipError_t e_ = (x);                                                   \
        if (e_ != hipSuccess) return e_ == hipErrorOutOfMemory ? AMG_ERR_OOM : AMG_ERR_HIP; \
    } while (0)

// fills n ints with v (used instead of a memset node, so the clears stay
// kernels of the caller's stream)
__global__ void k_fill(long n, int32_t *p, int32_t v) {
    for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) p[i] = v;
}

// The temporary arrays of one assembly, carved from one workspace: flags,
// chunk sums of the scans, row counts, the vertex -> element lists (vp, ve)
// and the mesh graph's row pointers (rp).
struct AsmScratch {
    int *flags = nullptr;      // [kFlags]
    long long *csum = nullptr; // [chunks]
    int32_t *cnt = nullptr, *vp = nullptr, *ve = nullptr, *rp = nullptr;
};

size_t round256(size_t b) { return (b + 255) & ~(size_t)255; }

size_t scratch_bytes(int dim, int32_t nv, int32_t ne) {
    const size_t nid = (size_t)ne * (dim + 1), nv1 = (size_t)nv + 1;
    const size_t chunks = ((size_t)nv + kScanChunk - 1) / kScanChunk;
    return round256(kFlags * sizeof(int)) + round256(chunks * sizeof(long long)) + 3 * round256(nv1 * sizeof(int32_t)) +
           round256(nid * sizeof(int32_t));
}

AsmScratch carve(void *base, int dim, int32_t nv, int32_t ne) {
    const size_t nid = (size_t)ne * (dim + 1), nv1 = (size_t)nv + 1;
    const size_t chunks = ((size_t)nv + kScanChunk - 1) / kScanChunk;
    char *p = static_cast<char *>(base);
    AsmScratch a;
    auto take = [&](size_t b) {
        char *q = p;
        p += round256(b);
        return q;
    };
    a.flags = (int *)take(kFlags * sizeof(int));
    a.csum = (long long *)take(chunks * sizeof(long long));
    a.cnt = (int32_t *)take(nv1 * sizeof(int32_t));
    a.vp = (int32_t *)take(nv1 * sizeof(int32_t));
    a.ve = (int32_t *)take(nid * sizeof(int32_t));
    a.rp = (int32_t *)take(nv1 * sizeof(int32_t));
    return a;
}

// A workspace from the process-wide cache of device blocks (a block of a
// little more than the size asked for, or a new allocation), handed back to
// the cache, not freed, once the stream has run the work that uses it: so
// repeated assemblies call neither hipMalloc nor hipFree (which waits for the
// whole device).
struct PoolBlock {
    int dev = -1;
    void *p = nullptr;
    size_t bytes = 0;
    hipStream_t s = nullptr;
    int get(size_t b, hipStream_t st) {
        s = st;
        ASM_HIP(hipGetDevice(&dev));
        auto got = DevPool::get().take(dev, b);
        if (!got.first) {
            void *q = nullptr;
            hipError_t e = hipMalloc(&q, b);
            if (e != hipSuccess) {  // once more without the cached blocks of this device
                (void)hipGetLastError();
                DevPool::get().release(dev);
                e = hipMalloc(&q, b);
            }
            if (e != hipSuccess) {
                (void)hipGetLastError();
                return e == hipErrorOutOfMemory ? AMG_ERR_OOM : AMG_ERR_HIP;
            }
            got = {q, b};
        }
        p = got.first;
        bytes = got.second;
        return AMG_OK;
    }
    ~PoolBlock() {
        if (!p) return;
        (void)hipStreamSynchronize(s);
        if (!DevPool::get().give(dev, p, bytes)) (void)hipFree(p);
    }
};

void scan(int32_t n, const int32_t *in, int32_t *out, int32_t *out2, long long *csum, int *flags, int most,
          hipStream_t s) {
    const int nchunks = (int)(((long)n + kScanChunk - 1) / kScanChunk);
    hipLaunchKernelGGL(k_scan_chunks, dim3(nchunks), dim3(kAsmBlock), 0, s, n, in, csum, flags + most);
    hipLaunchKernelGGL(k_scan_write, dim3(nchunks), dim3(kAsmBlock), 0, s, n, in, (const long long *)csum, out, out2,
                       flags);
}

// What the host reads back of a mesh's lists.
struct MeshInfo {
    int32_t total = 0, max_deg = 0, max_len = 0;
};

// vertex -> element lists (vp[nv+1], ve unordered per vertex) and the row
// lengths of the mesh graph with their scan (rp[nv+1])
template <int NL>
int mesh_lists_nl(int32_t nv, int32_t ne, const int32_t *elems, hipStream_t s, const AsmScratch &w, MeshInfo *info) {
    const int32_t nid = ne * NL;
    const int gl = (int)(((long)nid + kListIds - 1) / kListIds);
    hipLaunchKernelGGL(k_fill, dim3(1), dim3(64), 0, s, (long)kFlags, (int32_t *)w.flags, 0);
    hipLaunchKernelGGL(k_fill, dim3(blocks_for((long)nv + 1)), dim3(kAsmBlock), 0, s, (long)nv + 1, w.cnt, 0);
    // ids out of range are flagged and left out of the lists, so nothing below
    // indexes with them; the flag is read with the rest
    hipLaunchKernelGGL((k_vertex_lists<NL, false>), dim3(gl), dim3(kAsmBlock), 0, s, nid, elems, nv, w.cnt,
                       (int32_t *)nullptr, w.flags);
    scan(nv, w.cnt, w.vp, w.cnt, w.csum, w.flags, kMaxDeg, s);
    hipLaunchKernelGGL((k_vertex_lists<NL, true>), dim3(gl), dim3(kAsmBlock), 0, s, nid, elems, nv, w.cnt, w.ve,
                       w.flags);
    hipLaunchKernelGGL((k_row_count<NL>), dim3(std::min(blocks_for((long)nv * kRowLanes), 16384)), dim3(kAsmBlock), 0,
                       s, nv, elems, w.vp, w.ve, w.cnt);
    hipLaunchKernelGGL((k_row_pattern<false>), dim3(std::min(blocks_for(64L * nv), 2048)), dim3(kAsmBlock), 0, s, nv,
                       NL, elems, w.vp, w.ve, w.cnt, (const int32_t *)nullptr, (int32_t *)nullptr, kCountElems,
                       w.flags + kMaxDeg);
    scan(nv, w.cnt, w.rp, (int32_t *)nullptr, w.csum, w.flags, kMaxLen, s);
    ASM_HIP(hipGetLastError());
    int32_t h[kFlags] = {};
    ASM_HIP(hipMemcpyAsync(h, w.flags, kFlags * sizeof(int32_t), hipMemcpyDeviceToHost, s));
    ASM_HIP(hipStreamSynchronize(s));
    if (h[kBadId] || h[kOver]) return AMG_ERR_ARG;  // an id out of range, or more than 2^31 - 1 entries
    info->total = h[kTotal];
    info->max_deg = h[kMaxDeg];
    info->max_len = h[kMaxLen];
    return AMG_OK;
}

int mesh_lists(int dim, int32_t nv, int32_t ne, const int32_t *elems, hipStream_t s, const AsmScratch &w,
               MeshInfo *info) {
    return dim == 2 ? mesh_lists_nl<3>(nv, ne, elems, s, w, info) : mesh_lists_nl<4>(nv, ne, elems, s, w, info);
}

// the pattern and values into the caller's arrays, from the lists of mesh_lists
template <int DIM>
int fill_rows(int32_t nv, const double *coords, const int32_t *elems, const double *kappa, int32_t *rowptr,
              int32_t *col, double *valA, double *valM, hipStream_t s, const AsmScratch &w, const MeshInfo &info) {
    const int32_t *vp = w.vp, *ve = w.ve, *rp = w.rp;
    // 32 elements per row cover the meshes that are regular enough (24 around
    // a vertex of the Kuhn cube); the tables for 64 halve the occupancy
    const int32_t cap = info.max_deg <= 32 ? 32 : 64;
    const dim3 grid(std::min(blocks_for((long)nv * kRowLanes), 16384)), blk(kAsmBlock);
    if (cap == 32)
        hipLaunchKernelGGL((k_row_fill<DIM, 32>), grid, blk, 0, s, nv, coords, elems, kappa, vp, ve, rp, rowptr, col,
                           valA, valM);
    else
        hipLaunchKernelGGL((k_row_fill<DIM, 64>), grid, blk, 0, s, nv, coords, elems, kappa, vp, ve, rp, rowptr, col,
                           valA, valM);
    if (info.max_deg > cap || info.max_len > kFillLen) {
        hipLaunchKernelGGL(k_vertex_sort, dim3(blocks_for(nv)), blk, 0, s, nv, vp, w.ve, rp, cap);
        hipLaunchKernelGGL((k_row_pattern<true>), dim3(blocks_for(64L * nv)), blk, 0, s, nv, DIM + 1, elems, vp, ve,
                           (int32_t *)nullptr, rp, col, cap, (const int32_t *)nullptr);
        hipLaunchKernelGGL((k_row_values<DIM>), dim3(blocks_for(nv)), blk, 0, s, nv, coords, elems, kappa, vp, ve, rp,
                           (const int32_t *)col, valA, valM, cap);
    }
    ASM_HIP(hipGetLastError());
    ASM_HIP(hipStreamSynchronize(s));
    return AMG_OK;
}

int fill_rows(int dim, int32_t nv, const double *coords, const int32_t *elems, const double *kappa, int32_t *rowptr,
              int32_t *col, double *valA, double *valM, hipStream_t s, const AsmScratch &w, const MeshInfo &info) {
    return dim == 2 ? fill_rows<2>(nv, coords, elems, kappa, rowptr, col, valA, valM, s, w, info)
                    : fill_rows<3>(nv, coords, elems, kappa, rowptr, col, valA, valM, s, w, info);
}

// lists and fill (nnz checked against the mesh graph before anything is written)
int assemble_into(int dim, int32_t nv, const double *coords, int32_t ne, const int32_t *elems, const double *kappa,
                  int32_t nnz, int32_t *rowptr, int32_t *col, double *valA, double *valM, hipStream_t s,
                  const AsmScratch &w) {
    MeshInfo info;
    if (int e = mesh_lists(dim, nv, ne, elems, s, w, &info)) return e;
    if (info.total != nnz) return AMG_ERR_ARG;  // the caller's arrays do not fit this pattern
    return fill_rows(dim, nv, coords, elems, kappa, rowptr, col, valA, valM, s, w, info);
}

// ---- the allocation-free variant ----
// Its workspace is this file-scope device array: every device that runs the
// call holds one copy until the process ends, and every call on a device
// reuses that device's copy (so calls that overlap on one device race).
constexpr size_t kNoAllocBytes = size_t(32) << 20;
__device__ __align__(256) unsigned char scratch[kNoAllocBytes];

// The array's device address, looked up once per device with that device
// current; host code uses these addresses, never the array's name (which on
// the host is only a stand-in symbol).
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

int scratch_of_current_device(void **out) {
    int dev = -1;
    ASM_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return AMG_ERR_ARG;
    std::lock_guard<std::mutex> g(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        ASM_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return AMG_ERR_HIP;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return AMG_OK;
}

bool valid_args(int dim, int32_t nv, int32_t ne, const int32_t *elems) {
    return (dim == 2 || dim == 3) && nv > 0 && ne > 0 && elems && (long)ne * (dim + 1) <= INT_MAX;
}

}  // namespace
}  // namespace amg

// a mesh's lists, kept between the size query and the fill
struct amg_p1_plan {
    int dim = 0;
    int32_t nv = 0;
    amg::PoolBlock blk;
    amg::AsmScratch w;
    amg::MeshInfo info;
};

extern "C" int amg_p1_plan_device(int dim, int32_t nv, int32_t ne, const int32_t *elems, int32_t *nnz, void *stream,
                                  amg_p1_plan **plan) {
    using namespace amg;
    if (!plan) return AMG_ERR_ARG;
    *plan = nullptr;
    if (!nnz || !valid_args(dim, nv, ne, elems)) return AMG_ERR_ARG;
    amg_p1_plan *p = new (std::nothrow) amg_p1_plan;
    if (!p) return AMG_ERR_OOM;
    p->dim = dim;
    p->nv = nv;
    int e = p->blk.get(scratch_bytes(dim, nv, ne), (hipStream_t)stream);
    if (!e) {
        p->w = carve(p->blk.p, dim, nv, ne);
        e = mesh_lists(dim, nv, ne, elems, p->blk.s, p->w, &p->info);
    }
    if (e) {
        delete p;
        return e;
    }
    *nnz = p->info.total;
    *plan = p;
    return AMG_OK;
}

extern "C" int amg_p1_assemble_planned(amg_p1_plan *plan, const double *coords, const int32_t *elems,
                                       const double *kappa, int32_t *rowptr, int32_t *col, double *valA,
                                       double *valM) {
    using namespace amg;
    if (!plan || !coords || !elems || !kappa || !rowptr || !col || !valA || !valM) return AMG_ERR_ARG;
    return fill_rows(plan->dim, plan->nv, coords, elems, kappa, rowptr, col, valA, valM, plan->blk.s, plan->w,
                     plan->info);
}

extern "C" int amg_p1_plan_destroy(amg_p1_plan *plan) {
    delete plan;
    return AMG_OK;
}

extern "C" int amg_p1_pattern_device(int dim, int32_t nv, int32_t ne, const int32_t *elems, int32_t *nnz,
                                     void *stream) {
    using namespace amg;
    if (!nnz || !valid_args(dim, nv, ne, elems)) return AMG_ERR_ARG;
    const hipStream_t s = (hipStream_t)stream;
    PoolBlock blk;
    if (int e = blk.get(scratch_bytes(dim, nv, ne), s)) return e;
    MeshInfo info;
    if (int e = mesh_lists(dim, nv, ne, elems, s, carve(blk.p, dim, nv, ne), &info)) return e;
    *nnz = info.total;
    return AMG_OK;
}

extern "C" int amg_p1_assemble_device(int dim, int32_t nv, const double *coords, int32_t ne, const int32_t *elems,
                                      const double *kappa, int32_t nnz, int32_t *rowptr, int32_t *col,
                                      double *valA, double *valM, void *stream) {
    using namespace amg;
    if (!coords || !kappa || !rowptr || !col || !valA || !valM || !valid_args(dim, nv, ne, elems))
        return AMG_ERR_ARG;
    const hipStream_t s = (hipStream_t)stream;
    PoolBlock blk;
    if (int e = blk.get(scratch_bytes(dim, nv, ne), s)) return e;
    return assemble_into(dim, nv, coords, ne, elems, kappa, nnz, rowptr, col, valA, valM, s,
                         carve(blk.p, dim, nv, ne));
}

extern "C" int amg_p1_assemble_device_noalloc(int dim, int32_t nv, const double *coords, int32_t ne,
                                              const int32_t *elems, const double *kappa, int32_t nnz,
                                              int32_t *rowptr, int32_t *col, double *valA, double *valM,
                                              void *stream) {
    using namespace amg;
    if (!coords || !kappa || !rowptr || !col || !valA || !valM || !valid_args(dim, nv, ne, elems))
        return AMG_ERR_ARG;
    if (scratch_bytes(dim, nv, ne) > kNoAllocBytes) return AMG_ERR_ARG;  // beyond the static workspace
    void *base = nullptr;
    if (int e = scratch_of_current_device(&base)) return e;
    return assemble_into(dim, nv, coords, ne, elems, kappa, nnz, rowptr, col, valA, valM, (hipStream_t)stream,
                         carve(base, dim, nv, ne));
}
