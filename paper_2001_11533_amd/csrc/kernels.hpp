// Solve-phase device code for gfx950: row-blocked CSR SpMV/SpMM with fused
// epilogues, elementwise kernels with fused dot products, deterministic
// two-stage grid reductions, and the dense coarse-level apply.
//
// Layout: every work vector is row-major [n x NB] (entry (i, c) at i*NB + c),
// NB in {1, 2, 4, 8, 16}.  A row of a CSR matrix is handled by LPR = G NG
// consecutive lanes of one wavefront: NG = NB / CV groups of CV columns (CV = 1,
// 2 or 4 columns per lane, read as one contiguous piece), times G lanes that take
// the stored entries g, g + G, ... of the row; the G partial sums are combined
// across the lanes.  Every (column, value) entry is fetched once per row and
// column group for CV right-hand sides.
//
// Reductions are deterministic: each workgroup reduces its contribution in a
// fixed tree and writes one partial per (quantity, column); a one-workgroup
// kernel launched next (or the prologue of the next kernel that needs the
// result) sums the partials in a fixed order and runs a small "finalize" step, a
// thread per column (CG scalars, convergence flags).  Issuing a
// device-scope fence per workgroup instead (a "last workgroup" ticket) makes
// every workgroup write back its XCD's L2 and costs far more than the launch.
#pragma once

#include <type_traits>

#include "common.hpp"

namespace amg {

// ---------------------------------------------------------------------------
// per-column CG state kept in device memory
struct ColScal {
    double rho, alpha, beta, bb, tol2, rr, pq, rz;
    double rho_next;  // fused finalize: r.z of the latest residual, committed to rho by the update
    int conv, iters, bad, pad;
};

// What the host needs to steer a CG, written by the finalize kernels into
// pinned host memory (read after an event, no copy kernels).
struct Mail {
    int all_conv;
    int bad;
    int iters;       // largest iteration count over the columns
    int indefinite;
    int nlive;       // refinement: columns still refining
    int stagnated;
    int pad[2];
};

struct CgScal {
    ColScal s[16];
    int all_conv;
    int nb;          // live columns; columns >= nb are padding and stay frozen
    int indefinite;  // outer CG: p.q <= 0 or r.z <= 0 met on a live column
    int pad;
    Mail *mail;      // host-mapped mailbox of this CG
    void *xptr;      // where the CG accumulates its solution (set at start)
};

__device__ __forceinline__ void publish(CgScal *sc, int NBc) {
    int all = 1, bad = 0, it = 0;
    for (int c = 0; c < NBc; ++c) {
        all &= sc->s[c].conv;
        bad |= sc->s[c].bad;
        it = max(it, sc->s[c].iters);
    }
    sc->all_conv = all;
    Mail *m = sc->mail;
    m->iters = it;
    m->bad = bad;
    m->indefinite = sc->indefinite;
    m->all_conv = all;
}

// A workgroup's share of n units of work (slices, row blocks, blocks of
// elements): first, first + step, .. below end.  Workgroups are dispatched
// round-robin over the XCDs, whose L2s are separate; each XCD gets a contiguous
// run of units, so neighbouring rows share an L2, and when a launch has fewer
// workgroups than units its workgroups sweep that run side by side: what one
// gathers from its neighbours' rows is then at most a few steps old.  (A run of
// units per workgroup, taken before, spread an XCD over 128 places at once and
// fetched a gathered vector once per neighbour plane and line.)  The counts
// come from the host: dividing by the rows of a block took the kernel's first
// hundred cycles.  rot shifts the runs by rot XCDs.
struct Units {
    int n, run, step;  // units, units per XCD, workgroups per XCD
};
inline Units units(int n, int grid) { return {n, ceil_div(n, kXcd), grid / kXcd}; }
struct Share {
    int first, end, step;
};
__device__ __forceinline__ Share xcd_share(int n, int run, int step, int rot = 0) {
    const int x = (int)((blockIdx.x + (unsigned)rot) % kXcd);
    return {x * run + (int)(blockIdx.x / kXcd), min(n, (x + 1) * run), step};
}

// Small launches spend their time in a chain of waits (about 0.6 us each on a
// first touch): kernel arguments, stop flag, row pointers, entries, gathers.
// Scalar arguments therefore come first in every solve kernel, where the
// hardware preloads them into registers, and these helpers keep loads that
// need nothing but the arguments ahead of the test of the stop flag, so that
// the waits overlap: the compiler would otherwise move them behind the branch.
// pin: the loads of these values are issued, and waited for, here.
__device__ __forceinline__ void pin_s(int a, int b = 0, int c = 0, int d = 0) { asm volatile("" ::"s"(a), "s"(b), "s"(c), "s"(d)); }
template <class V> __device__ __forceinline__ void pin_v(V a, V b) { asm volatile("" ::"v"(a), "v"(b)); }
// the same for a functor's pointers and scalars
template <class F> __device__ __forceinline__ void pin_args(const F &f) {
    if constexpr (sizeof(F) % 8 == 0) {
        const unsigned long long *w = reinterpret_cast<const unsigned long long *>(&f);
#pragma unroll
        for (size_t i = 0; i < sizeof(F) / 8; ++i) asm volatile("" ::"s"(w[i]));
    }
}

// ---------------------------------------------------------------------------
// x plus its value OFF lanes away (lane index xor OFF), for OFF = NG, 2 NG, ..
// in ascending order: the sum over the lanes of a wavefront that agree modulo
// NG, left in all of them.  Within 16 lanes by DPP, across them by gfx950's
// row swaps; a shuffle through LDS per step costs about a hundred cycles.
// The mirrors stand in for xor 4 (NG = 1 only) once the lanes of a quad agree.
template <int CTRL> __device__ __forceinline__ int dpp_i(int x) {
    return __builtin_amdgcn_update_dpp(x, x, CTRL, 0xf, 0xf, false);
}
template <int OFF, int NG> __device__ __forceinline__ void lane_pair(int x, int &a, int &b) {
    a = x;
    if constexpr (OFF == 1) b = dpp_i<0xB1>(x);                      // quad_perm 1 0 3 2
    else if constexpr (OFF == 2) b = dpp_i<0x4E>(x);                 // quad_perm 2 3 0 1
    else if constexpr (OFF == 4 && NG == 1) b = dpp_i<0x141>(x);     // row_half_mirror
    else if constexpr (OFF == 4) b = __builtin_amdgcn_ds_swizzle(x, (4 << 10) | 0x1f);
    else if constexpr (OFF == 8) b = dpp_i<0x128>(x);                // row_ror 8
    else if constexpr (OFF == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        a = (int)r[0];
        b = (int)r[1];
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        a = (int)r[0];
        b = (int)r[1];
    }
}
template <int OFF, int NG> __device__ __forceinline__ float lane_add(float x) {
    int a, b;
    lane_pair<OFF, NG>(__float_as_int(x), a, b);
    return __int_as_float(a) + __int_as_float(b);
}
template <int OFF, int NG> __device__ __forceinline__ double lane_add(double x) {
    int al, bl, ah, bh;
    lane_pair<OFF, NG>(__double2loint(x), al, bl);
    lane_pair<OFF, NG>(__double2hiint(x), ah, bh);
    return __hiloint2double(ah, al) + __hiloint2double(bh, bl);
}
// over the lanes of groups of LIM (a power of two, the same for the wavefront)
template <int NG, typename T, int OFF = NG> __device__ __forceinline__ T group_add(T x, int lim) {
    if constexpr (OFF < 64) {
        if (OFF < lim) x = group_add<NG, T, 2 * OFF>(lane_add<OFF, NG>(x), lim);
    }
    return x;
}

// Columns per lane: a lane serves CV consecutive columns of the batch, so its
// gathers and stores are CV contiguous values.
template <int NB> constexpr int spmv_cv() { return NB >= 4 ? 4 : NB; }

// Lanes per row: NB / CV column groups x G lanes per (row, group), G a power
// of two chosen per matrix from its mean row length; LPR = (NB / CV) G <= 64.
struct Geo {
    int lg;   // log2 G
    int llpr; // log2 LPR
    __host__ __device__ int lpr() const { return 1 << llpr; }
    __host__ __device__ int rpb() const { return kBlock >> llpr; }
};

__host__ __device__ constexpr int ilog2(int x) {
    int l = 0;
    while ((1 << (l + 1)) <= x) ++l;
    return l;
}

// entries a lane loads together, and in large matrices of long rows (mid: whose
// rows leave the slots of eight half empty)
constexpr int kSpmvUnroll = 4, kSpmvUnrollMid = 6, kSpmvUnrollLong = 8;

// Whether a one-column product on a coarse matrix takes kSpmvUnrollLong entries
// per lane: rows of more than 16 entries, 10 MB or more of entries.  Such a
// launch is several rounds of wavefronts per CU, each round as long as its
// loads' latency, so twice the entries per lane halve the rounds (184344 rows
// of 46 entries in FP64: 34.2 -> 25.4 us; of 33 in float32: 15.1 -> 12.2 us);
// a smaller one is a single round that more lanes shorten (22748 rows of 32 in
// float32: 3.5 us, 3.8 us with eight entries).
template <int NB, typename T> inline bool long_rows(const DCsr &A) {
    return NB == 1 && A.nnz > 16L * A.n && (4.0 + sizeof(T)) * (double)A.nnz >= 1e7;
}

// Every slot of a round costs its loads whether a row fills it or not, and these
// launches are bound by the loads they issue: rows of at most 4.5 G entries, which
// a round of six per lane still takes nearly all of, take six (184344 rows of 33,
// G = 8: 12.7 -> 11.8 us in float32, 21.0 -> 19.2 us in FP64), longer ones eight
// (rows of 46: 22.0 us, 27.0 with six; 38: 19.4 us, 20.5 with six).
template <typename M> inline bool mid_rows(const M &A, int lg) { return 2L * A.nnz <= 9L * A.n << lg; }

// The fixed rule for G, from the mean row length m (measured over G = 1 .. 64 on
// every product of 2D and 3D hierarchies of 7e4 to 2.1e6 rows, 1 to 16 columns):
//   one or two columns: enough lanes that a row takes one round of U loads,
//     G = next power of two >= m / U; the float32 pass over T with U < m <= 2 U
//     takes one step more (its rows spread up to twice the mean: 65 -> 41 us at
//     2.1e6 rows, 10.7 -> 7.0 us at 2.7e5);
//   more columns: a lane's U loads are already CV columns each, so a lane serves
//     more entries, up to 6 (NB = 4), 8 (NB = 8) or 14 (NB = 16) of a row, but a
//     row of more than U entries gets two lanes up to NB = 8 (16 columns at
//     184344 rows of 33 entries: 33.6 us with G = 4, 39.2 us with m / U; the pass
//     over T at 2.1e6 rows: 252 us with G = 1, 266 with 2, 313 with 4); and small
//     matrices widen G, up to m / 2, until the launch has 2^17 lanes (16 columns
//     at 1742 rows of 94 entries: 3.5 us with G = 16, 5.3 us with 4).
template <int NB> inline Geo make_geo(long nnz, long rows, bool t32 = false, bool lrows = false) {
    constexpr int NG = NB / spmv_cv<NB>();
    const double m = rows > 0 ? (double)nnz / (double)rows : 1.0;
    constexpr double per = NB <= 2 ? kSpmvUnroll : NB == 4 ? 6.0 : NB == 8 ? 8.0 : 14.0;
    int g = 1;
    while (g < 64 && g < m / (lrows ? kSpmvUnrollLong : per)) g <<= 1;
    if (NB <= 8 && m > kSpmvUnroll) g = std::max(g, 2);
    if (NB <= 4 && t32 && m > kSpmvUnroll && m <= 2 * kSpmvUnroll) g = 4;
    if constexpr (NB > 2)
        while (rows * NG * g < (1L << 17) && 4 * g <= m) g <<= 1;
    while (g * NG > 64) g >>= 1;
    Geo geo;
    geo.lg = ilog2(g);
    geo.llpr = ilog2(g * NG);
    return geo;
}

// the geometry with G = 2^lg lanes per (row, column group)
template <int NB> __host__ __device__ inline Geo geo_from_lg(int lg) {
    Geo geo;
    geo.lg = lg;
    geo.llpr = lg + ilog2(NB / spmv_cv<NB>());
    return geo;
}

// largest log2 G a product on NB columns can take (LPR <= 64)
template <int NB> constexpr int max_lg() { return NB >= 4 ? 6 - (NB == 4 ? 0 : NB == 8 ? 1 : 2) : 6; }

// the autotuner's choice for this matrix, batch width and value type, else the
// default rule (fine: a matrix of the finest level; is_t: the fused pass over T = A S)
template <int NB, typename T> inline Geo geo_for(const DCsr &A, int fine, bool is_t = false) {
    constexpr bool f32 = std::is_same_v<T, float>;
    const int t = A.tuned_lg[ilog2(NB)][f32 ? 1 : 0];
    return t >= 0 ? geo_from_lg<NB>(t) : make_geo<NB>(A.nnz, A.n, is_t && f32, !is_t && fine == 0 && long_rows<NB, T>(A));
}

template <int NV, int NB> struct Reducer {
    double *partial;    // [NV*NB][gridDim.x]
};

constexpr int pow2floor(int x) {
    int p = 1;
    while (p * 2 <= x) p *= 2;
    return p;
}

// Block reduction of acc over the threads that serve the same columns: thread
// t serves column group t % NG (NG = NB / CV groups of CV consecutive columns;
// slot v of acc is column (t % NG) CV + v).  Each wavefront folds its lanes of
// one group by shuffles (xor offsets NG, 2 NG, .., 32), the wavefronts' sums are
// added in order through LDS, and thread t < NV NB writes partial (t / NB,
// t % NB) of this workgroup.  The totals are formed by fin_kernel, launched next
// on the same stream (a kernel boundary orders the partials; no device-scope
// fence is issued by the workgroups).
template <int NV, int NB, int CV>
__device__ void block_partials_cv(const double (&acc)[CV][NV], Reducer<NV, NB> r) {
    constexpr int NG = NB / CV, WV = kBlock / 64;
    __shared__ double wred[WV][NV][NB];
    const int t = threadIdx.x, lane = t & 63;
#pragma unroll
    for (int v = 0; v < CV; ++v)
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const double x = group_add<NG>(acc[v][q], 64);
            if (lane < NG) wred[t >> 6][q][lane * CV + v] = x;
        }
    __syncthreads();
    if (t < NV * NB) {
        double x = 0.0;
#pragma unroll
        for (int w = 0; w < WV; ++w) x += wred[w][t / NB][t % NB];
        r.partial[(size_t)t * gridDim.x + blockIdx.x] = x;
    }
}

template <int NV, int NB>
__device__ void block_partials(const double (&acc)[NV], Reducer<NV, NB> r) {
    const double(&a1)[1][NV] = *reinterpret_cast<const double(*)[1][NV]>(&acc);
    block_partials_cv<NV, NB, 1>(a1, r);
}

// Sums the partials of Q quantities in a fixed order with all BS threads of
// the workgroup: quantity q's partials are src(q, &ptr, &count).  LPS threads
// (a power of two) serve a quantity: each keeps eight running sums over the
// partials it strides through (eight loads in flight), then the LPS sums are
// folded by wavefront shuffles and, for LPS > 64, across the quantity's
// wavefronts through LDS.  The order depends only on the counts, so every
// workgroup that sums the same partials gets the same totals.  out (LDS,
// [Q]) holds the totals for every thread on return.
// between() runs behind the first round of loads.
struct NoBetween {
    __device__ void operator()() const {}
};
template <int Q, int BS, class SRC, class BTW = NoBetween>
__device__ void sum_quantities(SRC src, double *out, BTW between = BTW{}) {
    constexpr int LPS = pow2floor(BS / Q);
    constexpr int W = LPS < 64 ? LPS : 64;
    __shared__ double wsum[BS / 64];
    const int t = threadIdx.x;
    const int q = t / LPS, sub = t % LPS;
    double s = 0.0;
    if (q < Q) {
        const double *pp;
        int nblk;
        src(q, pp, nblk);
        // the first round: up to eight per lane, unconditional loads (clamped
        // index) added only where valid, so all are in flight together
        double a[8];
        {
            const int last = nblk > 0 ? nblk - 1 : 0;
            double v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = pp[min(sub + k * LPS, last)];
            between();
#pragma unroll
            for (int k = 0; k < 8; ++k) a[k] = sub + k * LPS < nblk ? v[k] : 0.0;
        }
        int b = sub + 8 * LPS;
        for (; b + 7 * LPS < nblk; b += 8 * LPS) {
            double v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = pp[b + k * LPS];
#pragma unroll
            for (int k = 0; k < 8; ++k) a[k] += v[k];
        }
        // at most seven left
        if (b < nblk) {
            double v[7];
#pragma unroll
            for (int k = 0; k < 7; ++k) v[k] = pp[min(b + k * LPS, nblk - 1)];
#pragma unroll
            for (int k = 0; k < 7; ++k) a[k] = b + k * LPS < nblk ? a[k] + v[k] : a[k];
        }
        s = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
    } else {
        between();
    }
    s = group_add<1>(s, W);
    if constexpr (LPS > 64) {
        if ((t & 63) == 0) wsum[t >> 6] = s;
        __syncthreads();
        if (sub == 0 && q < Q) {
            double v = 0.0;
#pragma unroll
            for (int w = 0; w < LPS / 64; ++w) v += wsum[(t >> 6) + w];
            out[q] = v;
        }
    } else {
        if (sub == 0 && q < Q) out[q] = s;
    }
    __syncthreads();
}

// The partials of NV quantities x NB columns, quantity-major ([NV*NB][nblk]).
template <int NV, int NB, int BS = kBlock, class BTW = NoBetween>
__device__ void sum_partials(const double *__restrict__ partial, int nblk, double (&tot)[NV][NB], BTW between = BTW{}) {
    sum_quantities<NV * NB, BS>(
        [&](int q, const double *&pp, int &n) {
            pp = partial + (size_t)q * nblk;
            n = nblk;
        },
        &tot[0][0], between);
}

// Two buffers of one quantity x NB columns each, summed together.
template <int NB, int BS = kBlock>
__device__ void sum_partials2(const double *__restrict__ pa, int na, const double *__restrict__ pb, int nb,
                              double (&ta)[1][NB], double (&tb)[1][NB]) {
    __shared__ double both[2 * NB];
    sum_quantities<2 * NB, BS>(
        [&](int q, const double *&pp, int &n) {
            if (q < NB) {
                pp = pa + (size_t)q * na;
                n = na;
            } else {
                pp = pb + (size_t)(q - NB) * nb;
                n = nb;
            }
        },
        both);
    if (threadIdx.x < NB) {
        ta[0][threadIdx.x] = both[threadIdx.x];
        tb[0][threadIdx.x] = both[NB + threadIdx.x];
    }
    __syncthreads();
}

// Convergence test and beta of one CG column after an update (r.r = rr) and
// the preconditioner (r.z = rz): the step of the finalize kernels, shared by
// the fused form below.  Returns the new beta (0 when the column stops).
__device__ __forceinline__ double cg_col_step(const ColScal &s, double rr, double rz, int &conv, int &bad) {
    conv = s.conv;
    bad = s.bad;
    if (conv) return 0.0;
    if (bad || rr <= s.tol2) {
        conv = 1;
        return 0.0;
    }
    if (!(rz > 0.0)) {
        bad = 1;
        conv = 1;
        return 0.0;
    }
    return rz / s.rho;
}

// The finalize of a captured CG iteration folded into the first kernel of the
// next one: every workgroup sums the partials of r.r (buffer p1, quantity 0)
// and r.z (Jacobi: p1, quantity 1; else buffer p2) in the same fixed order,
// so all reach the same beta and convergence decisions; workgroup 0 records
// them (rho_next = r.z, committed to rho by the update kernel that follows,
// so no workgroup here reads a value another one writes, conv and bad only
// ever switch on), counts the iteration and publishes the mailbox.
struct NoPro {
    static constexpr bool active = false;
};

template <int NB, bool JAC> struct FusedFin {
    static constexpr bool active = true;
    CgScal *sc;
    const double *p1;
    int n1;
    const double *p2;
    int n2;
};

// Returns whether every column has stopped; beta[c] (in LDS) holds the new betas.
template <int NB, bool JAC>
__device__ bool fused_fin(const FusedFin<NB, JAC> &f, const double *&beta) {
    __shared__ double t1[JAC ? 2 : 1][NB], t2[1][NB];
    __shared__ double sb[NB];
    __shared__ int sconv[NB];
    const int t = threadIdx.x;
    // the column scalars the step reads, thread c column c, loaded before the
    // partial sums so that both loads are in flight together (nothing written in
    // this kernel changes what the step decides from them: see above)
    ColScal pre;  // conv, bad, tol2 and rho only
    if (t < NB) {
        pre.conv = f.sc->s[t].conv;
        pre.bad = f.sc->s[t].bad;
        pre.tol2 = f.sc->s[t].tol2;
        pre.rho = f.sc->s[t].rho;
    }
    if constexpr (JAC) sum_partials<2, NB>(f.p1, f.n1, t1);
    else sum_partials2<NB>(f.p1, f.n1, f.p2, f.n2, t1, t2);
    if (t < NB) {
        ColScal &s = f.sc->s[t];
        const double rr = t1[0][t], rz = JAC ? t1[1][t] : t2[0][t];
        int conv, bad;
        const double b = cg_col_step(pre, rr, rz, conv, bad);
        if (blockIdx.x == 0 && !pre.conv) {
            s.iters += 1;
            s.rr = rr;
            s.rz = rz;
            s.beta = b;
            s.rho_next = rz;
            s.bad = bad;
            s.conv = conv;
        }
        sb[t] = b;
        sconv[t] = conv;
    }
    __syncthreads();
    if (blockIdx.x == 0 && t == 0) publish(f.sc, NB);
    int all = 1;
#pragma unroll
    for (int c = 0; c < NB; ++c) all &= sconv[c];
    beta = sb;
    return all != 0;
}

// The same step as a finalize kernel (after the last update a CG is allowed).
template <int NB, bool JAC> struct FinFusedTail {
    CgScal *sc;
    __device__ void head() const {}
    __device__ void col(int c, double rr, double rz) const {
        ColScal &s = sc->s[c];
        if (s.conv) return;
        int conv, bad;
        const double b = cg_col_step(s, rr, rz, conv, bad);
        s.iters += 1;
        s.rr = rr;
        s.rz = rz;
        s.beta = b;
        s.rho_next = rz;
        s.bad = bad;
        s.conv = conv;
    }
};

// Finalize functors that keep their CG's scalars in a member sc (CgScal *) have
// a step per column, col(c, totals of column c ..), and a head() for what
// belongs to the CG.  They run on a copy of the scalars in LDS, loaded at once
// and written back after the step, column c on thread c (thread 0 looping over
// the columns: 7.8 us per finalize of 16 columns and one quantity, 4.9 us so).
template <class F, class = void> struct fin_has_sc : std::false_type {};
template <class F>
struct fin_has_sc<F, std::void_t<decltype(std::declval<F &>().sc)>>
    : std::is_same<decltype(std::declval<F &>().sc), CgScal *> {};

constexpr int kScWords = (int)(sizeof(CgScal) / sizeof(unsigned long long));
static_assert(sizeof(CgScal) % sizeof(unsigned long long) == 0, "CgScal is copied in 8-byte words");

__device__ __forceinline__ unsigned long long sc_stage_load(const CgScal *sc) {
    const int t = threadIdx.x;
    return t < kScWords ? reinterpret_cast<const unsigned long long *>(sc)[t] : 0ull;
}

// the step on the LDS copy (loaded by sc_stage_load before the partial sums,
// so both loads are in flight together), then the copy back
template <int NB, class FIN, class STEP>
__device__ __forceinline__ void fin_staged(const FIN &fin, unsigned long long w, STEP step) {
    __shared__ CgScal lsc;
    const int t = threadIdx.x;
    if (t < kScWords) reinterpret_cast<unsigned long long *>(&lsc)[t] = w;
    __syncthreads();
    if (t < NB) {
        FIN f = fin;
        f.sc = &lsc;
        if (t == 0) f.head();
        step(f, t);
    }
    __syncthreads();
    if (t == 0) publish(&lsc, NB);
    __syncthreads();
    if (t < kScWords) reinterpret_cast<unsigned long long *>(fin.sc)[t] = reinterpret_cast<unsigned long long *>(&lsc)[t];
}

// One workgroup: totals of the partials, then the finalize step.
template <int NV, int NB, class FIN>
__global__ __launch_bounds__(kFinBlock) void fin_kernel(const double *__restrict__ partial, int nblk, FIN fin,
                                                        const int *__restrict__ stop) {
    __shared__ double tot[NV][NB];
    const int st = stop ? *stop : 0;  // tested after the sums, whose loads it does not hold up
    if constexpr (fin_has_sc<FIN>::value) {
        const unsigned long long w = sc_stage_load(fin.sc);
        sum_partials<NV, NB, kFinBlock>(partial, nblk, tot);
        if (st) return;
        fin_staged<NB>(fin, w, [&](const FIN &f, int c) {
            if constexpr (NV == 1) f.col(c, tot[0][c]);
            else f.col(c, tot[0][c], tot[1][c]);
        });
    } else {
        sum_partials<NV, NB, kFinBlock>(partial, nblk, tot);
        if (!st && threadIdx.x == 0) fin(tot);
    }
}

// The same with two partial buffers (one quantity each).
template <int NB, class FIN>
__global__ __launch_bounds__(kFinBlock) void fin2_kernel(const double *__restrict__ pa, int na,
                                                         const double *__restrict__ pb, int nb, FIN fin,
                                                         const int *__restrict__ stop) {
    __shared__ double ta[1][NB], tb[1][NB];
    const int st = stop ? *stop : 0;
    const unsigned long long w = sc_stage_load(fin.sc);
    sum_partials2<NB, kFinBlock>(pa, na, pb, nb, ta, tb);
    if (st) return;
    fin_staged<NB>(fin, w, [&](const FIN &f, int c) { f.col(c, ta[0][c], tb[0][c]); });
}

struct NoFin {
    template <int NV, int NB> __device__ void operator()(double (&)[NV][NB]) const {}
};

// ---------------------------------------------------------------------------
// CSR SpMV / SpMM with a gather functor (how x_k is formed) and an epilogue
// functor (what is written for row i); optional fused reductions.
// FINE = 1 marks launches on the finest level (a separate instantiation, so that
// profiles separate the fine-level kernels from the coarse-level ones).  CI =
// int16_t: columns relative to row_base (DCsr::c16), for the large coarse matrices
// (long_rows), whose products move little but their entries: 184344 rows of 46 in
// FP64 22.9 -> 22.0 us, of 33 in float32 12.2 -> 11.8 us.
template <typename T, int NB, int NV, class GX, class EP, int FINE, class PRO = NoPro, int U = kSpmvUnroll,
          typename CI = int>
__global__ __launch_bounds__(kBlock) void spmv_kernel(const int *__restrict__ stop, int un, int urun, int ustep,
                                                      int nrows, int lg, const int *__restrict__ rp,
                                                      const CI *__restrict__ ci, const T *__restrict__ av, GX gx,
                                                      EP ep, Reducer<(NV > 0 ? NV : 1), NB> red, PRO pro,
                                                      uint32_t scale) {
    constexpr int CV = spmv_cv<NB>(), NG = NB / CV;
    const Geo geo = geo_from_lg<NB>(lg);
    const int t = threadIdx.x;
    const int LPR = geo.lpr(), G = 1 << geo.lg;
    const int lane = t & (LPR - 1), c0 = (lane % NG) * CV, g = lane / NG, rl = t >> geo.llpr;
    const Share sh = xcd_share(un, urun, ustep);
    // the first block's row pointers beside the stop flag (a fused finalize
    // stops by itself)
    int row = sh.first * geo.rpb() + rl;
    int p0 = rp[min(row, nrows - 1)], p1 = rp[min(row, nrows - 1) + 1];
    if constexpr (!PRO::active) {
        const int st = *stop;
        pin_s(st);
        pin_args(gx);
        pin_args(ep);
        pin_v(p0, p1);
        if (st) return;
    }
    GX gxv[CV];
    EP epv[CV];
#pragma unroll
    for (int v = 0; v < CV; ++v) {
        gxv[v] = gx;
        gxv[v].prep(c0 + v);
        epv[v] = ep;
        epv[v].prep(c0 + v);
    }
    if constexpr (PRO::active) {  // the previous iteration's finalize, then this one
        const double *fb;
        if (fused_fin(pro, fb)) return;
#pragma unroll
        for (int v = 0; v < CV; ++v) {
            gxv[v].set_beta(fb[c0 + v]);
            epv[v].set_beta(fb[c0 + v]);
        }
    }
    constexpr int NVA = NV > 0 ? NV : 1;
    double acc[CV][NVA];
#pragma unroll
    for (int v = 0; v < CV; ++v)
#pragma unroll
        for (int q = 0; q < NVA; ++q) acc[v][q] = 0.0;
    for (int blk = sh.first; blk < sh.end; blk += sh.step) {
        const bool live = row < nrows;
        typename EP::P pr[CV];
        if (live && g == 0) {
#pragma unroll
            for (int v = 0; v < CV; ++v) pr[v] = epv[v].load(row, c0 + v);
        }
        T sum[CV];
#pragma unroll
        for (int v = 0; v < CV; ++v) sum[v] = T(0);
        // the next block's row pointers arrive while this one's entries do
        const int nrow = (blk + sh.step) * geo.rpb() + rl, nr = min(nrow, nrows - 1);
        const int n0 = rp[nr], n1 = rp[nr + 1];
        int kb = 0;
        if constexpr (!std::is_same_v<CI, int>) kb = row_base(row, scale);
        if (live) {
            for (int p = p0 + g; p < p1; p += U * G) {
                // unconditional loads (past the row's end: its last entry,
                // weighted by 0), so all U loads and gathers are in flight together
                int kk[U];
                T aa[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int q = p + u * G;
                    const int qc = min(q, p1 - 1);
                    kk[u] = kb + (int)ci[qc];
                    const T a = av[qc];
                    aa[u] = q < p1 ? a : T(0);
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
#pragma unroll
                    for (int v = 0; v < CV; ++v) sum[v] += aa[u] * gxv[v](kk[u], c0 + v);
                }
            }
        }
#pragma unroll
        for (int v = 0; v < CV; ++v) sum[v] = group_add<NG>(sum[v], LPR);
        if (live && g == 0) {
#pragma unroll
            for (int v = 0; v < CV; ++v) epv[v](row, c0 + v, sum[v], pr[v], acc[v]);
        }
        row = nrow;
        p0 = n0;
        p1 = n1;
    }
    if constexpr (NV > 0) block_partials_cv<NV, NB, CV>(acc, red);
}

// The same product over the sliced-ELL copy: NG lanes per row, CV columns each
// (one column: a wavefront per slice of 64 rows, a lane per row; 16 columns: a
// workgroup per slice).  A lane issues the loads of up to U entries of its row
// at once, with no dependence on row pointers, then their gathers.  U is 8 when
// no slice is wider (5- and 7-point rows) and for a batch, whose gathers are CV
// values each; one column takes wider rows in one round of 16.  Columns are
// 16-bit offsets from the slice's base column (6 bytes per float32 entry).
// xrot rotates the XCD-contiguous block ranges by xrot XCDs (0 in solves).
template <int NB> constexpr int sell_slices() { return kBlock / (NB / spmv_cv<NB>()) / 64; }  // per workgroup

template <typename T, int NB, int NV, class GX, class EP, class PRO = NoPro, int U = 16>
__global__ __launch_bounds__(kBlock) void sell_kernel(const int *__restrict__ stop, int un, int urun, int ustep,
                                                      int nrows, int nsl, const int *__restrict__ soff,
                                                      const int *__restrict__ sbase,
                                                      const uint16_t *__restrict__ cd, const T *__restrict__ av, GX gx,
                                                      EP ep, Reducer<(NV > 0 ? NV : 1), NB> red, PRO pro = PRO{},
                                                      int xrot = 0) {
    constexpr int CV = spmv_cv<NB>(), NG = NB / CV, SPB = sell_slices<NB>();
    const int c0 = (threadIdx.x % NG) * CV, rl = threadIdx.x / NG, lane = rl & 63;
    const Share sh = xcd_share(un, urun, ustep, xrot);
    // one slice per wavefront; the first one's place beside the stop flag
    const int wsl = __builtin_amdgcn_readfirstlane(rl >> 6);
    int sl = sh.first * SPB + wsl;
    int o = soff[min(sl, nsl - 1)], oe = soff[min(sl, nsl - 1) + 1], cb = sbase[min(sl, nsl - 1)];
    if constexpr (!PRO::active) {
        const int st = *stop;
        pin_s(st, o, oe, cb);
        pin_args(gx);
        pin_args(ep);
        if (st) return;
    }
    GX gxv[CV];
    EP epv[CV];
#pragma unroll
    for (int v = 0; v < CV; ++v) {
        gxv[v] = gx;
        gxv[v].prep(c0 + v);
        epv[v] = ep;
        epv[v].prep(c0 + v);
    }
    if constexpr (PRO::active) {  // the previous iteration's finalize, then this one
        const double *fb;
        if (fused_fin(pro, fb)) return;
#pragma unroll
        for (int v = 0; v < CV; ++v) {
            gxv[v].set_beta(fb[c0 + v]);
            epv[v].set_beta(fb[c0 + v]);
        }
    }
    constexpr int NVA = NV > 0 ? NV : 1;
    double acc[CV][NVA];
#pragma unroll
    for (int v = 0; v < CV; ++v)
#pragma unroll
        for (int q = 0; q < NVA; ++q) acc[v][q] = 0.0;
    for (int blk = sh.first; blk < sh.end; blk += sh.step) {
        if (SPB > 1 && sl >= nsl) break;
        const int row = sl * 64 + lane;
        const bool live = row < nrows;
        typename EP::P pr[CV] = {};
        if (live)
#pragma unroll
            for (int v = 0; v < CV; ++v) pr[v] = epv[v].load(row, c0 + v);
        const int w = (oe - o) >> 6;
        const int nsli = (blk + sh.step) * SPB + wsl, nx = min(nsli, nsl - 1);
        const int no = soff[nx], noe = soff[nx + 1], ncb = sbase[nx];
        T sum[CV];
#pragma unroll
        for (int v = 0; v < CV; ++v) sum[v] = T(0);
        for (int k0 = 0; k0 < w; k0 += U) {
            // Every load is unconditional (entries past the slice's width read
            // its last entry again, weighted by 0), so the U column and value
            // loads, then the U gathers, are in flight together; guarded loads
            // compile to one wait per entry.  A weight of exactly 0 leaves the
            // sum unchanged, and gathers what the row's last entry gathers.
            int kk[U];
            T aa[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const size_t q = (size_t)o + (size_t)min(k0 + u, w - 1) * 64 + lane;
                kk[u] = cb + (int)cd[q];
                const T a = av[q];
                aa[u] = k0 + u < w ? a : T(0);
            }
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int v = 0; v < CV; ++v) sum[v] += aa[u] * gxv[v](kk[u], c0 + v);
        }
        if (live)
#pragma unroll
            for (int v = 0; v < CV; ++v) epv[v](row, c0 + v, sum[v], pr[v], acc[v]);
        sl = nsli;
        o = no;
        oe = noe;
        cb = ncb;
    }
    if constexpr (NV > 0) block_partials_cv<NV, NB, CV>(acc, red);
}

// Elementwise kernel over n rows x NB columns with fused reductions.
template <int NB, int NV, class OP, int FINE>
__global__ __launch_bounds__(kBlock) void elem_kernel(int un, int urun, int ustep, int n, OP op,
                                                      Reducer<(NV > 0 ? NV : 1), NB> red) {
    const int t = threadIdx.x, c = t % NB;
    const long total = (long)n * NB;
    const Share sh = xcd_share(un, urun, ustep);
    op.prep(c);
    constexpr int NVA = NV > 0 ? NV : 1;
    double acc[NVA];
#pragma unroll
    for (int v = 0; v < NVA; ++v) acc[v] = 0.0;
    for (int blk = sh.first; blk < sh.end; blk += sh.step) {
        const long e = (long)blk * kBlock + t;
        if (e < total) op((int)(e / NB), c, acc);
    }
    if constexpr (NV > 0) block_partials<NV, NB>(acc, red);
}

// CG update: every workgroup first sums the p.q partials of the preceding
// operator kernel (same fixed order in all workgroups, so all agree on alpha),
// then x += alpha p, r -= alpha q (Jacobi: z = dinv r) on the live columns,
// with the partials of r.r (and r.z).  Workgroup 0 records alpha and flags a
// non-positive p.q (breakdown, or indefiniteness for the outer CG).  A CG whose
// columns have all stopped updates nothing (its scalars say so), so no stop
// flag is waited for; p, q and r of a thread's first element, which do not
// depend on alpha, are loaded behind the partials and beside their sums.
template <typename T, int NB, bool JAC, int FINE>
__global__ __launch_bounds__(kBlock) void cg_update_kernel(int un, int urun, int ustep, int n, int nblk_pq, int fused,
                                                           T *__restrict__ x, T *__restrict__ r,
                                                           const T *__restrict__ p, const T *__restrict__ q,
                                                           CgScal *sc, const double *__restrict__ part_pq,
                                                           T *__restrict__ z, float *__restrict__ r32,
                                                           float *__restrict__ x32, const float *__restrict__ d32,
                                                           double s0, const T *__restrict__ dinv, int outer,
                                                           Reducer<JAC ? 2 : 1, NB> red) {
    __shared__ double pq[1][NB];
    __shared__ double sh_a[NB];
    __shared__ int sh_live[NB];
    const int t = threadIdx.x;
    const long total = (long)n * NB;
    const Share sh = xcd_share(un, urun, ustep);
    // the column's scalars, loaded before the partial sums so that both loads
    // are in flight together (workgroup 0 writes only fields read here by no one)
    int conv0 = 0;
    double rho0 = 0.0;
    if (t < NB) {
        conv0 = sc->s[t].conv;
        rho0 = fused ? sc->s[t].rho_next : sc->s[t].rho;
    }
    T *xx = x ? x : static_cast<T *>(sc->xptr);
    const size_t of = std::min<size_t>((size_t)sh.first * kBlock + t, total - 1);
    T pf, qf, rf;
    auto first = [&] {
        pf = p[of];
        qf = q[of];
        rf = r[of];
    };
    if (nblk_pq > 0) sum_partials<1, NB>(part_pq, nblk_pq, pq, first);
    else first();
    if (nblk_pq == 0) {
        // alpha was formed by a finalize kernel (many partials)
        if (t < NB) {
            sh_a[t] = sc->s[t].alpha;
            sh_live[t] = !conv0;
        }
    } else if (t < NB) {
        ColScal &s = sc->s[t];
        const double v = pq[0][t];
        double a = 0.0;
        int live = !conv0;
        if (live) {
            if (v > 0.0) {
                a = rho0 / v;
            } else {
                live = 0;
                if (blockIdx.x == 0) {
                    s.bad = 1;
                    if (outer) sc->indefinite = 1;
                }
            }
        }
        sh_a[t] = a;
        sh_live[t] = live;
        if (blockIdx.x == 0 && !conv0) {
            s.alpha = a;
            s.pq = v;
            if (fused) s.rho = rho0;
        }
    }
    __syncthreads();
    const int c = t % NB;
    const T a = (T)sh_a[c];
    const int live = sh_live[c];
    double acc[JAC ? 2 : 1] = {};
    if (live) {
        for (int blk = sh.first; blk < sh.end; blk += sh.step) {
            const size_t o = (size_t)blk * kBlock + t;
            if ((long)o >= total) break;
            if (blk != sh.first) {
                pf = p[o];
                qf = q[o];
                rf = r[o];
            }
            xx[o] += a * pf;
            const T rv = rf - a * qf;
            r[o] = rv;
            acc[0] += (double)rv * (double)rv;
            if constexpr (JAC) {
                const T zz = dinv[o / NB] * rv;
                z[o] = zz;
                acc[1] += (double)rv * (double)zz;
            } else {
                // the V-cycle's first pre-sweep iterate x0 = D^{-1} r (in its precision)
                if (z) z[o] = (dinv[o / NB] * rv) * (T)s0;
                if (r32) {
                    const float rs = (float)rv;
                    r32[o] = rs;
                    if (x32) x32[o] = (d32[o / NB] * rs) * (float)s0;
                }
            }
        }
    }
    block_partials<JAC ? 2 : 1, NB>(acc, red);
}

// ---------------------------------------------------------------------------
// gathers
template <typename T, int NB> struct GPlain {  // x_k
    const T *x;
    __device__ void prep(int) {}
    __device__ T operator()(int k, int c) const { return x[(size_t)k * NB + c]; }
};

// z_k alone: the CG product formed as A z + beta q_old (ECgQR)
template <typename T, int NB, typename TZ = T> struct GZ {
    const TZ *z;
    __device__ void prep(int) {}
    __device__ void set_beta(double) {}
    __device__ T operator()(int k, int c) const { return (T)z[(size_t)k * NB + c]; }
};

// x_k = keep_k a_k + s b_k with keep_k = (mask == null || mask[k] == 0)
template <int NB> struct GLin {
    const double *a;
    const uint8_t *mask;
    const double *b;
    double s;
    __device__ void prep(int) {}
    __device__ double operator()(int k, int c) const {
        double v = a[(size_t)k * NB + c];
        if (mask && mask[k]) v = 0.0;
        if (b) v += s * b[(size_t)k * NB + c];
        return v;
    }
};

// ---------------------------------------------------------------------------
// epilogues: load(i, c) fetches the row's own operands before the entry loop
// (so their latency overlaps the gathers); operator() then writes the row.
struct NoPre {};

template <typename T, int NB> struct EStore {  // y_i = sum
    T *y;
    using P = NoPre;
    __device__ void prep(int) {}
    __device__ P load(int, int) const { return {}; }
    template <int NV> __device__ void operator()(int i, int c, T s, const P &, double (&)[NV]) const {
        y[(size_t)i * NB + c] = s;
    }
};

template <typename T, int NB> struct EAdd {  // y_i += sum
    T *y;
    struct P {
        T y0;
    };
    __device__ void prep(int) {}
    __device__ P load(int i, int c) const { return {y[(size_t)i * NB + c]}; }
    template <int NV> __device__ void operator()(int i, int c, T s, const P &pr, double (&)[NV]) const {
        y[(size_t)i * NB + c] = pr.y0 + s;
    }
};

// residual after the first pre-sweep, whose iterate x = dinv b the producer
// of b has written: r_i = b_i - (A x)_i
template <typename T, int NB> struct EResB {
    const T *b;
    T *r;
    struct P {
        T b;
    };
    __device__ void prep(int) {}
    __device__ P load(int i, int c) const { return {b[(size_t)i * NB + c]}; }
    template <int NV> __device__ void operator()(int i, int c, T s, const P &pr, double (&)[NV]) const {
        r[(size_t)i * NB + c] = pr.b - s;
    }
};

// restriction that also starts the next level's pre-smoothing: y_i = sum,
// x_i = (dinv_i sum) s0 (s0 = 1 for l1-Jacobi, 1/theta for Chebyshev)
template <typename T, int NB> struct EStoreX {
    T *y;
    const T *dinv;
    T *x;
    T s0;
    struct P {
        T d;
    };
    __device__ void prep(int) {}
    __device__ P load(int i, int) const { return {dinv[i]}; }
    template <int NV> __device__ void operator()(int i, int c, T s, const P &pr, double (&)[NV]) const {
        const size_t o = (size_t)i * NB + c;
        y[o] = s;
        x[o] = (pr.d * s) * s0;
    }
};

// Chebyshev smoothing (degree 2, l1 diagonal), second step from the first
// iterate x1 = (dinv b) / theta: out_i = x1_i + (c1 x1_i + c2 dinv_i (b_i - (A x1)_i))
template <typename T, int NB> struct EChebPre {
    const T *b;
    const T *dinv;
    const T *x1;
    T *out;
    T c1, c2;
    struct P {
        T b, d, x;
    };
    __device__ void prep(int) {}
    __device__ P load(int i, int c) const {
        const size_t o = (size_t)i * NB + c;
        return {b[o], dinv[i], x1[o]};
    }
    template <int NV> __device__ void operator()(int i, int c, T s, const P &pr, double (&)[NV]) const {
        const T r = pr.d * (pr.b - s);
        const T d = c1 * pr.x + c2 * r;
        out[(size_t)i * NB + c] = pr.x + d;
    }
};

// Chebyshev smoothing from an iterate y0, first step:
// y1_i = y0_i + (dinv_i (b_i - (A y0)_i)) s0
template <typename T, int NB> struct EChebPost1 {
    const T *b;
    const T *dinv;
    const T *y0;
    T *y1;
    T s0;
    struct P {
        T b, d, y;
    };
    __device__ void prep(int) {}
    __device__ P load(int i, int c) const {
        const size_t o = (size_t)i * NB + c;
        return {b[o], dinv[i], y0[o]};
    }
    template <int NV> __device__ void operator()(int i, int c, T s, const P &pr, double (&)[NV]) const {
        y1[(size_t)i * NB + c] = pr.y + (pr.d * (pr.b - s)) * s0;
    }
};

// second step: out_i = y1_i + (c1 (y1_i - y0_i) + c2 dinv_i (b_i - (A y1)_i));
// optionally acc += b_i out_i
template <typename T, int NB, bool DOT> struct EChebPost2 {
    const T *b;
    const T *dinv;
    const T *y0;
    const T *y1;
    T *out;
    T c1, c2;
    struct P {
        T b, d, y0, y1;
    };
    __device__ void prep(int) {}
    __device__ P load(int i, int c) const {
        const size_t o = (size_t)i * NB + c;
        return {b[o], dinv[i], y0[o], y1[o]};
    }
    template <int NV> __device__ void operator()(int i, int c, T s, const P &pr, double (&acc)[NV]) const {
        const T r = pr.d * (pr.b - s);
        const T d = c1 * (pr.y1 - pr.y0) + c2 * r;
        const T v = pr.y1 + d;
        out[(size_t)i * NB + c] = v;
        if constexpr (DOT) acc[0] += (double)pr.b * (double)v;
    }
};

// post-smoothing: out_i = x_i + dinv_i (b_i - (A x)_i); optionally acc += b_i out_i
template <typename T, int NB, bool DOT> struct EPost {
    const T *dinv;
    const T *b;
    const T *x;
    T *out;
    struct P {
        T b, x, d;
    };
    __device__ void prep(int) {}
    __device__ P load(int i, int c) const {
        const size_t o = (size_t)i * NB + c;
        return {b[o], x[o], dinv[i]};
    }
    template <int NV> __device__ void operator()(int i, int c, T s, const P &pr, double (&acc)[NV]) const {
        const T v = pr.x + pr.d * (pr.b - s);
        out[(size_t)i * NB + c] = v;
        if constexpr (DOT) acc[0] += (double)pr.b * (double)v;
    }
};

// Prolongation fused into the first post-smoothing step.  The corrected
// iterate x + S e and the residual it leaves, b - A (x + S e) = r - T e with
// r = b - A x from the pre-smoothing and T = A S (the Galerkin intermediate,
// whose pattern contains that of S), come from one pass over T's pattern that
// carries S's values aligned to it (zero where S has no entry): per row i and
// column c, se = (S e)_i and te = (T e)_i, both gathered from the coarse
// vector e.  LPR = G NG lanes per row as in spmv_kernel: G groups over the
// entries, NG groups of CV consecutive columns, so a gather of e is CV
// contiguous values; the epilogue receives both sums.  Columns are int32 or,
// when the coarse level has at most 65536 nodes, 16-bit (CI = uint16_t), or
// relative to row_base (CI = int16_t, larger coarse levels: 2146689 rows 58.9 -> 53.6 us).
template <typename T, int NB, int NV, class EP, typename CI = int>
__global__ __launch_bounds__(kBlock) void tpro_kernel(const int *__restrict__ stop, int un, int urun, int ustep,
                                                      int nrows, int lg, const int *__restrict__ rp,
                                                      const CI *__restrict__ ci, const T *__restrict__ tv,
                                                      const T *__restrict__ sv, const T *__restrict__ e, EP ep,
                                                      Reducer<(NV > 0 ? NV : 1), NB> red, uint32_t scale) {
    constexpr int CV = spmv_cv<NB>(), NG = NB / CV;
    const Geo geo = geo_from_lg<NB>(lg);
    const int t = threadIdx.x, LPR = geo.lpr(), G = 1 << geo.lg;
    const int lane = t & (LPR - 1), c0 = (lane % NG) * CV, g = lane / NG, rl = t >> geo.llpr;
    const Share sh = xcd_share(un, urun, ustep);
    int row = sh.first * geo.rpb() + rl;
    int p0 = rp[min(row, nrows - 1)], p1 = rp[min(row, nrows - 1) + 1];
    {
        const int st = *stop;
        pin_s(st);
        pin_args(ep);
        pin_v(p0, p1);
        if (st) return;
    }
    EP epv = ep;
    epv.prep(c0);  // the epilogues of this kernel hold nothing per column
    constexpr int NVA = NV > 0 ? NV : 1;
    double acc[CV][NVA];
#pragma unroll
    for (int v = 0; v < CV; ++v)
#pragma unroll
        for (int q = 0; q < NVA; ++q) acc[v][q] = 0.0;
    constexpr int U = kSpmvUnroll;
    for (int blk = sh.first; blk < sh.end; blk += sh.step) {
        const bool live = row < nrows;
        typename EP::P pr[CV];
        if (live && g == 0) {
#pragma unroll
            for (int v = 0; v < CV; ++v) pr[v] = epv.load(row, c0 + v);
        }
        T se[CV], te[CV];
#pragma unroll
        for (int v = 0; v < CV; ++v) se[v] = te[v] = T(0);
        const int nrow = (blk + sh.step) * geo.rpb() + rl, nr = min(nrow, nrows - 1);
        const int n0 = rp[nr], n1 = rp[nr + 1];
        int kb = 0;
        if constexpr (std::is_same_v<CI, int16_t>) kb = row_base(row, scale);
        if (live) {
            for (int p = p0 + g; p < p1; p += U * G) {
                // unconditional loads, as in spmv_kernel
                int kk[U];
                T ta[U], sa[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    const int q = p + u * G;
                    const int qc = min(q, p1 - 1);
                    kk[u] = kb + (int)ci[qc];
                    const T a = tv[qc], s = sv[qc];
                    ta[u] = q < p1 ? a : T(0);
                    sa[u] = q < p1 ? s : T(0);
                }
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int v = 0; v < CV; ++v) {
                        const T ev = e[(size_t)kk[u] * NB + c0 + v];
                        se[v] += sa[u] * ev;
                        te[v] += ta[u] * ev;
                    }
            }
        }
#pragma unroll
        for (int v = 0; v < CV; ++v) {  // the G groups of a row and column group
            se[v] = group_add<NG>(se[v], LPR);
            te[v] = group_add<NG>(te[v], LPR);
        }
        if (live && g == 0) {
#pragma unroll
            for (int v = 0; v < CV; ++v) epv(row, c0 + v, se[v], te[v], pr[v], acc[v]);
        }
        row = nrow;
        p0 = n0;
        p1 = n1;
    }
    if constexpr (NV > 0) block_partials_cv<NV, NB, CV>(acc, red);
}

// Chebyshev, first post step: y0 = t + S e (in place of t),
// y1 = y0 + (dinv (r - T e)) s0, i.e. y0 + (dinv (b - A y0)) s0
template <typename T, int NB> struct EProCheb {
    T *t;
    const T *r;
    const T *dinv;
    T *y1;
    T s0;
    struct P {
        T t, r, d;
    };
    __device__ void prep(int) {}
    __device__ P load(int i, int c) const {
        const size_t o = (size_t)i * NB + c;
        return {t[o], r[o], dinv[i]};
    }
    template <int NV>
    __device__ void operator()(int i, int c, T se, T te, const P &pr, double (&)[NV]) const {
        const size_t o = (size_t)i * NB + c;
        const T y0 = pr.t + se;
        t[o] = y0;
        y1[o] = y0 + (pr.d * (pr.r - te)) * s0;
    }
};

// l1-Jacobi post-sweep: out = (x + S e) + dinv (r - T e), i.e.
// x1 + dinv (b - A x1) with x1 = x + S e; optionally acc += b out
template <typename T, int NB, bool DOT> struct EProJac {
    const T *x;
    const T *r;
    const T *b;
    const T *dinv;
    T *out;
    struct P {
        T x, r, b, d;
    };
    __device__ void prep(int) {}
    __device__ P load(int i, int c) const {
        const size_t o = (size_t)i * NB + c;
        return {x[o], r[o], DOT ? b[o] : T(0), dinv[i]};
    }
    template <int NV>
    __device__ void operator()(int i, int c, T se, T te, const P &pr, double (&acc)[NV]) const {
        const T x1 = pr.x + se;
        const T v = x1 + pr.d * (pr.r - te);
        out[(size_t)i * NB + c] = v;
        if constexpr (DOT) acc[0] += (double)pr.b * (double)v;
    }
};

// CG direction and its product without gathering the direction:
// p_i = z_i + beta pold_i and q_i = (A z)_i + beta qold_i, which is (A p)_i
// since qold = A pold; q is updated in place (row i reads and writes only its
// own entry), and beta = 0 takes (A z)_i alone; acc p.q
template <typename T, int NB, typename TZ = T> struct ECgQR {
    const TZ *z;
    const T *pold;
    T *p;
    T *q;
    const CgScal *sc;
    T beta;
    struct P {
        T z, po, qo;
    };
    __device__ void prep(int c) { beta = (T)sc->s[c].beta; }
    __device__ void set_beta(double b) { beta = (T)b; }
    __device__ P load(int i, int c) const {
        const size_t o = (size_t)i * NB + c;
        return {(T)z[o], pold[o], q[o]};
    }
    template <int NV> __device__ void operator()(int i, int c, T s, const P &pr, double (&acc)[NV]) const {
        const size_t o = (size_t)i * NB + c;
        const T pi = pr.z + beta * pr.po;
        const T qi = beta != T(0) ? s + beta * pr.qo : s;
        p[o] = pi;
        q[o] = qi;
        acc[0] += (double)pi * (double)qi;
    }
};

// out_i = s1 keep_i sum + s2 y_i + s3 w_i (+ acc x_i out_i)
template <int NB> struct ELin {
    double *out;
    const uint8_t *mask;
    double s1;
    const double *y;
    double s2;
    const double *w;
    double s3;
    const double *dotx;  // acc[0] += dotx_i * out_i when not null
    struct P {
        double y0, w0, dx;
        int keep;
    };
    __device__ void prep(int) {}
    __device__ P load(int i, int c) const {
        const size_t o = (size_t)i * NB + c;
        return {y ? y[o] : 0.0, w ? w[o] : 0.0, dotx ? dotx[o] : 0.0, !(mask && mask[i])};
    }
    template <int NV> __device__ void operator()(int i, int c, double s, const P &pr, double (&acc)[NV]) const {
        double v = pr.keep ? s1 * s : 0.0;
        if (y) v += s2 * pr.y0;
        if (w) v += s3 * pr.w0;
        out[(size_t)i * NB + c] = v;
        if (dotx) acc[0] += pr.dx * v;
    }
};

// residual for refinement: r_i = f_i - (A x)_i (FP64), acc r.r
template <int NB> struct EResid {
    const double *f;
    double *r;
    struct P {
        double f;
    };
    __device__ void prep(int) {}
    __device__ P load(int i, int c) const { return {f[(size_t)i * NB + c]}; }
    template <int NV> __device__ void operator()(int i, int c, double s, const P &pr, double (&acc)[NV]) const {
        const double v = pr.f - s;
        r[(size_t)i * NB + c] = v;
        acc[0] += v * v;
    }
};

// ---------------------------------------------------------------------------
// finalize steps
template <int NB> struct FinAlpha {  // alpha = rho / p.q on live columns
    CgScal *sc;
    int outer;  // 1: flag indefiniteness instead of treating it as breakdown
    int fused;  // 1: rho is the rho_next of the fused finalize, committed here
    __device__ void head() const {}
    __device__ void col(int c, double pq) const {
        ColScal &s = sc->s[c];
        if (fused && !s.conv) s.rho = s.rho_next;
        s.pq = pq;
        s.alpha = 0.0;
        if (s.conv) return;
        if (!(pq > 0.0)) {
            s.bad = 1;
            if (outer) sc->indefinite = 1;
            s.conv = 1;
            return;
        }
        s.alpha = s.rho / pq;
    }
};

template <int NB, bool JAC> struct FinUpd {  // convergence test on r.r (and Jacobi beta)
    CgScal *sc;
    __device__ void head() const {}
    __device__ void col(int c, double rr, double rz = 0.0) const {
        ColScal &s = sc->s[c];
        if (s.conv) return;
        s.iters += 1;
        s.rr = rr;
        if (rr <= s.tol2 || s.bad) s.conv = 1;
        if constexpr (JAC) {
            s.rz = rz;
            s.beta = s.conv ? 0.0 : rz / s.rho;
            s.rho = rz;
        }
    }
};

// Inner V-cycle CG, once per iteration after the preconditioner: convergence
// test on r.r (partials of the update kernel), then beta from r.z (partials of
// the V-cycle's last kernel).
template <int NB> struct FinUB {
    CgScal *sc;
    __device__ void head() const {}
    __device__ void col(int c, double rr, double rz) const {
        ColScal &s = sc->s[c];
        if (s.conv) return;
        s.iters += 1;
        s.rr = rr;
        if (s.bad || rr <= s.tol2) {
            s.conv = 1;
            s.beta = 0.0;
        } else if (!(rz > 0.0)) {
            s.bad = 1;
            s.conv = 1;
        } else {
            s.rz = rz;
            s.beta = rz / s.rho;
            s.rho = rz;
        }
    }
};

// Inner V-cycle CG, between the update and the preconditioner where a column
// is expected to have converged: the convergence test on r.r alone.  A column
// that stops here is recorded as the finalize after the preconditioner would
// record it (that step no longer touches it); the others are left alone.
template <int NB> struct FinConv {
    CgScal *sc;
    __device__ void head() const {}
    __device__ void col(int c, double rr) const {
        ColScal &s = sc->s[c];
        if (s.conv || !(s.bad || rr <= s.tol2)) return;
        s.iters += 1;
        s.rr = rr;
        s.beta = 0.0;
        s.conv = 1;
    }
};

// Inner V-cycle CG start: rho = r.z of the first preconditioner application.
template <int NB> struct FinRho0 {
    CgScal *sc;
    __device__ void head() const {}
    __device__ void col(int c, double rz) const {
        ColScal &s = sc->s[c];
        s.beta = 0.0;
        if (s.conv) return;
        if (!(rz > 0.0)) {
            s.bad = 1;
            s.conv = 1;
        } else {
            s.rho = rz;
            s.rz = rz;
        }
    }
};

template <int NB> struct FinBeta {  // beta = r.z / rho after the preconditioner
    CgScal *sc;
    int outer;
    __device__ void head() const {}
    __device__ void col(int c, double rz) const {
        ColScal &s = sc->s[c];
        if (s.conv) {
            s.beta = 0.0;
            return;
        }
        if (!(rz > 0.0)) {
            s.bad = 1;
            if (outer) sc->indefinite = 1;
            s.conv = 1;
            s.beta = 0.0;
            return;
        }
        s.rz = rz;
        s.beta = rz / s.rho;
        s.rho = rz;
    }
};

// CG in the mass-matrix inner product (the coarsest Hessian level): after the
// preconditioner z = M^{-1} r, stop on r.z <= tol2 (tol2 = rtol^2 b.M^{-1}b, set
// by FinOuterInit from b.z), else beta = r.z / rho
template <int NB> struct FinRzConv {
    CgScal *sc;
    __device__ void head() const {}
    __device__ void col(int c, double rz) const {
        ColScal &s = sc->s[c];
        if (s.conv) {
            s.beta = 0.0;
            return;
        }
        s.iters += 1;
        s.rz = rz;
        s.rr = rz;
        if (s.bad || rz <= s.tol2) {
            s.conv = 1;
            s.beta = 0.0;
        } else if (!(rz > 0.0)) {
            s.bad = 1;
            s.conv = 1;
            s.beta = 0.0;
        } else {
            s.beta = rz / s.rho;
            s.rho = rz;
        }
    }
};

// initial state: bb = b.b, tol2 = rtol^2 bb, conv = (bb == 0); Jacobi: rho = r.z
template <int NB, bool JAC> struct FinInit {
    CgScal *sc;
    double rtol;
    int nlive;
    void *x;
    int fused;  // the first fused finalize then gives beta = 0, rho_next = r.z and iteration 0
    __device__ void head() const {
        sc->xptr = x;
        sc->nb = nlive;
        sc->indefinite = 0;
    }
    __device__ void col(int c, double bb, double rz = 0.0) const {
        ColScal &s = sc->s[c];
        s.bb = bb;
        s.tol2 = rtol * rtol * bb;
        s.rr = bb;
        s.iters = 0;
        s.bad = 0;
        s.alpha = 0.0;
        s.beta = 0.0;
        s.rho = 1.0;
        s.conv = c >= nlive || !(bb > 0.0);
        if constexpr (JAC) {
            s.rz = rz;
            s.rho = s.conv ? 1.0 : rz;
        }
        if (fused) {
            s.rho = __builtin_huge_val();
            s.iters = -1;
        }
    }
};

template <int NB> struct FinStore {  // plain reduction result into out[v*NB + c]
    double *out;
    template <int NV> __device__ void operator()(double (&tot)[NV][NB]) const {
        for (int v = 0; v < NV; ++v)
            for (int c = 0; c < NB; ++c) out[v * NB + c] = tot[v][c];
    }
};

// ---------------------------------------------------------------------------
// elementwise operations
// r = b, x = 0, pold = 0; Jacobi: z = dinv r; else, when z is given, the
// V-cycle's first pre-sweep iterate z = dinv r, and with r32 the float32
// residual and its iterate x32 = d32 r32
template <typename T, int NB, bool JAC> struct OpInit {
    const T *b;
    T *r, *x, *pold, *z;
    const T *dinv;
    float *r32;
    float *x32;
    const float *d32;
    double s0;  // scale of the first smoothing iterate (1, or 1/theta for Chebyshev)
    __device__ void prep(int) {}
    template <int NV> __device__ void operator()(int i, int c, double (&acc)[NV]) const {
        const size_t o = (size_t)i * NB + c;
        const T v = b[o];
        r[o] = v;
        if constexpr (!JAC) {
            if (z) z[o] = (dinv[i] * v) * (T)s0;
            if (r32) {
                const float rf = (float)v;
                r32[o] = rf;
                if (x32) x32[o] = (d32[i] * rf) * (float)s0;
            }
        }
        x[o] = T(0);
        pold[o] = T(0);
        acc[0] += (double)v * (double)v;
        if constexpr (JAC) {
            const T zz = dinv[i] * v;
            z[o] = zz;
            acc[1] += (double)v * (double)zz;
        }
    }
};

template <int NB> struct OpDot {  // acc[v] += x_v . y_v (up to 2 pairs)
    const double *x0, *y0, *x1, *y1;
    __device__ void prep(int) {}
    template <int NV> __device__ void operator()(int i, int c, double (&acc)[NV]) const {
        const size_t o = (size_t)i * NB + c;
        acc[0] += x0[o] * y0[o];
        if constexpr (NV > 1) acc[1] += x1[o] * y1[o];
    }
};

template <int NB> struct OpAxpby {  // out = a x + b y (a, b per column or scalar), out may alias x or y
    double *out;
    const double *x, *y;
    double a, b;
    __device__ void prep(int) {}
    template <int NV> __device__ void operator()(int i, int c, double (&)[NV]) const {
        const size_t o = (size_t)i * NB + c;
        double v = a * x[o];
        if (y) v += b * y[o];
        out[o] = v;
    }
};

// out = x - (y + b w)
template <int NB> struct OpSubSum {
    double *out;
    const double *x, *y, *w;
    double b;
    __device__ void prep(int) {}
    template <int NV> __device__ void operator()(int i, int c, double (&)[NV]) const {
        const size_t o = (size_t)i * NB + c;
        out[o] = x[o] - (y[o] + b * w[o]);
    }
};

// outer CG direction update: p = z + beta_c p
template <int NB> struct OpPUpd {
    double *p;
    const double *z;
    const CgScal *sc;
    double beta;
    int live;
    __device__ void prep(int c) {
        beta = sc->s[c].beta;
        live = !sc->s[c].conv;
    }
    template <int NV> __device__ void operator()(int i, int c, double (&)[NV]) const {
        if (!live) return;
        const size_t o = (size_t)i * NB + c;
        p[o] = z[o] + beta * p[o];
    }
};

// FP64 refinement state per column, kept on the device
struct RefScal {
    double fn[16];  // ||f||
    double s[16];   // current ||r||
    int live[16];
    int nlive;
    int stagnated;
    double rtol;
    Mail *mail;     // host-mapped: nlive, stagnated
};

template <int NB> struct OpCopyNorm {  // r = f, x = 0, acc f.f
    const double *f;
    double *r, *x;
    __device__ void prep(int) {}
    template <int NV> __device__ void operator()(int i, int c, double (&acc)[NV]) const {
        const size_t o = (size_t)i * NB + c;
        const double v = f[o];
        r[o] = v;
        x[o] = 0.0;
        acc[0] += v * v;
    }
};

template <int NB> struct FinRefInit {
    RefScal *rs;
    double rtol;
    int nlive;
    __device__ void operator()(double (&tot)[1][NB]) const {
        int nl = 0;
        rs->rtol = rtol;
        rs->stagnated = 0;
        for (int c = 0; c < 16; ++c) {
            const double fn = c < NB ? sqrt(tot[0][c]) : 0.0;
            rs->fn[c] = fn;
            rs->s[c] = fn;
            rs->live[c] = (c < nlive) && fn > 0.0;
            nl += rs->live[c];
        }
        rs->nlive = nl;
        rs->mail->nlive = nl;
        rs->mail->stagnated = rs->stagnated;
    }
};

// after r = f - A x: a live column finishes at ||r|| <= rtol ||f||; it has
// stagnated when the residual did not at least halve
template <int NB> struct FinRefine {
    RefScal *rs;
    __device__ void operator()(double (&tot)[1][NB]) const {
        int nl = 0;
        for (int c = 0; c < NB; ++c) {
            if (!rs->live[c]) continue;
            const double r = sqrt(tot[0][c]);
            if (r <= rs->rtol * rs->fn[c]) {
                rs->live[c] = 0;
                continue;
            }
            if (!(r <= 0.5 * rs->s[c])) rs->stagnated = 1;
            rs->s[c] = r;
            ++nl;
        }
        rs->nlive = nl;
        rs->mail->nlive = nl;
        rs->mail->stagnated = rs->stagnated;
    }
};

template <int NB> struct OpRefAdd {  // x64 += s_c d32 on live columns
    double *x;
    const float *d;
    const RefScal *rs;
    double sc;
    int on;
    __device__ void prep(int c) {
        sc = rs->s[c];
        on = rs->live[c];
    }
    template <int NV> __device__ void operator()(int i, int c, double (&)[NV]) const {
        if (!on) return;
        const size_t o = (size_t)i * NB + c;
        x[o] += sc * (double)d[o];
    }
};

template <int NB> struct OpCastScale {  // b32 = fp32(r / s_c), zero on finished columns
    float *b;
    const double *r;
    const RefScal *rs;
    double inv;
    __device__ void prep(int c) { inv = rs->live[c] ? 1.0 / rs->s[c] : 0.0; }
    template <int NV> __device__ void operator()(int i, int c, double (&)[NV]) const {
        const size_t o = (size_t)i * NB + c;
        b[o] = (float)(r[o] * inv);
    }
};

// outer CG start: bb = b.b, rr = r.r
template <int NB> struct FinOuterInit {
    CgScal *sc;
    double rtol;
    int nlive;
    __device__ void head() const {
        sc->nb = nlive;
        sc->indefinite = 0;
    }
    __device__ void col(int c, double bb, double rr) const {
        ColScal &s = sc->s[c];
        s.bb = bb;
        s.rr = rr;
        s.tol2 = rtol * rtol * bb;
        s.iters = 0;
        s.bad = 0;
        s.alpha = s.beta = 0.0;
        s.rho = 1.0;
        s.conv = c >= nlive || !(bb > 0.0) || rr <= s.tol2;
    }
};

template <int NB> struct FinRho {  // rho = r.z at the start of the outer CG
    CgScal *sc;
    __device__ void head() const {}
    __device__ void col(int c, double rz) const {
        ColScal &s = sc->s[c];
        if (s.conv) return;
        if (!(rz > 0.0)) {
            s.bad = 1;
            sc->indefinite = 1;
            return;
        }
        s.rho = rz;
        s.rz = rz;
    }
};

// V-cycle input from a packed FP64 vector: b = T(in) (zero on padding
// columns) and the first smoothing iterate x = (dinv b) s0 that the producer
// of a V-cycle's right-hand side writes
template <typename T, int NB> struct OpVcIn {
    T *b, *x;
    const double *in;
    const T *dinv;
    T s0;
    int nb;
    __device__ void prep(int) {}
    template <int NV> __device__ void operator()(int i, int c, double (&)[NV]) const {
        const size_t o = (size_t)i * NB + c;
        const T v = c < nb ? (T)in[(size_t)i * nb + c] : T(0);
        b[o] = v;
        if (x) x[o] = (dinv[i] * v) * s0;
    }
};

template <typename T, int NB> struct OpVcOut {  // out[i*nb + c] = double(z[i*NB + c]), c < nb
    double *out;
    const T *z;
    int nb;
    __device__ void prep(int) {}
    template <int NV> __device__ void operator()(int i, int c, double (&)[NV]) const {
        if (c < nb) out[(size_t)i * nb + c] = (double)z[(size_t)i * NB + c];
    }
};

template <int NB> struct OpPack {  // out[i*NB + c] = c < nb ? in[i*nb + c] : 0
    double *out;
    const double *in;
    int nb;
    __device__ void prep(int) {}
    template <int NV> __device__ void operator()(int i, int c, double (&)[NV]) const {
        out[(size_t)i * NB + c] = c < nb ? in[(size_t)i * nb + c] : 0.0;
    }
};

template <int NB> struct OpUnpack {  // out[i*nb + c] = in[i*NB + c], c < nb
    double *out;
    const double *in;
    int nb;
    __device__ void prep(int) {}
    template <int NV> __device__ void operator()(int i, int c, double (&)[NV]) const {
        if (c < nb) out[(size_t)i * nb + c] = in[(size_t)i * NB + c];
    }
};

// ---------------------------------------------------------------------------
// dense coarse-level apply: x = Inv b with Inv row-major (stride ld, a
// multiple of 64 entries, zero padded), entries TM (FP64 or float32), one
// wavefront per row, 16-byte loads four deep per lane, FP64 accumulation.
template <typename TM> struct Vec16;
template <> struct Vec16<double> {
    using type = double2;
    static constexpr int n = 2;
    __device__ static double get(const double2 &v, int e) { return e == 0 ? v.x : v.y; }
};
template <> struct Vec16<float> {
    using type = float4;
    static constexpr int n = 4;
    __device__ static double get(const float4 &v, int e) {
        return e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w;
    }
};

// At most four columns, b of the matrix's type and 16-byte aligned (a workspace,
// whose storage is allocated in 256-byte units; callers' vectors are packed into
// one): b is read in 16-byte vectors like the matrix rows, NB of them per vector of the
// row, eight (four with four columns) row vectors and theirs in flight per lane
// (a float32 row of up to 2048 entries is one round).  Every load is
// unconditional (guarded loads compile to a wait each): vectors past the last
// that holds an entry re-read it, and entries past n are zeroed in both.  In
// float32 every lane takes part in every round, with nothing but such vectors past
// the end: a round of at most 16 lanes takes far longer over its conversions to FP64
// (64 rows or fewer: 3.8, 5.5 and 4.9 us for one, two and four columns, 2.5, 2.7 and
// 2.6 us with all lanes; 65 rows took that before).  In FP64, without conversions,
// lanes past the end stay out (600 rows, four columns: 3.3 us, 4.1 with all).  The
// last vector of b may reach past its entries, within the 16 bytes that hold
// the last of them.  The stop flag is tested before the store, so no load waits
// for it, and the few wavefronts per SIMD of such a launch may use the registers
// that keep all loads in flight.
template <typename TM, int NB>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(1, 4))) void dense_vec_kernel(
    const int *__restrict__ stop, int n, int ld, const TM *__restrict__ inv, const TM *__restrict__ b,
    TM *__restrict__ x) {
    using V = Vec16<TM>;
    using VT = typename V::type;
    constexpr int W = V::n, D = NB < 4 ? 8 : 4;
    constexpr bool whole = sizeof(TM) == 4;
    const int lane = threadIdx.x % 64;
    const int i = (blockIdx.x * kBlock + threadIdx.x) / 64;
    if (i >= n) return;
    const int st = *stop;
    const int last = (n - 1) / W * W;         // the vector that holds entry n - 1
    const int lastb = (n * NB - 1) / W * W;  // and the last one of the batch
    double acc[NB];
#pragma unroll
    for (int c = 0; c < NB; ++c) acc[c] = 0.0;
    const TM *row = inv + (size_t)i * ld;
    for (int base = whole ? 0 : lane * W; base < n; base += 64 * W * D) {
        const int k0 = whole ? base + lane * W : base;
        VT m[D], bv[D][NB];
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int k = min(k0 + u * 64 * W, last);
            m[u] = *reinterpret_cast<const VT *>(row + k);
#pragma unroll
            for (int q = 0; q < NB; ++q) bv[u][q] = *reinterpret_cast<const VT *>(b + min(k * NB + q * W, lastb));
        }
        // keep the scheduler from interleaving the loads with their uses
        // (it would otherwise issue them one at a time)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < D; ++u)
#pragma unroll
            for (int e = 0; e < W; ++e) {
                const bool on = k0 + u * 64 * W + e < n;
                const double a = on ? V::get(m[u], e) : 0.0;
#pragma unroll
                for (int c = 0; c < NB; ++c) {
                    const int t = e * NB + c;
                    acc[c] += a * (on ? V::get(bv[u][t / W], t % W) : 0.0);
                }
            }
    }
#pragma unroll
    for (int c = 0; c < NB; ++c) acc[c] = group_add<1>(acc[c], 64);
    if (lane < NB && !st) {
        double v = acc[0];
#pragma unroll
        for (int c = 1; c < NB; ++c)
            if (lane == c) v = acc[c];
        x[(size_t)i * NB + lane] = (TM)v;
    }
}

// Several columns: x = Inv B on the FP64 matrix cores.  A workgroup forms `rows`
// (at most 16) rows by all columns; its 16 wavefronts take the 16-entry chunks
// of the rows in turn, each chunk four v_mfma_f64_16x16x4f64 (lane l: row l % 16,
// the entries 4 (l / 16) .. + 3 of the chunk in one 16-byte load per four floats;
// step e multiplies entry e of each lane, so the matrix operand's k and the
// batch operand's k are permuted alike), the loads of D chunks in flight, and their
// sums are added through LDS in wavefront order.  The
// accumulation is FP64 whatever T.  Lanes past `rows`, columns past NB and rows
// past n are computed from clamped reads and dropped; the batch's entries past n
// (the ragged chunk's, and those of chunks past the last, which re-read it) are
// zeroed: the matrix's entries there are finite, the batch's need not be.  Bound by the latency of the matrix's and the batch's loads:
// `rows` is what fills the 256 CUs (dense_mm_rows), matrix-core work done for
// the lanes past it is not what is waited for.  n = 1639, float32, 16 columns:
// 9.2 us with 8 rows per workgroup, 9.5 us with 16 (103 workgroups), 29.2 us
// with a wavefront per row on the vector ALUs, whose lanes each read every
// column of the batch.  Slots past a wavefront's chunks cost their loads, so D is
// the chunks it has, up to eight (float32) or four: 597 rows, float32, 8 columns:
// 4.6 us with three, 9.0 us with eight; 149 rows, FP64, 16 columns: 3.6 us with one,
// 4.8 us with four.
inline int dense_mm_rows(int n) {
    int r = 1;
    while (r < 16 && ceil_div(n, r) > 256) r <<= 1;
    return r;
}
constexpr int kMmWaves = 16;
typedef double mm_v4d __attribute__((ext_vector_type(4)));
template <typename T, int NB, int D>
__global__ __launch_bounds__(64 * kMmWaves) void dense_mm_kernel(const int *__restrict__ stop, int n, int ld,
                                                                 int rows, const T *__restrict__ inv,
                                                                 const T *__restrict__ b, T *__restrict__ x) {
    const int st = *stop;  // tested before the store: no load waits for it
    using V = Vec16<T>;
    using VT = typename V::type;
    const int l = threadIdx.x & 63, wv = threadIdx.x >> 6, kq = (l >> 4) * 4;
    const int row0 = blockIdx.x * rows;
    const T *row = inv + (size_t)min(row0 + min(l & 15, rows - 1), n - 1) * ld;
    const int col = min(l & 15, NB - 1);
    const int nk = (n + 15) / 16;
    mm_v4d acc = {0.0, 0.0, 0.0, 0.0};
    for (int c0 = wv; c0 < nk; c0 += kMmWaves * D) {
        VT m[D][4 / V::n];
        T v[D][4];
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int k = min(c0 + u * kMmWaves, nk - 1) * 16 + kq;
#pragma unroll
            for (int q = 0; q < 4 / V::n; ++q) m[u][q] = *reinterpret_cast<const VT *>(row + k + q * V::n);
#pragma unroll
            for (int e = 0; e < 4; ++e) v[u][e] = b[(size_t)min(k + e, n - 1) * NB + col];
        }
        __builtin_amdgcn_sched_barrier(0);  // the loads stay together, ahead of their uses
#pragma unroll
        for (int u = 0; u < D; ++u) {
            const int k = (c0 + u * kMmWaves) * 16 + kq;  // past n in the chunks past the last
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const T bk = k + e < n ? v[u][e] : T(0);
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(V::get(m[u][e / V::n], e % V::n), (double)bk, acc, 0, 0, 0);
            }
        }
    }
    __shared__ double red[kMmWaves][4][64];
#pragma unroll
    for (int r = 0; r < 4; ++r) red[wv][r][l] = acc[r];
    __syncthreads();
    if (threadIdx.x >= 256) return;
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < kMmWaves; ++w) s += red[w][wv][l];
    const int k = (l >> 4) + 4 * wv, i = row0 + k;  // result r of lane l: row l / 16 + 4 r, column l % 16
    if (!st && k < rows && i < n && (l & 15) < NB) x[(size_t)i * NB + (l & 15)] = (T)s;
}

}  // namespace amg
