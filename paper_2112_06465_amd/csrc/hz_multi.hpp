// Shared-pattern batched BiCGStab: B systems A_j x_j = b_j with one sparsity
// pattern, e.g. a frequency sweep A(k_j) = K - k_j^2 M + i k_j B on one mesh.
// Each system runs Section 7's preconditioned BiCGStab with its own scalars,
// convergence test and exit; the systems share the launches, the row_ptr /
// col_idx reads and the gathers' cache lines.
//
// Layout (system-minor): entry p of system j is vals[p*B + j]; element i of
// a vector of system j is v[i*B + j].  A block owns a contiguous row chunk
// (XCD-aware mapping as in the single solve) and takes kBlock/BL rows per
// step with one lane per system (BL = a power of two >= B; lanes j >= B
// idle).  A row's values and gathered x of all systems are then contiguous
// B*16-byte runs: every load is coalesced, col_idx is read once for all
// systems, and no cross-lane row reduction is needed.
//
// Iteration (the one-system iteration with s formed by itself, four kernels):
//   A1: v = A p; partial <rhat, v>
//   S:  the end of iteration i - 1 per system; alpha = rho / <rhat, v>; s = r - alpha v
//   B1: t = A s; partials ||s||^2, <t, s>, ||t||^2, <rhat, t>, <rhat, s>
//   C:  half-step test; omega = <t, s> / <t, t>; rho and beta of the next
//       iteration; x += alpha p + omega s; r = s - omega t;
//       p = r + beta (p - omega v); partial ||r||^2
// Partials are per (component, block, lane), reduced over the row slots of a
// block by a fixed tree and finished at the consumer's head by every block
// in a fixed order: reruns are bitwise identical, and system j's arithmetic
// does not depend on the other systems (permuting the batch permutes the
// results bitwise).  A head reads K G BL doubles in every block, so a launch
// has one block per CU (G <= kMultiMaxGrid) and each component is added by
// waves of its own, two systems a lane: with 490 blocks of the same 31k rows
// and all threads adding all components the heads read 250 KB a block and
// took half of S, C and a fifth kernel, P, which C now contains.  Measured,
// 16 systems K - k^2 M + i k B of 31,429 rows: 85 -> 58 us an iteration.
#pragma once

#include "hz_kernels.hpp"

namespace hz {

constexpr int kMultiMax = 256;      // most systems per shared-pattern launch
constexpr int kMultiMaxGrid = 256;  // most blocks: one per CU
#define HZ_MULTI_BOUNDS __launch_bounds__(kBlock)  // one block per CU: <= 128 VGPRs

// Where the row product takes system j's entry p from.
enum : int {
    VS_EXPLICIT = 0,  // vals[p*B + j] (column-scaled by D_j^{-1} under Jacobi)
    VS_KMB = 1        // K[p] - k_j^2 M[p] + i k_j Bm[p] (a frequency sweep; never scaled)
};

struct MultiArgs {
    int n;     // rows of the shared pattern
    int B;     // systems
    Geom geo;  // row chunks of the geo.G blocks
    const int* __restrict__ row_ptr;
    const int* __restrict__ col_idx;
    const double2* __restrict__ vals;  // VS_EXPLICIT: [nnz][B]
    const double* __restrict__ K;      // VS_KMB: three real [nnz] arrays and the wavenumbers [B]
    const double* __restrict__ M;
    const double* __restrict__ Bm;
    const double* __restrict__ kw;
    const double* kd;     // VS_KMB with Jacobi, else null: row i's diagonal K, M, Bm at kd[4 i .. 4 i + 2]; the
                          // products act on q = D^{-1} p and u = D^{-1} s
    const double2* b;     // [n][B]
    double2* r;
    double2* rh;
    double2* p;
    double2* v;
    double2* s;
    double2* t;
    double2* q;  // the vector A1 gathers: p itself, or D^{-1} p written by C
    double2* u;  // the vector B1 gathers: s itself, or D^{-1} s written by S
    double2* x;
    double* part;    // [kParts][G][BL]
    SolverScal* sc;  // [B]
    int* ndone;      // systems finished so far
};

// The block's partials of K components: region[(k*G + lb)*BL + lane], the sums
// over the block's row slots separately for every lane: over a wave's slots by
// rotations, over the waves through LDS.
template <int BL, int K, int TAG = 0>
__device__ __forceinline__ void mstore(double* region, int G, int lb, double (&e)[K]) {
    constexpr int NW = kBlock / kWave, LN = BL < kWave ? BL : kWave, WS = BL / LN;  // WS: waves per slot
    __shared__ double red[K][NW][LN];
    const int lane = threadIdx.x % kWave;
    if constexpr (BL < kWave) {
#pragma unroll
        for (int k = 0; k < K; ++k) e[k] = wave_sum<BL>(e[k]);
    }
    if (lane < LN) {
#pragma unroll
        for (int k = 0; k < K; ++k) red[k][wave_id()][lane] = e[k];
    }
    __syncthreads();
    for (int o = threadIdx.x; o < K * BL; o += kBlock) {
        const int k = o / BL, j = o % BL;
        double t = red[k][j / LN][j % LN];
#pragma unroll
        for (int w = WS; w < NW; w += WS) t += red[k][w + j / LN][j % LN];
        region[((size_t)k * G + lb) * BL + j] = t;
    }
}

// Totals of K components over all G blocks for every lane: component k by
// the W = head_waves waves k W .., a lane adding two neighbouring systems'
// partials of blocks in turn; totals per wave in LDS, at() adds the W of them.
// load() issues the first NV rounds' loads, store() waits and adds the rest.
template <int BL, int K> struct MSum {
    static constexpr int W = head_waves(K, kBlock / kWave), NV = 32 / W;
    static constexpr int P = BL / 2 < kWave ? BL / 2 : kWave;  // pairs of systems that a wave's lanes hold
    static_assert(BL <= 2 * kWave || W % 2 == 0, "a lane keeps its systems from round to round");
    typedef double2 Tot[kBlock / kWave][P];
    const double2* p;
    int m, f0;
    double2 v[NV];

    static __device__ __forceinline__ int comp() { return wave_id() / W; }
    __device__ __forceinline__ void load(const double* region, int G) {
        p = reinterpret_cast<const double2*>(region);
        m = G * (BL / 2);
        f0 = wave_id() % W * kWave + (int)(threadIdx.x % kWave);
#pragma unroll
        for (int r = 0; r < NV; ++r) v[r] = p[f0 + r * W * kWave < m ? f0 + r * W * kWave : m - 1];
    }
    __device__ __forceinline__ void store(Tot& tot) {
        double2 t = mk<double>(0.0, 0.0);
        for (int g = 0; g < m; g += NV * W * kWave) {  // uniform
            if (g > 0) {
#pragma unroll
                for (int r = 0; r < NV; ++r) {
                    const int f = g + f0 + r * W * kWave;
                    v[r] = p[f < m ? f : m - 1];
                }
            }
#pragma unroll
            for (int r = 0; r < NV; ++r) {
                const bool in = g + f0 + r * W * kWave < m;
                t.x += in ? v[r].x : 0.0;
                t.y += in ? v[r].y : 0.0;
            }
        }
        if constexpr (P < kWave) t = mk<double>(wave_sum<P>(t.x), wave_sum<P>(t.y));
        if ((int)(threadIdx.x % kWave) < P) tot[wave_id()][threadIdx.x % kWave] = t;
    }
    static __device__ __forceinline__ double at(const Tot& tot, int k, int j) {
        constexpr int H = BL / 2 / P;  // lane groups: a wave holds pairs h P .. h P + P - 1, h = its share mod H
        const int h = j / 2 / P, q = j / 2 % P;
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < W; w += H) {
            const double2 d = tot[k * W + w + h][q];
            t += j % 2 ? d.y : d.x;
        }
        return t;
    }
};

// Totals of K components for the kernels of one block.
template <int BL, int K>
__device__ __forceinline__ void mhead(const double* region, int G, double (&out)[K]) {
    __shared__ typename MSum<BL, K>::Tot tot;
    MSum<BL, K> ms;
    if (ms.comp() < K) {
        ms.load(region + (size_t)ms.comp() * G * BL, G);
        ms.store(tot);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) out[k] = MSum<BL, K>::at(tot, k, threadIdx.x % BL);
}

// True when every system has ended.  (The products, during which no system
// ends, read it in every wave; S and C, whose leaders end systems, read it
// once per block and broadcast it with the head's barrier.)
__device__ __forceinline__ bool all_done(const MultiArgs& a) { return *a.ndone >= a.B; }

template <int BL> __device__ __forceinline__ double* mregion(const MultiArgs& a, int comp) {
    return a.part + (size_t)comp * a.geo.G * BL;
}

// Entry p of system j.  k = (k_j, k_j^2) for VS_KMB.
template <int VS>
__device__ __forceinline__ double2 mval(const MultiArgs& a, int p, int j, double2 k) {
    if constexpr (VS == VS_EXPLICIT) {
        return a.vals[(size_t)p * a.B + j];
    } else {
        return mk<double>(__builtin_fma(-k.y, a.M[p], a.K[p]), k.x * a.Bm[p]);
    }
}

template <int VS> __device__ __forceinline__ double2 mwave(const MultiArgs& a, int j) {
    if constexpr (VS == VS_KMB) {
        const double kj = a.kw[j];
        return mk<double>(kj, kj * kj);
    } else {
        return mk<double>(0.0, 0.0);
    }
}

// Row i of A times X for lane j: entries in order, U loads of each kind in flight.
template <int U, int VS>
__device__ __forceinline__ double2 mrow(const MultiArgs& a, int64_t i, int j, const double2* __restrict__ X,
                                        double2 k) {
    const size_t B = (size_t)a.B;
    const int beg = a.row_ptr[i], end = a.row_ptr[i + 1];
    double2 acc = mk<double>(0.0, 0.0);
    int p = beg;
    for (; p + U <= end; p += U) {
        int c[U];
        double2 av[U], xv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) c[u] = a.col_idx[p + u];
#pragma unroll
        for (int u = 0; u < U; ++u) av[u] = mval<VS>(a, p + u, j, k);
#pragma unroll
        for (int u = 0; u < U; ++u) xv[u] = X[(size_t)c[u] * B + j];
#pragma unroll
        for (int u = 0; u < U; ++u) acc = cfma<double>(av[u], xv[u], acc);
    }
    for (; p < end; ++p) acc = cfma<double>(mval<VS>(a, p, j, k), X[(size_t)a.col_idx[p] * B + j], acc);
    return acc;
}

// The products stage a tile's column indices (and, for K/M/B, its K, M, Bm
// entries) in LDS: every lane of a row (one per system) needs the same ones,
// and loading them per lane costs one 64-lane load instruction per entry and
// kind for BL times fewer distinct values.  Explicit values differ per system
// and are still loaded per lane.  Tiles with more entries than kMTileCap read
// everything per lane as mrow does.
constexpr int kMTileCap = 1536;

// Row i of A_j times X for lane j, entries [b, e) of the staged tile (tile
// offsets; the tile starts at entry e0), in batches of U straight-line gathers:
// an entry past the row's end is read at its last one and dropped by a select
// (four at a time and the rest singly, a 15-entry row waited for six gathers,
// one after the other; A1 13.8 -> 13.4 us with half the waves).
template <int U, int VS>
__device__ __forceinline__ double2 mrow_lds(const MultiArgs& a, int e0, const unsigned* cs, const double* ks,
                                            const double* ms, const double* bs, int b, int e, int j, size_t B,
                                            const double2* __restrict__ X, double2 k) {
    const double2* __restrict__ Xj = X + j;
    auto val = [&](int p) {
        if constexpr (VS == VS_KMB) {
            return mk<double>(__builtin_fma(-k.y, ms[p], ks[p]), k.x * bs[p]);
        } else {
            return ld_mat(a.vals + (size_t)(e0 + p) * B + j);
        }
    };
    double2 acc = mk<double>(0.0, 0.0);
    for (int p = b; p < e; p += U) {
        double2 xv[U], av[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int pu = p + u < e ? p + u : e - 1;
            if constexpr (VS != VS_KMB) av[u] = val(pu);
            xv[u] = Xj[cs[pu]];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const double2 nx = cfma<double>(VS == VS_KMB ? val(p + u < e ? p + u : e - 1) : av[u], xv[u], acc);
            acc = mk<double>(p + u < e ? nx.x : acc.x, p + u < e ? nx.y : acc.y);
        }
    }
    return acc;
}

// A thread's part of a tile: the tile's first entry and their number, its
// row's entries (tile offsets), and the shared entries that it stages.
template <int VS> struct MTile {
    static constexpr int R = (kMTileCap + kBlock - 1) / kBlock, RK = VS == VS_KMB ? R : 1;
    int e0, ne, rb, re;
    int c[R];
    double kv[RK], mv[RK], bv[RK];
};
// The tile of S rows from r0 on.
template <int VS, int S>
__device__ __forceinline__ MTile<VS> m_fetch(const MultiArgs& a, const RowRange& rr, int64_t r0) {
    MTile<VS> t{};
    const int* __restrict__ rp = a.row_ptr;
    const int64_t re = r0 + S < rr.rw.x1 ? r0 + S : rr.rw.x1;
    const int64_t i = r0 + threadIdx.x / (kBlock / S), ic = i < re ? i : re - 1;  // an in-bounds row of the tile
    t.e0 = rp[r0];
    t.ne = rp[re] - t.e0;
    t.rb = rp[ic] - t.e0;
    t.re = rp[ic + 1] - t.e0;
    if (t.ne > 0 && t.ne <= kMTileCap) {  // uniform
#pragma unroll
        for (int r = 0; r < MTile<VS>::R; ++r) {
            const int q = (int)threadIdx.x + r * kBlock, at = t.e0 + (q < t.ne ? q : t.ne - 1);
            t.c[r] = a.col_idx[at];
            if constexpr (VS == VS_KMB) {
                t.kv[r] = a.K[at];
                t.mv[r] = a.M[at];
                t.bv[r] = a.Bm[at];
            }
        }
    }
    return t;
}

// f(i, acc, w) for every row i of the block on lane j when `on`, acc = row i
// of A_j times X and w = pre(i), the operands of the epilogue.  The block walks
// its rows in tiles of kBlock / BL consecutive rows (the rows and order of
// HZ_MROWS); a tile's shared entries are loaded once, contiguously by the
// whole block, into registers while the tile before is computed, and from
// there into LDS.  w is loaded before the row's gathers, so it adds no wait.
template <int BL, int U, int VS, typename P, typename F>
__device__ __forceinline__ void m_tiles(const MultiArgs& a, const RowRange& rr, bool on, const double2* __restrict__ X,
                                        double2 k, P&& pre, F&& f) {
    constexpr int S = kBlock / BL;
    constexpr bool kmb = VS == VS_KMB;
    constexpr int KC = kmb ? kMTileCap : 1;  // K, M, Bm staged only for K/M/B
    constexpr int R = MTile<VS>::R;
    __shared__ unsigned cs[kMTileCap];  // col B: n B vector elements of 16 bytes fit into memory only below 2^32
    __shared__ double ks[KC], ms[KC], bs[KC];
    const int g = threadIdx.x / BL, j = threadIdx.x % BL;
    int64_t r0 = rr.rw.x0 + (int64_t)rr.rw.k * S;
    MTile<VS> nx{};
    if (r0 < rr.rw.x1) nx = m_fetch<VS, S>(a, rr, r0);
    while (r0 < rr.rw.x1) {  // uniform
        const int64_t i = r0 + g, end = r0 + S < rr.rw.x1 ? r0 + S : rr.rw.x1;
        const bool staged = nx.ne <= kMTileCap;
        const int e0 = nx.e0, rb = nx.rb, re = nx.re;
        if (staged) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int q = (int)threadIdx.x + r * kBlock;
                if (q < nx.ne) {
                    cs[q] = (unsigned)nx.c[r] * (unsigned)a.B;
                    if constexpr (kmb) {
                        ks[q] = nx.kv[r];
                        ms[q] = nx.mv[r];
                        bs[q] = nx.bv[r];
                    }
                }
            }
            __syncthreads();
        }
        r0 += (int64_t)rr.rw.K * S;
        if (r0 < rr.rw.x1) nx = m_fetch<VS, S>(a, rr, r0);
        if (on && i < end) {
            const auto w = pre(i);
            const double2 acc = staged ? mrow_lds<U, VS>(a, e0, cs, ks, ms, bs, rb, re, j, (size_t)a.B, X, k)
                                       : mrow<2, VS>(a, i, j, X, k);
            f(i, acc, w);
        }
        if (staged) __syncthreads();  // the tile's entries have been read
    }
}

// 1 / (K_ii - k^2 M_ii + i k Bm_ii) from the row's diagonal triple, with the
// operations of k_m_jacobi_kmb (bitwise the value it stores in dinv).
struct MDiag {
    double2 km;
    double b;
    __device__ __forceinline__ void load(const double* __restrict__ kd, int64_t i) {
        if (kd == nullptr) return;  // uniform
        km = reinterpret_cast<const double2*>(kd)[2 * i];
        b = kd[4 * i + 2];
    }
    __device__ __forceinline__ double2 inverse(double kj) const {
        const double2 d = mk<double>(__builtin_fma(-kj * kj, km.y, km.x), kj * b);
        const double q = d.x * d.x + d.y * d.y;
        return mk<double>(d.x / q, -d.y / q);
    }
};

#define HZ_MULTI_ROWS                                       \
    constexpr int S = kBlock / BL;                          \
    const RowRange rr = rows_of_block(a.n, a.geo);          \
    const int g = threadIdx.x / BL, j = threadIdx.x % BL;   \
    const size_t Bz = (size_t)a.B;                          \
    (void)Bz

// The block's rows for slot g: its tiles of S rows (see struct Rows).
#define HZ_MROWS(i) \
    for (int64_t i = rr.rw.x0 + (int64_t)rr.rw.k * S + g; i < rr.rw.x1; i += (int64_t)rr.rw.K * S)

// Solve set-up: r = rhat = p = src, q = D^{-1} p; partials <rhat,r>, ||r||^2 (C), ||b||^2 (I).
template <int BL>
__global__ HZ_MULTI_BOUNDS void k_m_init(const MultiArgs a, const double2* src) {
    HZ_MULTI_ROWS;
    double e[3] = {0.0, 0.0, 0.0}, eb[1] = {0.0};
    const double kj = a.kd && j < a.B ? a.kw[j] : 0.0;
    if (j < a.B)
        HZ_MROWS(i) {
            const size_t q = (size_t)i * Bz + j;
            const double2 bv = a.b[q], rv = src[q];
            if (a.r != src) a.r[q] = rv;
            a.rh[q] = rv;
            a.p[q] = rv;
            MDiag d{};
            d.load(a.kd, i);
            if (a.kd) a.q[q] = cmul<double>(d.inverse(kj), rv);
            eb[0] = __builtin_fma(bv.x, bv.x, eb[0]);
            eb[0] = __builtin_fma(bv.y, bv.y, eb[0]);
            const double2 c = cdotacc(rv.x, rv.y, rv.x, rv.y, mk<double>(e[0], e[1]));
            e[0] = c.x;
            e[1] = c.y;
            e[2] = __builtin_fma(rv.x, rv.x, e[2]);
            e[2] = __builtin_fma(rv.y, rv.y, e[2]);
        }
    mstore<BL, 3>(mregion<BL>(a, kPartC), a.geo.G, rr.lb, e);
    mstore<BL, 1>(mregion<BL>(a, kPartI), a.geo.G, rr.lb, eb);
}

// ||b||, initial convergence test of every system (one block).
template <int BL>
__global__ HZ_MULTI_BOUNDS void k_m_fin_init(const MultiArgs a) {
    double hb[1], hr[3];
    mhead<BL, 1>(mregion<BL>(a, kPartI), a.geo.G, hb);
    mhead<BL, 3>(mregion<BL>(a, kPartC), a.geo.G, hr);
    const int j = threadIdx.x;
    if (j >= a.B) return;  // lanes of slot 0 only (B <= BL)
    SolverScal* sc = a.sc + j;
    const double bn = __builtin_sqrt(hb[0]);
    sc->bnorm = bn;
    sc->iter = 1;
    sc->cur = 0;
    sc->done = 0;
    sc->zero_x = 0;
    sc->iters = 0;
    sc->pending = 0;
    sc->why = BD_NONE;
    sc->status = ST_NOT_CONVERGED;
    sc->alpha = sc->omega = sc->beta = mk<double>(1.0, 0.0);
    sc->rho2[1] = mk<double>(hr[0], hr[1]);
    if (!__builtin_isfinite(bn) || !__builtin_isfinite(hr[2])) return finish(sc, a.ndone, ST_NONFINITE, 0);
    if (bn == 0.0) {
        sc->zero_x = 1;
        sc->relres = 0.0;
        return finish(sc, a.ndone, ST_OK, 0);
    }
    const double rel = __builtin_sqrt(hr[2]) / bn;
    sc->relres = rel;
    if (rel <= sc->rtol) finish(sc, a.ndone, ST_OK, 0);
    else if (sc->maxiter <= 0) finish(sc, a.ndone, ST_NOT_CONVERGED, 0);
}

// A1-kernel: v = A p; partial <rhat, v>.
template <int BL, int U, int VS>
__global__ HZ_MULTI_BOUNDS void k_m_A1(const MultiArgs a) {
    HZ_MULTI_ROWS;
    double e[2] = {0.0, 0.0};
    const bool on = j < a.B && !a.sc[j].done && !a.sc[j].pending;
    const double2 kj = j < a.B ? mwave<VS>(a, j) : mk<double>(0.0, 0.0);
    if (all_done(a)) return;
    auto pre = [&](int64_t i) { return a.rh[(size_t)i * Bz + j]; };
    auto row = [&](int64_t i, double2 acc, double2 w) {
        a.v[(size_t)i * Bz + j] = acc;
        const double2 c = cdotacc(w.x, w.y, acc.x, acc.y, mk<double>(e[0], e[1]));
        e[0] = c.x;
        e[1] = c.y;
    };
    m_tiles<BL, U, VS>(a, rr, on, a.q, kj, pre, row);
    mstore<BL, 2>(mregion<BL>(a, kPartA), a.geo.G, rr.lb, e);
}

// S-kernel: the end of iteration i-1 and alpha per system (as in the
// one-system solve), then s = r - alpha v on the system's lanes.
template <int BL>
__global__ HZ_MULTI_BOUNDS void k_m_S(const MultiArgs a) {
    __shared__ typename MSum<BL, 3>::Tot tot;
    __shared__ double2 al[BL];
    __shared__ int go[BL];
    __shared__ int over;
    HZ_MULTI_ROWS;
    if (threadIdx.x == 0) over = all_done(a);
    MSum<BL, 3> ms;
    const int c = ms.comp();  // <rhat, v>, then ||r||^2
    if (c < 3) ms.load(mregion<BL>(a, c < 2 ? kPartA + c : kPartC + 2), a.geo.G);
    SolverScal* sc = a.sc + (j < a.B ? j : 0);
    const int done = sc->done, pending = sc->pending, it = sc->iter;
    const double2 rho_0 = sc->rho2[0], rho_1 = sc->rho2[1];
    const EndIn z{sc->bnorm, sc->rtol, sc->omega, (it & 1) ? rho_1 : rho_0, sc->beta, sc->maxiter};
    const int64_t step = (int64_t)rr.rw.K * S;
    int64_t i = rr.rw.x0 + (int64_t)rr.rw.k * S + g;
    if (j >= a.B) i = rr.rw.x1;
    const double kj = a.kd && j < a.B ? a.kw[j] : 0.0;
    double2 v0 = mk<double>(0.0, 0.0), r0 = v0;  // the first row's, in flight during the head
    MDiag d0{};
    if (i < rr.rw.x1) {
        v0 = a.v[(size_t)i * Bz + j];
        r0 = a.r[(size_t)i * Bz + j];
        d0.load(a.kd, i);
    }
    if (c < 3) ms.store(tot);
    __syncthreads();
    if (over) return;
    if (threadIdx.x < BL) {
        const bool lead = rr.lb == 0;
        double2 alpha = mk<double>(0.0, 0.0);
        auto decide = [&]() -> int {
            if (j >= a.B || done) return 0;
            if (pending) {  // the half step's x += alpha p is complete everywhere
                if (lead) finish(sc, a.ndone, ST_OK, pending);
                return 0;
            }
            if (it > 1) {
                double rel;
                int sit, why;
                const int st = iteration_end(it, ms.at(tot, 2, j), z, rel, sit, why);
                if (lead) sc->relres = rel;
                if (st >= 0) {
                    if (lead) finish(sc, a.ndone, st, sit, why);
                    return 0;
                }
            }
            const double2 sigma = mk<double>(ms.at(tot, 0, j), ms.at(tot, 1, j));
            if (!zfinite(sigma) || zzero(sigma)) {
                if (lead) finish(sc, a.ndone, zzero(sigma) ? ST_BREAKDOWN : ST_NONFINITE, it, zzero(sigma) ? BD_RHAT_V : BD_NONE);
                return 0;
            }
            alpha = zdiv(z.rho, sigma);
            if (lead) {
                sc->alpha = alpha;
                sc->cur = it;
            }
            return 1;
        };
        go[threadIdx.x] = decide();
        al[threadIdx.x] = alpha;
    }
    __syncthreads();
    if (!go[j]) return;
    const double2 nal = mk<double>(-al[j].x, -al[j].y);
    while (i < rr.rw.x1) {
        const size_t q = (size_t)i * Bz + j;
        const double2 sv = cfma<double>(nal, v0, r0);
        const MDiag d = d0;
        i += step;
        if (i < rr.rw.x1) {
            v0 = a.v[(size_t)i * Bz + j];
            r0 = a.r[(size_t)i * Bz + j];
            d0.load(a.kd, i);
        }
        a.s[q] = sv;
        if (a.kd) a.u[q] = cmul<double>(d.inverse(kj), sv);
    }
}

// B1-kernel: t = A s and its dot products.
template <int BL, int U, int VS>
__global__ HZ_MULTI_BOUNDS void k_m_B1(const MultiArgs a) {
    HZ_MULTI_ROWS;
    double e[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    const bool on = j < a.B && !a.sc[j].done;
    const double2 kj = j < a.B ? mwave<VS>(a, j) : mk<double>(0.0, 0.0);
    if (all_done(a)) return;
    struct Ops {
        double2 s, rh;
    };
    auto pre = [&](int64_t i) { return Ops{a.s[(size_t)i * Bz + j], a.rh[(size_t)i * Bz + j]}; };
    auto row = [&](int64_t i, double2 acc, const Ops& w) {
        a.t[(size_t)i * Bz + j] = acc;
        b_terms<double>(e, w.s, acc, w.rh);
    };
    m_tiles<BL, U, VS>(a, rr, on, a.u, kj, pre, row);
    mstore<BL, 8>(mregion<BL>(a, kPartB), a.geo.G, rr.lb, e);
}

// C-kernel: half-step test on ||s||; omega; rho and beta of the next iteration;
// x += alpha p + omega s; r = s - omega t; p and q = D^{-1} p; partial ||r||^2.
template <int BL>
__global__ HZ_MULTI_BOUNDS void k_m_C(const MultiArgs a) {
    enum : int { STOP = 0, HALF = 1, FULL = 2 };
    __shared__ typename MSum<BL, 8>::Tot tot;
    __shared__ double2 cal[BL], com[BL], cbt[BL];  // alpha, omega, beta
    __shared__ int mode[BL];
    __shared__ int over;
    HZ_MULTI_ROWS;
    if (threadIdx.x == 0) over = all_done(a);
    MSum<BL, 8> ms;
    ms.load(mregion<BL>(a, kPartB + ms.comp()), a.geo.G);
    SolverScal* sc = a.sc + (j < a.B ? j : 0);
    // pending is written by this kernel's leader, so only done is read here
    // (a pending exit of the previous iteration was concluded by S)
    const int done = sc->done, it = sc->cur;
    const double bnorm = sc->bnorm, rtol = sc->rtol;
    const double2 alpha = sc->alpha, rho_0 = sc->rho2[0], rho_1 = sc->rho2[1], rho = (it & 1) ? rho_1 : rho_0;
    const int64_t step = (int64_t)rr.rw.K * S;
    int64_t i = rr.rw.x0 + (int64_t)rr.rw.k * S + g;
    if (j >= a.B) i = rr.rw.x1;
    const double kj = a.kd && j < a.B ? a.kw[j] : 0.0;
    double2 s0 = mk<double>(0.0, 0.0), t0 = s0, p0 = s0, v0 = s0, x0 = s0;
    MDiag d0{};
    auto fetch = [&]() HZ_INLINE {
        const size_t q = (size_t)i * Bz + j;
        s0 = a.s[q];
        t0 = a.t[q];
        p0 = a.p[q];
    };
    auto fetch2 = [&]() HZ_INLINE {  // for the first row, when the partials' registers are free
        const size_t q = (size_t)i * Bz + j;
        v0 = a.v[q];
        x0 = a.x[q];
        d0.load(a.kd, i);
    };
    if (i < rr.rw.x1) fetch();
    ms.store(tot);
    if (i < rr.rw.x1) fetch2();
    __syncthreads();
    if (over) return;
    if (threadIdx.x < BL) {
        const bool lead = rr.lb == 0;
        double2 om = mk<double>(0.0, 0.0), beta = om;
        auto decide = [&]() -> int {
            if (j >= a.B || done) return STOP;
            double h[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) h[k] = ms.at(tot, k, j);
            const double rel = __builtin_sqrt(h[0]) / bnorm;
            if (!__builtin_isfinite(rel)) {
                if (lead) finish(sc, a.ndone, ST_NONFINITE, it);
                return STOP;
            }
            if (rel <= rtol) {  // concluded by the next S-kernel
                if (lead) {
                    sc->relres = rel;
                    sc->pending = it;
                }
                return HALF;
            }
            const double2 ts = mk<double>(h[1], h[2]);
            const double tt = h[3];
            int st = -1, why = BD_NONE;
            if (!zfinite(ts) || !__builtin_isfinite(tt)) st = ST_NONFINITE;
            else if (tt == 0.0) st = ST_BREAKDOWN, why = BD_TT;
            else {
                om = zdiv(ts, mk<double>(tt, 0.0));
                if (!zfinite(om)) st = ST_NONFINITE;
            }
            if (st >= 0) {
                if (lead) finish(sc, a.ndone, st, it, why);
                return STOP;
            }
            // omega = 0, rho = 0 or a non-finite beta end the solve in the next S, after its test on ||r||
            const double2 ort = zmul(om, mk<double>(h[4], h[5]));
            const double2 rho_n = mk<double>(h[6] - ort.x, h[7] - ort.y);
            beta = zmul(zdiv(rho_n, rho), zdiv(alpha, om));
            if (lead) {
                sc->omega = om;
                sc->rho2[(it + 1) & 1] = rho_n;
                sc->beta = beta;
                sc->iter = it + 1;
            }
            return FULL;
        };
        mode[threadIdx.x] = decide();
        cal[threadIdx.x] = alpha;
        com[threadIdx.x] = om;
        cbt[threadIdx.x] = beta;
    }
    __syncthreads();
    double e[1] = {0.0};
    if (mode[j] == HALF) {  // half-step exit: x += alpha p
        for (; i < rr.rw.x1; i += step) {
            const size_t q = (size_t)i * Bz + j;
            a.x[q] = cfma<double>(cal[j], a.p[q], a.x[q]);
        }
    } else if (mode[j] == FULL) {
        const double2 al = cal[j], om = com[j], bt = cbt[j], nom = mk<double>(-om.x, -om.y);
        while (i < rr.rw.x1) {
            const size_t q = (size_t)i * Bz + j;
            double2 x = cfma<double>(al, p0, x0);
            x = cfma<double>(om, s0, x);
            const double2 r = cfma<double>(nom, t0, s0);
            const double2 pn = p_update<double>(bt, om, r, p0, v0);
            const MDiag d = d0;
            i += step;
            if (i < rr.rw.x1) {
                fetch();
                fetch2();
            }
            a.x[q] = x;
            a.r[q] = r;
            a.p[q] = pn;
            if (a.kd) a.q[q] = cmul<double>(d.inverse(kj), pn);
            e[0] = __builtin_fma(r.x, r.x, e[0]);
            e[0] = __builtin_fma(r.y, r.y, e[0]);
        }
    }
    mstore<BL, 1>(mregion<BL>(a, kPartC + 2), a.geo.G, rr.lb, e);
}

// After the last iteration of a limited solve: conclude it (one block).
template <int BL>
__global__ HZ_MULTI_BOUNDS void k_m_end(const MultiArgs a) {
    double h[1];
    mhead<BL, 1>(mregion<BL>(a, kPartC + 2), a.geo.G, h);
    const int j = threadIdx.x;
    if (j >= a.B) return;
    SolverScal* sc = a.sc + j;
    if (sc->done) return;
    if (sc->pending) return finish(sc, a.ndone, ST_OK, sc->pending);
    const int it = sc->iter;
    if (it <= 1) return;
    const EndIn z{sc->bnorm, sc->rtol, sc->omega, sc->rho2[it & 1], sc->beta, sc->maxiter};
    double rel;
    int sit, why;
    const int st = iteration_end(it, h[0], z, rel, sit, why);
    sc->relres = rel;
    if (st >= 0) finish(sc, a.ndone, st, sit, why);
}

// y = b - A xin for every system (explicit values `vals`, or K, M, Bm);
// partial ||y||^2 (I).
template <int BL, int U, int VS>
__global__ HZ_MULTI_BOUNDS void k_m_resid(const MultiArgs a, const double2* __restrict__ vals,
                                           const double2* __restrict__ xin, double2* __restrict__ y) {
    HZ_MULTI_ROWS;
    MultiArgs a2 = a;
    a2.vals = vals;
    double e[1] = {0.0};
    const double2 k = j < a.B ? mwave<VS>(a, j) : mk<double>(0.0, 0.0);
    auto pre = [&](int64_t i) { return a.b[(size_t)i * Bz + j]; };
    auto row = [&](int64_t i, double2 acc, double2 bv) {
        const double2 d = mk<double>(bv.x - acc.x, bv.y - acc.y);
        y[(size_t)i * Bz + j] = d;
        e[0] = __builtin_fma(d.x, d.x, e[0]);
        e[0] = __builtin_fma(d.y, d.y, e[0]);
    };
    m_tiles<BL, U, VS>(a2, rr, j < a.B, xin, k, pre, row);
    mstore<BL, 1>(mregion<BL>(a, kPartI), a.geo.G, rr.lb, e);
}

// relres_true of every system from region I (one block).
template <int BL>
__global__ HZ_MULTI_BOUNDS void k_m_fin_true(const MultiArgs a) {
    double h[1];
    mhead<BL, 1>(mregion<BL>(a, kPartI), a.geo.G, h);
    const int j = threadIdx.x;
    if (j >= a.B) return;
    SolverScal* sc = a.sc + j;
    sc->relres_true = sc->bnorm > 0.0 ? __builtin_sqrt(h[0]) / sc->bnorm : 0.0;
}

// x = 0 for the systems whose right-hand side is zero.
template <int BL>
__global__ HZ_MULTI_BOUNDS void k_m_zero_if(const MultiArgs a) {
    HZ_MULTI_ROWS;
    if (j >= a.B || !a.sc[j].zero_x) return;
    HZ_MROWS(i) a.x[(size_t)i * Bz + j] = mk<double>(0.0, 0.0);
}

// dinv[i*B + j] = 1 / A_j(i, i); a missing or zero diagonal flags sc[j].bad_diag.
__global__ __launch_bounds__(kBlock) void k_m_jacobi(int n, int B, const int* __restrict__ rp,
                                                     const int* __restrict__ ci, const double2* __restrict__ vals,
                                                     double2* __restrict__ dinv, SolverScal* sc) {
    const int64_t f = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (f >= (int64_t)n * B) return;
    const int64_t i = f / B;
    const int j = (int)(f % B);
    double2 d = mk<double>(0.0, 0.0);
    for (int p = rp[i]; p < rp[i + 1]; ++p)
        if (ci[p] == i) d = vals[(size_t)p * B + j];
    if (d.x == 0.0 && d.y == 0.0) {
        sc[j].bad_diag = 1;  // every writer stores 1
        dinv[f] = mk<double>(0.0, 0.0);
        return;
    }
    const double q = d.x * d.x + d.y * d.y;
    dinv[f] = mk<double>(d.x / q, -d.y / q);
}

// dinv[i*B + j] = 1 / (K_ii - k_j^2 M_ii + i k_j Bm_ii); a missing or zero
// diagonal flags sc[j].bad_diag.
__global__ __launch_bounds__(kBlock) void k_m_jacobi_kmb(int n, int B, const int* __restrict__ rp,
                                                         const int* __restrict__ ci, const double* __restrict__ K,
                                                         const double* __restrict__ M, const double* __restrict__ Bm,
                                                         const double* __restrict__ kw, double2* __restrict__ dinv,
                                                         SolverScal* sc) {
    const int64_t f = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (f >= (int64_t)n * B) return;
    const int64_t i = f / B;
    const int j = (int)(f % B);
    const double kj = kw[j];
    double2 d = mk<double>(0.0, 0.0);
    for (int p = rp[i]; p < rp[i + 1]; ++p)
        if (ci[p] == i) d = mk<double>(__builtin_fma(-kj * kj, M[p], K[p]), kj * Bm[p]);
    if (d.x == 0.0 && d.y == 0.0) {
        sc[j].bad_diag = 1;  // every writer stores 1
        dinv[f] = mk<double>(0.0, 0.0);
        return;
    }
    const double q = d.x * d.x + d.y * d.y;
    dinv[f] = mk<double>(d.x / q, -d.y / q);
}

// kd[4 i .. 4 i + 3] = (K_ii, M_ii, Bm_ii, 0): the last diagonal entry of row i
// (the one k_m_jacobi_kmb uses), zeros if the row has none.
__global__ __launch_bounds__(kBlock) void k_m_diag_kmb(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                                       const double* __restrict__ K, const double* __restrict__ M,
                                                       const double* __restrict__ Bm, double* __restrict__ kd) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    double k = 0.0, m = 0.0, b = 0.0;
    for (int p = rp[i]; p < rp[i + 1]; ++p)
        if (ci[p] == i) k = K[p], m = M[p], b = Bm[p];
    reinterpret_cast<double2*>(kd)[2 * i] = mk<double>(k, m);
    reinterpret_cast<double2*>(kd)[2 * i + 1] = mk<double>(b, 0.0);
}

// out[p*B + j] = vals[p*B + j] * dinv[col_p*B + j]   (A_j D_j^{-1})
__global__ __launch_bounds__(kBlock) void k_m_colscale(int64_t nnz, int B, const int* __restrict__ ci,
                                                       const double2* __restrict__ vals,
                                                       const double2* __restrict__ dinv, double2* __restrict__ out) {
    const int64_t f = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (f >= nnz * B) return;
    const int64_t p = f / B;
    const int j = (int)(f % B);
    out[f] = cmul<double>(vals[f], dinv[(size_t)ci[p] * B + j]);
}

// Conjugate transposes of every system: tvals[q*B + j] = conj(vals[tsrc[q]*B + j]).
__global__ __launch_bounds__(kBlock) void k_m_conj_vals(int64_t nnz, int B, const int* __restrict__ tsrc,
                                                        const double2* __restrict__ vals,
                                                        double2* __restrict__ tvals) {
    const int64_t f = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (f >= nnz * B) return;
    const int64_t q = f / B;
    const int j = (int)(f % B);
    const double2 a = vals[(size_t)tsrc[q] * B + j];
    tvals[f] = mk<double>(a.x, -a.y);
}

// Entry gradients of every system: grad[p*B + j] = -lam_j[row_p] conj(x_j[col_p]).
template <int BL>
__global__ HZ_STREAM_BOUNDS void k_m_grad_vals(const MultiArgs a, const double2* __restrict__ lam,
                                               const double2* __restrict__ xs, double2* __restrict__ grad) {
    HZ_MULTI_ROWS;
    if (j >= a.B) return;
    HZ_MROWS(i) {
        const double2 l = lam[(size_t)i * Bz + j];
        const double2 nl = mk<double>(-l.x, -l.y);
        for (int p = a.row_ptr[i]; p < a.row_ptr[i + 1]; ++p) {
            const double2 xv = xs[(size_t)a.col_idx[p] * Bz + j];
            grad[(size_t)p * Bz + j] = cmul<double>(nl, mk<double>(xv.x, -xv.y));
        }
    }
}

// Columns of a system-minor [n][B] array for a group of Bg <= kSweepGroup
// systems: gather (dir 0) dst[i*Bg + k] = src[i*B + idx[k]], or scatter
// (dir 1) dst[i*B + idx[k]] = src[i*Bg + k].
constexpr int kSweepGroup = 16;
// Ordering key of system j for grouping a batch: the sum of Re(A_j(i, i))
// over up to kBlock evenly spaced rows i (duplicates of a diagonal entry
// all count; a row without one adds nothing), in a fixed order.  For a
// frequency sweep K - k^2 M + i k B it decreases with k.  One block per
// system.
__global__ __launch_bounds__(kBlock) void k_m_diag_key(int n, int B, const int* __restrict__ rp,
                                                       const int* __restrict__ ci, const double2* __restrict__ vals,
                                                       double* __restrict__ key) {
    __shared__ double red[kBlock];
    const int j = blockIdx.x, t = threadIdx.x;
    const int m = n < kBlock ? n : kBlock;
    double v = 0.0;
    if (t < m) {
        const int i = (int)((int64_t)t * n / m);
        for (int p = rp[i]; p < rp[i + 1]; ++p)
            if (ci[p] == i) v += vals[(size_t)p * B + j].x;
    }
    red[t] = v;
    __syncthreads();
    for (int w = kBlock / 2; w >= 1; w /= 2) {
        if (t < w) red[t] += red[t + w];
        __syncthreads();
    }
    if (t == 0) key[j] = red[0];
}

struct GroupCols {
    int j[kSweepGroup];
};
__global__ __launch_bounds__(kBlock) void k_m_cols(int n, int B, int Bg, GroupCols idx, const double2* __restrict__ src,
                                                   double2* __restrict__ dst, int dir) {
    const int64_t f = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (f >= (int64_t)n * Bg) return;
    const int64_t i = f / Bg;
    const int k = (int)(f % Bg);
    const int64_t w = i * B + idx.j[k];
    if (dir == 0) dst[f] = src[w];
    else dst[w] = src[f];
}

}  // namespace hz
