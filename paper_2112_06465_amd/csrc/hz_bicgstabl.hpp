// BiCGstab(l): the paper's P-BiCGSTAB(l) (Section 7, iterative Krylov
// methods; l = 8 in its speed-up tables), in the form of Sleijpen and
// Fokkema.  One system, on the one-system work map of the BiCGStab kernels
// and with the same device scalars (SolverScal) and partial regions.
//
// A cycle is l Bi-CG steps (j = 0 .. l-1), which in the textbook update every
// vector found so far:
//   u_i = r_i - beta_j u_i (i <= j);   u_{j+1} = A u_j;
//   r_i -= alpha_j u_{i+1} (i <= j);   r_{j+1} = A r_j;   x += alpha_j u_0
// Only u_j and r_j are needed for the step itself, the others not before the
// cycle's end, so a step updates these two and the rest is caught up element
// by element, in registers, where it is used (l_catch_up; the same operations
// in the same order, so the same bits).  That leaves 6 vector passes of a
// step's 6 j + 9 and 37 of the cycle's end: 89 + 3 l instead of 271 + 3 l
// passes at l = 8 (with the operands of the products' epilogues).  Launches
// of step j:
//   U : rho_1 = <r~, r_j> (partials from the previous launch); at j = 0 the
//       cycle's convergence test on ||r_0|| and rho_0 = -omega rho_0;
//       beta_j = alpha rho_1 / rho_0; u_j = r_j - beta_j u_j
//   AU: u_{j+1} = A u_j; partial <r~, u_{j+1}>
//   R : alpha_j = rho_1 / <r~, u_{j+1}>; r_j -= alpha_j u_{j+1}
//   AR: r_{j+1} = A r_j; partial <r~, r_{j+1}> (rho of step j + 1)
// then the minimal-residual part, three launches:
//   gram  : partials of G_pq = <r_p, r_q>, 0 <= p <= q <= l, q > 0
//   mr    : one block sums them and solves the normal equations
//           (R^H R) gamma = R^H r_0 (R = [r_1 .. r_l]) by Cholesky after
//           scaling to unit diagonal; omega = gamma_l
//   update: x += sum_j alpha_j u_0 (of step j) + sum_j gamma_j r_{j-1};
//           r_0 -= sum_j gamma_j r_j; u_0 -= sum_j gamma_j u_j;
//           partials <r~, r_0>, ||r_0||^2
// A solve that ends inside a cycle leaves x with the steps that were complete
// (k_l_late).  Measured, l = 8 on the 260k-row cabin: a cycle 505 -> 337 us,
// U and R 11.5 -> 5.2 us, gram 19.5 -> 16, mr 22 -> 10, update 15 with the
// catching up, the products 15 -> 12.6 us on the sliced operator.
// ("A" is the column-scaled matrix under Jacobi, as for BiCGStab.)  rho of
// global step s = (cycle - 1) l + j lives in rho2[s & 1]: the U-launch of
// step s reads slot (s - 1) & 1 and writes slot s & 1, which no block of the
// same launch reads.
#pragma once

#include "hz_kernels.hpp"
#include "hz_slices.hpp"
#include "hz_soltile.hpp"

namespace hz {

constexpr int kLMax = 8;                                   // largest l
constexpr int kGramPairs = (kLMax + 1) * (kLMax + 2) / 2;  // pairs p <= q of r_0 .. r_l
constexpr int kGramBlock = 512;                            // threads of a Gram block: two waves per SIMD
constexpr int kGramMaxGrid = 256;                          // Gram blocks: one per CU
constexpr int kLUpBlock = 256;                             // threads and blocks of the update
constexpr int kLUpMaxGrid = 1024;
enum : int { BD_MR = 5 };                                  // the minimal-residual system is singular

struct LScal {
    double2 al[kLMax], be[kLMax];  // alpha_j and beta_j of the cycle
    int late;                      // complete steps of a cycle that the solve ended in (0: none)
    int spare;
};

struct LArgs {
    int G, stride;  // one-system map of the solver launches
    OneMap one;
    int* ndone;
    const int* __restrict__ row_ptr;
    const int* __restrict__ col_idx;
    const double2* __restrict__ vals;
    const int* __restrict__ soff;  // the sliced operator's offsets and columns, or null
    const short* __restrict__ scol;
    const double2* rt;  // shadow residual r~
    // u_j and r_j for j < l, as step j leaves them, and the l-th ones as their products leave them
    double2* r[kLMax + 1];
    double2* u[kLMax + 1];
    // the products' results, by turns: u_j in up[j & 1] and r_j in rp[j & 1] until step j has updated them
    double2* up[2];
    double2* rp[2];
    double2* x;       // iterate of the (column-scaled) system
    double* part;     // kParts x stride (regions as for BiCGStab)
    double* gpart;    // Gram partials: component c of block g at [g * 2 kGramPairs + c]
    double2* gam;     // gamma_1 .. gamma_l at [1 .. l]
    LScal* ls;
    SolverScal* sc;
    int n, ell;       // rows, l
    int j, reg;       // the Bi-CG step of this launch; a product's partial region
    // a launch's vectors: U and R dst = add + c src, products dst = A src
    const double2* src;
    const double2* add;
    double2* dst;
    int gG, uG;       // blocks of the Gram and of the update launch
    int pf = 1;       // CSR products: blocks per block of the map (sol_subs(G) when they run as sub-blocks)
    int np = 0;       // partial slots that the products write
};

__device__ __forceinline__ SysBlock lblock(const LArgs& a, int F = 1) {
    return map_block(a.one, nullptr, nullptr, a.G, F, blockIdx.x);
}

__device__ __forceinline__ double2 zneg_mul(double2 a, double2 b) {  // -(a b)
    return mk<double>(-(a.x * b.x - a.y * b.y), -(a.x * b.y + a.y * b.x));
}

// The step's scalar from K partial components and dst = add - c src: the
// element-wise part of U and R.  The first elements are loaded with the
// partials, the scalar arithmetic runs in the first wave.  decide(totals, c)
// returns whether the solve goes on.
template <int K, typename F>
__device__ __forceinline__ void l_step(const LArgs& a, const SysBlock& q, const double* part, int cnt, F decide) {
    __shared__ double tot[kBlock / kWave];
    __shared__ double2 coef;
    __shared__ int go;
    PartSum<K> ps;
    if (ps.comp() < K) ps.load(part + ps.comp() * a.stride, cnt);
    const double2* __restrict__ src = a.src;
    const double2* __restrict__ add = a.add;
    int64_t i = q.rw.x0 + (int64_t)q.rw.k * kBlock + threadIdx.x;
    const int64_t step = (int64_t)q.rw.K * kBlock;
    double2 s0 = mk<double>(0.0, 0.0), a0 = s0;
    if (i < q.rw.x1) {
        s0 = src[i];
        a0 = add[i];
    }
    if (ps.comp() < K) ps.store(tot);
    __syncthreads();
    if (wave_id() == 0) {
        double h[K];
#pragma unroll
        for (int k = 0; k < K; ++k) h[k] = ps.at(tot, k);
        double2 c = mk<double>(0.0, 0.0);
        const int g = decide(h, c);
        if (threadIdx.x == 0) {
            coef = c;
            go = g;
        }
    }
    __syncthreads();
    if (!go) return;
    const double2 nc = mk<double>(-coef.x, -coef.y);
    while (i < q.rw.x1) {
        const int64_t at = i;
        const double2 d = cfma<double>(nc, s0, a0);
        i += step;
        if (i < q.rw.x1) {
            s0 = src[i];
            a0 = add[i];
        }
        a.dst[at] = d;
    }
}

// U: beta_j, u_j = r_j - beta_j u_j
__global__ HZ_STREAM_BOUNDS void k_l_U(const LArgs a) {
    const SysBlock q = lblock(a);
    SolverScal* sc = a.sc;
    const int done = sc->done, it = sc->iter;  // cycle (1-based)
    const double bnorm = sc->bnorm, rtol = sc->rtol;
    const int maxc = sc->maxiter;
    const double2 alpha = sc->alpha, omega = sc->omega, ra = sc->rho2[0], rb = sc->rho2[1];
    // region C holds the partials of AR (step j - 1), or of the update or the set-up (j = 0)
    int cnt = a.np;
    if (a.j == 0) cnt = it == 1 ? a.G : a.uG;
    auto decide = [&](const double* h, double2& beta) -> int {
        if (done) return 0;
        const int s = (it - 1) * a.ell + a.j;
        const double2 rho_prev = s == 0 ? mk<double>(1.0, 0.0) : ((s + 1) & 1 ? rb : ra);
        const double2 rho1 = mk<double>(h[0], h[1]);
        double2 rho0 = rho_prev;
        if (a.j == 0) {  // a cycle starts: test the residual of the previous one
            const double rel = __builtin_sqrt(h[2]) / bnorm;
            int st = -1;
            if (!__builtin_isfinite(rel)) st = ST_NONFINITE;
            else if (rel <= rtol) st = ST_OK;
            else if (it - 1 >= maxc) st = ST_NOT_CONVERGED;
            if (sys_leader(q)) {
                sc->relres = rel;
                sc->cur = it;
            }
            if (st >= 0) {
                if (sys_leader(q)) finish(sc, a.ndone, st, it - 1);
                return 0;
            }
            rho0 = zneg_mul(omega, rho_prev);
        }
        int st = -1, why = BD_NONE;
        if (!zfinite(rho1)) st = ST_NONFINITE;
        else if (zzero(rho0) || zzero(rho1)) st = ST_BREAKDOWN, why = BD_RHO;
        else {
            beta = zmul(alpha, zdiv(rho1, rho0));
            if (!zfinite(beta)) st = ST_NONFINITE;
        }
        if (sys_leader(q)) {
            if (st >= 0) {
                a.ls->late = a.j;
                finish(sc, a.ndone, st, it - 1, why);
            } else {
                sc->rho2[s & 1] = rho1;
                a.ls->be[a.j] = beta;
            }
        }
        return st < 0;
    };
    const double* part = a.part + kPartC * a.stride;
    if (a.j == 0) l_step<3>(a, q, part, cnt, decide);
    else l_step<2>(a, q, part, cnt, decide);
}

// R: alpha_j, r_j -= alpha_j u_{j+1}
__global__ HZ_STREAM_BOUNDS void k_l_R(const LArgs a) {
    const SysBlock q = lblock(a);
    SolverScal* sc = a.sc;
    const int done = sc->done, it = sc->iter;
    const double2 ra = sc->rho2[0], rb = sc->rho2[1];
    l_step<2>(a, q, a.part + kPartA * a.stride, a.np, [&](const double* h, double2& alpha) -> int {
        if (done) return 0;
        const double2 rho1 = ((it - 1) * a.ell + a.j) & 1 ? rb : ra;
        const double2 g = mk<double>(h[0], h[1]);
        int st = -1, why = BD_NONE;
        if (!zfinite(g)) st = ST_NONFINITE;
        else if (zzero(g)) st = ST_BREAKDOWN, why = BD_RHAT_V;
        else {
            alpha = zdiv(rho1, g);
            if (!zfinite(alpha)) st = ST_NONFINITE;
        }
        if (sys_leader(q)) {
            if (st >= 0) {
                a.ls->late = a.j;
                finish(sc, a.ndone, st, it - 1, why);
            } else {
                sc->alpha = alpha;
                a.ls->al[a.j] = alpha;
            }
        }
        return st < 0;
    });
}

// AU and AR: dst = A src; partial <r~, dst>.  On vector rows,
template <int L, int U>
__global__ HZ_STREAM_BOUNDS void k_l_A(const LArgs a) {
    const SysBlock q = lblock(a);
    if (a.sc->done) return;
    const double2* __restrict__ x = a.src;
    double2* __restrict__ y = a.dst;
    const double2* __restrict__ rt = a.rt;
    double e[2] = {0.0, 0.0};
    for_rows<double, L, U>(q.rw, a.row_ptr, a.col_idx, a.vals, [x](int c) { return x[c]; },
                           [&](int64_t row, double2 acc) {
                               y[row] = acc;
                               const double2 w = rt[row];
                               const double2 c = cdotacc(w.x, w.y, acc.x, acc.y, mk<double>(e[0], e[1]));
                               e[0] = c.x;
                               e[1] = c.y;
                           });
    store_sys_partials<2, epi_stride(L)>(a.part + a.reg * a.stride, a.stride, q.lb, e);
}

// on the tile loop of the standalone product, as pf = sol_subs(G) blocks of
// kSpBlock threads per block of the map (r~ loaded with the tile, the product
// held in the LDS ring), one partial slot per sub-block,
__global__ __launch_bounds__(kSpBlock) void k_l_At(const LArgs a) {
    const SysBlock q = lblock(a, a.pf);
    if (a.sc->done) return;
    const double2* __restrict__ x = a.src;
    double2* __restrict__ y = a.dst;
    const double2* __restrict__ rt = a.rt;
    double e[2] = {0.0, 0.0};
    tile_loop<double, kHold>(
        q.rw, a.row_ptr, a.col_idx, a.vals, [x](int c) { return x[c]; }, [rt](int64_t row) { return rt[row]; },
        [&](int64_t, double2 acc, double2 w) {
            const double2 c = cdotacc(w.x, w.y, acc.x, acc.y, mk<double>(e[0], e[1]));
            e[0] = c.x;
            e[1] = c.y;
        },
        [y](int64_t row, double2 acc) { y[row] = acc; });
    store_sys_partials<2, kTileLanes, 0, kSpBlock>(a.part + a.reg * a.stride, a.stride, q.lb, e);
}

// and on the sliced operator (15 -> 12.6 us on the 260k-row cabin).
template <bool NT>
__global__ HZ_SLICE_BOUNDS void k_l_As(const LArgs a) {
    const SliceRows q = slice_rows_of(a.one, a.np);
    const Sliced<double> m{a.soff, a.scol, a.vals};
    const FirstSlice f = first_slice(m, q);
    if (a.sc->done) return;
    const double2* __restrict__ x = a.src;
    double2* __restrict__ y = a.dst;
    const double2* __restrict__ rt = a.rt;
    double e[2] = {0.0, 0.0};
    slice_rows<double, NT>(
        m, q, f, a.one.n, [x](int c) { return x[c]; }, [rt](int row) { return rt[row]; },
        [&](int64_t row, double2 acc, double2, double2 w) {
            y[row] = acc;
            const double2 c = cdotacc(w.x, w.y, acc.x, acc.y, mk<double>(e[0], e[1]));
            e[0] = c.x;
            e[1] = c.y;
        });
    slice_store<2>(a.part + a.reg * a.stride, a.stride, q.lb, e);
}

// An element's r_0 .. r_{l-1} and u_0 .. u_{l-1}, as their own steps left
// them, brought to the end of the cycle; op(alpha_j, u_0 of step j) for every
// step.  (U0 = 0 leaves out u_0, which no r_i depends on.)
template <int ELL, int U0, typename Op>
__device__ __forceinline__ void l_catch_up(const LScal* __restrict__ ls, double2 (&r)[ELL + 1], double2 (&u)[ELL + 1],
                                           Op op) {
    if constexpr (U0) op(ls->al[0], u[0]);
#pragma unroll
    for (int j = 1; j < ELL; ++j) {
        const double2 al = ls->al[j], be = ls->be[j];  // uniform: scalar loads
        const double2 na = mk<double>(-al.x, -al.y), nb = mk<double>(-be.x, -be.y);
#pragma unroll
        for (int i = U0 ? 0 : 1; i < j; ++i) u[i] = cfma<double>(nb, u[i], r[i]);
#pragma unroll
        for (int i = 0; i < j; ++i) r[i] = cfma<double>(na, u[i + 1], r[i]);
        if constexpr (U0) op(al, u[0]);
    }
}

template <int ELL>
__device__ __forceinline__ double2 gram_at(const double* g, int p, int qq) {  // <r_p, r_q>, any p, q
    const bool sw = p > qq;
    const int lo = sw ? qq : p, hi = sw ? p : qq;
    const int c = lo * (ELL + 1) - lo * (lo - 1) / 2 + (hi - lo);
    return mk<double>(g[2 * c], sw ? -g[2 * c + 1] : g[2 * c + 1]);
}

// Gram partials of <r_p, r_q>, 0 <= p <= q <= ELL, pair index in row-major
// order of the upper triangle (of the real <r_p, r_p> the real part alone, and
// not <r_0, r_0>: the system does not use the rest); each of the gG blocks sums
// a contiguous chunk of rows in a fixed order.  The threads' sums are added
// through LDS, 16 components at a time (butterflies of 80 sums in every wave
// took about as long as the loads).
template <int ELL>
__global__ __launch_bounds__(kGramBlock) void k_l_gram(const LArgs a) {
    constexpr int NP = (ELL + 1) * (ELL + 2) / 2, PASS = 16, LPC = kGramBlock / PASS, PAD = 16;
    if (a.sc->done) return;  // uniform: one system
    double acc[2 * NP];
#pragma unroll
    for (int c = 0; c < 2 * NP; ++c) acc[c] = 0.0;
    const int64_t chunk = ((int64_t)a.n + a.gG - 1) / a.gG;
    const int64_t i0 = (int64_t)blockIdx.x * chunk, i1 = i0 + chunk < a.n ? i0 + chunk : a.n;
    for (int64_t i = i0 + threadIdx.x; i < i1; i += kGramBlock) {
        double2 r[ELL + 1], u[ELL + 1];
#pragma unroll
        for (int p = 0; p <= ELL; ++p) r[p] = a.r[p][i];
#pragma unroll
        for (int p = 1; p < ELL; ++p) u[p] = a.u[p][i];
        l_catch_up<ELL, 0>(a.ls, r, u, [](double2, double2) {});
        int c = 0;
#pragma unroll
        for (int p = 0; p <= ELL; ++p)
#pragma unroll
            for (int qq = p; qq <= ELL; ++qq, ++c) {
                if (qq == 0) continue;
                if (qq == p) {
                    acc[2 * c] = __builtin_fma(r[p].x, r[p].x, acc[2 * c]);
                    acc[2 * c] = __builtin_fma(r[p].y, r[p].y, acc[2 * c]);
                    continue;
                }
                const double2 d = cdotacc(r[p].x, r[p].y, r[qq].x, r[qq].y, mk<double>(acc[2 * c], acc[2 * c + 1]));
                acc[2 * c] = d.x;
                acc[2 * c + 1] = d.y;
            }
    }
    __shared__ double lds[PASS][kGramBlock + PAD];
    const int mc = threadIdx.x / LPC, ml = threadIdx.x % LPC;
#pragma unroll
    for (int c0 = 0; c0 < 2 * NP; c0 += PASS) {
        if (c0 > 0) __syncthreads();  // lds may be rewritten
#pragma unroll
        for (int c = c0; c < c0 + PASS && c < 2 * NP; ++c) lds[c - c0][threadIdx.x] = acc[c];
        __syncthreads();
        if (c0 + mc < 2 * NP) {  // groups of LPC lanes
            double t = lds[mc][ml];
#pragma unroll
            for (int k = 1; k < PASS; ++k) t += lds[mc][ml + k * LPC];
            t = group_sum<LPC>(t);
            if (ml == 0) a.gpart[(int64_t)blockIdx.x * (2 * kGramPairs) + c0 + mc] = t;
        }
    }
}

// The Gram matrix, then the minimal-residual coefficients by Cholesky of the
// unit-diagonal scaled normal equations.  One block: eight groups of 128
// threads add the Gram blocks' partials (a component per thread, group l the
// blocks l, l + 8, ...), then the first wave factors with an entry of the
// matrix per lane, a column per step (one thread alone took 15 us).
template <int ELL>
__global__ __launch_bounds__(kBlock) void k_l_mr(const LArgs a) {
    constexpr int NP = (ELL + 1) * (ELL + 2) / 2, W = 128, NG = kBlock / W;
    static_assert(2 * NP <= W && ELL <= 8, "a thread per component, a lane per entry");
    SolverScal* sc = a.sc;
    if (sc->done) return;  // uniform: one system
    __shared__ double part[NG][W];
    __shared__ double g[W];
    {
        const int c = threadIdx.x % W, l = threadIdx.x / W, cc = c < 2 * NP ? c : 0;
        double sum = 0.0;
        for (int b0 = l; b0 < a.gG; b0 += 16 * NG) {
            double v[16];
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int b = b0 + k * NG;
                v[k] = a.gpart[(int64_t)(b < a.gG ? b : b0) * (2 * kGramPairs) + cc];
            }
#pragma unroll
            for (int k = 0; k < 16; ++k) sum += b0 + k * NG < a.gG ? v[k] : 0.0;
        }
        part[l][c] = sum;
    }
    __syncthreads();
    if (threadIdx.x < W) {
        double sum = part[0][threadIdx.x];
        for (int l = 1; l < NG; ++l) sum += part[l][threadIdx.x];
        g[threadIdx.x] = sum;
    }
    __syncthreads();
    if (wave_id() != 0) return;
    // lane 8 p + q: entry (p, q) of the scaled system M'_pq = d_p G_pq d_q, d_p = 1 / sqrt(G_pp), p, q = 1 .. ELL;
    // every lane of row p: c'_p = d_p <r_p, r_0>
    const int it = sc->iter, p = threadIdx.x / 8, q = threadIdx.x % 8;
    const int pc = p < ELL ? p : 0, qc = q < ELL ? q : 0;
    const double gpp = gram_at<ELL>(g, pc + 1, pc + 1).x, gqq = gram_at<ELL>(g, qc + 1, qc + 1).x;
    bool ok = __all(__builtin_isfinite(gpp) && gpp > 0.0);
    const double dp = ok ? 1.0 / __builtin_sqrt(gpp) : 0.0, dq = ok ? 1.0 / __builtin_sqrt(gqq) : 0.0;
    double2 M = gram_at<ELL>(g, pc + 1, qc + 1), y = gram_at<ELL>(g, pc + 1, 0);
    M = mk<double>(M.x * dp * dq, M.y * dp * dq);
    y = mk<double>(y.x * dp, y.y * dp);
    auto from = [](double2 v, int lane) { return mk<double>(__shfl(v.x, lane), __shfl(v.y, lane)); };
#pragma unroll
    for (int k = 0; k < ELL; ++k) {  // M' = L L^H, and L z = c' with it
        const double mkk = __shfl(M.x, 9 * k);
        ok = ok && __builtin_isfinite(mkk) && mkk > 0.0;
        const double lkk = ok ? __builtin_sqrt(mkk) : 1.0;
        if (q == k) M = p == k ? mk<double>(lkk, 0.0) : mk<double>(M.x / lkk, M.y / lkk);
        const double2 lp = from(M, 8 * p + k), lq = from(M, 8 * q + k);
        if (q > k) {  // M_pq -= L_pk conj(L_qk)
            M.x -= lp.x * lq.x + lp.y * lq.y;
            M.y -= lp.y * lq.x - lp.x * lq.y;
        }
        if (p == k) y = mk<double>(y.x / lkk, y.y / lkk);
        const double2 t = zmul(lp, from(y, 8 * k));
        if (p > k) y = mk<double>(y.x - t.x, y.y - t.y);
    }
    if (!ok) {
        if (threadIdx.x == 0) {
            a.ls->late = ELL;
            finish(sc, a.ndone, ST_BREAKDOWN, it - 1, BD_MR);
        }
        return;
    }
#pragma unroll
    for (int k = ELL - 1; k >= 0; --k) {  // L^H gamma' = z
        const double lkk = __shfl(M.x, 9 * k);
        if (p == k) y = mk<double>(y.x / lkk, y.y / lkk);
        const double2 l = from(M, 8 * k + pc), z = from(y, 8 * k);  // (L^H)_pk = conj(L_kp)
        if (p < k) {
            y.x -= l.x * z.x + l.y * z.y;
            y.y -= l.x * z.y - l.y * z.x;
        }
    }
    const double2 gm = mk<double>(y.x * dp, y.y * dp);  // gamma = D gamma'
    const bool fin = __all(p >= ELL || zfinite(gm));
    if (p < ELL && q == 0) a.gam[p + 1] = gm;
    const double2 om = from(gm, 8 * (ELL - 1));
    if (threadIdx.x != 0) return;
    if (!fin || zzero(om)) {
        a.ls->late = ELL;
        if (!fin) finish(sc, a.ndone, ST_NONFINITE, it - 1);
        else finish(sc, a.ndone, ST_BREAKDOWN, it, BD_OMEGA);
        return;
    }
    sc->omega = om;
    sc->iter = it + 1;
    sc->iters = it;
}

// The cycle's end: x, r_0 and u_0 of the next one; partials <r~, r_0>, ||r_0||^2 for its first step
template <int ELL>
__global__ __launch_bounds__(kLUpBlock, 4) void k_l_update(const LArgs a) {
    if (a.sc->done) return;
    double e[3] = {0.0, 0.0, 0.0};
    for (int64_t i = (int64_t)blockIdx.x * kLUpBlock + threadIdx.x; i < a.n; i += (int64_t)a.uG * kLUpBlock) {
        double2 r[ELL + 1], u[ELL + 1];
#pragma unroll
        for (int p = 0; p <= ELL; ++p) r[p] = a.r[p][i];
#pragma unroll
        for (int p = 0; p <= ELL; ++p) u[p] = a.u[p][i];
        double2 x = a.x[i];
        const double2 w = a.rt[i];
        l_catch_up<ELL, 1>(a.ls, r, u, [&](double2 al, double2 u0) { x = cfma<double>(al, u0, x); });
        double2 r0 = r[0], u0 = u[0];
#pragma unroll
        for (int p = 1; p <= ELL; ++p) {
            const double2 gm = a.gam[p], ng = mk<double>(-gm.x, -gm.y);  // uniform: scalar loads
            x = cfma<double>(gm, r[p - 1], x);
            r0 = cfma<double>(ng, r[p], r0);
            u0 = cfma<double>(ng, u[p], u0);
        }
        a.x[i] = x;
        a.rp[0][i] = r0;
        a.up[0][i] = u0;
        const double2 c = cdotacc(w.x, w.y, r0.x, r0.y, mk<double>(e[0], e[1]));
        e[0] = c.x;
        e[1] = c.y;
        e[2] = __builtin_fma(r0.x, r0.x, e[2]);
        e[2] = __builtin_fma(r0.y, r0.y, e[2]);
    }
    store_sys_partials<3, 1, 0, kLUpBlock>(a.part + kPartC * a.stride, a.stride, blockIdx.x, e);
}

// After the loop: x += sum_j alpha_j u_0 over the complete steps of a cycle
// that ended the solve (a breakdown or a non-finite scalar).
__global__ __launch_bounds__(kLUpBlock) void k_l_late(const LArgs a) {
    const int m = a.ls->late;
    if (m <= 0) return;
    for (int64_t i = (int64_t)blockIdx.x * kLUpBlock + threadIdx.x; i < a.n; i += (int64_t)gridDim.x * kLUpBlock) {
        double2 x = cfma<double>(a.ls->al[0], a.u[0][i], a.x[i]);
        for (int j = 1; j < m; ++j) {
            const double2 al = a.ls->al[j], be = a.ls->be[j];
            const double2 na = mk<double>(-al.x, -al.y), nb = mk<double>(-be.x, -be.y);
            for (int p = 0; p < j; ++p) a.u[p][i] = cfma<double>(nb, a.u[p][i], a.r[p][i]);
            for (int p = 0; p < j; ++p) a.r[p][i] = cfma<double>(na, a.u[p + 1][i], a.r[p][i]);
            x = cfma<double>(al, a.u[0][i], x);
        }
        a.x[i] = x;
    }
}

}  // namespace hz
