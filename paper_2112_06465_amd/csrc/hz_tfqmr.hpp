// TFQMR: the paper's P-TFQMR (Section 7, iterative Krylov methods), Freund's
// transpose-free QMR in the form of Saad's book.  One system, on the
// one-system work map of the BiCGStab kernels, their device scalars
// (SolverScal: rho, alpha, bnorm, rtol, status ...) and partial regions.
//
// Full iteration k (half steps m = 2k - 2, even, and m + 1, odd), four
// launches:
//   K1 (element-wise): alpha = rho / <r~, v>; u' = u - alpha v
//   K2 (product): A u' and, per row: w1 = w - alpha A u, w = w1 - alpha A u';
//       partials ||w1||^2, ||w||^2, <r~, w>
//   K3 (element-wise): theta, c, tau, eta of both half steps from ||w1||^2
//       and ||w||^2 and their quasi-residual tests; beta = rho_new / rho;
//       d1 = u + (theta_m^2 / alpha) eta_m d; x += eta d1;
//       d = u' + (theta^2 / alpha) eta d1;    x += eta d;   u = w + beta u'
//   K4 (product): Au = A u, v = A u + beta (A u' + beta v); partial <r~, v>
// Nothing of the first half step but ||w1||^2 is needed before the second, so
// its vector work waits for K3: 23 vector passes, where K1 and K2 each
// finishing their own half step took 29 and a head in the product.  On small
// systems K1 runs in K2 and K3 in K4, which then gather two vectors and form
// u' or u of a column on the fly (choose_fused); the same arithmetic per
// element.  Measured on the 210k-row cylinder with Jacobi (sliced operator):
// 49.3 -> 38.7 us an iteration.
// tau, theta, eta of the end of iteration k live in slot k & 1 of the TFQMR
// scalars, rho of iteration k in rho2[(k - 1) & 1]: a launch never reads a
// slot its own leader writes.  K1 reads the iteration number `iter` and
// publishes it as `cur`; K3 reads `cur` and advances `iter`.  An exit found by
// K3 still needs every block's share of the last x updates, so it is recorded
// (half_exit, end_exit) instead of ending the solve, and the next K1 (or
// k_q_conclude after the last chunk) concludes it: a block that has not
// started when the leader writes the record must still do its rows.
#pragma once

#include "hz_kernels.hpp"
#include "hz_slices.hpp"

namespace hz {

struct TScal {
    double tau[2], theta[2];  // per parity of the iteration
    double2 eta[2];
    int half_exit;  // iteration whose first half step converged (0: none)
    int end_exit;   // iteration that ended at its second half step (0: none)
    int end_status, end_why;
};

struct QArgs {
    int G, stride;
    OneMap one;
    int* ndone;
    const int* __restrict__ row_ptr;
    const int* __restrict__ col_idx;
    const double2* __restrict__ vals;
    const int* __restrict__ soff;  // the sliced operator's offsets and columns, or null
    const short* __restrict__ scol;
    const double2* rt;  // shadow residual r~
    double2* w;
    double2* u;    // u of the even half step
    double2* u1;   // u' = u - alpha v
    double2* au;   // A u
    double2* au1;  // A u'
    double2* v;
    double2* d;
    double2* x;
    double* part;
    SolverScal* sc;
    TScal* tq;
    int np;  // blocks and partial slots of the products
    int spare;
};

__device__ __forceinline__ SysBlock qblock(const QArgs& a) {
    return map_block(a.one, nullptr, nullptr, a.G, 1, blockIdx.x);
}

// theta, c, tau, eta of a half step from ||w||^2, the previous tau and alpha
struct QStep {
    double theta, tau;
    double2 eta;
};
__device__ __forceinline__ QStep q_step(double ww, double tau_prev, double2 alpha) {
    QStep st;
    st.theta = __builtin_sqrt(ww) / tau_prev;
    const double c2 = 1.0 / (1.0 + st.theta * st.theta);
    st.tau = tau_prev * st.theta * __builtin_sqrt(c2);
    st.eta = mk<double>(c2 * alpha.x, c2 * alpha.y);
    return st;
}

// (theta^2 / alpha) eta
__device__ __forceinline__ double2 q_dcoef(double theta, double2 eta, double2 alpha) {
    const double2 t = zdiv(eta, alpha);
    return mk<double>(theta * theta * t.x, theta * theta * t.y);
}

// TFQMR set-up: rho_0 = <r~, r_0>, tau_0 = ||r_0|| from the set-up partials
__global__ __launch_bounds__(kBlock) void k_q_fin_init(const QArgs a) {
    double h[3];
    sys_sum<3>(a.part + kPartC * a.stride, a.stride, 0, a.G, h);
    if (threadIdx.x != 0) return;
    a.sc->rho2[0] = mk<double>(h[0], h[1]);
    a.tq->tau[0] = __builtin_sqrt(h[2]);
    a.tq->theta[0] = 0.0;
    a.tq->eta[0] = mk<double>(0.0, 0.0);
    a.tq->half_exit = 0;
    a.tq->end_exit = 0;
    a.tq->end_status = ST_NOT_CONVERGED;
    a.tq->end_why = BD_NONE;
}

// Leader of system 0: end the solve recorded by K2 or K3.  Returns whether
// one was recorded (then every block of the launch returns).
__device__ __forceinline__ bool q_conclude(const QArgs& a, bool leader) {
    const int he = a.tq->half_exit, ee = a.tq->end_exit;
    if (he == 0 && ee == 0) return false;
    if (leader) {
        if (he) finish(a.sc, a.ndone, ST_OK, he);
        else finish(a.sc, a.ndone, a.tq->end_status, ee, a.tq->end_why);
    }
    return true;
}

// After the last chunk: conclude an exit recorded by its last launches.
__global__ void k_q_conclude(const QArgs a) {
    if (a.sc->done) return;
    q_conclude(a, threadIdx.x == 0);
}

// Head of K1, and of K2 where it contains K1: alpha.  run() returns false when
// the solve has ended (every block returns); the leader records it.  Scalars
// in the first wave only, as in the BiCGStab heads.
template <int NT = kBlock> struct QAlpha {
    PartSum<2, NT, head_shares(2, NT)> ps;  // (both forms add in one order)
    int done, it;
    double2 rho;

    __device__ __forceinline__ void load(const QArgs& a) {
        done = a.sc->done;
        it = a.sc->iter;
        const double2 r0 = a.sc->rho2[0], r1 = a.sc->rho2[1];
        rho = (it & 1) ? r0 : r1;
        if (ps.comp() < 2) ps.load(a.part + (kPartA + ps.comp()) * a.stride, a.np);
    }
    __device__ __forceinline__ bool run(const QArgs& a, bool leader, double2& alpha) {
        __shared__ double tot[decltype(ps)::TOT];
        __shared__ double2 al;
        __shared__ int go;
        if (ps.comp() < 2) ps.store(tot);
        __syncthreads();
        if (wave_id() == 0) {
            double2 c = mk<double>(0.0, 0.0);
            const int g = decide(a, leader, mk<double>(ps.at(tot, 0), ps.at(tot, 1)), c);
            if (threadIdx.x == 0) {
                al = c;
                go = g;
            }
        }
        __syncthreads();
        alpha = al;
        return go != 0;
    }
    __device__ __forceinline__ int decide(const QArgs& a, bool leader, double2 sigma, double2& alpha) {
        if (done || q_conclude(a, leader)) return 0;
        int st = -1, why = BD_NONE;
        if (!zfinite(sigma) || !zfinite(rho)) st = ST_NONFINITE;
        else if (zzero(sigma)) st = ST_BREAKDOWN, why = BD_RHAT_V;
        else if (zzero(rho)) st = ST_BREAKDOWN, why = BD_RHO;
        else {
            alpha = zdiv(rho, sigma);
            if (!zfinite(alpha)) st = ST_NONFINITE;
        }
        if (leader) {
            if (st >= 0) {
                finish(a.sc, a.ndone, st, it - 1, why);
            } else {
                a.sc->alpha = alpha;
                a.sc->cur = it;
            }
        }
        return st < 0;
    }
};

// K1: u' = u - alpha v
__global__ HZ_STREAM_BOUNDS void k_q_dir1(const QArgs a) {
    const SysBlock q = qblock(a);
    QAlpha<> hd;
    hd.load(a);
    int64_t i = q.rw.x0 + (int64_t)q.rw.k * kBlock + threadIdx.x;
    const int64_t step = (int64_t)q.rw.K * kBlock;
    double2 u0 = mk<double>(0.0, 0.0), v0 = u0;
    if (i < q.rw.x1) {
        u0 = a.u[i];
        v0 = a.v[i];
    }
    double2 alpha;
    if (!hd.run(a, sys_leader(q), alpha)) return;
    const double2 na = mk<double>(-alpha.x, -alpha.y);
    while (i < q.rw.x1) {
        const int64_t at = i;
        const double2 d = cfma<double>(na, v0, u0);
        i += step;
        if (i < q.rw.x1) {
            u0 = a.u[i];
            v0 = a.v[i];
        }
        a.u1[at] = d;
    }
}

// Scalars of K3, and what an element needs of them.
enum : int { Q_STOP = 0, Q_HALF = 1, Q_LAST1 = 2, Q_LAST = 3, Q_FULL = 4 };  // HALF: to d1; LAST1: x of d1 only; LAST: both
struct QCoef {
    double2 dc0, eta1, dc1, eta2, beta;
    int mode, spare;
};
template <int NT = kBlock> struct QEnd {
    PartSum<4, NT, head_shares(4, NT)> ps;
    int done, it, maxit;
    double bnorm, rtol, tau0, theta0;
    double2 alpha, rho_old, eta0;

    __device__ __forceinline__ void load(const QArgs& a) {
        const SolverScal* sc = a.sc;
        done = sc->done;
        it = sc->cur;
        maxit = sc->maxiter;
        bnorm = sc->bnorm;
        rtol = sc->rtol;
        alpha = sc->alpha;
        if (ps.comp() < 4) ps.load(a.part + (kPartB + ps.comp()) * a.stride, a.np);
        const double2 r0 = sc->rho2[0], r1 = sc->rho2[1];
        rho_old = (it & 1) ? r0 : r1;
        const TScal* t = a.tq;
        const bool odd = (it & 1) != 0;  // iteration k reads the slot (k - 1) & 1
        tau0 = odd ? t->tau[0] : t->tau[1];
        theta0 = odd ? t->theta[0] : t->theta[1];
        eta0 = odd ? t->eta[0] : t->eta[1];
    }
    __device__ __forceinline__ const QCoef& run(const QArgs& a, bool leader) {
        __shared__ double tot[decltype(ps)::TOT];
        __shared__ QCoef cf;
        if (ps.comp() < 4) ps.store(tot);
        __syncthreads();
        if (wave_id() == 0) {
            QCoef c;
            c.mode = decide(a, leader, ps.at(tot, 0), ps.at(tot, 1), mk<double>(ps.at(tot, 2), ps.at(tot, 3)), c);
            if (threadIdx.x == 0) cf = c;
        }
        __syncthreads();
        return cf;
    }
    __device__ __forceinline__ int decide(const QArgs& a, bool leader, double ww1, double ww2, double2 rho_new,
                                          QCoef& c) {
        c.dc0 = c.eta1 = c.dc1 = c.eta2 = c.beta = mk<double>(0.0, 0.0);
        c.spare = 0;
        if (done) return Q_STOP;
        SolverScal* sc = a.sc;
        const QStep s1 = q_step(ww1, tau0, alpha);
        const int m1 = 2 * it - 1;  // the first half step's index + 1 (m + 1 with m = 2 it - 2)
        const double bound1 = __builtin_sqrt((double)(m1 + 1)) * s1.tau / bnorm;
        if (!__builtin_isfinite(bound1)) {  // no block writes x: ending at once is safe
            if (leader) finish(sc, a.ndone, ST_NONFINITE, it);
            return Q_STOP;
        }
        c.dc0 = q_dcoef(theta0, eta0, alpha);
        c.eta1 = s1.eta;
        if (bound1 <= rtol) {  // x_{m+1} = x_m + eta d solves: apply, and record a half-step exit
            if (leader) {
                sc->relres = bound1;
                a.tq->half_exit = it;
            }
            return Q_HALF;
        }
        const QStep s2 = q_step(ww2, s1.tau, alpha);
        c.dc1 = q_dcoef(s1.theta, s1.eta, alpha);
        c.eta2 = s2.eta;
        const int m2 = 2 * it;  // half step index + 1 of the iterate this launch completes
        const double bound = __builtin_sqrt((double)(m2 + 1)) * s2.tau / bnorm;
        int st = -1, why = BD_NONE;
        if (!__builtin_isfinite(bound) || !zfinite(rho_new)) st = ST_NONFINITE;
        else if (bound <= rtol) st = ST_OK;
        else if (it >= maxit) st = ST_NOT_CONVERGED;
        else if (zzero(rho_old)) st = ST_BREAKDOWN, why = BD_RHO;
        else {
            c.beta = zdiv(rho_new, rho_old);
            if (!zfinite(c.beta)) st = ST_NONFINITE;
        }
        if (leader) {
            sc->relres = bound;
            if (st >= 0) {  // the next K1 ends the solve
                a.tq->end_status = st;
                a.tq->end_why = why;
                a.tq->end_exit = it;
            } else {
                a.tq->tau[it & 1] = s2.tau;
                a.tq->theta[it & 1] = s2.theta;
                a.tq->eta[it & 1] = s2.eta;
                sc->rho2[it & 1] = rho_new;
                sc->beta = c.beta;
                sc->iter = it + 1;
                sc->iters = it;
            }
        }
        if (st < 0) return Q_FULL;
        return st == ST_NONFINITE ? Q_LAST1 : Q_LAST;  // x_{m+2} = x_{m+1} + eta d is the last iterate
    }
};
// The x and d updates of an element.
__device__ __forceinline__ void q_update(const QCoef& c, double2 u, double2 u1, double2& d, double2& x) {
    d = cfma<double>(c.dc0, d, u);
    x = cfma<double>(c.eta1, d, x);
    if (c.mode < Q_LAST) return;
    d = cfma<double>(c.dc1, d, u1);
    x = cfma<double>(c.eta2, d, x);
}
// The last x of a solve that ends.
__device__ __forceinline__ void q_last(const QArgs& a, const QCoef& c, int64_t i0, int64_t step, int64_t end) {
    for (int64_t i = i0; i < end; i += step) {
        double2 d = a.d[i], x = a.x[i];
        q_update(c, a.u[i], a.u1[i], d, x);
        a.x[i] = x;
    }
}

// K3: x, d and u = w + beta u'
__global__ HZ_STREAM_BOUNDS void k_q_dir2(const QArgs a) {
    const SysBlock q = qblock(a);
    QEnd<> hd;
    hd.load(a);
    // the first element's d, x and u are in flight during the head (all five: 16 of 64 registers spilled)
    const int i0 = (int)q.rw.x0 + q.rw.k * kBlock + threadIdx.x, step = q.rw.K * kBlock, end = (int)q.rw.x1;
    double2 d = mk<double>(0.0, 0.0), x = d, u = d;
    if (i0 < end) {
        d = a.d[i0];
        x = a.x[i0];
        u = a.u[i0];
    }
    const QCoef& c = hd.run(a, sys_leader(q));
    if (c.mode == Q_STOP) return;
    if (c.mode != Q_FULL) return q_last(a, c, i0, step, end);
    for (int i = i0; i < end;) {
        const int j = i;
        const double2 u1 = a.u1[j], w = a.w[j];
        double2 dn = d, xn = x;
        q_update(c, u, u1, dn, xn);
        i = i < end - step ? i + step : end;
        if (i < end) {
            d = a.d[i];
            x = a.x[i];
            u = a.u[i];
        }
        a.x[j] = xn;
        a.d[j] = dn;
        a.u[j] = cfma<double>(c.beta, u1, w);
    }
}

// The products.  A row's part of K2: w, A u'; sums ||w1||^2, ||w||^2, <r~, w>
struct QRow2 {
    double2 w, au, rt;
};
__device__ __forceinline__ QRow2 q_row2(const QArgs& a, int64_t row) { return QRow2{a.w[row], a.au[row], a.rt[row]}; }
__device__ __forceinline__ void q_end2(const QArgs& a, int64_t row, double2 na, double2 acc, const QRow2& p,
                                       double (&e)[4]) {
    const double2 w1 = cfma<double>(na, p.au, p.w);
    const double2 w = cfma<double>(na, acc, w1);
    a.w[row] = w;
    a.au1[row] = acc;
    e[0] = __builtin_fma(w1.x, w1.x, e[0]);
    e[0] = __builtin_fma(w1.y, w1.y, e[0]);
    e[1] = __builtin_fma(w.x, w.x, e[1]);
    e[1] = __builtin_fma(w.y, w.y, e[1]);
    const double2 c = cdotacc(p.rt.x, p.rt.y, w.x, w.y, mk<double>(e[2], e[3]));
    e[2] = c.x;
    e[3] = c.y;
}
// A row's part of K4: A u and v; sum <r~, v>
struct QRow4 {
    double2 v, au1, rt;
};
__device__ __forceinline__ QRow4 q_row4(const QArgs& a, int64_t row) { return QRow4{a.v[row], a.au1[row], a.rt[row]}; }
__device__ __forceinline__ void q_end4(const QArgs& a, int64_t row, double2 beta, double2 acc, const QRow4& p,
                                       double (&e)[2]) {
    a.au[row] = acc;
    const double2 inner = cfma<double>(beta, p.v, p.au1);  // A u' + beta v
    const double2 vv = cfma<double>(beta, inner, acc);
    a.v[row] = vv;
    const double2 c = cdotacc(p.rt.x, p.rt.y, vv.x, vv.y, mk<double>(e[0], e[1]));
    e[0] = c.x;
    e[1] = c.y;
}
// A row's part of the set-up: u = w = r_0, v = Au = A r_0, d = 0; sum <r~, v>
__device__ __forceinline__ void q_end0(const QArgs& a, int64_t row, double2 r0, double2 acc, double (&e)[2]) {
    a.u[row] = r0;
    a.w[row] = r0;
    a.au[row] = acc;
    a.v[row] = acc;
    a.d[row] = mk<double>(0.0, 0.0);
    const double2 t = a.rt[row];
    const double2 c = cdotacc(t.x, t.y, acc.x, acc.y, mk<double>(e[0], e[1]));
    e[0] = c.x;
    e[1] = c.y;
}

// On the CSR operator.
template <int L, int U>
__global__ HZ_STREAM_BOUNDS void k_q_init(const QArgs a, const double2* __restrict__ r0) {
    const SysBlock q = qblock(a);
    double e[2] = {0.0, 0.0};
    for_rows<double, L, U>(q.rw, a.row_ptr, a.col_idx, a.vals, [r0](int c) { return r0[c]; },
                           [&](int64_t row, double2 acc) { q_end0(a, row, r0[row], acc, e); });
    store_sys_partials<2, epi_stride(L)>(a.part + kPartA * a.stride, a.stride, q.lb, e);
}

template <int L, int U, bool FUSED>
__global__ HZ_STREAM_BOUNDS void k_q_prod2(const QArgs a) {
    const SysBlock q = qblock(a);
    double2 alpha;
    if constexpr (FUSED) {
        QAlpha<> hd;
        hd.load(a);
        if (!hd.run(a, sys_leader(q), alpha)) return;
    } else {
        if (a.sc->done) return;
        alpha = a.sc->alpha;
    }
    const double2 na = mk<double>(-alpha.x, -alpha.y);
    const double2* __restrict__ u = a.u;
    const double2* __restrict__ v = a.v;
    const double2* __restrict__ u1 = a.u1;
    auto col = [=](int c) {
        if constexpr (FUSED) return cfma<double>(na, v[c], u[c]);
        else return u1[c];
    };
    double e[4] = {0.0, 0.0, 0.0, 0.0};
    for_rows<double, L, U>(q.rw, a.row_ptr, a.col_idx, a.vals, col, [&](int64_t row, double2 acc) {
        if constexpr (FUSED) a.u1[row] = col((int)row);
        q_end2(a, row, na, acc, q_row2(a, row), e);
    });
    store_sys_partials<4, epi_stride(L)>(a.part + kPartB * a.stride, a.stride, q.lb, e);
}

template <int L, int U, bool FUSED>
__global__ HZ_STREAM_BOUNDS void k_q_prod4(const QArgs a) {
    const SysBlock q = qblock(a);
    if constexpr (FUSED) {
        QEnd<> hd;
        hd.load(a);
        const QCoef& c = hd.run(a, sys_leader(q));
        if (c.mode == Q_STOP) return;
        if (c.mode != Q_FULL)
            return q_last(a, c, q.rw.x0 + (int64_t)q.rw.k * kBlock + threadIdx.x, (int64_t)q.rw.K * kBlock, q.rw.x1);
        const double2 beta = c.beta;
        const double2* __restrict__ w = a.w;
        const double2* __restrict__ u1 = a.u1;
        auto col = [=](int k) { return cfma<double>(beta, u1[k], w[k]); };
        double e[2] = {0.0, 0.0};
        for_rows<double, L, U>(q.rw, a.row_ptr, a.col_idx, a.vals, col, [&](int64_t row, double2 acc) {
            double2 d = a.d[row], x = a.x[row];
            q_update(c, a.u[row], u1[row], d, x);
            a.x[row] = x;
            a.d[row] = d;
            a.u[row] = col((int)row);
            q_end4(a, row, beta, acc, q_row4(a, row), e);
        });
        store_sys_partials<2, epi_stride(L)>(a.part + kPartA * a.stride, a.stride, q.lb, e);
    } else {
        if (a.sc->done || a.tq->half_exit || a.tq->end_exit) return;
        const double2 beta = a.sc->beta;
        const double2* __restrict__ u = a.u;
        double e[2] = {0.0, 0.0};
        for_rows<double, L, U>(q.rw, a.row_ptr, a.col_idx, a.vals, [u](int c) { return u[c]; },
                               [&](int64_t row, double2 acc) { q_end4(a, row, beta, acc, q_row4(a, row), e); });
        store_sys_partials<2, epi_stride(L)>(a.part + kPartA * a.stride, a.stride, q.lb, e);
    }
}

// On the sliced operator.  (The fused ones without a register limit, as
// BiCGStab's.)
__device__ __forceinline__ Sliced<double> sliced_of(const QArgs& a) { return Sliced<double>{a.soff, a.scol, a.vals}; }
__device__ __forceinline__ bool slice_leader(const SliceRows& q) { return q.lb == 0 && threadIdx.x == 0; }

__global__ HZ_SLICE_BOUNDS void k_q_inits(const QArgs a, const double2* __restrict__ r0) {
    const SliceRows q = slice_rows_of(a.one, a.np);
    double e[2] = {0.0, 0.0};
    slice_rows<double, false>(
        sliced_of(a), q, first_slice(sliced_of(a), q), a.one.n, [r0](int c) { return r0[c]; }, [](int) { return 0; },
        [&](int64_t row, double2 acc, double2 self, int) { q_end0(a, row, self, acc, e); });
    slice_store<2>(a.part + kPartA * a.stride, a.stride, q.lb, e);
}

template <bool NT>
__global__ HZ_SLICE_BOUNDS void k_q_prod2s(const QArgs a) {
    const SliceRows q = slice_rows_of(a.one, a.np);
    const FirstSlice f = first_slice(sliced_of(a), q);
    if (a.sc->done) return;
    const double2 alpha = a.sc->alpha, na = mk<double>(-alpha.x, -alpha.y);
    const double2* __restrict__ u1 = a.u1;
    double e[4] = {0.0, 0.0, 0.0, 0.0};
    slice_rows<double, NT>(
        sliced_of(a), q, f, a.one.n, [u1](int c) { return u1[c]; }, [&a](int row) { return q_row2(a, row); },
        [&](int64_t row, double2 acc, double2, const QRow2& p) { q_end2(a, row, na, acc, p, e); });
    slice_store<4>(a.part + kPartB * a.stride, a.stride, q.lb, e);
}

__global__ __launch_bounds__(kSlBlock) void k_q_prod2sf(const QArgs a) {
    const SliceRows q = slice_rows_of(a.one, a.np);
    const FirstSlice f = first_slice(sliced_of(a), q);
    QAlpha<kSlBlock> hd;
    hd.load(a);
    double2 alpha;
    if (!hd.run(a, slice_leader(q), alpha)) return;
    const double2 na = mk<double>(-alpha.x, -alpha.y);
    const double2* __restrict__ u = a.u;
    const double2* __restrict__ v = a.v;
    double e[4] = {0.0, 0.0, 0.0, 0.0};
    slice_rows<double, false>(
        sliced_of(a), q, f, a.one.n, [=](int c) { return cfma<double>(na, v[c], u[c]); },
        [&a](int row) { return q_row2(a, row); },
        [&](int64_t row, double2 acc, double2 self, const QRow2& p) {
            a.u1[row] = self;
            q_end2(a, row, na, acc, p, e);
        });
    slice_store<4>(a.part + kPartB * a.stride, a.stride, q.lb, e);
}

template <bool NT>
__global__ HZ_SLICE_BOUNDS void k_q_prod4s(const QArgs a) {
    const SliceRows q = slice_rows_of(a.one, a.np);
    const FirstSlice f = first_slice(sliced_of(a), q);
    if (a.sc->done || a.tq->half_exit || a.tq->end_exit) return;
    const double2 beta = a.sc->beta;
    const double2* __restrict__ u = a.u;
    double e[2] = {0.0, 0.0};
    slice_rows<double, NT>(
        sliced_of(a), q, f, a.one.n, [u](int c) { return u[c]; }, [&a](int row) { return q_row4(a, row); },
        [&](int64_t row, double2 acc, double2, const QRow4& p) { q_end4(a, row, beta, acc, p, e); });
    slice_store<2>(a.part + kPartA * a.stride, a.stride, q.lb, e);
}

__global__ __launch_bounds__(kSlBlock) void k_q_prod4sf(const QArgs a) {
    const SliceRows q = slice_rows_of(a.one, a.np);
    const FirstSlice f = first_slice(sliced_of(a), q);
    QEnd<kSlBlock> hd;
    hd.load(a);
    const QCoef& c = hd.run(a, slice_leader(q));
    if (c.mode == Q_STOP) return;
    if (c.mode != Q_FULL)  // its rows are those of the grid's stride
        return q_last(a, c, (int64_t)blockIdx.x * kSlBlock + threadIdx.x, (int64_t)a.np * kSlBlock, a.one.n);
    const double2 beta = c.beta;
    const double2* __restrict__ w = a.w;
    const double2* __restrict__ u1 = a.u1;
    double e[2] = {0.0, 0.0};
    slice_rows<double, false>(
        sliced_of(a), q, f, a.one.n, [=](int k) { return cfma<double>(beta, u1[k], w[k]); },
        [&a](int row) { return q_row4(a, row); },
        [&](int64_t row, double2 acc, double2 self, const QRow4& p) {
            double2 d = a.d[row], x = a.x[row];
            q_update(c, a.u[row], u1[row], d, x);
            a.x[row] = x;
            a.d[row] = d;
            a.u[row] = self;
            q_end4(a, row, beta, acc, p, e);
        });
    slice_store<2>(a.part + kPartA * a.stride, a.stride, q.lb, e);
}

}  // namespace hz
