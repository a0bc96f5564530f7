// Mixed precision with reliable updates.
//
// The refinement of zbicgstab_solve_mixed restarts a complex64 BiCGStab for
// every correction, and each restart throws the Krylov space away.  This
// variant keeps one complex64 BiCGStab running on the scaled problem
// A D^{-1} y = b / ||b||, accumulates its iterate y in complex64, and every
// time its recursive residual has fallen by a factor delta (or the inner
// iteration has ended) performs a reliable update (Sleijpen and van der
// Vorst, reliable updated residuals in hybrid Bi-CG methods): the FP64
// iterate takes x += ||b|| D^{-1} y and y restarts from zero, the true
// residual r64 = b - A x is formed in FP64, and the complex64 recursive
// residual is replaced by r64 / ||b|| (with <rhat, r>, ||r||^2 and the
// direction p that were formed from the old one) while v, rhat and the other
// scalars carry on.  Convergence is decided on the
// FP64 true residual only.
#pragma once

#include "hz_kernels.hpp"

namespace hz {

// out = in / ||b||  (complex64), ||b|| from the outer scalars
__global__ __launch_bounds__(kBlock) void k_ru_demote(int n, const double2* __restrict__ in, const SolverScal* sc,
                                                      float2* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const double inv = 1.0 / sc->bnorm;
    const double2 v = in[i];
    out[i] = mk<float>((float)(v.x * inv), (float)(v.y * inv));
}

// x += ||b|| D^{-1} y in FP64 (D^{-1} as the complex64 operator uses it), then y = 0
__global__ __launch_bounds__(kBlock) void k_ru_promote(int n, float2* __restrict__ y, const float2* __restrict__ dinv,
                                                       const SolverScal* sc, double2* __restrict__ x) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const double bn = sc->bnorm;
    double2 d = mk<double>((double)y[i].x, (double)y[i].y);
    if (dinv != nullptr) d = zmul(mk<double>((double)dinv[i].x, (double)dinv[i].y), d);
    double2 xv = x[i];
    xv.x = __builtin_fma(bn, d.x, xv.x);
    xv.y = __builtin_fma(bn, d.y, xv.y);
    x[i] = xv;
    y[i] = mk<float>(0.0f, 0.0f);
}

// Replace the complex64 recursive residual by r64 / ||b||, in three launches
// between iterations (the next iteration's p, rho and beta were formed from
// the old residual).  First the new residual into s (free here) with its
// partials <rhat, r>, ||r||^2 (region C) ...
__global__ HZ_STREAM_BOUNDS void k_ru_replace(const BicgArgs<float> a, const double2* __restrict__ r64,
                                              const SolverScal* outer) {
    const SysBlock q = sys_block(a);
    if (q.sys < 0) return;
    const double inv = 1.0 / outer->bnorm;
    double e[3] = {0.0, 0.0, 0.0};
    HZ_FOR_ELEMS(i, q.rw) {
        const double2 v = r64[i];
        const float2 r = mk<float>((float)(v.x * inv), (float)(v.y * inv));
        a.s[i] = r;
        const float2 w = a.rh[i];
        const double2 c = cdotacc(w.x, w.y, r.x, r.y, mk<double>(e[0], e[1]));
        e[0] = c.x;
        e[1] = c.y;
        e[2] = __builtin_fma((double)r.x, (double)r.x, e[2]);
        e[2] = __builtin_fma((double)r.y, (double)r.y, e[2]);
    }
    store_sys_partials<3>(a.part + kPartC * a.stride, a.stride, q.lb, e);
}

// ... then p = r_new + (rho_new / rho_old) (p - r_old), which is r_new + beta
// (p_prev - omega v) with the beta of the new rho = <rhat, r_new>; the old
// direction is dropped where rho_old is zero ...
__device__ __forceinline__ double2 ru_factor(const double2 rho_new, const double2 rho_old) {
    if (zzero(rho_old) || !zfinite(rho_old)) return mk<double>(0.0, 0.0);
    return zdiv(rho_new, rho_old);
}
__global__ HZ_STREAM_BOUNDS void k_ru_direction(const BicgArgs<float> a) {
    const SysBlock q = sys_block(a);
    if (q.sys < 0) return;
    const SolverScal* sc = a.sc + q.sys;
    const double2 rho_old = sc->rho2[sc->iter & 1];
    double h[2];
    sys_sum<2>(a.part + kPartC * a.stride, a.stride, q.gbeg, q.gcnt, h);
    const float2 f = narrow<float>(ru_factor(mk<double>(h[0], h[1]), rho_old));
    HZ_FOR_ELEMS(i, q.rw) {
        const float2 rn = a.s[i], ro = a.r[i], p = a.p[i];
        a.p[i] = cfma<float>(f, mk<float>(p.x - ro.x, p.y - ro.y), rn);
        a.r[i] = rn;
    }
}

// ... and last rho and beta of the next iteration (one block).
__global__ HZ_STREAM_BOUNDS void k_ru_rho(const BicgArgs<float> a) {
    double h[2];
    const SysMap sm = sys_range(a, 0);
    sys_sum<2>(a.part + kPartC * a.stride, a.stride, sm.gbeg, sm.gcnt, h);
    if (threadIdx.x != 0) return;
    SolverScal* sc = a.sc;
    const double2 rho = mk<double>(h[0], h[1]);
    sc->beta = zmul(ru_factor(rho, sc->rho2[sc->iter & 1]), sc->beta);
    sc->rho2[sc->iter & 1] = rho;
}

}  // namespace hz
