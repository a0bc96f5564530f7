// The two row products of the BiCGStab iteration (Section 7: v = A p with
// <rhat, v>, and t = A s with its dot products) in the standalone product's
// tile form, for one large system in CSR: without Jacobi, or with a matrix
// that is not sliced (BiCGstab(l)'s product, with the same structure, is in
// hz_bicgstabl.hpp).
//
// The solver's other kernels run 1024-thread blocks, at most kMaxGrid of
// them, and under their 64-VGPR budget a product could not hold its results
// back without spilling; its stores then sat in front of the next tile's
// loads (one in-order counter tracks both).  These kernels run each logical
// block of the solver's map as F = sol_subs(G) blocks of kSpBlock threads
// (half the waves per CU at most, twice the registers per wave) through
// tile_loop with its LDS ring: the epilogue operands of each row (rhat, or s
// and rhat) are loaded with the tile's matrix entries and the row's terms go into the block's dot products
// as soon as the tile is summed, while the totals v (or t) are held for kHold
// tiles and stored when the ring is flushed.  Sub-block j of logical block lb
// takes 64-row tiles j, j + F K, ... of its group's rows, and writes its
// partials to a slot of its own; the regions' readers sum F slots per block
// (BicgArgs::np = F G).  Sums are taken in a fixed order: results are bitwise
// reproducible.
#pragma once

#include "hz_spmv.hpp"

namespace hz {

constexpr int kSolSlots = 1024;  // partial slots per component that the sub-blocks of a launch may take

// Product blocks per logical block of a map of G blocks: enough for about
// kSolSlots blocks (four per CU, the residency that the tile loop's 36 KB of
// LDS allows), at least 2 and at most 4, and F G <= max(2 G, kSolSlots).
__host__ __device__ constexpr int sol_subs(int G) {
    const int f = G > 0 ? kSolSlots / G : 4;
    return f < 2 ? 2 : (f > 4 ? 4 : f);
}

template <typename T, bool PAST> __device__ __forceinline__ void bicg_At(const BicgArgs<T>& a) {
    const SysBlock q = map_block(a.one, a.bmap, a.smap, a.G, a.pf, blockIdx.x);
    if (q.sys < 0) return;
    if (ended<PAST>(a.sc + q.sys, sys_leader(q))) return;
    zero_slots(a, kPartA, 2, q.lb, a.pf * a.G, threadIdx.x == 0);
    const cx<T>* __restrict__ p = a.p;
    cx<T>* __restrict__ v = a.v;
    const cx<T>* __restrict__ rh = a.rh;
    double e[2] = {0.0, 0.0};
    tile_loop<T, kHold>(
        q.rw, a.row_ptr, a.col_idx, a.vals, [p](int c) { return p[c]; }, [rh](int64_t row) { return rh[row]; },
        [&](int64_t, cx<T> acc, cx<T> w) {
            const double2 c = cdotacc(w.x, w.y, acc.x, acc.y, mk<double>(e[0], e[1]));
            e[0] = c.x;
            e[1] = c.y;
        },
        [v](int64_t row, cx<T> acc) { v[row] = acc; });
    store_sys_partials<2, kTileLanes, 0, kSpBlock>(a.part + kPartA * a.stride, a.stride, q.lb, e);
}

template <typename T, bool PAST = false>
__global__ __launch_bounds__(kSpBlock) void k_bicg_At(const BicgArgs<T> a) {
    if (!past_end<PAST>(a)) bicg_At<T, PAST>(a);
}

template <typename T> __device__ __forceinline__ void bicg_Bt(const BicgArgs<T>& a) {
    const SysBlock q = map_block(a.one, a.bmap, a.smap, a.G, a.pf, blockIdx.x);
    if (q.sys < 0) return;
    if (a.sc[q.sys].done) return;
    zero_slots(a, kPartB, 8, q.lb, a.pf * a.G, threadIdx.x == 0);
    const cx<T>* __restrict__ sv = a.s;
    const cx<T>* __restrict__ rh = a.rh;
    cx<T>* __restrict__ tv = a.t;
    double e[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    tile_loop<T, kHold>(
        q.rw, a.row_ptr, a.col_idx, a.vals, [sv](int c) { return sv[c]; },
        [sv, rh](int64_t row) { return BRow<T>{sv[row], rh[row]}; },
        [&](int64_t, cx<T> acc, BRow<T> m) { b_terms<T>(e, m.s, acc, m.w); },
        [tv](int64_t row, cx<T> acc) { tv[row] = acc; });
    store_sys_partials<8, kTileLanes, 0, kSpBlock>(a.part + kPartB * a.stride, a.stride, q.lb, e);
}
template <typename T, bool PAST = false>
__global__ __launch_bounds__(kSpBlock) void k_bicg_Bt(const BicgArgs<T> a) {
    if (!past_end<PAST>(a)) bicg_Bt<T>(a);
}

}  // namespace hz
