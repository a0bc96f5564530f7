// The sliced operator of a Jacobi solve, and the row products on it.
//
// A one-system solve under Jacobi scales the matrix once, so it is free to
// store A D^{-1} as its products read it best: slices of 64 consecutive rows,
// entry k of a slice's row g at off + 64 k + g (sliced ELLPACK with slices of
// a wave, rows in order), every row padded to the slice's longest.  One lane
// computes one row, so
//  - a wave's load of entry k is 1 KB of values and 128 bytes of columns,
//    contiguous, and a slice is one contiguous stream;
//  - the entries k of 64 consecutive rows of a mesh have nearly consecutive
//    columns, so a gather touches about 17 cache lines where 64 consecutive
//    entries of four rows touch about 60 (the tile loop's gathers kept the L1
//    busy for half of its time, and its waves waited 74 % of theirs);
//  - no row sum crosses lanes: no LDS, no barrier, a quarter of the
//    instructions of the tile loop.
// The diagonal of A D^{-1} is 1 and is left out, and columns are 16-bit
// offsets from the slice's first row: 18 bytes for 13.6 entries a row of the
// P1 meshes plus 1.6-3.2 % padding, instead of 20 bytes for 14.6 entries.
// Measured: v = A p with its dot product on the 1.24 M-row cabin 82.3 -> 70 us
// (5.6 TB/s of 390 MB), on the 210k-row cylinder 12.7 -> 11.3 us.
//
// A matrix is not sliced when a column is more than 32,767 rows from its
// slice, a row has no diagonal or one without a proper reciprocal
// (k_jacobi_diag), or the padding exceeds the room (irregular rows): the
// set-up kernels find that on the device and leave it in the word
// after the done-counter (slice_no).  The host of a synchronous solve reads
// it with the set-up's other results and launches one form's product kernels;
// an asynchronous solve's contain both forms and read the word themselves
// (hz_either.hpp).
//
// Rows are taken in order, so it is for meshes whose rows are even, as those of
// split hexahedra: a Delaunay mesh of 32,768 jittered points in
// Cuthill-McKee order (16.3 entries a row, the longest 48) would need 1.40 nnz
// slots (0.94 with its rows sorted by length) and stays in CSR.
//
// A row's entries are summed in the order they are stored, every other one of
// a batch in a chain of its own, and added to the diagonal; a padded slot is a
// zero value at the row's own column.  Batches of slots are straight-line (a
// slot past the slice's width reads its last slot and is dropped by a uniform
// branch): with the loads themselves behind uniform branches the compiler
// spilled 60 registers and the product took twice as long.
#pragma once

#include "hz_kernels.hpp"

namespace hz {

constexpr int kSlBlock = 256;            // threads: four waves, one slice each at a time
constexpr int kSlMaxGrid = 1024;         // blocks (= partials) at most: four per CU
constexpr int kSlWaves = kSlBlock / kWave;
#define HZ_SLICE_BOUNDS __launch_bounds__(256, 4)  // four blocks per CU: <= 128 VGPRs

// ------------------------------------------------------------------ set-up

// off[s + 1] = slots of slice s: 64 x (longest row - 1), off[0] = 0.  A row of
// more than kSlLongest entries beside the diagonal repeats columns (16 bits
// tell 65,536 apart) and is not sliced: *no = 1.  So a slice has at most 2^22
// slots, which an int holds (64 x an arbitrary row length it does not).
constexpr int kSlLongest = 1 << 16;
__global__ __launch_bounds__(kSlBlock) void k_slice_width(int n, const int* __restrict__ rp, int* __restrict__ off,
                                                          int* no) {
    const int64_t i = (int64_t)blockIdx.x * kSlBlock + threadIdx.x;
    int len = i < n ? rp[i + 1] - rp[i] - 1 : 0;
    if (len > kSlLongest) {
        *no = 1;  // every writer stores 1
        len = kSlLongest;
    }
#pragma unroll
    for (int s = 1; s < kWave; s *= 2) {
        const int o = __shfl_xor(len, s);
        len = len > o ? len : o;
    }
    if (i == 0) off[0] = 0;
    if (i < n && threadIdx.x % kWave == 0) off[i / kWave + 1] = kWave * (len > 0 ? len : 0);  // i / 64 < 2^25
}

// In-place inclusive scan of off[1 .. ns] by one block; *no = 1 if the slots
// exceed `room` (the offsets are then not used).
__global__ __launch_bounds__(kBlock) void k_slice_scan(int ns, int* __restrict__ off, int64_t room, int* no) {
    __shared__ long long wsum[kBlock / kWave];
    const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
    long long run = 0;
    for (int64_t c = 0; c < ns; c += kBlock) {  // uniform
        const int64_t s = c + threadIdx.x;
        long long v = s < ns ? off[s + 1] : 0;
#pragma unroll
        for (int d = 1; d < kWave; d *= 2) {
            const long long o = __shfl_up(v, d);
            v += lane >= d ? o : 0;
        }
        if (lane == kWave - 1) wsum[wid] = v;
        __syncthreads();
        long long before = run, all = run;
        for (int w = 0; w < kBlock / kWave; ++w) {
            before += w < wid ? wsum[w] : 0;
            all += wsum[w];
        }
        if (s < ns) off[s + 1] = (int)(before + v);
        run = all;
        __syncthreads();  // wsum may be rewritten
    }
    if (threadIdx.x == 0 && run > room) *no = 1;
}

// The slices' values A D^{-1} (rounded to TO for the complex64 iteration) and
// columns; one lane per row.  The diagonal entry that dinv came from (the
// row's last) is left out.  A matrix that is not sliced keeps its pattern
// (k_colscale's work, without a launch more).  Entries go in batches whose loads
// are in flight together, a slot past the row's end read at an entry in bounds
// and dropped: 84 -> 34 us on the 210k-row cylinder and 566 -> 202 us on the
// 1.24 M-row cabin against an entry at a time.
template <typename TO>
__global__ __launch_bounds__(kSlBlock) void k_slice_fill(int n, int nnz, const int* __restrict__ rp,
                                                         const int* __restrict__ ci,
                                                         const double2* __restrict__ vals,
                                                         const double2* __restrict__ dinv,
                                                         const int* __restrict__ off, cx<TO>* __restrict__ out,
                                                         short* __restrict__ col, const int* no) {
    constexpr int U = 8;
    const int64_t i = (int64_t)blockIdx.x * kSlBlock + threadIdx.x;
    if (*no != 0) {
        for (int64_t p = i; p < nnz; p += (int64_t)gridDim.x * kSlBlock) {
            const double2 v = cmul<double>(vals[p], dinv[ci[p]]);
            out[p] = mk<TO>((TO)v.x, (TO)v.y);
        }
        return;
    }
    const int64_t s = i / kWave;
    if (s * kWave >= n) return;  // whole waves
    const int lane = threadIdx.x % kWave, o = off[s], w = (off[s + 1] - o) / kWave;
    const int base = (int)(s * kWave), row = (int)(i < n ? i : n - 1);
    const int beg = rp[row], end = rp[row + 1], last = end - 1;  // a sliced row holds its diagonal: end > beg
    int diag = last;
    for (int p = beg; p < end; p += U) {
        int c[U];
#pragma unroll
        for (int u = 0; u < U; ++u) c[u] = ci[p + u < end ? p + u : last];
#pragma unroll
        for (int u = 0; u < U; ++u) diag = c[u] == row ? (p + u < end ? p + u : last) : diag;
    }
    const int stop = i < n ? last - beg : 0;  // entries beside the diagonal
    for (int k0 = 0; k0 < w; k0 += U) {       // uniform
        int c[U];
        double2 a[U], d[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = beg + k0 + u, p = q < diag ? q : q + 1;
            c[u] = ci[p < end ? p : last];
            a[u] = vals[p < end ? p : last];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) d[u] = dinv[c[u]];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (k0 + u >= w) continue;  // uniform
            const bool in = k0 + u < stop;
            const double2 v = cmul<double>(a[u], d[u]);
            const int64_t at = (int64_t)o + (int64_t)(k0 + u) * kWave + lane;
            out[at] = mk<TO>(in ? (TO)v.x : TO(0), in ? (TO)v.y : TO(0));
            col[at] = (short)(in ? c[u] - base : row - base);  // the padding's column: the row's own
        }
    }
}

// ------------------------------------------------------------------ row products

template <typename T> struct Sliced {
    const int* __restrict__ off;
    const short* __restrict__ col;
    const cx<T>* __restrict__ v;
};

// The rows of a block of a launch of `sg` sliced product blocks over the
// one-system map: group x's blocks take its slices four at a time in turn.
// A kernel of TB > kSlBlock threads does the work of V <= TB / kSlBlock such
// blocks in each of its own (lb < 0: threads beyond, and past the group's last).
struct SliceRows {
    int lb;              // the block's partial slot
    int64_t s, step, s1; // this wave's first slice, the step, the group's end
};
template <int TB = kSlBlock> __device__ __forceinline__ SliceRows slice_rows_of(const OneMap& one, int sg, int V = 1) {
    constexpr bool many = TB > kSlBlock;
    SliceRows q;
    const int b = blockIdx.x, x = one.groups == kXcd ? b % kXcd : 0, v = many ? wave_id() / kSlWaves : 0;
    const int k = (one.groups == kXcd ? b / kXcd : b) * (many ? V : 1) + v;
    const int K = sg / one.groups;
    const int64_t x0 = (int64_t)x * one.gr, x1 = x0 + one.gr < one.n ? x0 + one.gr : one.n;
    q.lb = x * K + k;
    q.s = x0 / kWave + (int64_t)k * kSlWaves + wave_id() % kSlWaves;
    q.step = (int64_t)K * kSlWaves;
    q.s1 = (x1 + kWave - 1) / kWave;
    if (many && (v >= V || k >= K)) {
        q.lb = -1;
        q.s = q.s1;
    }
    return q;
}

template <bool NT, typename P> __device__ __forceinline__ auto ld_if(const P* p) {
    if constexpr (NT) return ld_mat(p);
    else return *p;
}

// A slice's row sums in batches of U slots, all of a batch's loads issued
// before any is used, in two chains that start at zero, added to the diagonal
// at the end: with one chain from the diagonal on, BiCGstab(8), whose residual
// drifts by what its products round, ended at a true residual of 3e-11 on the
// 260k-row cabin (mean of eight systems) instead of 1.4e-11 (1.8e-11 with the
// tile loop's sums); a sum per batch drifts as little and took 1-4 % longer.
// (Issuing the next batch's loads with a batch's gathers gained nothing where
// it fitted the registers, complex64, and spilled in FP64.)
template <typename T, int U, bool NT, typename Op>
__device__ __forceinline__ cx<T> slice_sum(const short* __restrict__ cp, const cx<T>* __restrict__ vp, int base, int w,
                                           cx<T> acc, Op op) {
    cx<T> even = mk<T>(T(0), T(0)), odd = even;
    for (int k0 = 0; k0 < w; k0 += U) {  // uniform
        short c[U];
        cx<T> v[U], g[U];
#pragma unroll
        for (int u = 0; u < U; ++u) c[u] = ld_if<NT>(cp + (k0 + u < w ? k0 + u : w - 1) * kWave);
#pragma unroll
        for (int u = 0; u < U; ++u) v[u] = ld_if<NT>(vp + (k0 + u < w ? k0 + u : w - 1) * kWave);
#pragma unroll
        for (int u = 0; u < U; ++u) g[u] = op(base + c[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (k0 + u >= w) continue;  // uniform
            if (u % 2 == 0) even = cfma<T>(v[u], g[u], even);
            else odd = cfma<T>(v[u], g[u], odd);
        }
    }
    return mk<T>(acc.x + (even.x + odd.x), acc.y + (even.y + odd.y));
}

// The offset and width of a wave's first slice, loaded ahead of a kernel's head.
struct FirstSlice {
    int o = 0, w = 0;
};
template <typename T> __device__ __forceinline__ FirstSlice first_slice(const Sliced<T>& m, const SliceRows& q) {
    FirstSlice f;
    if (q.s < q.s1) {  // uniform
        f.o = m.off[q.s];
        f.w = (m.off[q.s + 1] - f.o) / kWave;
    }
    return f;
}

// epi(row, total, operand of the row, pre(row)) for every row of the wave's
// slices, one lane per row; op(col) is the gathered operand.  A slice's width
// is split into equal batches of 4 to 7 slots.  NT: streaming loads, for
// operators that do not stay in the Infinity Cache (cabin 73 -> 66 us;
// 12.0 -> 12.8 us on the cylinder, which does).
template <typename T, bool NT, typename Op, typename Pre, typename Epi>
__device__ __forceinline__ void slice_rows(const Sliced<T>& m, const SliceRows& q, FirstSlice f, int n, Op op, Pre pre,
                                           Epi epi) {
    const int lane = threadIdx.x % kWave;
    for (int64_t s = q.s; s < q.s1; s += q.step) {  // uniform in the wave
        const int o = f.o, w = f.w;
        if (s + q.step < q.s1) {
            f.o = m.off[s + q.step];
            f.w = (m.off[s + q.step + 1] - f.o) / kWave;
        }
        const int base = (int)(s * kWave), row = base + lane < n ? base + lane : n - 1;
        const cx<T> self = op(row);
        const auto pr = pre(row);
        const short* cp = m.col + (int64_t)o + lane;
        const cx<T>* vp = m.v + (int64_t)o + lane;
        const int nb = (w + 6) / 7, u = nb > 0 ? (w + nb - 1) / nb : 0;
        cx<T> acc = self;
        switch (u) {  // uniform
            case 0: break;
            case 7: acc = slice_sum<T, 7, NT>(cp, vp, base, w, acc, op); break;
            case 6: acc = slice_sum<T, 6, NT>(cp, vp, base, w, acc, op); break;
            case 5: acc = slice_sum<T, 5, NT>(cp, vp, base, w, acc, op); break;
            default: acc = slice_sum<T, 4, NT>(cp, vp, base, w, acc, op); break;
        }
        if (base + lane < n) epi((int64_t)row, acc, self, pr);
    }
}

// The block's totals of K doubles to slot lb of each component, summed through
// LDS (the values of 256 threads per component, then one wave per component at
// a time): with every row in a lane of its own the wave butterflies of eight
// sums would take about 1 us of the SIMDs.  PASS components at a time are in
// LDS; TB > kSlBlock: for each of a thread block's blocks.
template <int K, int TB = kSlBlock, int PASS = K>
__device__ __forceinline__ void slice_store(double* __restrict__ part, int stride, int lb, double (&e)[K]) {
    constexpr int V = TB / kSlBlock;
    __shared__ double l[V][PASS][kSlBlock];
    const int lane = threadIdx.x % kWave, w = wave_id() % kSlWaves, v = V > 1 ? wave_id() / kSlWaves : 0;
#pragma unroll
    for (int p0 = 0; p0 < K; p0 += PASS) {
        if (p0 > 0) __syncthreads();  // l may be rewritten
#pragma unroll
        for (int k = p0; k < p0 + PASS && k < K; ++k) l[v][k - p0][threadIdx.x % kSlBlock] = e[k];
        __syncthreads();
#pragma unroll
        for (int k0 = p0; k0 < p0 + PASS && k0 < K; k0 += kSlWaves) {
            const int k = k0 + w;
            if (k < K && k < p0 + PASS && (V == 1 || lb >= 0)) {
                const double* p = l[v][k - p0] + lane;
                const double t = wave_sum<1>((p[0] + p[kWave]) + (p[2 * kWave] + p[3 * kWave]));
                if (lane == 0) part[k * stride + lb] = t;
            }
        }
    }
}

// ------------------------------------------------------------------ BiCGStab's products on it

template <typename T> __device__ __forceinline__ Sliced<T> sliced_of(const BicgArgs<T>& a) {
    return Sliced<T>{a.soff, a.scol, a.vals};
}
// The first thread of a block (zero_slots).
__device__ __forceinline__ bool slice_first(const SliceRows& q) { return threadIdx.x % kSlBlock == 0 && q.lb >= 0; }

// v = A p; partial <rhat, v>
template <typename T, bool NT, bool PAST = false, int TB = kSlBlock, int PASS = 2>
__device__ __forceinline__ void bicg_As(const BicgArgs<T>& a) {
    const SliceRows q = slice_rows_of<TB>(a.one, a.sg, a.sv);
    const FirstSlice f = first_slice(sliced_of(a), q);
    if (ended<PAST>(a.sc, q.lb == 0 && threadIdx.x == 0)) return;
    zero_slots(a, kPartA, 2, q.lb, a.sg, slice_first(q));
    const cx<T>* __restrict__ p = a.p;
    const cx<T>* __restrict__ rh = a.rh;
    cx<T>* __restrict__ v = a.v;
    double e[2] = {0.0, 0.0};
    slice_rows<T, NT>(
        sliced_of(a), q, f, a.one.n, [p](int c) { return p[c]; }, [rh](int row) { return rh[row]; },
        [&](int64_t row, cx<T> acc, cx<T>, cx<T> w) {
            v[row] = acc;
            const double2 c = cdotacc(w.x, w.y, acc.x, acc.y, mk<double>(e[0], e[1]));
            e[0] = c.x;
            e[1] = c.y;
        });
    slice_store<2, TB, PASS>(a.part + kPartA * a.stride, a.stride, q.lb, e);
}
template <typename T, bool NT>
__global__ HZ_SLICE_BOUNDS void k_bicg_As(const BicgArgs<T> a) {
    bicg_As<T, NT>(a);
}

// t = A s and its dot products
template <typename T, bool NT, int TB = kSlBlock, int PASS = 8>
__device__ __forceinline__ void bicg_Bs(const BicgArgs<T>& a) {
    const SliceRows q = slice_rows_of<TB>(a.one, a.sg, a.sv);
    const FirstSlice f = first_slice(sliced_of(a), q);
    if (a.sc->done) return;
    zero_slots(a, kPartB, 8, q.lb, a.sg, slice_first(q));
    const cx<T>* __restrict__ sv = a.s;
    const cx<T>* __restrict__ rh = a.rh;
    cx<T>* __restrict__ tv = a.t;
    double e[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    slice_rows<T, NT>(
        sliced_of(a), q, f, a.one.n, [sv](int c) { return sv[c]; }, [rh](int row) { return rh[row]; },
        [&](int64_t row, cx<T> acc, cx<T> s, cx<T> w) {
            tv[row] = acc;
            b_terms<T>(e, s, acc, w);
        });
    slice_store<8, TB, PASS>(a.part + kPartB * a.stride, a.stride, q.lb, e);
}
template <typename T, bool NT>
__global__ HZ_SLICE_BOUNDS void k_bicg_Bs(const BicgArgs<T> a) {
    bicg_Bs<T, NT>(a);
}

// p[i]; N32: by a byte offset of 32 bits (i below 2^32 / sizeof), one register
// an address, for the kernels that may have no more than 128 of them (64-bit
// addresses of two vectors' gathers take a batch of 7 to 136).  Where there is
// no such limit 64-bit ones are 1 % faster.
template <bool N32, typename P> __device__ __forceinline__ P& at(P* __restrict__ p, int i) {
    if constexpr (!N32) return p[i];
    using B = std::conditional_t<std::is_const_v<P>, const char, char>;
    return *reinterpret_cast<P*>(reinterpret_cast<B*>(p) + (unsigned)i * (unsigned)sizeof(P));
}

// The same with the S-kernel's head, s formed for every gathered column and stored.
// (No register limit: it gathers two vectors, and runs on systems that do not
// fill the chip; 9 spilled registers cost 1.5 us.)
template <typename T, bool N32 = false, int TB = kSlBlock, int PASS = 8>
__device__ __forceinline__ void bicg_SBs(const BicgArgs<T>& a) {
    const SliceRows q = slice_rows_of<TB>(a.one, a.sg, a.sv);
    const FirstSlice f = first_slice(sliced_of(a), q);
    zero_slots(a, kPartB, 8, q.lb, a.sg, slice_first(q));
    SysBlock sb{};
    sb.sys = 0;
    sb.local = q.lb;
    sb.gbeg = 0;
    sb.gcnt = a.G;
    AlphaHead<kSlBlock> hd;
    hd.load(a, sb);
    double2 alpha;
    if (!hd.run(a, sb, alpha)) return;
    const cx<T> nal = mk<T>((T)-alpha.x, (T)-alpha.y);
    const cx<T>* __restrict__ r = a.r;
    const cx<T>* __restrict__ v = a.v;
    const cx<T>* __restrict__ rh = a.rh;
    cx<T>* __restrict__ sv = a.s;
    cx<T>* __restrict__ tv = a.t;
    double e[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    slice_rows<T, false>(
        sliced_of(a), q, f, a.one.n, [=](int c) { return cfma<T>(nal, at<N32>(v, c), at<N32>(r, c)); },
        [rh](int row) { return at<N32>(rh, row); },
        [&](int64_t row, cx<T> acc, cx<T> s, cx<T> w) {
            at<N32>(sv, (int)row) = s;
            at<N32>(tv, (int)row) = acc;
            b_terms<T>(e, s, acc, w);
        });
    slice_store<8, TB, PASS>(a.part + kPartB * a.stride, a.stride, q.lb, e);
}
template <typename T>
__global__ __launch_bounds__(kSlBlock) void k_bicg_SBs(const BicgArgs<T> a) {
    bicg_SBs<T>(a);
}

}  // namespace hz
