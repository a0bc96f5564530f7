// Device kernels of the helmz library (gfx950 / CDNA4, wave64).
//
// Reductions: every reducing kernel writes one fixed-order partial per block
// (component-major, stride kMaxGrid).  The kernel that needs the total sums
// the partials itself, redundantly in every block and in a fixed order, so
// all blocks hold bitwise the same scalar and no single-block finaliser
// kernel sits between two streaming kernels.  No floating-point atomics:
// results are bitwise reproducible run to run.
//
// Row ownership: a launch of G blocks splits the rows into G contiguous
// chunks.  Hardware dispatches block b to XCD (b mod 8); block b works on
// logical chunk (b mod 8) * (G/8) + b/8, so each XCD owns one contiguous
// eighth of the rows.  The x-gathers of a banded FE matrix then stay inside
// that XCD's L2, and every kernel of a solve maps the same rows to the same
// XCD.
#pragma once

#include <hip/hip_runtime.h>

#include <limits>
#include <type_traits>
#include <stdint.h>

#define HZ_INLINE __attribute__((always_inline))

namespace hz {

constexpr int kWave = 64;
constexpr int kXcd = 8;
constexpr int kBlock = 1024;   // threads per block (16 waves)
constexpr int kMaxGrid = 512;  // bound on blocks (= partials) of a reducing launch: 2 blocks per CU
#define HZ_STREAM_BOUNDS __launch_bounds__(1024, 8)  // 8 waves per SIMD (two blocks per CU): <= 64 VGPRs

// partial-sum regions (component index; component c lives at part[c * kMaxGrid + block])
constexpr int kPartA = 0;   // <rhat, v>                                             (2)
constexpr int kPartB = 2;   // ||s||^2, <t, s>, ||t||^2, <rhat, t>, <rhat, s>          (8)
constexpr int kPartC = 10;  // <rhat, r>, ||r||^2                                    (3)
constexpr int kPartI = 13;  // ||b||^2 / residual norms                              (1)
constexpr int kParts = 14;

// ------------------------------------------------------------------ complex

template <typename T> struct cplx_of;
template <> struct cplx_of<double> { using type = double2; };
template <> struct cplx_of<float> { using type = float2; };
template <typename T> using cx = typename cplx_of<T>::type;

template <typename T> __device__ __forceinline__ cx<T> mk(T re, T im) {
    cx<T> z;
    z.x = re;
    z.y = im;
    return z;
}
__device__ __forceinline__ double fmaT(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fmaT(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// c + a b
template <typename T> __device__ __forceinline__ cx<T> cfma(cx<T> a, cx<T> b, cx<T> c) {
    c.x = fmaT(a.x, b.x, c.x);
    c.x = fmaT(-a.y, b.y, c.x);
    c.y = fmaT(a.x, b.y, c.y);
    c.y = fmaT(a.y, b.x, c.y);
    return c;
}
// a b
template <typename T> __device__ __forceinline__ cx<T> cmul(cx<T> a, cx<T> b) {
    return mk<T>(fmaT(a.x, b.x, -a.y * b.y), fmaT(a.x, b.y, a.y * b.x));
}
// c + conj(a) b, accumulated in double
__device__ __forceinline__ double2 cdotacc(double ar, double ai, double br, double bi, double2 c) {
    c.x = __builtin_fma(ar, br, c.x);
    c.x = __builtin_fma(ai, bi, c.x);
    c.y = __builtin_fma(ar, bi, c.y);
    c.y = __builtin_fma(-ai, br, c.y);
    return c;
}
__device__ __forceinline__ double2 zdiv(double2 a, double2 b) {
    double d = b.x * b.x + b.y * b.y;
    double2 q;
    q.x = (a.x * b.x + a.y * b.y) / d;
    q.y = (a.y * b.x - a.x * b.y) / d;
    return q;
}
__device__ __forceinline__ double2 zmul(double2 a, double2 b) {
    double2 q;
    q.x = a.x * b.x - a.y * b.y;
    q.y = a.x * b.y + a.y * b.x;
    return q;
}
__device__ __forceinline__ bool zfinite(double2 a) { return __builtin_isfinite(a.x) && __builtin_isfinite(a.y); }
__device__ __forceinline__ bool zzero(double2 a) { return a.x == 0.0 && a.y == 0.0; }
template <typename T> __device__ __forceinline__ cx<T> narrow(double2 a) { return mk<T>((T)a.x, (T)a.y); }

// Streaming (non-temporal) loads of matrix arrays, for kernels whose every
// load instruction covers whole cache lines of consecutive entries (the block
// tiles of the standalone product): the data is read once, and on this part
// such streaming loads sustain 5-10 % more HBM bandwidth than ordinary ones.
// Row-split accesses (L lanes per row, a line shared by neighbouring rows) and
// the solvers' products, whose matrix is re-read every iteration, measured
// slower with them and use ordinary loads.  HZ_STREAM_MATRIX=0 at build time
// makes these ordinary loads too.
#ifndef HZ_STREAM_MATRIX
#define HZ_STREAM_MATRIX 1
#endif
typedef double hz_d2v __attribute__((ext_vector_type(2)));
typedef float hz_f2v __attribute__((ext_vector_type(2)));
__device__ __forceinline__ int ld_mat(const int* p) {
#if HZ_STREAM_MATRIX
    return __builtin_nontemporal_load(p);
#else
    return *p;
#endif
}
__device__ __forceinline__ short ld_mat(const short* p) {
#if HZ_STREAM_MATRIX
    return __builtin_nontemporal_load(p);
#else
    return *p;
#endif
}
__device__ __forceinline__ double2 ld_mat(const double2* p) {
#if HZ_STREAM_MATRIX
    const hz_d2v v = __builtin_nontemporal_load(reinterpret_cast<const hz_d2v*>(p));
    return mk<double>(v.x, v.y);
#else
    return *p;
#endif
}
__device__ __forceinline__ float2 ld_mat(const float2* p) {
#if HZ_STREAM_MATRIX
    const hz_f2v v = __builtin_nontemporal_load(reinterpret_cast<const hz_f2v*>(p));
    return mk<float>(v.x, v.y);
#else
    return *p;
#endif
}

// ------------------------------------------------------------------ lane exchange (DPP / ds_swizzle)

struct I2 {
    int lo, hi;
};

template <int CTRL> __device__ __forceinline__ int dpp_i32(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
template <int PAT> __device__ __forceinline__ int swz_i32(int v) { return __builtin_amdgcn_ds_swizzle(v, PAT); }

template <int CTRL> __device__ __forceinline__ double dpp(double v) {
    I2 w = __builtin_bit_cast(I2, v);
    w.lo = dpp_i32<CTRL>(w.lo);
    w.hi = dpp_i32<CTRL>(w.hi);
    return __builtin_bit_cast(double, w);
}
template <int CTRL> __device__ __forceinline__ float dpp(float v) {
    return __builtin_bit_cast(float, dpp_i32<CTRL>(__builtin_bit_cast(int, v)));
}
template <int PAT> __device__ __forceinline__ double swz(double v) {
    I2 w = __builtin_bit_cast(I2, v);
    w.lo = swz_i32<PAT>(w.lo);
    w.hi = swz_i32<PAT>(w.hi);
    return __builtin_bit_cast(double, w);
}
template <int PAT> __device__ __forceinline__ float swz(float v) {
    return __builtin_bit_cast(float, swz_i32<PAT>(__builtin_bit_cast(int, v)));
}

// DPP controls (gfx9 encoding)
constexpr int kQuadXor1 = 0xB1;     // quad_perm(1,0,3,2)
constexpr int kQuadXor2 = 0x4E;     // quad_perm(2,3,0,1)
constexpr int kHalfMirror = 0x141;  // lane i <-> 7-i inside each group of 8
constexpr int kMirror = 0x140;      // lane i <-> 15-i inside each row of 16
constexpr int kSwzXor16 = 0x401F;   // ds_swizzle bit mode: lane ^ 16 within 32

// Sum over aligned groups of L lanes; every lane of a group receives the same
// bitwise value (each step adds a value and its partner's, a + b == b + a).
// All 64 lanes must be active.
template <int L, typename T> __device__ __forceinline__ T group_sum(T v) {
    static_assert(L == 1 || L == 2 || L == 4 || L == 8 || L == 16 || L == 32 || L == 64, "L");
    if constexpr (L >= 2) v += dpp<kQuadXor1>(v);
    if constexpr (L >= 4) v += dpp<kQuadXor2>(v);
    if constexpr (L >= 8) v += dpp<kHalfMirror>(v);
    if constexpr (L >= 16) v += dpp<kMirror>(v);
    if constexpr (L >= 32) v += swz<kSwzXor16>(v);
    if constexpr (L >= 64) v += __shfl_xor(v, 32);
    return v;
}

// Block sum of K doubles over a block of NT threads; the result is valid in
// thread 0 only.  Waves are combined in a fixed order.  Safe to call
// repeatedly in one kernel.
template <int K, int NT = kBlock> __device__ __forceinline__ void block_sum(double (&v)[K]) {
    __shared__ double lds[NT / kWave][K];
    const int wid = threadIdx.x / kWave, lane = threadIdx.x % kWave;
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = group_sum<64>(v[k]);
    __syncthreads();  // a previous call's reader is done with lds
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < K; ++k) lds[wid][k] = v[k];
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            double s = lds[0][k];
            for (int w = 1; w < NT / kWave; ++w) s += lds[w][k];
            v[k] = s;
        }
    }
}

// Sum over a wave of values that only the lanes l = 0 mod STRIDE hold (the
// others hold 0), in the lanes l = 0 mod STRIDE: the steps below STRIDE are
// left out.  Rotations within a row of 16 pair every lane with the one s away.
template <int S> __device__ __forceinline__ double row_ror(double v) { return dpp<0x120 + S>(v); }
template <int STRIDE> __device__ __forceinline__ double wave_sum(double v) {
    if constexpr (STRIDE <= 1) v += row_ror<1>(v);
    if constexpr (STRIDE <= 2) v += row_ror<2>(v);
    if constexpr (STRIDE <= 4) v += row_ror<4>(v);
    if constexpr (STRIDE <= 8) v += row_ror<8>(v);
    if constexpr (STRIDE <= 16) v += swz<kSwzXor16>(v);
    if constexpr (STRIDE <= 32) v += __shfl_xor(v, 32);
    return v;
}

// The block's totals of K doubles to out[k * stride], k < K: wave sums to LDS,
// one barrier, then the first wave adds the NW wave sums of 64 / NW components
// at a time.  STRIDE: the lanes that hold values (wave_sum).  TAG separates
// the LDS of several calls in one kernel.
template <int K, int STRIDE = 1, int TAG = 0, int NT = kBlock>
__device__ __forceinline__ void block_store(double* __restrict__ out, int stride, double (&v)[K]) {
    constexpr int NW = NT / kWave, PER = kWave / NW;
    __shared__ double lds[K][NW];
    const int wid = threadIdx.x / kWave, lane = threadIdx.x % kWave;
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = wave_sum<STRIDE>(v[k]);
    if (lane == 0) {
#pragma unroll
        for (int k = 0; k < K; ++k) lds[k][wid] = v[k];
    }
    __syncthreads();
    if (wid == 0) {
#pragma unroll
        for (int k0 = 0; k0 < K; k0 += PER) {
            const int k = k0 + lane / NW;
            const double t = group_sum<NW>(lds[k < K ? k : K - 1][lane % NW]);
            if (k < K && lane % NW == 0) out[k * stride] = t;
        }
    }
}

// Sum of K partial components (component k at part[k*kMaxGrid + g], g < G)
// in a fixed order, delivered to every thread of the block.
// (G <= kMaxGrid <= kBlock: one partial per thread, the K loads issued
// together; idle waves load nothing, as in sys_sum.)
template <int K> __device__ __forceinline__ void head_sum(const double* __restrict__ part, int G, double (&out)[K]) {
    static_assert(kMaxGrid <= kBlock, "one partial per thread");
    __shared__ double bc[K];
    const int t = threadIdx.x;
#pragma unroll
    for (int k = 0; k < K; ++k) out[k] = 0.0;
    if ((__builtin_amdgcn_readfirstlane((int)threadIdx.x) & ~(kWave - 1)) < G) {
        const bool mine = t < G;
        const int g0 = mine ? t : G - 1;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const double v = part[k * kMaxGrid + g0];
            out[k] = mine ? v : 0.0;
        }
    }
    block_sum<K>(out);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < K; ++k) bc[k] = out[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) out[k] = bc[k];
}

// Store a block's K partials (thread 0 holds them after block_sum).
template <int K> __device__ __forceinline__ void store_partials(double* __restrict__ part, int lb, double (&e)[K]) {
    block_sum<K>(e);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < K; ++k) part[k * kMaxGrid + lb] = e[k];
    }
}

// ------------------------------------------------------------------ launch geometry

// Chunked row ownership of a launch (see the file comment).
struct Geom {
    int G;  // blocks: a multiple of 8 when there are at least 8
};

__device__ __forceinline__ int logical_block(int b, int G) {
    return (G % kXcd == 0) ? (b % kXcd) * (G / kXcd) + b / kXcd : b;
}

// The rows of a block.  The block is the k-th of the K blocks that share the
// row range [x0, x1) of its group and takes that range's tiles k, k + K,
// k + 2K, ... (a tile is kBlock/L rows in a row product, kBlock rows in an
// element-wise pass).  A launch of G >= 8 blocks has 8 groups, one per XCD,
// each owning an eighth of the rows; the K blocks of an XCD then advance
// through its range side by side, so the part of x their gathers touch at
// any time is a few tiles plus the matrix bandwidth, small enough for the
// XCD's L2 (with one contiguous chunk per block it would be K separate
// windows).  A system of a batch with its own chunk per block is K = 1.
struct Rows {
    int64_t x0, x1;
    int k, K;
};
__device__ __forceinline__ Rows group_rows(int n, int G, int lb) {
    Rows r;
    const int groups = (G % kXcd == 0) ? kXcd : 1;
    r.K = G / groups;
    const int x = lb / r.K;
    r.k = lb % r.K;
    r.x0 = (int64_t)n * x / groups;
    r.x1 = (int64_t)n * (x + 1) / groups;
    return r;
}

struct RowRange {
    int lb;
    Rows rw;
};
__device__ __forceinline__ RowRange rows_of_block(int n, Geom geo) {
    RowRange r;
    r.lb = logical_block(blockIdx.x, geo.G);
    r.rw = group_rows(n, geo.G, r.lb);
    return r;
}

// Element-wise pass over the rows of a block (tiles of kBlock rows).
#define HZ_FOR_ELEMS(i, rw) \
    for (int64_t i = (rw).x0 + (int64_t)(rw).k * kBlock + threadIdx.x; i < (rw).x1; i += (int64_t)(rw).K * kBlock)

// ------------------------------------------------------------------ row product (vector CSR)

// sum_p vals_p * op(col_p) over one row, computed by L lanes: lane l takes
// entries beg+l, beg+l+L, ...; each lane issues U (col, value) loads, then U
// operand gathers, then U complex FMAs, so U independent loads of each kind
// are in flight per lane.  The loads are straight-line: an entry past the
// row's end is read at the row's last entry (in bounds, since the loop runs
// only while base < end) and its product is dropped by selects on the
// accumulator, so no load is exec-masked (a masked load makes the compiler
// wait for every load in flight).  Returns the lane's partial (the caller
// sums the group).  Entry order per lane is sequential, so results are
// deterministic.
template <typename T, int L, int U, typename Op>
__device__ __forceinline__ cx<T> row_partial(int beg, int end, int lane, const int* __restrict__ ci,
                                             const cx<T>* __restrict__ vals, Op op,
                                             cx<T> acc = mk<T>(T(0), T(0))) {
    for (int base = beg + lane; base < end; base += L * U) {
        int c[U];
        cx<T> a[U], o[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int p = base + u * L < end ? base + u * L : end - 1;
            c[u] = ci[p];
            a[u] = vals[p];
        }
#pragma unroll
        for (int u = 0; u < U; ++u) o[u] = op(c[u]);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool in = base + u * L < end;
            const cx<T> nx = cfma<T>(a[u], o[u], acc);
            acc.x = in ? nx.x : acc.x;
            acc.y = in ? nx.y : acc.y;
        }
    }
    return acc;
}

// Block-tile form of the row loop (the lane count L = 1 selects it): tiles
// of kSolTileRows rows; the block loads a tile's entries [rp[r0], rp[r0 +
// kSolTileRows]) contiguously (thread t takes entries e0 + t + k kBlock,
// straight-line, clamped into the tile), multiplies them by the gathered
// operand op(col), writes the products to LDS, and kSolTileLanes threads per
// row sum the row out of LDS in entry order; epi(row, total) runs in the
// first thread of each row.  Each load instruction reads kBlock consecutive
// entries, whole cache lines, where the vector form reads a row's few
// entries per lane group, so its loads carry the streaming hint (ld_mat).  A
// tile with more than kSolTileCap entries is done as vector rows.  The trip
// count is uniform across the block.
constexpr int kSolTileLanes = 4;
constexpr int kSolTileRows = kBlock / kSolTileLanes;
constexpr int kSolTilePer = 4;
constexpr int kSolTileCap = kBlock * kSolTilePer;

// No epilogue operand: epi(row, total).  With a `pre` functor the epilogue is
// epi(row, total, pre(row)).  The vector form issues that load before the
// row's product, so that its latency overlaps the product's loads; the tile
// form loads it at the epilogue (its kernels use all 64 VGPRs, and an early
// load spilled: 241 -> 250 us per cabin iteration).
struct NoPre {
    __device__ int operator()(int64_t) const { return 0; }
};

template <typename T, typename Op, typename Epi, typename Pre = NoPre>
__device__ __forceinline__ void for_tiles(const Rows& rw, const int* __restrict__ rp, const int* __restrict__ ci,
                                          const cx<T>* __restrict__ vals, Op op, Epi epi, Pre pre = Pre{}) {
    constexpr bool kPre = !std::is_same_v<Pre, NoPre>;
    constexpr int L = kSolTileLanes;
    __shared__ cx<T> prod[kSolTileCap];
    const int t = threadIdx.x, g = t / L, lane = t % L;
    const int64_t first = rw.x0 + (int64_t)rw.k * kSolTileRows, step = (int64_t)rw.K * kSolTileRows;
    const int64_t r1 = rw.x1;
    for (int64_t r0 = first; r0 < r1; r0 += step) {
        const int64_t re = r0 + kSolTileRows < r1 ? r0 + kSolTileRows : r1;
        const int e0 = rp[r0], e1 = rp[re];
        const int64_t row = r0 + g;
        const int b = rp[row < re ? row : re], e = rp[row + 1 < re ? row + 1 : re];
        cx<T> acc = mk<T>(T(0), T(0));
        if (e1 > e0 && e1 - e0 <= kSolTileCap) {  // (a tile of empty rows loads nothing: block-uniform)
            const int last = e1 - 1;
            int c[kSolTilePer];
            cx<T> v[kSolTilePer], o[kSolTilePer];
#pragma unroll
            for (int k = 0; k < kSolTilePer; ++k) {
                const int p = e0 + t + k * kBlock;
                c[k] = ld_mat(ci + (p < last ? p : last));
            }
#pragma unroll
            for (int k = 0; k < kSolTilePer; ++k) {
                const int p = e0 + t + k * kBlock;
                v[k] = ld_mat(vals + (p < last ? p : last));
            }
#pragma unroll
            for (int k = 0; k < kSolTilePer; ++k) o[k] = op(c[k]);
#pragma unroll
            for (int k = 0; k < kSolTilePer; ++k) {
                const bool ok = e0 + t + k * kBlock < e1;
                const cx<T> pr = cmul<T>(v[k], o[k]);
                prod[t + k * kBlock] = mk<T>(ok ? pr.x : T(0), ok ? pr.y : T(0));
            }
            __syncthreads();
            for (int q = b - e0 + lane; q < e - e0; q += L) {
                const cx<T> pv = prod[q];
                acc.x += pv.x;
                acc.y += pv.y;
            }
            __syncthreads();
        } else if (e1 > e0 && row < re) {
            acc = row_partial<T, L, 1>(b, e, lane, ci, vals, op);
        }
        acc.x = group_sum<L>(acc.x);
        acc.y = group_sum<L>(acc.y);
        if (row < re && lane == 0) {
            if constexpr (kPre) {
                epi(row, acc, pre(row));
            } else {
                epi(row, acc);
            }
        }
    }
}

// A thread's share of the block's first tile of rows, loaded ahead of a
// kernel's head (whose loads, reduction and scalar arithmetic then run while
// these are in flight): the bounds of its row and, with UP = U, its first U
// entries.  (The chain row_ptr -> entries -> gathers is three round trips to
// memory, most of the time of a small system's product.)
template <typename T, int UP> struct FirstRow {
    int beg = 0, end = 0;
    int c[UP > 0 ? UP : 1];
    cx<T> a[UP > 0 ? UP : 1];
};
template <typename T, int L, int UP>
__device__ __forceinline__ void first_row(FirstRow<T, UP>& f, const Rows& rw, const int* __restrict__ rp,
                                          const int* __restrict__ ci, const cx<T>* __restrict__ vals) {
    if constexpr (L > 1) {
        constexpr int RPS = kBlock / L;
        const int64_t row = rw.x0 + (int64_t)rw.k * RPS + threadIdx.x / L;
        if (row < rw.x1) {
            f.beg = rp[row];
            f.end = rp[row + 1];
        }
        if constexpr (UP > 0) {
            const int lane = threadIdx.x % L;
#pragma unroll
            for (int u = 0; u < UP; ++u) {
                f.c[u] = 0;
                f.a[u] = mk<T>(T(0), T(0));
            }
            if (f.beg + lane < f.end) {
#pragma unroll
                for (int u = 0; u < UP; ++u) {
                    const int p = f.beg + lane + u * L < f.end ? f.beg + lane + u * L : f.end - 1;
                    f.c[u] = ci[p];
                    f.a[u] = vals[p];
                }
            }
        }
    }
}

// Row loop of a block over its tiles of RPS = kBlock/L rows (g = thread / L
// picks the row of the tile).  The next step's row_ptr pair is loaded before
// the current row's product, so that load's latency overlaps the current
// step.  `f` holds the first tile's bounds, and its entries if UP = U (first_row).
// epi(row, total) runs in lane 0 of each row's group after
// the group sum.  The trip count is uniform across the block.
template <typename T, int L, int U, int UP, typename Op, typename Epi, typename Pre = NoPre>
__device__ __forceinline__ void for_rows(const FirstRow<T, UP>& f, const Rows& rw, const int* __restrict__ rp,
                                         const int* __restrict__ ci, const cx<T>* __restrict__ vals, Op op, Epi epi,
                                         Pre pre = Pre{}) {
    constexpr bool kPre = !std::is_same_v<Pre, NoPre>;
    if constexpr (L == 1) {
        for_tiles<T>(rw, rp, ci, vals, op, epi, pre);
        return;
    }
    constexpr int RPS = kBlock / L;
    const int g = threadIdx.x / L, lane = threadIdx.x % L;
    const int64_t first = rw.x0 + (int64_t)rw.k * RPS, step = (int64_t)rw.K * RPS, r1 = rw.x1;
    int64_t row = first + g;
    int beg = f.beg, end = f.end;
    for (int64_t base = first; base < r1; base += step) {
        const int64_t nrow = row + step;
        int nbeg = 0, nend = 0;
        if (nrow < r1) {
            nbeg = rp[nrow];
            nend = rp[nrow + 1];
        }
        const bool ok = row < r1;
        cx<T> acc = mk<T>(T(0), T(0));
        decltype(pre(row)) w{};
        if (ok) {
            if constexpr (kPre) w = pre(row);
            if (UP > 0 && base == first) {  // uniform: the prefetched entries, in the order of row_partial
                if (beg + lane < end) {
                    cx<T> o[UP > 0 ? UP : 1];
#pragma unroll
                    for (int u = 0; u < UP; ++u) o[u] = op(f.c[u]);
#pragma unroll
                    for (int u = 0; u < UP; ++u) {
                        const bool in = beg + lane + u * L < end;
                        const cx<T> nx = cfma<T>(f.a[u], o[u], acc);
                        acc.x = in ? nx.x : acc.x;
                        acc.y = in ? nx.y : acc.y;
                    }
                }
                acc = row_partial<T, L, U>(beg + L * U, end, lane, ci, vals, op, acc);
            } else {
                acc = row_partial<T, L, U>(beg, end, lane, ci, vals, op);
            }
        }
        acc.x = group_sum<L>(acc.x);
        acc.y = group_sum<L>(acc.y);
        if (ok && lane == 0) {
            if constexpr (kPre) {
                epi(row, acc, w);
            } else {
                epi(row, acc);
            }
        }
        row = nrow;
        beg = nbeg;
        end = nend;
    }
}

// The same without a head to hide the first loads behind.
template <typename T, int L, int U, typename Op, typename Epi, typename Pre = NoPre>
__device__ __forceinline__ void for_rows(const Rows& rw, const int* __restrict__ rp, const int* __restrict__ ci,
                                         const cx<T>* __restrict__ vals, Op op, Epi epi, Pre pre = Pre{}) {
    FirstRow<T, 0> f;
    first_row<T, L, 0>(f, rw, rp, ci, vals);
    for_rows<T, L, U, 0>(f, rw, rp, ci, vals, op, epi, pre);
}

// ------------------------------------------------------------------ solver scalars (device resident)

// One block per system.  Written only by thread 0 of the system's first
// block, and read only by later kernels (never by other blocks of the
// writing kernel), except `done`, whose early read by other blocks of the
// system leads to the exit they would compute themselves.
struct alignas(256) SolverScal {
    double2 rho2[2];  // rho of iteration i in slot i & 1
    double2 alpha;    // alpha of the current iteration
    double2 omega;    // omega of the last completed iteration
    double2 beta;
    double bnorm;  // ||b||
    double rtol;
    double relres;       // last recursive ||r|| / ||b|| (or ||s|| / ||b||)
    double relres_true;  // filled by the final residual check
    double outer_rn;     // refinement: ||b - A x|| of the current outer step
    int iter;            // next iteration to run (1-based); written by the last kernel of an iteration
    int cur;             // iteration in progress; written by the first kernel of an iteration
    int maxiter;
    int status;  // solver status once done
    int done;    // 1 once the solve has ended (all later kernels are no-ops)
    int iters;   // reported iteration count
    int zero_x;  // ||b|| = 0: the solution is x = 0
    int bad_diag;  // Jacobi requested with a zero diagonal entry
    int pending;   // half-step exit taken in iteration `pending`; the next first kernel concludes
    int why;       // for a breakdown: which scalar vanished (BD_*)
    int closed;    // 1 once an A-kernel has seen done (asynchronous solves; past_end)
};

enum : int { ST_OK = 0, ST_NOT_CONVERGED = 1, ST_BREAKDOWN = 2, ST_NONFINITE = 3 };
enum : int { BD_NONE = 0, BD_RHO = 1, BD_RHAT_V = 2, BD_TT = 3, BD_OMEGA = 4 };

// Reset the scalar blocks of nsys systems before a solve.
__global__ void k_sc_init(SolverScal* sc, int nsys, double rtol, int maxiter) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= nsys) return;
    SolverScal z = {};
    z.rtol = rtol;
    z.maxiter = maxiter;
    z.status = ST_NOT_CONVERGED;
    sc[j] = z;
}

// ------------------------------------------------------------------ work map of a solver launch

// Logical block lb of a solver launch belongs to system `sys`, takes the rows
// that (x0, x1, k, K) describe (as in struct Rows) of the (block-diagonal)
// matrix and is the `local`-th block of its system; sys < 0 marks padding.  System j owns the contiguous logical block
// range [gbeg, gbeg + gcnt).  A single solve is the one-system case.
struct BlockMap {
    int sys, x0, x1, k, K, local;  // rows as in struct Rows
};
struct SysMap {
    int gbeg, gcnt, row0, row1;
};

// The map of a one-system launch by value: groups of K blocks, one per XCD
// (or one group of fewer than 8 blocks), each owning gr rows.  A block finds
// its rows from its index and these arguments; from the BlockMap and SysMap
// arrays of a batch it takes two dependent loads, each a round trip past the
// L2 that the kernel boundary has emptied, before any other load can start.
struct OneMap {
    int n = 0;       // rows; 0: a batch, take the arrays
    int groups = 1;  // 8 or 1
    int K = 1, gr = 0;
};

template <typename T> struct BicgArgs {
    int G;       // blocks of every solver launch (a multiple of 8, or < 8)
    int stride;  // partial component stride (>= np)
    int pf = 1;  // product blocks per block of the map (sol_subs(G) when the products run as sub-blocks)
    OneMap one;
    int np = 0;      // one system: partial slots that the products write (regions A and B)
    int sg = 0;      // blocks of the sliced products
    int either = 0;  // the products choose the operator's form on the device
    int sv = 1;      // blocks of the sliced form that one block of theirs stands for
    int s_csr = 0;   // the S-kernel runs for the CSR operator only (either form, the sliced one fused)
    // (no padding bytes: the graph cache compares these structs bytewise)
    const BlockMap* bmap;
    const SysMap* smap;
    int* ndone;  // systems finished so far
    const int* __restrict__ row_ptr;
    const int* __restrict__ col_idx;
    const cx<T>* __restrict__ vals;
    const int* __restrict__ soff;    // the sliced operator's offsets and columns (vals its values), or null
    const short* __restrict__ scol;
    const cx<T>* b;
    cx<T>* r;
    const cx<T>* rh;
    cx<T>* p;
    cx<T>* v;
    cx<T>* s;
    cx<T>* t;
    cx<T>* x;
    double* part;
    SolverScal* sc;
};

struct SysBlock {
    int lb, sys, local;
    Rows rw;
    int gbeg, gcnt;
};
// Block `b` of a launch of F G blocks over the map: F sub-blocks share the
// rows of each logical block, lb counts them, and partials [gbeg, gbeg +
// gcnt) are those of the launch's own blocks.
__device__ __forceinline__ SysBlock map_block(const OneMap& one, const BlockMap* bmap, const SysMap* smap, int G,
                                              int F, int b) {
    SysBlock q;
    if (one.n > 0) {
        const int x = one.groups == kXcd ? b % kXcd : 0, k = one.groups == kXcd ? b / kXcd : b;
        q.rw.k = k;
        q.rw.K = F * one.K;
        q.rw.x0 = (int64_t)x * one.gr;
        q.rw.x1 = q.rw.x0 + one.gr < one.n ? q.rw.x0 + one.gr : one.n;
        q.lb = q.local = x * F * one.K + k;
        q.sys = 0;
        q.gbeg = 0;
        q.gcnt = F * G;
        return q;
    }
    q.lb = logical_block(b, F * G);
    const BlockMap m = bmap[q.lb / F];
    q.sys = m.sys;
    q.local = F * m.local + q.lb % F;
    q.rw.x0 = m.x0;
    q.rw.x1 = m.x1;
    q.rw.k = F * m.k + q.lb % F;
    q.rw.K = F * m.K;
    if (m.sys >= 0) {
        const SysMap sm = smap[m.sys];
        q.gbeg = F * sm.gbeg;
        q.gcnt = F * sm.gcnt;
    } else {
        q.gbeg = q.gcnt = 0;
    }
    return q;
}
template <typename T> __device__ __forceinline__ SysBlock sys_block(const BicgArgs<T>& a) {
    return map_block(a.one, a.bmap, a.smap, a.G, 1, blockIdx.x);
}
// Partials of the block's system in the products' regions A and B.
template <typename T> __device__ __forceinline__ int prod_parts(const BicgArgs<T>& a, const SysBlock& q) {
    return a.one.n > 0 ? a.np : q.gcnt;
}
// The word after the done-counter: 1 if the operator is not sliced.
__device__ __forceinline__ int* slice_no(int* ndone) { return ndone + 1; }
// A product of `cnt` blocks where either form may run: zeros to the slots past
// its own that the readers also add.
template <typename A>
__device__ __forceinline__ void zero_slots(const A& a, int region, int K, int lb, int cnt, bool first) {
    if (a.either == 0 || !first) return;
    for (int g = lb + cnt; g < a.np; g += cnt)
        for (int k = 0; k < K; ++k) a.part[(region + k) * a.stride + g] = 0.0;
}
// Partial range of system j (for the one-block-per-system kernels).
template <typename T> __device__ __forceinline__ SysMap sys_range(const BicgArgs<T>& a, int j) {
    return a.one.n > 0 ? SysMap{0, a.G, 0, a.one.n} : a.smap[j];
}

__device__ __forceinline__ bool sys_leader(const SysBlock& q) { return q.local == 0 && threadIdx.x == 0; }

// Record the end of system q's solve (its leader thread only).
__device__ __forceinline__ void finish(SolverScal* sc, int* ndone, int status, int iterations, int why = BD_NONE) {
    sc->status = status;
    sc->iters = iterations;
    sc->why = why;
    sc->done = 1;
    atomicAdd(ndone, 1);
}

__device__ __forceinline__ int wave_id() { return __builtin_amdgcn_readfirstlane((int)threadIdx.x) / kWave; }

// The sum of K components of partials by the NW waves of a block: component
// k by the W = NW / K (rounded down to a power of two) waves k W .. k W + W - 1,
// wave i of them taking its partials i, i + W, ... in rounds of 64.  load()
// issues the loads of the first kHeadNV rounds of each wave, all at once;
// store() waits for them, adds the rest if any, and puts the wave's sum into
// tot; after a barrier at() adds the W sums.  The order is fixed.  With one
// partial of every component per thread, and all waves adding all components,
// the eight sums of a head took the SIMDs about 1 us (7.3 us for the C-kernel of
// 8,000 rows, 4.3 us with a wave per component).
// V > 1: each wave does the work of V, so that a smaller block adds in the
// order of one with V times its waves.
constexpr int kHeadNV = 4;
constexpr int head_waves(int K, int NW) { return 2 * K > NW ? 1 : 2 * head_waves(K, NW / 2); }
template <int K, int NT = kBlock, int V = 1> struct PartSum {
    static constexpr int RW = head_waves(K, NT / kWave);  // waves per component,
    static constexpr int W = RW * V;                      // and the shares they add
    static_assert(K * RW <= NT / kWave, "K RW waves");
    static constexpr int TOT = V * NT / kWave;  // totals in LDS
    double v[V][kHeadNV];
    const double* part;
    int cnt, w0;
    // the component of this wave (a uniform value; K or more: none)
    static __device__ __forceinline__ int comp() { return wave_id() / RW; }
    // p: the first partial of this wave's component, c >= 1 of them
    __device__ __forceinline__ void load(const double* __restrict__ p, int c) {
        part = p;
        cnt = c;
        w0 = wave_id() % RW * V;
        const int lane = threadIdx.x % kWave;
#pragma unroll
        for (int s = 0; s < V; ++s)
#pragma unroll
            for (int j = 0; j < kHeadNV; ++j) {
                v[s][j] = 0.0;
                const int r = (w0 + s + j * W) * kWave;
                if (V > 1 || r < cnt) v[s][j] = p[r + lane < cnt ? r + lane : cnt - 1];  // uniform; masked in store()
            }
    }
    __device__ __forceinline__ void store(double* tot) {
        const int lane = threadIdx.x % kWave;
        double t[V];
#pragma unroll
        for (int s = 0; s < V; ++s) t[s] = masked(s, 0, lane);
        for (int g = kHeadNV * W * kWave; g < cnt; g += kHeadNV * W * kWave) {  // uniform
#pragma unroll
            for (int s = 0; s < V; ++s) {
#pragma unroll
                for (int j = 0; j < kHeadNV; ++j) {
                    const int r = g + (w0 + s + j * W) * kWave;
                    if (r < cnt) v[s][j] = part[r + lane < cnt ? r + lane : cnt - 1];
                }
                t[s] += masked(s, g, lane);
            }
        }
#pragma unroll
        for (int s = 0; s < V; ++s) t[s] = wave_sum<1>(t[s]);
#pragma unroll
        for (int s = 0; s < V; ++s)
            if (lane == 0) tot[wave_id() * V + s] = t[s];
    }
    // the sum of v[s], whose rounds start at partial g
    __device__ __forceinline__ double masked(int s, int g, int lane) const {
        double m[kHeadNV];
#pragma unroll
        for (int j = 0; j < kHeadNV; ++j) m[j] = g + (w0 + s + j * W) * kWave + lane < cnt ? v[s][j] : 0.0;
        return (m[0] + m[1]) + (m[2] + m[3]);
    }
    static __device__ __forceinline__ double at(const double* tot, int k) {
        double t = tot[k * W];
#pragma unroll
        for (int i = 1; i < W; ++i) t += tot[k * W + i];
        return t;
    }
};
// The shares per wave with which a head of NT threads adds in the order of one of kBlock.
constexpr int head_shares(int K, int NT) { return head_waves(K, kBlock / kWave) / head_waves(K, NT / kWave); }

// Sum of K components over one system's partials [gbeg, gbeg + gcnt), in a
// fixed order, delivered to every thread of the block (component k at
// part[k * stride + g]).  One barrier.
template <int K, int TAG = 0>
__device__ __forceinline__ void sys_sum(const double* __restrict__ part, int stride, int gbeg, int gcnt,
                                        double (&out)[K]) {
    __shared__ double tot[kBlock / kWave];
    const int c = PartSum<K>::comp();
    if (c < K) {
        PartSum<K> ps;
        ps.load(part + c * stride + gbeg, gcnt);
        ps.store(tot);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < K; ++k) out[k] = PartSum<K>::at(tot, k);
}

// The block's totals to slot lb of each component.
template <int K, int STRIDE = 1, int TAG = 0, int NT = kBlock>
__device__ __forceinline__ void store_sys_partials(double* __restrict__ part, int stride, int lb, double (&e)[K]) {
    block_store<K, STRIDE, TAG, NT>(part + lb, stride, e);
}

// The lanes of a row loop's epilogue with lane code L (L = 1: the tiles' kSolTileLanes).
constexpr int epi_stride(int L) { return L == 1 ? kSolTileLanes : L; }

// ------------------------------------------------------------------ standalone SpMV with residual epilogue

enum : int {
    EPI_NONE = 0,  // y = A x
    EPI_RESID = 1  // y = w - A x; partial ||y||^2 (1 component)
};

template <typename T> struct SpmvArgs {
    int n;
    Geom geo;
    const int* __restrict__ row_ptr;
    const int* __restrict__ col_idx;
    const cx<T>* __restrict__ vals;
    const cx<T>* __restrict__ x;
    cx<T>* __restrict__ y;
    const cx<T>* __restrict__ w;  // b for EPI_RESID
    double* __restrict__ part;    // region for EPI_RESID's partial
};

template <typename T, int L, int U, int EPI>
__global__ HZ_STREAM_BOUNDS void k_spmv(const SpmvArgs<T> a) {
    const RowRange rr = rows_of_block(a.n, a.geo);
    const cx<T>* __restrict__ xv = a.x;
    auto op = [xv](int c) { return xv[c]; };
    double e[1] = {0.0};
    for_rows<T, L, U>(rr.rw, a.row_ptr, a.col_idx, a.vals, op, [&](int64_t row, cx<T> acc) {
        if constexpr (EPI == EPI_RESID) {
            const cx<T> bw = a.w[row];
            acc.x = bw.x - acc.x;
            acc.y = bw.y - acc.y;
            e[0] = __builtin_fma((double)acc.x, (double)acc.x, e[0]);
            e[0] = __builtin_fma((double)acc.y, (double)acc.y, e[0]);
        }
        a.y[row] = acc;
    });
    if constexpr (EPI == EPI_RESID) store_partials<1>(a.part, rr.lb, e);
}

// y = b - A x over the solver's work map, per-system partial ||y||^2 in
// region I (the initial residual and the final true residual of a solve).
template <typename T, int L, int U>
__global__ HZ_STREAM_BOUNDS void k_sys_resid(const BicgArgs<T> a, const cx<T>* __restrict__ vals,
                                             const cx<T>* __restrict__ xin, cx<T>* __restrict__ y) {
    const SysBlock q = sys_block(a);
    if (q.sys < 0) return;
    auto op = [xin](int c) { return xin[c]; };
    double e[1] = {0.0};
    for_rows<T, L, U>(q.rw, a.row_ptr, a.col_idx, vals, op, [&](int64_t row, cx<T> acc) {
        const cx<T> bw = a.b[row];
        acc.x = bw.x - acc.x;
        acc.y = bw.y - acc.y;
        e[0] = __builtin_fma((double)acc.x, (double)acc.x, e[0]);
        e[0] = __builtin_fma((double)acc.y, (double)acc.y, e[0]);
        y[row] = acc;
    });
    store_sys_partials<1, epi_stride(L)>(a.part + kPartI * a.stride, a.stride, q.lb, e);
}

// ------------------------------------------------------------------ BiCGStab: three or four kernels per iteration
//
// Iteration i (Section 7's P-BiCGSTAB, right-preconditioned; A here is the
// column-scaled matrix under Jacobi), for every system of the launch:
//   A-kernel: v = A p; partial <rhat, v>.  No scalars: it starts on its rows at once.
//   S-kernel: the end of iteration i-1 decided from ||r||; alpha = rho / <rhat, v>;
//             s = r - alpha v.
//   B-kernel: t = A s; partials ||s||^2, <t, s>, ||t||^2, <rhat, t>, <rhat, s>.
//   C-kernel: half-step test on ||s||; omega = <t, s>/<t, t>;
//             rho_{i+1} = <rhat, s> - omega <rhat, t>; beta;
//             x += alpha p + omega s; r = s - omega t; p = r + beta (p - omega v);
//             partial ||r||^2.
// rho of the next iteration comes from sums that the B-kernel takes beside
// the others (<rhat, r> by linearity; <rhat, s> vanishes but for rounding, so
// no cancellation is added), which lets one pass update x, r and p: a kernel
// that read r, p, v again and wrote p is gone, with its launch (48 n bytes an
// iteration), and rhat is read by the two products only.
//
// On a small system the S-kernel is folded into the B-kernel, which forms s
// for every gathered column (k_bicg_SB), so an iteration is three
// launches; see choose_fused.
//
// Systems of a batch share nothing but the launches: each has its own
// scalars, partial range and exit.  The heads issue every load (scalars,
// partials, first rows or elements) before the reduction's one barrier, so
// their latencies overlap; decisions are taken after it.

// The end of iteration it - 1 (it >= 2) from ||r||^2: convergence, breakdown,
// iteration limit, in the order of the textbook loop.  Returns the status
// that ends the solve, or -1.
struct EndIn {
    double bnorm, rtol;
    double2 omega, rho, beta;  // omega of iteration it - 1; rho and beta of iteration it
    int maxiter;
};
__device__ __forceinline__ int iteration_end(int it, double rr, const EndIn& z, double& rel, int& sit, int& why) {
    rel = __builtin_sqrt(rr) / z.bnorm;
    why = BD_NONE;
    sit = it - 1;
    if (!__builtin_isfinite(rel)) return ST_NONFINITE;
    if (rel <= z.rtol) return ST_OK;
    if (zzero(z.omega)) {
        why = BD_OMEGA;
        return ST_BREAKDOWN;
    }
    if (it - 1 >= z.maxiter) {
        sit = z.maxiter;
        return ST_NOT_CONVERGED;
    }
    sit = it;
    if (!zfinite(z.rho)) return ST_NONFINITE;
    if (zzero(z.rho)) {
        why = BD_RHO;
        return ST_BREAKDOWN;
    }
    if (!zfinite(z.beta)) return ST_NONFINITE;
    return -1;
}

// Head of the S-kernel and of the B-kernel that contains it: conclude a
// half-step exit or iteration it - 1, then alpha = rho / <rhat, v>.  load()
// issues the loads; run() returns false when the system's solve has ended
// (every block of the system returns); its leader records the decision.  The
// scalar arithmetic (FP64 divisions and a square root) runs in the first wave
// only and is broadcast: in all 16 waves it kept the SIMDs busy for longer
// than the extra barrier costs.
template <int NT = kBlock> struct AlphaHead {
    PartSum<3, NT> ps;
    int done, pending, it;
    EndIn z;

    template <typename T> __device__ __forceinline__ void load(const BicgArgs<T>& a, const SysBlock& q) {
        const SolverScal* sc = a.sc + q.sys;
        done = sc->done;
        pending = sc->pending;
        it = sc->iter;
        z.bnorm = sc->bnorm;
        z.rtol = sc->rtol;
        z.maxiter = sc->maxiter;
        z.omega = sc->omega;
        z.beta = sc->beta;
        const double2 r0 = sc->rho2[0], r1 = sc->rho2[1];
        z.rho = (it & 1) ? r1 : r0;
        const int c = ps.comp();  // <rhat, v>, then ||r||^2
        if (c < 3)
            ps.load(a.part + (c < 2 ? kPartA + c : kPartC + 2) * a.stride + q.gbeg, c < 2 ? prod_parts(a, q) : q.gcnt);
    }
    template <typename T> __device__ __forceinline__ bool run(const BicgArgs<T>& a, const SysBlock& q, double2& alpha) {
        __shared__ double tot[NT / kWave];
        __shared__ double2 al;
        __shared__ int go;
        if (ps.comp() < 3) ps.store(tot);
        __syncthreads();
        if (wave_id() == 0) {
            const double s0 = ps.at(tot, 0), s1 = ps.at(tot, 1), rr = ps.at(tot, 2);
            const int g = decide(a, q, s0, s1, rr, alpha);
            if (threadIdx.x == 0) {
                al = alpha;
                go = g;
            }
        }
        __syncthreads();
        alpha = al;
        return go != 0;
    }
    template <typename T>
    __device__ __forceinline__ bool decide(const BicgArgs<T>& a, const SysBlock& q, double s0, double s1, double rr,
                                           double2& alpha) {
        SolverScal* sc = a.sc + q.sys;
        alpha = mk<double>(0.0, 0.0);
        if (done) return false;
        if (pending) {  // every block of the previous kernel has applied x += alpha p
            if (sys_leader(q)) finish(sc, a.ndone, ST_OK, pending);
            return false;
        }
        if (it > 1) {
            double rel;
            int sit, why;
            const int st = iteration_end(it, rr, z, rel, sit, why);
            if (sys_leader(q)) sc->relres = rel;
            if (st >= 0) {
                if (sys_leader(q)) finish(sc, a.ndone, st, sit, why);
                return false;
            }
        }
        const double2 sigma = mk<double>(s0, s1);
        if (!zfinite(sigma) || zzero(sigma)) {
            if (sys_leader(q))
                finish(sc, a.ndone, zzero(sigma) ? ST_BREAKDOWN : ST_NONFINITE, it, zzero(sigma) ? BD_RHAT_V : BD_NONE);
            return false;
        }
        alpha = zdiv(z.rho, sigma);
        if (sys_leader(q)) {
            sc->alpha = alpha;
            sc->cur = it;
        }
        return true;
    }
};

// After the last iteration of a limited solve: conclude it (one block per system).
template <typename T> __global__ HZ_STREAM_BOUNDS void k_bicg_end(const BicgArgs<T> a) {
    const int j = blockIdx.x;
    const SysMap sm = sys_range(a, j);
    SolverScal* sc = a.sc + j;
    double h[1];
    sys_sum<1>(a.part + (kPartC + 2) * a.stride, a.stride, sm.gbeg, sm.gcnt, h);
    if (threadIdx.x != 0 || sc->done) return;
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

// PAST kernels (asynchronous solves) first ask whether the solve's end lies
// behind them: such a call launches its limit of iterations, most of them past
// the end as a rule, and a block with loads in flight stays until they return.
// An iteration past the end takes 4.8 us in three launches (up to 131,072
// rows) and 6.5 us in four; without the question, and with one launch for each
// form of a product, 9.3 to 18 us.  In a synchronous solve, which stops within a
// chunk, the question costs 0.2 us of a small iteration.  (`done` would not do:
// S, SB and C set it themselves, and waves that return on it would be missing
// at the barriers of waves that have read it before.)
template <bool PAST, typename T> __device__ __forceinline__ bool past_end(const BicgArgs<T>& a) {
    if constexpr (PAST) return a.sc->closed != 0;
    else return false;
}
// Whether an A-kernel, which is no part of deciding the end, has nothing to do.
template <bool PAST> __device__ __forceinline__ bool ended(SolverScal* sc, bool leader) {
    const int done = sc->done;
    if (PAST && done != 0 && leader) sc->closed = 1;
    return done != 0 || sc->pending != 0;
}

// v = A p; partial <rhat, v>
template <typename T, int L, int U, bool PAST> __device__ __forceinline__ void bicg_A(const BicgArgs<T>& a) {
    const SysBlock q = sys_block(a);
    if (q.sys < 0) return;
    FirstRow<T, 0> f;
    first_row<T, L, 0>(f, q.rw, a.row_ptr, a.col_idx, a.vals);
    if (ended<PAST>(a.sc + q.sys, sys_leader(q))) return;
    zero_slots(a, kPartA, 2, q.lb, a.G, threadIdx.x == 0);
    const cx<T>* __restrict__ p = a.p;
    cx<T>* __restrict__ v = a.v;
    const cx<T>* __restrict__ rh = a.rh;
    double e[2] = {0.0, 0.0};
    for_rows<T, L, U, 0>(
        f, q.rw, a.row_ptr, a.col_idx, a.vals, [p](int c) { return p[c]; },
        [&](int64_t row, cx<T> acc, cx<T> w) {
            v[row] = acc;
            const double2 c = cdotacc(w.x, w.y, acc.x, acc.y, mk<double>(e[0], e[1]));
            e[0] = c.x;
            e[1] = c.y;
        },
        [rh](int64_t row) { return rh[row]; });
    store_sys_partials<2, epi_stride(L)>(a.part + kPartA * a.stride, a.stride, q.lb, e);
}
template <typename T, int L, int U, bool PAST = false>
__global__ HZ_STREAM_BOUNDS void k_bicg_A(const BicgArgs<T> a) {
    if (!past_end<PAST>(a)) bicg_A<T, L, U, PAST>(a);
}

// s = r - alpha v
template <typename T, bool PAST = false>
__global__ HZ_STREAM_BOUNDS void k_bicg_S(const BicgArgs<T> a) {
    if (past_end<PAST>(a)) return;
    const SysBlock q = sys_block(a);
    if (q.sys < 0 || (a.s_csr && *slice_no(a.ndone) == 0)) return;
    AlphaHead<> hd;
    hd.load(a, q);
    const cx<T>* __restrict__ v = a.v;
    const cx<T>* __restrict__ r = a.r;
    int64_t i = q.rw.x0 + (int64_t)q.rw.k * kBlock + threadIdx.x;
    const int64_t step = (int64_t)q.rw.K * kBlock;
    cx<T> v0 = mk<T>(T(0), T(0)), r0 = v0;
    if (i < q.rw.x1) {
        v0 = v[i];
        r0 = r[i];
    }
    double2 alpha;
    if (!hd.run(a, q, alpha)) return;
    const cx<T> nal = mk<T>((T)-alpha.x, (T)-alpha.y);
    while (i < q.rw.x1) {
        const int64_t at = i;
        const cx<T> s = cfma<T>(nal, v0, r0);
        i += step;
        if (i < q.rw.x1) {
            v0 = v[i];
            r0 = r[i];
        }
        a.s[at] = s;
    }
}

// The dot products of a row of t = A s: ||s||^2, <t, s>, ||t||^2, <rhat, t>, <rhat, s>.
template <typename T> __device__ __forceinline__ void b_terms(double (&e)[8], cx<T> s, cx<T> t, cx<T> w) {
    e[0] = __builtin_fma((double)s.x, (double)s.x, e[0]);
    e[0] = __builtin_fma((double)s.y, (double)s.y, e[0]);
    double2 c = cdotacc(t.x, t.y, s.x, s.y, mk<double>(e[1], e[2]));
    e[1] = c.x;
    e[2] = c.y;
    e[3] = __builtin_fma((double)t.x, (double)t.x, e[3]);
    e[3] = __builtin_fma((double)t.y, (double)t.y, e[3]);
    c = cdotacc(w.x, w.y, t.x, t.y, mk<double>(e[4], e[5]));
    e[4] = c.x;
    e[5] = c.y;
    c = cdotacc(w.x, w.y, s.x, s.y, mk<double>(e[6], e[7]));
    e[6] = c.x;
    e[7] = c.y;
}

// The epilogue operands of a row of t = A s: s and rhat.
template <typename T> struct BRow {
    cx<T> s, w;
};

// t = A s and its dot products
template <typename T, int L, int U> __device__ __forceinline__ void bicg_B(const BicgArgs<T>& a) {
    const SysBlock q = sys_block(a);
    if (q.sys < 0) return;
    FirstRow<T, 0> f;
    first_row<T, L, 0>(f, q.rw, a.row_ptr, a.col_idx, a.vals);
    if (a.sc[q.sys].done) return;
    zero_slots(a, kPartB, 8, q.lb, a.G, threadIdx.x == 0);
    const cx<T>* __restrict__ sv = a.s;
    const cx<T>* __restrict__ rh = a.rh;
    cx<T>* __restrict__ tv = a.t;
    double e[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for_rows<T, L, U, 0>(
        f, q.rw, a.row_ptr, a.col_idx, a.vals, [sv](int c) { return sv[c]; },
        [&](int64_t row, cx<T> acc, BRow<T> m) {
            tv[row] = acc;
            b_terms<T>(e, m.s, acc, m.w);
        },
        [sv, rh](int64_t row) { return BRow<T>{sv[row], rh[row]}; });
    store_sys_partials<8, epi_stride(L)>(a.part + kPartB * a.stride, a.stride, q.lb, e);
}
template <typename T, int L, int U, bool PAST = false>
__global__ HZ_STREAM_BOUNDS void k_bicg_B(const BicgArgs<T> a) {
    if (!past_end<PAST>(a)) bicg_B<T, L, U>(a);
}

// The same with the S-kernel's head: s = r - alpha v is formed for every
// gathered column and stored.  One block per CU: the head, the prefetched
// entries and eight sums need more than the 64 registers of two.
template <typename T, int L, int U> __device__ __forceinline__ void bicg_SB(const BicgArgs<T>& a) {
    const SysBlock q = sys_block(a);
    if (q.sys < 0) return;
    zero_slots(a, kPartB, 8, q.lb, a.G, threadIdx.x == 0);
    AlphaHead<> hd;
    hd.load(a, q);
    FirstRow<T, U> f;
    first_row<T, L, U>(f, q.rw, a.row_ptr, a.col_idx, a.vals);
    double2 alpha;
    if (!hd.run(a, q, alpha)) return;
    const cx<T> nal = mk<T>((T)-alpha.x, (T)-alpha.y);
    const cx<T>* __restrict__ r = a.r;
    const cx<T>* __restrict__ v = a.v;
    const cx<T>* __restrict__ rh = a.rh;
    cx<T>* __restrict__ sv = a.s;
    cx<T>* __restrict__ tv = a.t;
    auto scol = [=](int c) { return cfma<T>(nal, v[c], r[c]); };
    double e[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    for_rows<T, L, U, U>(
        f, q.rw, a.row_ptr, a.col_idx, a.vals, scol,
        [&](int64_t row, cx<T> acc, BRow<T> m) {
            sv[row] = m.s;
            tv[row] = acc;
            b_terms<T>(e, m.s, acc, m.w);
        },
        [=](int64_t row) { return BRow<T>{scol((int)row), rh[row]}; });
    store_sys_partials<8, epi_stride(L)>(a.part + kPartB * a.stride, a.stride, q.lb, e);
}
template <typename T, int L, int U, bool PAST = false>
__global__ __launch_bounds__(kBlock) void k_bicg_SB(const BicgArgs<T> a) {
    if (!past_end<PAST>(a)) bicg_SB<T, L, U>(a);
}

// p_{i+1} = r_{i+1} + beta (p_i - omega v_i)
template <typename T>
__device__ __forceinline__ cx<T> p_update(cx<T> bt, cx<T> omt, cx<T> rc, cx<T> pc, cx<T> vc) {
    const cx<T> d = mk<T>(pc.x - fmaT(omt.x, vc.x, -omt.y * vc.y), pc.y - fmaT(omt.x, vc.y, omt.y * vc.x));
    return cfma<T>(bt, d, rc);
}

template <typename T, bool PAST = false>
__global__ HZ_STREAM_BOUNDS void k_bicg_C(const BicgArgs<T> a) {
    enum : int { STOP = 0, HALF = 1, FULL = 2 };
    __shared__ double tot[kBlock / kWave];
    __shared__ double2 coef[3];  // alpha, omega, beta
    __shared__ int mode;
    if (past_end<PAST>(a)) return;
    const SysBlock q = sys_block(a);
    if (q.sys < 0) return;
    SolverScal* sc = a.sc + q.sys;
    const int done = sc->done, it = sc->cur;
    const double bnorm = sc->bnorm, rtol = sc->rtol;
    const double2 alpha = sc->alpha, rho_0 = sc->rho2[0], rho_1 = sc->rho2[1];
    const double2 rho = (it & 1) ? rho_1 : rho_0;
    PartSum<8> ps;
    ps.load(a.part + (kPartB + ps.comp()) * a.stride + q.gbeg, prod_parts(a, q));
    // the first element's s, t and p are in flight during the head (32-bit
    // indices: with 64-bit ones the kernel spilled two of its 64 registers)
    cx<T> s0 = mk<T>(T(0), T(0)), t0 = s0, p0 = s0;
    int i = (int)q.rw.x0 + q.rw.k * kBlock + threadIdx.x;
    const int step = q.rw.K * kBlock, end = (int)q.rw.x1;
    if (i < end) {
        s0 = a.s[i];
        t0 = a.t[i];
        p0 = a.p[i];
    }
    ps.store(tot);
    __syncthreads();
    if (wave_id() == 0) {  // the decision and the scalars, once per block
        double h[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) h[k] = ps.at(tot, k);
        auto decide = [&]() -> int {
            if (done) return STOP;
            const bool lead = sys_leader(q);
            const double rel = __builtin_sqrt(h[0]) / bnorm;
            if (!__builtin_isfinite(rel)) {
                if (lead) finish(sc, a.ndone, ST_NONFINITE, it);
                return STOP;
            }
            if (rel <= rtol) {  // concluded by the next head
                if (lead) {
                    sc->relres = rel;
                    sc->pending = it;
                }
                return HALF;
            }
            const double2 ts = mk<double>(h[1], h[2]);
            const double tt = h[3];
            int st = -1, why = BD_NONE;
            double2 om = mk<double>(0.0, 0.0);
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
            // rho and beta of the next iteration; omega = 0, rho = 0 or a non-finite
            // beta end the solve in the next head, after its test on ||r||
            const double2 ort = zmul(om, mk<double>(h[4], h[5]));
            const double2 rho_n = mk<double>(h[6] - ort.x, h[7] - ort.y);
            const double2 beta = zmul(zdiv(rho_n, rho), zdiv(alpha, om));
            if (lead) {
                sc->omega = om;
                sc->rho2[(it + 1) & 1] = rho_n;
                sc->beta = beta;
                sc->iter = it + 1;
            }
            if (threadIdx.x == 0) {
                coef[1] = om;
                coef[2] = beta;
            }
            return FULL;
        };
        const int md = decide();
        if (threadIdx.x == 0) {
            coef[0] = alpha;
            mode = md;
        }
    }
    __syncthreads();
    if (mode == STOP) return;
    const cx<T> al = narrow<T>(coef[0]);
    if (mode == HALF) {  // half-step exit: x += alpha p
        HZ_FOR_ELEMS(j, q.rw) a.x[j] = cfma<T>(al, a.p[j], a.x[j]);
        return;
    }
    const cx<T> omt = narrow<T>(coef[1]), nom = mk<T>(-omt.x, -omt.y), bt = narrow<T>(coef[2]);
    double e[1] = {0.0};
    while (i < end) {
        const int j = i;
        const cx<T> v = a.v[j];
        cx<T> x = cfma<T>(al, p0, a.x[j]);
        x = cfma<T>(omt, s0, x);
        const cx<T> r = cfma<T>(nom, t0, s0);
        const cx<T> p = p_update<T>(bt, omt, r, p0, v);
        i = i < end - step ? i + step : end;
        if (i < end) {
            s0 = a.s[i];
            t0 = a.t[i];
            p0 = a.p[i];
        }
        a.x[j] = x;
        a.r[j] = r;
        a.p[j] = p;
        e[0] = __builtin_fma((double)r.x, (double)r.x, e[0]);
        e[0] = __builtin_fma((double)r.y, (double)r.y, e[0]);
    }
    store_sys_partials<1>(a.part + (kPartC + 2) * a.stride, a.stride, q.lb, e);
}

// Locality of a CSR matrix: count of entries with |col - row| > W (integer atomics).
__global__ __launch_bounds__(kBlock) void k_far_count(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                                      int W, unsigned long long* __restrict__ count) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    double c = 0.0;  // exact: counts stay far below 2^53
    if (i < n)
        for (int p = rp[i]; p < rp[i + 1]; ++p) {
            const int64_t d = (int64_t)ci[p] - i;
            c += (d > W || d < -W) ? 1.0 : 0.0;
        }
    c = group_sum<64>(c);
    if (threadIdx.x % kWave == 0 && c != 0.0) atomicAdd(count, (unsigned long long)c);
}

// Solve set-up: r = src (b, or the residual b - A x0), rhat = r;
// partials <rhat, r>, ||r||^2 (region C) and ||b||^2 (region I).
template <typename T>
__global__ __launch_bounds__(kBlock) void k_init(const BicgArgs<T> a, const cx<T>* src) {
    const SysBlock q = sys_block(a);
    if (q.sys < 0) return;
    double e[3] = {0.0, 0.0, 0.0}, eb[1] = {0.0};
    HZ_FOR_ELEMS(i, q.rw) {
        const cx<T> bv = a.b[i], rv = src[i];
        if (a.r != src) a.r[i] = rv;
        const_cast<cx<T>*>(a.rh)[i] = rv;
        if (a.p != nullptr) a.p[i] = rv;  // p_1 = r_0 (BiCGStab)
        eb[0] = __builtin_fma((double)bv.x, (double)bv.x, eb[0]);
        eb[0] = __builtin_fma((double)bv.y, (double)bv.y, eb[0]);
        double2 c = cdotacc(rv.x, rv.y, rv.x, rv.y, mk<double>(e[0], e[1]));
        e[0] = c.x;
        e[1] = c.y;
        e[2] = __builtin_fma((double)rv.x, (double)rv.x, e[2]);
        e[2] = __builtin_fma((double)rv.y, (double)rv.y, e[2]);
    }
    store_sys_partials<3>(a.part + kPartC * a.stride, a.stride, q.lb, e);
    store_sys_partials<1, 1, 1>(a.part + kPartI * a.stride, a.stride, q.lb, eb);
}

// ||b||, initial convergence test, per system (one block per system); iteration 1 comes next.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_fin_init(const BicgArgs<T> a) {
    const int j = blockIdx.x;
    const SysMap sm = sys_range(a, j);
    SolverScal* sc = a.sc + j;
    double hb[1], hr[3];
    sys_sum<1>(a.part + kPartI * a.stride, a.stride, sm.gbeg, sm.gcnt, hb);
    sys_sum<3>(a.part + kPartC * a.stride, a.stride, sm.gbeg, sm.gcnt, hr);
    if (threadIdx.x != 0) return;
    const double bn = __builtin_sqrt(hb[0]);
    sc->bnorm = bn;
    sc->iter = 1;
    sc->cur = 0;
    sc->done = 0;
    sc->zero_x = 0;
    sc->iters = 0;
    sc->pending = 0;
    sc->closed = 0;
    sc->why = BD_NONE;
    sc->status = ST_NOT_CONVERGED;
    sc->alpha = sc->omega = sc->beta = mk<double>(1.0, 0.0);
    sc->rho2[1] = mk<double>(hr[0], hr[1]);  // rho of iteration 1
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

// relres_true = sqrt(region I over the system) / ||b||, one block per system
template <typename T>
__global__ __launch_bounds__(kBlock) void k_fin_true(const BicgArgs<T> a) {
    const int j = blockIdx.x;
    const SysMap sm = sys_range(a, j);
    double h[1];
    sys_sum<1>(a.part + kPartI * a.stride, a.stride, sm.gbeg, sm.gcnt, h);
    SolverScal* sc = a.sc + j;
    if (threadIdx.x == 0) sc->relres_true = sc->bnorm > 0.0 ? __builtin_sqrt(h[0]) / sc->bnorm : 0.0;
}

// x = 0 on the rows of systems whose right-hand side is zero
template <typename T>
__global__ __launch_bounds__(kBlock) void k_zero_if(const BicgArgs<T> a) {
    const SysBlock q = sys_block(a);
    if (q.sys < 0 || !a.sc[q.sys].zero_x) return;
    HZ_FOR_ELEMS(i, q.rw) a.x[i] = mk<T>(T(0), T(0));
}

// ------------------------------------------------------------------ Jacobi folding: A D^{-1}

// dinv_i = 1 / A_ii (the last diagonal entry of the row); flags a missing or
// zero diagonal and, with no != null, what the sliced operator cannot hold: a
// column too far from the row's slice, a row without a diagonal, or one whose
// reciprocal is not its inverse (|A_ii|^2 a NaN, or outside the normal range),
// so that the diagonal of A D^{-1} is not 1.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_jacobi_diag(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                                        const cx<T>* __restrict__ vals, cx<T>* __restrict__ dinv,
                                                        SolverScal* sc, int* no) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    cx<T> d = mk<T>(T(0), T(0));
    const int base = (int)i & ~(kWave - 1);
    bool far = false, has = false;
    for (int p = rp[i]; p < rp[i + 1]; ++p) {
        const int c = ci[p];
        if (c == i) {
            d = vals[p];
            has = true;
        }
        far = far || c - base > 32767 || base - c > 32768;
    }
    if (no != nullptr && (far || !has)) *no = 1;  // every writer stores 1
    if (d.x == T(0) && d.y == T(0)) {
        sc->bad_diag = 1;  // every writer stores 1
        dinv[i] = mk<T>(T(0), T(0));
        return;
    }
    const T q = d.x * d.x + d.y * d.y;
    using lim = std::numeric_limits<T>;
    if (no != nullptr && !(q >= lim::min() && q <= lim::max())) *no = 1;
    dinv[i] = mk<T>(d.x / q, -d.y / q);
}

// out_p = vals_p * dinv[col_p]   (column scaling A D^{-1}, rounded to TO for
// the complex64 iteration)
template <typename TO>
__global__ __launch_bounds__(kBlock) void k_colscale(int64_t nnz, const int* __restrict__ ci,
                                                     const double2* __restrict__ vals,
                                                     const double2* __restrict__ dinv, cx<TO>* __restrict__ out) {
    const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (p >= nnz) return;
    const double2 a = cmul<double>(vals[p], dinv[ci[p]]);
    out[p] = mk<TO>((TO)a.x, (TO)a.y);
}

// y_i = d_i x_i with d = 1 / dinv (the preconditioned initial iterate), or x_i = dinv_i y_i at the end
template <typename T>
__global__ __launch_bounds__(kBlock) void k_diag_apply(int n, const cx<T>* __restrict__ dinv, cx<T>* __restrict__ x,
                                                       int invert) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    cx<T> d = dinv[i];
    if (invert) {
        const T q = d.x * d.x + d.y * d.y;
        d = mk<T>(d.x / q, -d.y / q);
    }
    x[i] = cmul<T>(d, x[i]);
}


// ------------------------------------------------------------------ standalone BLAS-1

template <int MODE>  // 0: conj(x) y  (2 comps), 1: |x|^2 (1 comp)
__global__ __launch_bounds__(kBlock) void k_dot_part(int n, Geom geo, const double2* __restrict__ x,
                                                     const double2* __restrict__ y, double* __restrict__ part) {
    const RowRange rr = rows_of_block(n, geo);
    constexpr int K = MODE == 0 ? 2 : 1;
    double e[K];
#pragma unroll
    for (int k = 0; k < K; ++k) e[k] = 0.0;
    HZ_FOR_ELEMS(i, rr.rw) {
        const double2 xv = x[i];
        if constexpr (MODE == 0) {
            const double2 yv = y[i];
            double2 c = cdotacc(xv.x, xv.y, yv.x, yv.y, mk<double>(e[0], e[1]));
            e[0] = c.x;
            e[1] = c.y;
        } else {
            e[0] = __builtin_fma(xv.x, xv.x, e[0]);
            e[0] = __builtin_fma(xv.y, xv.y, e[0]);
        }
    }
    store_partials<K>(part, rr.lb, e);
}

template <int MODE>
__global__ __launch_bounds__(kBlock) void k_dot_fin(const double* __restrict__ part, int G, void* out) {
    constexpr int K = MODE == 0 ? 2 : 1;
    double s[K];
    head_sum<K>(part, G, s);
    if (threadIdx.x != 0) return;
    if constexpr (MODE == 0) {
        static_cast<double2*>(out)[0] = mk<double>(s[0], s[1]);
    } else {
        static_cast<double*>(out)[0] = __builtin_sqrt(s[0]);
    }
}

__global__ __launch_bounds__(kBlock) void k_zaxpy(int64_t n, double2 alpha, const double2* __restrict__ x,
                                                  double2* __restrict__ y) {
    const int64_t stride = (int64_t)gridDim.x * kBlock;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += stride) y[i] = cfma<double>(alpha, x[i], y[i]);
}

// ------------------------------------------------------------------ CSR validation

__global__ __launch_bounds__(kBlock) void k_validate(int n, int nnz, const int* __restrict__ rp, const int* __restrict__ ci,
                                                     int* __restrict__ bad) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i > n) return;
    const int a = rp[i];
    if (i == 0 && a != 0) *bad = 1;
    if (i == n) {
        if (a != nnz) *bad = 1;
        return;
    }
    const int b = rp[i + 1];
    if (b < a || a < 0 || b > nnz) {
        *bad = 1;
        return;
    }
    for (int p = a; p < b; ++p)
        if (ci[p] < 0 || ci[p] >= n) {
            *bad = 1;
            return;
        }
}

}  // namespace hz

// ================================================================== mixed precision (complex64 inner solve)
namespace hz {

// out32_p = complex64(vals_p)
__global__ __launch_bounds__(kBlock) void k_demote_vals(int64_t nnz, const double2* __restrict__ vals,
                                                        float2* __restrict__ out) {
    const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (p >= nnz) return;
    const double2 v = vals[p];
    out[p] = mk<float>((float)v.x, (float)v.y);
}

__global__ __launch_bounds__(kBlock) void k_demote_vec(int n, const double2* __restrict__ in, float2* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const double2 v = in[i];
    out[i] = mk<float>((float)v.x, (float)v.y);
}

// Outer scalars of the refinement live in a second SolverScal: bnorm, relres,
// status/done, and outer_rn = ||r|| of the current outer residual.
__global__ __launch_bounds__(kBlock) void k_fin_bnorm(const double* __restrict__ part, int G, SolverScal* sc) {
    double s[1];
    head_sum<1>(part, G, s);
    if (threadIdx.x == 0) sc->bnorm = __builtin_sqrt(s[0]);
}

// After r = b - A x: decide convergence; otherwise record ||r|| for the next correction.
__global__ __launch_bounds__(kBlock) void k_fin_outer(const double* __restrict__ part, int G, SolverScal* sc,
                                                      int outer, int max_outer) {
    double s[1];
    head_sum<1>(part, G, s);
    if (threadIdx.x != 0) return;
    const double rn = __builtin_sqrt(s[0]), bn = sc->bnorm;
    sc->outer_rn = rn;
    int st = -1;
    if (!__builtin_isfinite(rn) || !__builtin_isfinite(bn)) st = ST_NONFINITE;
    else if (bn == 0.0) {
        sc->zero_x = 1;
        sc->relres = 0.0;
        st = ST_OK;
    } else {
        const double rel = rn / bn;
        sc->relres = rel;
        sc->relres_true = rel;
        if (rel <= sc->rtol) st = ST_OK;
        else if (outer >= max_outer) st = ST_NOT_CONVERGED;
    }
    if (st >= 0) {
        sc->status = st;
        sc->iters = outer;
        sc->done = 1;
    }
}

// b32 = complex64(r / ||r||)
__global__ __launch_bounds__(kBlock) void k_demote_scaled(int n, const double2* __restrict__ r, const SolverScal* sc,
                                                          float2* __restrict__ out) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const double inv = 1.0 / sc->outer_rn;
    const double2 v = r[i];
    out[i] = mk<float>((float)(v.x * inv), (float)(v.y * inv));
}

// x += ||r|| * D^{-1} d  (FP64 update of the FP64 iterate)
__global__ __launch_bounds__(kBlock) void k_promote_add(int n, const float2* __restrict__ d, const float2* __restrict__ dinv,
                                                        const SolverScal* sc, double2* __restrict__ x) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const double rn = sc->outer_rn;
    double2 dv = mk<double>((double)d[i].x, (double)d[i].y);
    if (dinv != nullptr) dv = zmul(mk<double>((double)dinv[i].x, (double)dinv[i].y), dv);
    double2 xv = x[i];
    xv.x = __builtin_fma(rn, dv.x, xv.x);
    xv.y = __builtin_fma(rn, dv.y, xv.y);
    x[i] = xv;
}

}  // namespace hz
