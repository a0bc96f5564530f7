// Adjoint (backward) kernels of the helmz library.
//
// For x = A^{-1} b and a real loss L with real-pair gradient g = dL/dRe x +
// i dL/dIm x, the adjoint state lambda solves A^H lambda = g; then
// dL/db = lambda and dL/dA_ij = -lambda_i conj(x_j) on A's pattern.
//
// A^H is formed on the device in CSR (count, scan, scatter, per-row sort),
// deterministically: the scatter order is fixed afterwards by sorting each
// row by column index, and columns are unique.  When the caller asserts
// A = A^T (HZ_SYMMETRIC), A^H = conj(A) and the adjoint solve is the forward
// solve on conjugated data: A conj(lambda) = conj(g).
#pragma once

#include "hz_kernels.hpp"

namespace hz {

// counts[col_p + 1] += 1 for every entry (integer atomics: exact)
__global__ __launch_bounds__(kBlock) void k_tr_count(int64_t nnz, const int* __restrict__ ci, int* __restrict__ cnt) {
    const int64_t p = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (p < nnz) atomicAdd(&cnt[ci[p] + 1], 1);
}

// In-place inclusive scan of a[0..m) (16-byte aligned) with one block: rounds
// of 16 consecutive elements a thread, thread totals by a wave scan, wave
// totals through LDS.  Used once per adjoint set-up.  (A contiguous segment per
// thread, an element at a time, took 265 us at 92,478 elements; 21 us so.)
__global__ __launch_bounds__(1024) void k_scan_1block(int m, int* __restrict__ a) {
    constexpr int E = 16;
    __shared__ int wsum[1024 / kWave];
    const int lane = threadIdx.x % kWave, wid = threadIdx.x / kWave;
    int run = 0;
    for (int64_t c = 0; c < m; c += 1024 * E) {  // uniform
        const int64_t i0 = c + (int64_t)threadIdx.x * E;
        int v[E];
        if (i0 + E <= m) {
#pragma unroll
            for (int k = 0; k < E; k += 4) {
                const int4 q = *reinterpret_cast<const int4*>(a + i0 + k);
                v[k] = q.x;
                v[k + 1] = q.y;
                v[k + 2] = q.z;
                v[k + 3] = q.w;
            }
        } else {
#pragma unroll
            for (int k = 0; k < E; ++k) v[k] = i0 + k < m ? a[i0 + k] : 0;
        }
#pragma unroll
        for (int k = 1; k < E; ++k) v[k] += v[k - 1];
        int t = v[E - 1];
#pragma unroll
        for (int d = 1; d < kWave; d *= 2) {
            const int o = __shfl_up(t, d);
            t += lane >= d ? o : 0;
        }
        if (lane == kWave - 1) wsum[wid] = t;
        __syncthreads();
        int before = run + t - v[E - 1];
        for (int w = 0; w < 1024 / kWave; ++w) {
            before += w < wid ? wsum[w] : 0;
            run += wsum[w];
        }
        if (i0 + E <= m) {
#pragma unroll
            for (int k = 0; k < E; k += 4)
                *reinterpret_cast<int4*>(a + i0 + k) =
                    make_int4(before + v[k], before + v[k + 1], before + v[k + 2], before + v[k + 3]);
        } else {
#pragma unroll
            for (int k = 0; k < E; ++k)
                if (i0 + k < m) a[i0 + k] = before + v[k];
        }
        __syncthreads();  // wsum may be rewritten
    }
}

// scatter (i, j, a) -> row j of A^H with value conj(a); fill[] starts as a copy of t_row_ptr
__global__ __launch_bounds__(kBlock) void k_tr_scatter(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                                       const double2* __restrict__ v, int* __restrict__ fill,
                                                       int* __restrict__ tci, double2* __restrict__ tv) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    for (int p = rp[i]; p < rp[i + 1]; ++p) {
        const int q = atomicAdd(&fill[ci[p]], 1);
        tci[q] = (int)i;
        const double2 a = v[p];
        tv[q] = mk<double>(a.x, -a.y);
    }
}

// scatter entry p = (i, j) to row j of the transpose as column i, recording
// its source index p (the values of several systems are gathered by it later)
__global__ __launch_bounds__(kBlock) void k_tr_scatter_idx(int n, const int* __restrict__ rp,
                                                           const int* __restrict__ ci, int* __restrict__ fill,
                                                           int* __restrict__ tci, int* __restrict__ tsrc) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    for (int p = rp[i]; p < rp[i + 1]; ++p) {
        const int q = atomicAdd(&fill[ci[p]], 1);
        tci[q] = (int)i;
        tsrc[q] = p;
    }
}

// sort each row of a CSR matrix by column, carrying a payload per entry (the
// values, or source entry indices), stably.  Used for the transpose and for
// P A P^T.  A row belongs to kSortLanes lanes, which hold up to four entries
// each, find every entry's rank by passing the columns round, and store it
// there; longer rows are sorted by insertion, by one lane.  (Insertion in
// every row, a thread per row, took 3.1 ms on the 1.24 M-row cabin and 0.28 ms
// on 92k rows; 0.18 and 0.027 so.  Long rows gain too, since a wave waits for
// four rows' scattered accesses instead of 64: csr_zpermute of 20,000 rows of 120
// entries 11.2 -> 2.6 ms, of 200,000 rows of 300 317 -> 146 ms.)
// A launch holds fewer than 2^32 threads, 2^28 rows of 16 lanes: row_sort
// launches kSortRows rows at a time, from row j0 on.  (A loop over rows in the
// kernel took 9 % longer on 1 M rows of 15.)
constexpr int kSortLanes = 16, kSortBlock = 256, kSortRows = 1 << 24;
template <typename V>
__global__ __launch_bounds__(kSortBlock) void k_row_sort(int n, int j0, const int* __restrict__ trp, int* tci, V* tv) {
    constexpr int E = 4;
    const int64_t j = j0 + ((int64_t)blockIdx.x * kSortBlock + threadIdx.x) / kSortLanes;
    const int lane = threadIdx.x % kSortLanes;
    const int lo = j < n ? trp[j] : 0, len = j < n ? trp[j + 1] - lo : 0;
    const bool byrank = len <= E * kSortLanes;
    int c[E], rank[E];
    V v[E];
#pragma unroll
    for (int u = 0; u < E; ++u) {
        const int q = lane + u * kSortLanes;
        rank[u] = 0;
        c[u] = 0;
        if (byrank && q < len) {
            c[u] = tci[lo + q];
            v[u] = tv[lo + q];
        }
    }
#pragma unroll
    for (int w = 0; w < E; ++w) {
        if (!__any(byrank && w * kSortLanes < len)) break;  // uniform in the wave
        for (int l = 0; l < kSortLanes; ++l) {
            const int k = w * kSortLanes + l, ck = __shfl(c[w], l, kSortLanes);
#pragma unroll
            for (int u = 0; u < E; ++u) {
                const int q = lane + u * kSortLanes;
                rank[u] += k < len && (ck < c[u] || (ck == c[u] && k < q)) ? 1 : 0;
            }
        }
    }
    __syncthreads();  // every entry is in registers
#pragma unroll
    for (int u = 0; u < E; ++u)
        if (byrank && lane + u * kSortLanes < len) {
            tci[lo + rank[u]] = c[u];
            tv[lo + rank[u]] = v[u];
        }
    if (byrank || lane != 0) return;
    for (int q = lo + 1; q < lo + len; ++q) {
        const int cq = tci[q];
        const V a = tv[q];
        int k = q - 1;
        while (k >= lo && tci[k] > cq) {
            tci[k + 1] = tci[k];
            tv[k + 1] = tv[k];
            --k;
        }
        tci[k + 1] = cq;
        tv[k + 1] = a;
    }
}
template <typename V> void row_sort(hipStream_t s, int n, const int* trp, int* tci, V* tv) {
    for (int64_t j0 = 0; j0 < n; j0 += kSortRows) {
        const int64_t rows = n - j0 < kSortRows ? n - j0 : kSortRows;
        hipLaunchKernelGGL(k_row_sort<V>, dim3(unsigned((rows * kSortLanes + kSortBlock - 1) / kSortBlock)),
                           dim3(kSortBlock), 0, s, n, int(j0), trp, tci, tv);
    }
}

// out = conj(in); in and out may be the same array
__global__ __launch_bounds__(kBlock) void k_conj(int n, const double2* in, double2* out) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) {
        const double2 a = in[i];
        out[i] = mk<double>(a.x, -a.y);
    }
}

// grad_vals[p] = -lambda_i conj(x_{col p}) for the entries p of row i (L lanes per row)
template <int L>
__global__ __launch_bounds__(kBlock) void k_grad_vals(int n, Geom geo, const int* __restrict__ rp,
                                                      const int* __restrict__ ci, const double2* __restrict__ lam,
                                                      const double2* __restrict__ x, double2* __restrict__ gv) {
    constexpr int RPS = kBlock / L;
    const Rows rw = rows_of_block(n, geo).rw;
    const int g = threadIdx.x / L, lane = threadIdx.x % L;
    for (int64_t row = rw.x0 + (int64_t)rw.k * RPS + g; row < rw.x1; row += (int64_t)rw.K * RPS) {
        const double2 l = lam[row];
        for (int p = rp[row] + lane; p < rp[row + 1]; p += L) {
            const double2 xv = x[ci[p]];
            // -(l * conj(xv))
            gv[p] = mk<double>(-__builtin_fma(l.x, xv.x, l.y * xv.y), -__builtin_fma(l.y, xv.x, -l.x * xv.y));
        }
    }
}

}  // namespace hz
