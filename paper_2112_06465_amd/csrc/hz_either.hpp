// BiCGStab's products of an asynchronous Jacobi solve, which choose the
// operator's form on the device.
//
// Whether a matrix is sliced is known after the set-up kernels, in the word
// after the done-counter; a synchronous solve reads it and launches the sliced
// or the CSR products.  An asynchronous one may not wait, and a launch for each
// form, one of which returns at once, costs a launch more per product in every
// iteration, and most of a call's iterations lie past the solve's end.  So these
// kernels hold both forms, in blocks of the CSR form's size: 1,024 threads for
// vector rows, which do the work of up to four of the sliced form's blocks (same
// rows, same slots, same order of every sum, so the same bits as the synchronous
// solve), and 256 for tiles.  Streaming loads only with the tiles, which are for
// matrices that do not stay in the Infinity Cache either.
// Measured, Jacobi, us an iteration of the asynchronous solve (and past its end),
// two launches a product / these: 7,953 rows 17.3 (9.3) / 15.1 (4.8), 67,689 rows
// 25.3 (13.0) / 23.4 (5.3), 209,777 rows 41.0 (13.4) / 39.2 (6.8), 1.24 M rows 187
// (18) / 184 (6.7); one far column, 393,625 rows 66.6 (15.4) / 69.5 (6.8): the CSR
// form has one block per CU here.  No registers are to spare in Bx and SBx: with
// seven spilled, an iteration past the end took 0.5 us longer.
#pragma once

#include "hz_slices.hpp"
#include "hz_soltile.hpp"

namespace hz {

// Blocks of the sliced form, sg of them, that a block of kBlock threads stands
// for: as few as leave one block per CU, so that small systems are spread as
// widely as in the sliced form itself.
inline int either_share(int sg) {
    const int v = (sg + kMaxGrid / 2 - 1) / (kMaxGrid / 2);
    return v < kBlock / kSlBlock ? v : kBlock / kSlBlock;
}
// Blocks of a launch, with `share` blocks of the sliced form or one of the CSR form's in each.
inline int either_grid(const OneMap& one, int sg, int share, int csr) {
    const int K = (sg / one.groups + share - 1) / share;
    return one.groups * K > csr ? one.groups * K : csr;
}

// The form to run (or neither, past the solve's end), from two loads in flight together.
enum class Form { kNone, kCsr, kSliced };
template <typename T> __device__ __forceinline__ Form form_of(const BicgArgs<T>& a, int csr_blocks) {
    const int no = *slice_no(a.ndone), closed = a.sc->closed;
    if (closed != 0) return Form::kNone;
    if (no == 0) return Form::kSliced;
    return (int)blockIdx.x < csr_blocks ? Form::kCsr : Form::kNone;
}

template <typename T, int L, int U>
__global__ __launch_bounds__(kBlock) void k_bicg_Ax(const BicgArgs<T> a) {
    const Form f = form_of(a, a.G);
    if (f == Form::kSliced) bicg_As<T, false, true, kBlock, kSlWaves>(a);
    else if (f == Form::kCsr) bicg_A<T, L, U, true>(a);
}

// t = A s; FS: the sliced form forms s itself
template <typename T, int L, int U, bool FS>
__global__ __launch_bounds__(kBlock) void k_bicg_Bx(const BicgArgs<T> a) {
    const Form f = form_of(a, a.G);
    if (f == Form::kCsr) bicg_B<T, L, U>(a);
    if (f != Form::kSliced) return;
    if constexpr (FS) bicg_SBs<T, true, kBlock, kSlWaves>(a);
    else bicg_Bs<T, false, kBlock, kSlWaves>(a);
}

// both forms form s
template <typename T, int L, int U>
__global__ __launch_bounds__(kBlock) void k_bicg_SBx(const BicgArgs<T> a) {
    const Form f = form_of(a, a.G);
    if (f == Form::kSliced) bicg_SBs<T, true, kBlock, kSlWaves>(a);
    else if (f == Form::kCsr) bicg_SB<T, L, U>(a);
}

// The tiles leave 4 KB of LDS a block with four blocks per CU: the sliced
// form's sums are stored a component at a time.
template <typename T>
__global__ HZ_SLICE_BOUNDS void k_bicg_Atx(const BicgArgs<T> a) {
    const Form f = form_of(a, a.pf * a.G);
    if (f == Form::kCsr) bicg_At<T, true>(a);
    else if (f == Form::kSliced && (int)blockIdx.x < a.sg) bicg_As<T, true, true, kSlBlock, 1>(a);
}
template <typename T, bool FS>
__global__ HZ_SLICE_BOUNDS void k_bicg_Btx(const BicgArgs<T> a) {
    const Form f = form_of(a, a.pf * a.G);
    if (f == Form::kCsr) bicg_Bt<T>(a);
    if (f != Form::kSliced || (int)blockIdx.x >= a.sg) return;
    if constexpr (FS) bicg_SBs<T, true, kSlBlock, 1>(a);
    else bicg_Bs<T, true, kSlBlock, 1>(a);
}

}  // namespace hz
