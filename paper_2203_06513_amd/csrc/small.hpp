// The wave partials of a particle pass summed per cell, for the field updates that open the
// kernels of small grids (small_field_I, small_field_II): NS slots a partial, of which with
// RES the last two are a maximum and flag bits.  Thread t of SMALL_THREADS takes values
// t, t + SMALL_THREADS, ... of the M x NS totals.
#pragma once

#include "common.hpp"

namespace ecpic {

constexpr int SMALL_Q = 6;   // values a thread loads with the status words

template <int NS, bool RES>
__device__ __forceinline__ double combine(int slot, double a, double b) {
    if (RES && slot == NS - 2) return fmax(a, b);
    if (RES && slot == NS - 1) return (double)((int)a | (int)b);
    return a + b;
}

// Values first + q SMALL_THREADS, q < SMALL_Q, when item c is cell c (in bounds whatever
// the list holds): every load of a thread is in flight before it adds.
template <int NS, bool RES, int WPI>
__device__ __forceinline__ void cell_totals(const double *part, int M, int first, double (&v)[SMALL_Q]) {
    double u[SMALL_Q][WPI];
    int slot[SMALL_Q];
#pragma unroll
    for (int q = 0; q < SMALL_Q; ++q) {
        const int i = min(first + q * SMALL_THREADS, M * NS - 1), c = i / NS;
        slot[q] = i - c * NS;
#pragma unroll
        for (int w = 0; w < WPI; ++w) u[q][w] = part[(c * WPI + w) * NS + slot[q]];
    }
#pragma unroll
    for (int q = 0; q < SMALL_Q; ++q) {
        v[q] = 0.0;
#pragma unroll
        for (int w = 0; w < WPI; ++w) v[q] = combine<NS, RES>(slot[q], v[q], u[q][w]);
    }
}

template <int NS, bool RES>
__device__ __forceinline__ void cell_totals(const double *part, int wpi, int M, int first, double (&v)[SMALL_Q]) {
    switch (wpi) {
        case 1: cell_totals<NS, RES, 1>(part, M, first, v); break;
        case 2: cell_totals<NS, RES, 2>(part, M, first, v); break;
        case 3: cell_totals<NS, RES, 3>(part, M, first, v); break;
        default: cell_totals<NS, RES, 4>(part, M, first, v); break;
    }
}

// All totals into LDS.  v: this thread's first values as cell_totals loads them; lists with
// other than one item per cell are followed instead.
template <int NS, bool RES>
__device__ __forceinline__ void stage_totals(double *raw, const double *part, const ItemList &it, bool one_each,
                                             int wpi, int M, const double (&v)[SMALL_Q]) {
    const int t = threadIdx.x, len = M * NS;
    if (one_each) {
#pragma unroll
        for (int q = 0; q < SMALL_Q; ++q)
            if (t + q * SMALL_THREADS < len) raw[t + q * SMALL_THREADS] = v[q];
        for (int i = t + SMALL_Q * SMALL_THREADS; i < len; i += SMALL_Q * SMALL_THREADS) {
            double x[SMALL_Q];
            cell_totals<NS, RES>(part, wpi, M, i, x);
#pragma unroll
            for (int q = 0; q < SMALL_Q; ++q)
                if (i + q * SMALL_THREADS < len) raw[i + q * SMALL_THREADS] = x[q];
        }
        return;
    }
    for (int i = t; i < len; i += SMALL_THREADS) {
        const int c = i / NS, slot = i - c * NS, u1 = it.cell_first[c + 1] * wpi;
        double x = 0.0;
        for (int u = it.cell_first[c] * wpi; u < u1; ++u) x = combine<NS, RES>(slot, x, part[u * NS + slot]);
        raw[i] = x;
    }
}

}  // namespace ecpic
