// Reduced 2D model (Sections 2.2, 3.2 and 4.3), without and with the spin terms
// (hbar): kernels, spectral solves and the C ABI of include/ecpic2d.h.
//
// Data layout in HBM (one context):
//   particles  SoA, grouped by tile (TW cells of one row) in tile order, double
//              buffered: xi_k = x_k / dx_k in [0, M_k) (f64), p1, p2 (f64), id
//              (i32, the index given at set_particles).  Inside a tile the
//              cell-sorted sequence is stored transposed (see tile_pos), so a
//              coalesced read hands the lanes of a wave particles of different
//              cells.  start[c] is where cell c's share of its tile begins in the
//              sorted count (start[first cell of a tile] is the tile's offset).
//              The Picard iterate d = x^{n+1} - x^n (physical units) and p^{k+1}
//              live in more buffers; with spin, sx, sy, sz (f64) are double
//              buffered with the particles.
//   fields     row-major M1 x M2 coefficient grids, index i1 M2 + i2 (no halo;
//              the tile kernels wrap indices while staging).
//   spectra    M1 x M2 complex grids for the linear solves.
//
// Tiles.  A tile is TW consecutive cells of one row (x1 fixed); its particles
// are contiguous in the sorted order.  One thread block per tile stages the
// field coefficients the tile's particles can touch (rows r-p-1 .. r+1, columns
// c0-p-1 .. c0+TW, enough for a step of less than one cell) in LDS, gathers
// from there, accumulates its deposits in LDS with atomics, and adds the patch
// to the global grid with atomics at the end.
//
// Linear solves.  Every linear operator of the 2D scheme is a sum of tensor
// products of circulants (periodic B-spline mass matrices and differences), so
// the 2D discrete Fourier transform diagonalises it: M0 + dt^2 K/4 and the Maxwell
// system are solved exactly by a forward transform, a division by the symbol and an
// inverse transform.  M1 is one tensor product a component, so its inverse is two 1D
// circulant convolutions, with rows cut below 1e-18 of their largest entry.  The
// transforms are Stockham FFTs with the values in registers (radix 8) and LDS between
// stages (rows in one kernel, columns with the spectral step fused in the next, inverse
// rows with an epilogue).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <map>
#include <string>
#include <thread>
#include <vector>

#include "../../include/ecpic2d.h"
#include "coef.hpp"
#include "common.hpp"
#include "hostcopy.hpp"
#include "inverse_row.hpp"
#include "spline.hpp"

namespace ecpic2d {

using ecpic::basis_values;
using ecpic::frcp;
using ecpic::fsqrt;
using ecpic::piece_means;
using ecpic::wave_sum_dpp;

constexpr int WAVE = 64;
constexpr int BLOCK = 256;
constexpr int TWMAX = 64;        // tile width (cells along x2)
constexpr int MAXM = 512;        // largest grid size per direction (LDS of the transforms)
constexpr int MAXK = 64;         // residual slots per substep (Picard cap)
constexpr int FLAG_NONFINITE = 1, FLAG_CFL = 2;

__device__ __forceinline__ int wrapi(int j, int M) {
    const int w = j < 0 ? j + M : (j >= M ? j - M : j);
    if (w >= 0 && w < M) return w;
    const int r = j % M;
    return r < 0 ? r + M : r;
}

__device__ __forceinline__ unsigned long long bitsd(double v) { return (unsigned long long)__double_as_longlong(v); }

// Max of v >= 0 over the block, then one atomic max (as bits) into *slot.
__device__ __forceinline__ void block_max_to(double v, unsigned long long *slot) {
    __shared__ double red[1024 / WAVE];
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, WAVE));
    const int lane = threadIdx.x & (WAVE - 1), wid = threadIdx.x / WAVE;
    if (lane == 0) red[wid] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double m = red[0];
        for (int w = 1; w < (int)(blockDim.x / WAVE); ++w) m = fmax(m, red[w]);
        if (m > 0.0) atomicMax(slot, bitsd(m));
    }
}

// The vector memory operations this thread has issued are complete (device-scope
// atomics then have been performed where every block sees them).
__device__ __forceinline__ void wait_memory() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
}

// Sum over the block in a fixed order; thread 0 writes it to *out.
__device__ __forceinline__ void block_sum_to(double v, double *out) {
    __shared__ double red[BLOCK / WAVE];
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, WAVE);
    const int lane = threadIdx.x & (WAVE - 1), wid = threadIdx.x / WAVE;
    if (lane == 0) red[wid] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
        for (int w = 0; w < (int)(blockDim.x / WAVE); ++w) s += red[w];
        *out = s;
    }
}

// Block -> tile, keeping each XCD (blocks are dealt to the 8 XCDs round robin)
// on a contiguous band of rows so neighbouring tiles share its L2.
__device__ __forceinline__ int tile_of_block() {
    const int b = blockIdx.x, n = gridDim.x;
    if (n % 8 != 0) return b;
    return (b % 8) * (n / 8) + b / 8;
}

// The same with `split` blocks per tile (all on one XCD): the tile, and which share of
// its rows of 64 particles the block takes (wave w of part q takes every
// split * waves-th row from row q * waves + w on).
__device__ __forceinline__ int tile_of_block(int split, int &part) {
    const int b = tile_of_block(), t = b / split;
    part = b - t * split;
    return t;
}

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & (WAVE - 1)); }

// Number of lanes below this one set in mask.
__device__ __forceinline__ int rank_in(unsigned long long mask) {
    return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(mask >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)mask, 0u));
}

// Walk over a tile's particles.  The sort stores each tile transposed: with
// cnt = 64 Q + R particles, the particle of rank t = l Q + j (t < 64 Q) in the
// cell-sorted order sits at position j 64 + l, the last R in order.  Reading
// position j 64 + lane is then coalesced, while lane l works through the run of
// ranks [l Q, (l+1) Q), so the lanes of one wave sit in different cells and
// their LDS deposits rarely hit the same address.  Waves take j = wave, wave +
// waves, ... while j 64 < cnt (the last pass holds the R remaining particles).
__device__ __forceinline__ int tile_pos(int t, int cnt) {
    const int Q = cnt / WAVE;
    return t < WAVE * Q ? (t % Q) * WAVE + t / Q : t;
}

// Slot of this lane in the range of its cell, one atomic per run of equal
// consecutive cells: the first lane of a run adds the run's length to
// cursor[c] and hands the old value to the run (ds_bpermute).  Live lanes must be
// a prefix of the wave; every lane must execute this.
__device__ __forceinline__ int claim_slot(int c, bool live, int32_t *cursor) {
    const int lane = lane_id();
    const int prev = __shfl_up(c, 1, WAVE);
    const bool head = live && (lane == 0 || prev != c);
    const unsigned long long heads = __builtin_amdgcn_ballot_w64(head);
    const unsigned long long lives = __builtin_amdgcn_ballot_w64(live);
    const unsigned long long upto = lane == WAVE - 1 ? ~0ull : ((2ull << lane) - 1ull);   // lanes <= this one
    const int leader = WAVE - 1 - __builtin_clzll((heads & upto) | 1ull);
    int b = 0;
    if (head) {
        const unsigned long long later = (heads & ~upto) | ~lives;   // next head or first dead lane
        const int next = later ? __builtin_ctzll(later) : WAVE;
        b = atomicAdd(&cursor[c], next - lane);
    }
    b = __builtin_amdgcn_ds_bpermute(leader << 2, b);
    return b + lane - leader;
}

// Slot of this lane in counter[key] for the lanes with flag set, one atomic per
// distinct key among them (the lowest such lane adds the key's lane count and
// hands the old value on); lanes without flag get an unspecified value.
__device__ __forceinline__ int wave_claim(int32_t *counter, int key, bool flag) {
    unsigned long long rem = __builtin_amdgcn_ballot_w64(flag);
    int slot = 0;
    while (rem) {
        const int leader = __builtin_ctzll(rem);
        const int lk = __shfl(key, leader, WAVE);
        const bool mine = flag && key == lk;
        const unsigned long long m = __builtin_amdgcn_ballot_w64(mine);
        int b = 0;
        if (lane_id() == leader) b = atomicAdd(&counter[lk], __builtin_popcountll(m));
        b = __shfl(b, leader, WAVE);
        if (mine) slot = b + rank_in(m);
        rem &= ~m;
    }
    return slot;
}

// Gauss-Legendre rule with P points on [0, 1] (exact to degree 2P - 1, the degree
// of a product of a degree-P and a degree-(P-1) spline along a straight path).
template <int P>
struct GL;
template <> struct GL<2> {
    static constexpr double x[2] = {0.21132486540518713, 0.7886751345948129};
    static constexpr double w[2] = {0.5, 0.5};
};
template <> struct GL<3> {
    static constexpr double x[3] = {0.1127016653792583, 0.5, 0.8872983346207417};
    static constexpr double w[3] = {0.27777777777777785, 0.4444444444444444, 0.27777777777777785};
};
template <> struct GL<4> {
    static constexpr double x[4] = {0.06943184420297371, 0.33000947820757187, 0.6699905217924281,
                                    0.9305681557970262};
    static constexpr double w[4] = {0.17392742256872684, 0.3260725774312731, 0.3260725774312731,
                                    0.17392742256872684};
};
template <> struct GL<5> {
    static constexpr double x[5] = {0.04691007703066802, 0.23076534494715845, 0.5, 0.7692346550528415,
                                    0.9530899229693319};
    static constexpr double w[5] = {0.11846344252809471, 0.2393143352496831, 0.2844444444444445,
                                    0.2393143352496831, 0.11846344252809471};
};

// ---------------------------------------------------------------------------
// Small grid and particle kernels
// ---------------------------------------------------------------------------

__global__ void k2_fill(double *a, int64_t n, double v) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        a[i] = v;
}

__global__ void k2_fill_u64(unsigned long long *a, int n) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) a[i] = 0ull;
}

__global__ void k2_fill_i32(int32_t *a, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        a[i] = 0;
}

// (G a)_1 = (a_{i1,i2} - a_{i1-1,i2}) / dx1, (G a)_2 = (a_{i1,i2} - a_{i1,i2-1}) / dx2.
__global__ void k2_grad(const double *__restrict__ a, double *__restrict__ g1, double *__restrict__ g2, int M1,
                        int M2, double inv_dx1, double inv_dx2) {
    const int N = M1 * M2;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < N; i += gridDim.x * blockDim.x) {
        const int i1 = i / M2, i2 = i - i1 * M2;
        const double v = a[i];
        g1[i] = (v - a[wrapi(i1 - 1, M1) * M2 + i2]) * inv_dx1;
        g2[i] = (v - a[i1 * M2 + wrapi(i2 - 1, M2)]) * inv_dx2;
    }
}

// Start of Subsystem I: G a_z, the field iterates e^(0) = e^n and their mean with e^n,
// the current accumulators, residual slots, flags and gate, in one pass.
struct BeginI {
    const double *az, *e1, *e2;
    double *g1, *g2, *ek1, *ek2, *eb1, *eb2, *J1, *J2;
    unsigned long long *res;
    int nres, *flags, *gate;
    int M1, M2;
    double inv_dx1, inv_dx2;
};

__global__ void k2_begin_I(BeginI a) {
    const int N = a.M1 * a.M2, t0 = blockIdx.x * blockDim.x + threadIdx.x, nt = gridDim.x * blockDim.x;
    for (int i = t0; i < a.nres; i += nt) a.res[i] = 0ull;
    if (t0 == 0) *a.flags = *a.gate = 0;
    for (int i = t0; i < N; i += nt) {
        const int i1 = i / a.M2, i2 = i - i1 * a.M2;
        const double v = a.az[i];
        a.g1[i] = (v - a.az[wrapi(i1 - 1, a.M1) * a.M2 + i2]) * a.inv_dx1;
        a.g2[i] = (v - a.az[i1 * a.M2 + wrapi(i2 - 1, a.M2)]) * a.inv_dx2;
        const double e1 = a.e1[i], e2 = a.e2[i];
        a.ek1[i] = e1;
        a.ek2[i] = e2;
        a.eb1[i] = e1;
        a.eb2[i] = e2;
        a.J1[i] = 0.0;
        a.J2[i] = 0.0;
    }
}

// Start of Subsystem III: e^n and the iterate e^(0) = e^n, the accumulator, residual
// slots and gate.
__global__ void k2_begin_III(const double *__restrict__ ez, double *__restrict__ ezn, double *__restrict__ ezk,
                             double *__restrict__ S, int N, unsigned long long *res, int nres, int *gate) {
    const int t0 = blockIdx.x * blockDim.x + threadIdx.x, nt = gridDim.x * blockDim.x;
    for (int i = t0; i < nres; i += nt) res[i] = 0ull;
    if (t0 == 0) *gate = 0;
    for (int i = t0; i < N; i += nt) {
        const double e = ez[i];
        ezn[i] = e;
        ezk[i] = e;
        S[i] = 0.0;
    }
}

// Positions of new particles: wrap into [0, M) (cell units), record the cell and
// count it.
__global__ __launch_bounds__(BLOCK) void k2_bin_new(const double *__restrict__ x1, const double *__restrict__ x2,
                                                    double *__restrict__ xi1, double *__restrict__ xi2,
                                                    int32_t *__restrict__ cell, int32_t *__restrict__ count, int64_t n,
                                                    int M1, int M2, double inv_dx1, double inv_dx2, int *flags) {
    for (int64_t base = blockIdx.x * (int64_t)blockDim.x; base < n; base += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = base + threadIdx.x;
        const bool live = i < n;
        int c = 0;
        if (live) {
            double u1 = x1[i] * inv_dx1, u2 = x2[i] * inv_dx2;
            if (!isfinite(u1) || !isfinite(u2)) { atomicOr(flags, FLAG_NONFINITE); u1 = 0.0; u2 = 0.0; }
            u1 = fmod(u1, (double)M1);
            u2 = fmod(u2, (double)M2);
            if (u1 < 0.0) u1 += (double)M1;
            if (u2 < 0.0) u2 += (double)M2;
            if (u1 >= (double)M1) u1 = 0.0;
            if (u2 >= (double)M2) u2 = 0.0;
            xi1[i] = u1;
            xi2[i] = u2;
            c = (int)u1 * M2 + (int)u2;
            cell[i] = c;
        }
        claim_slot(c, live, count);
    }
}

// Exclusive scan of count[0..Nc) into start[0..Nc], count <- 0, in three passes:
// block sums (SCAN_TILE cells per block), a scan of the block sums (one block),
// and the block-local scans plus their offsets.
constexpr int SCAN_THREADS = 1024, SCAN_PER = 4, SCAN_TILE = SCAN_THREADS * SCAN_PER;

__device__ __forceinline__ int block_exscan1024(int v, int *total) {
    __shared__ int wsum[SCAN_THREADS / WAVE];
    const int lane = lane_id(), wid = threadIdx.x / WAVE;
    int x = v;
#pragma unroll
    for (int o = 1; o < WAVE; o <<= 1) {
        const int y = __shfl_up(x, o, WAVE);
        if (lane >= o) x += y;
    }
    if (lane == WAVE - 1) wsum[wid] = x;
    __syncthreads();
    int pre = 0, tot = 0;
    for (int w = 0; w < (int)(blockDim.x / WAVE); ++w) {
        pre += w < wid ? wsum[w] : 0;
        tot += wsum[w];
    }
    __syncthreads();
    *total = tot;
    return pre + x - v;
}

__global__ __launch_bounds__(SCAN_THREADS) void k2_scan_sums(const int32_t *__restrict__ count, int32_t *bsum,
                                                             int Nc) {
    const int c0 = blockIdx.x * SCAN_TILE + threadIdx.x * SCAN_PER;
    int v = 0;
#pragma unroll
    for (int q = 0; q < SCAN_PER; ++q) v += c0 + q < Nc ? count[c0 + q] : 0;
    int tot;
    block_exscan1024(v, &tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

__global__ __launch_bounds__(SCAN_THREADS) void k2_scan_top(int32_t *bsum, int nb, int32_t *start_end) {
    // nb <= SCAN_THREADS (Nc <= 512 * 512 = 64 tiles)
    const int v = (int)threadIdx.x < nb ? bsum[threadIdx.x] : 0;
    int tot;
    const int pre = block_exscan1024(v, &tot);
    if ((int)threadIdx.x < nb) bsum[threadIdx.x] = pre;
    if (threadIdx.x == 0) *start_end = tot;
}

__global__ __launch_bounds__(SCAN_THREADS) void k2_scan_apply(int32_t *__restrict__ count, int32_t *__restrict__ start,
                                                              const int32_t *__restrict__ bsum, int Nc) {
    const int c0 = blockIdx.x * SCAN_TILE + threadIdx.x * SCAN_PER;
    int k[SCAN_PER], v = 0;
#pragma unroll
    for (int q = 0; q < SCAN_PER; ++q) {
        k[q] = c0 + q < Nc ? count[c0 + q] : 0;
        v += k[q];
    }
    int tot;
    int off = bsum[blockIdx.x] + block_exscan1024(v, &tot);
#pragma unroll
    for (int q = 0; q < SCAN_PER; ++q)
        if (c0 + q < Nc) {
            start[c0 + q] = off;
            off += k[q];
            count[c0 + q] = 0;
        }
}

// Move every particle to its cell's range of the destination buffers.
__global__ __launch_bounds__(BLOCK) void k2_scatter(const double *__restrict__ s1, const double *__restrict__ s2,
                                                    const double *__restrict__ q1, const double *__restrict__ q2,
                                                    const int32_t *__restrict__ sid, double *__restrict__ d1,
                                                    double *__restrict__ d2, double *__restrict__ r1,
                                                    double *__restrict__ r2, int32_t *__restrict__ did,
                                                    const int32_t *__restrict__ cell, const int32_t *__restrict__ start,
                                                    int32_t *__restrict__ cursor, int64_t n, int M2, int TW) {
    for (int64_t base = blockIdx.x * (int64_t)blockDim.x; base < n; base += (int64_t)gridDim.x * blockDim.x) {
        const int64_t i = base + threadIdx.x;
        const bool live = i < n;
        const int c = live ? cell[i] : 0;
        const int slot = claim_slot(c, live, cursor);
        if (live) {
            const int r = c / M2, first = r * M2 + ((c - r * M2) / TW) * TW;   // tile's first cell
            const int tb = start[first], cnt = start[first + TW] - tb;
            const int j = tb + tile_pos(start[c] - tb + slot, cnt);
            d1[j] = s1[i];
            d2[j] = s2[i];
            r1[j] = q1[i];
            r2[j] = q2[i];
            did[j] = sid[i];
        }
    }
}

// out[id[i]] = v[i] (positions back to physical units when scale != 1).
__global__ void k2_unsort(const double *__restrict__ v, const int32_t *__restrict__ id, double *__restrict__ out,
                          int64_t n, double scale) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        out[id[i]] = v[i] * scale;
}

__global__ void k2_iota(int32_t *id, int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        id[i] = (int32_t)i;
}

// Value of the degree (P, P) field at a point in cell (c1, c2), local (t1, t2),
// from the global grid.
template <int P>
__device__ __forceinline__ double gather00(const double *__restrict__ f, int M1, int M2, int c1, int c2, double t1,
                                           double t2) {
    double b1[P + 1], b2[P + 1];
    basis_values<P>(t1, b1);
    basis_values<P>(t2, b2);
    double s = 0.0;
#pragma unroll
    for (int m1 = 0; m1 <= P; ++m1) {
        const double *row = f + wrapi(c1 - m1, M1) * M2;
        double t = 0.0;
#pragma unroll
        for (int m2 = 0; m2 <= P; ++m2) t += b2[m2] * row[wrapi(c2 - m2, M2)];
        s += b1[m1] * t;
    }
    return s;
}

// sum f_{i1,i2} N^{D1}_{i1}(x1) N^{D2}_{i2}(x2) at a point of cell (c1, c2), from
// global memory (diagnostics).
template <int D1, int D2>
__device__ __forceinline__ double gatherg(const double *__restrict__ f, int M1, int M2, int c1, int c2, double t1,
                                          double t2) {
    double b1[D1 + 1], b2[D2 + 1];
    basis_values<D1>(t1, b1);
    basis_values<D2>(t2, b2);
    double s = 0.0;
#pragma unroll
    for (int m1 = 0; m1 <= D1; ++m1) {
        const double *row = f + wrapi(c1 - m1, M1) * M2;
        double t = 0.0;
#pragma unroll
        for (int m2 = 0; m2 <= D2; ++m2) t += b2[m2] * row[wrapi(c2 - m2, M2)];
        s += b1[m1] * t;
    }
    return s;
}

// Zeeman sum w s . B_h(x) over the particles (times hbar on the host), B_h =
// (dA_z/dx2, -dA_z/dx1, B_z) from G a_z (g1, g2) and b_z.
template <int P>
__global__ __launch_bounds__(BLOCK) void k2_zeeman(const double *__restrict__ xi1, const double *__restrict__ xi2,
                                                   const double *__restrict__ sx, const double *__restrict__ sy,
                                                   const double *__restrict__ sz, const double *__restrict__ g1,
                                                   const double *__restrict__ g2, const double *__restrict__ bz,
                                                   int64_t n, int M1, int M2, double w, double *__restrict__ partial) {
    double s = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double u1 = xi1[i], u2 = xi2[i];
        const int c1 = (int)u1, c2 = (int)u2;
        const double t1 = u1 - c1, t2 = u2 - c2;
        const double Bx = gatherg<P, P - 1>(g2, M1, M2, c1, c2, t1, t2);
        const double By = -gatherg<P - 1, P>(g1, M1, M2, c1, c2, t1, t2);
        const double Bz = gatherg<P - 1, P - 1>(bz, M1, M2, c1, c2, t1, t2);
        s += w * (sx[i] * Bx + sy[i] * By + sz[i] * Bz);
    }
    block_sum_to(s, &partial[blockIdx.x]);
}

// out[i] = in[id[i]]: values given in the caller's order, put into the sorted order.
__global__ void k2_gather_id(const double *__restrict__ in, const int32_t *__restrict__ id, double *__restrict__ out,
                             int64_t n) {
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        out[i] = in[id[i]];
}

// Spin deposits over tiles (no motion): mode 0: Dx += w s_x N^P(x1) N^{P-1}(x2) and
// Dy += w s_y N^{P-1}(x1) N^P(x2) (Lambda1*^T W S_xy); mode 1: Dz += w s_z
// N^{P-1}(x1) N^{P-1}(x2) (Lambda2^T W S_z).  Targets zero on entry.
template <int P>
__global__ __launch_bounds__(BLOCK) void k2_deposit_spin(const double *__restrict__ xi1,
                                                         const double *__restrict__ xi2,
                                                         const double *__restrict__ sx,
                                                         const double *__restrict__ sy,
                                                         const double *__restrict__ sz,
                                                         const int32_t *__restrict__ start, double *__restrict__ Dx,
                                                         double *__restrict__ Dy, double *__restrict__ Dz, int M1,
                                                         int M2, int TW, double w, int mode, int split) {
    constexpr int PR = P + 1, PCM = TWMAX + P, PS = PR * PCM;
    __shared__ double sX[PS], sY[PS];
    const int nseg = M2 / TW;
    int part;
    const int tile = tile_of_block(split, part);
    const int r = tile / nseg, c0 = (tile - r * nseg) * TW;
    const int PC = TW + P;
    const int R0 = r - P, C0 = c0 - P;
    for (int t = threadIdx.x; t < PR * PC; t += blockDim.x) {
        sX[t] = 0.0;
        sY[t] = 0.0;
    }
    __syncthreads();
    const int begin = start[tile], end = start[tile + 1];
    for (int i = begin + part * BLOCK + threadIdx.x; i < end; i += split * BLOCK) {
        const double u1 = xi1[i], u2 = xi2[i];
        const int c2 = (int)u2;
        double a1[P + 1], a2[P + 1], b1[P], b2[P];
        basis_values<P>(u1 - r, a1);
        basis_values<P>(u2 - c2, a2);
        basis_values<P - 1>(u1 - r, b1);
        basis_values<P - 1>(u2 - c2, b2);
        if (mode == 0) {
            const double qx = w * sx[i], qy = w * sy[i];
#pragma unroll
            for (int m1 = 0; m1 <= P; ++m1)
#pragma unroll
                for (int m2 = 0; m2 <= P; ++m2) {
                    const int k = (r - m1 - R0) * PC + c2 - m2 - C0;
                    if (m2 < P) atomicAdd(&sX[k], qx * a1[m1] * b2[m2]);
                    if (m1 < P) atomicAdd(&sY[k], qy * b1[m1] * a2[m2]);
                }
        } else {
            const double qz = w * sz[i];
#pragma unroll
            for (int m1 = 0; m1 < P; ++m1)
#pragma unroll
                for (int m2 = 0; m2 < P; ++m2) atomicAdd(&sX[(r - m1 - R0) * PC + c2 - m2 - C0], qz * b1[m1] * b2[m2]);
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < PR * PC; t += blockDim.x) {
        const int i = t / PC, j = t - i * PC;
        const int g = wrapi(R0 + i, M1) * M2 + wrapi(C0 + j, M2);
        if (mode == 0) {
            if (sX[t] != 0.0) atomicAdd(&Dx[g], sX[t]);
            if (sY[t] != 0.0) atomicAdd(&Dy[g], sY[t]);
        } else if (sX[t] != 0.0) {
            atomicAdd(&Dz[g], sX[t]);
        }
    }
}

// src = G*^T (Dx, Dy) = G2^T Dx - G1^T Dy, the transposes of the backward
// differences: (G1^T u)_i = (u_{i1,i2} - u_{i1+1,i2}) / dx1, likewise in x2.
__global__ __launch_bounds__(BLOCK) void k2_spin_src(const double *__restrict__ Dx, const double *__restrict__ Dy,
                                                     double *__restrict__ src, int M1, int M2, double inv_dx1,
                                                     double inv_dx2) {
    const int N = M1 * M2;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < N; i += gridDim.x * blockDim.x) {
        const int i1 = i / M2, i2 = i - i1 * M2;
        src[i] = (Dx[i] - Dx[i1 * M2 + wrapi(i2 + 1, M2)]) * inv_dx2 -
                 (Dy[i] - Dy[wrapi(i1 + 1, M1) * M2 + i2]) * inv_dx1;
    }
}

// ---------------------------------------------------------------------------
// Subsystem I sweep (Section 4.3): gather, push, deposit, one tile per block
// ---------------------------------------------------------------------------
struct SweepArgs {
    const double *xi1, *xi2, *p1, *p2;   // sorted particles
    double *d1, *d2;                     // increment d^(k) (physical); formed and stored by sweep 0
    double *dn1, *dn2;                   // increment d^(k+1)
    double *pk1, *pk2;                   // momentum p^(k+1)
    const int32_t *start;                // first particle of each tile (ntiles + 1)
    const double *eb1, *eb2;             // (e^n + e^(k)) / 2
    const double *az, *g1a, *g2a;        // a_z and G a_z
    double *J1, *J2;                     // current of d^(k) (accumulated, zero on entry)
    unsigned long long *res;             // max |d^(k+1) - d^(k)|, as bits
    int *flags;
    const int *gate;                     // nonzero: an earlier sweep converged, nothing to do
    int M1, M2, TW;
    double inv_dx1, inv_dx2, dt, w;
    const double *sx, *sy, *sz, *bz;     // spins and b_z (the sweep with spin)
    double hbar;
    double *azn, *gamn;                  // A_z(x^n) and gamma(x^n, p^n): formed by sweep 0, read by the rest
    int keep_p;                          // store p^(k+1)
    int split;                           // blocks per tile
};

// Line mean of the V1 basis (degree P-1) along one leg of the step, from t0 in
// [0, 1) of cell c0 to t1 in (-1, 2) (cell units, c0 frame); s = +1 / -1 / 0
// tells whether t1 lies in cell c0+1 / c0-1 / c0, and rlen is 1 / |t1 - t0|
// (used only when s != 0).  lb[k], k = 0..P+1, is the mean of Lambda1_{c0-P+k}:
// the mean over each piece of the leg (the part in c0 and the part in c0+s),
// weighted by the piece's share of the length.
template <int P>
__device__ __forceinline__ void leg_mean_v1(double t0, double t1, int s, double rlen, double (&lb)[P + 2]) {
    constexpr int D = P - 1;
    const double t1c = fmin(fmax(t1, 0.0), 1.0);
    double avgA[D + 1], avgB[D + 1];
    piece_means<D>(fmin(t0, t1c), fmax(t0, t1c), avgA);
    // the piece in the neighbour cell: [0, t1 - 1] (s = +1) or [t1 + 1, 1] (s = -1)
    const double as = s < 0 ? t1 + 1.0 : 0.0, bs = s > 0 ? t1 - 1.0 : (s < 0 ? 1.0 : 0.0);
    piece_means<D>(as, bs, avgB);
    const double wB = s != 0 ? (bs - as) * rlen : 0.0, wA = 1.0 - wB;
#pragma unroll
    for (int k = 0; k <= P + 1; ++k) {
        const double v = (k >= 1 && k <= P) ? wA * avgA[P - k] : 0.0;   // index c0 - m, k = P - m
        double vb = 0.0;                                                 // index c0 + s - m
        if (s > 0 && P + 1 - k >= 0 && P + 1 - k <= D) vb = avgB[P + 1 - k < 0 ? 0 : (P + 1 - k > D ? D : P + 1 - k)];
        if (s < 0 && P - 1 - k >= 0 && P - 1 - k <= D) vb = avgB[P - 1 - k < 0 ? 0 : (P - 1 - k > D ? D : P - 1 - k)];
        lb[k] = v + wB * vb;
    }
}

// The mean along a leg that stays in cell c0: the same vector, from one piece
// (entries 0 and P + 1 are zero).
template <int P>
__device__ __forceinline__ void leg_mean_cell(double t0, double t1, double (&lb)[P + 2]) {
    double avg[P];
    piece_means<P - 1>(t0, t1, avg);   // symmetric in its two ends
    lb[0] = 0.0;
    lb[P + 1] = 0.0;
#pragma unroll
    for (int k = 1; k <= P; ++k) lb[k] = avg[P - k];
}

// 1 / |s| for a leg of s cells, with |s| raised to a tiny normal floor: a leg
// that crosses a grid line is longer than that unless it starts within the
// floor of the line, where the split of its (vanishing) length does not matter.
__device__ __forceinline__ double leg_rcp(double s) { return frcp(fmax(fabs(s), 1.0e-290)); }

// Path integrals of one V1 component on one piece of the straight step (between
// two grid-line crossings), by the P-point Gauss-Legendre rule in the frame of the
// piece's cell: W[u][v] is the integral over the piece (parameter from sa, length
// len) of N^{DA}_{-DA+u}(x1) N^{DB}_{-DB+v}(x2), with (DA, DB) = (P-1, P) or
// (P, P-1) and the step starting at (t1, t2) with slope (s1, s2).  The two
// components use disjoint basis values, so taking them in turn costs nothing and
// halves the registers the integrals hold.
template <int P, int DA, int DB>
__device__ __forceinline__ void piece_integrals(double t1, double t2, double s1, double s2, double sa, double len,
                                                double (&W)[DA + 1][DB + 1]) {
#pragma unroll
    for (int u = 0; u <= DA; ++u)
#pragma unroll
        for (int v = 0; v <= DB; ++v) W[u][v] = 0.0;
#pragma unroll
    for (int q = 0; q < P; ++q) {
        const double s = sa + len * GL<P>::x[q];
        const double g = len * GL<P>::w[q];
        double bx[DA + 1], by[DB + 1];
        basis_values<DA>(t1 + s * s1, bx);   // bx[m]: N^{DA}_{-m}
        basis_values<DB>(t2 + s * s2, by);
#pragma unroll
        for (int u = 0; u <= DA; ++u) {
            const double gx = g * bx[DA - u];
#pragma unroll
            for (int v = 0; v <= DB; ++v) W[u][v] += gx * by[DB - v];
        }
    }
}

// The field patch of a tile in LDS (rows r-P-1 .. r+1, columns c0-P-1 .. c0+TW),
// rows PC apart for every tile width, so that offsets inside it are constants.
template <int P>
struct Patch {
    static constexpr int PC = TWMAX + P + 2, PR = P + 3, SIZE = PR * PC;
    double *E1, *E2, *A, *G1, *G2, *J1, *J2, *Bz;
    int R0, C0, r;
};

// One particle's step (cell units): the start in its own cell (r, c2) as t in
// [0, 1), the increment s (D in physical units) and the end u in that cell's
// frame, the cell change e of the end point, and the momentum q.  A crossing
// step also has the path parameters lo <= hi of its grid-line crossings (1 when
// there is none).
struct Step {
    double t1, t2, s1, s2, u1, u2, D1, D2, q1, q2, lo, hi;
    int c2, e1, e2;
};

__device__ __forceinline__ Step make_step(const SweepArgs &a, double x1, double x2, double q1, double q2, double D1,
                                          double D2, int r) {
    Step g;
    g.c2 = (int)x2;
    g.t1 = x1 - r;
    g.t2 = x2 - g.c2;
    g.s1 = D1 * a.inv_dx1;
    g.s2 = D2 * a.inv_dx2;
    g.u1 = (x1 + g.s1) - r;
    g.u2 = (x2 + g.s2) - g.c2;
    g.D1 = D1;
    g.D2 = D2;
    g.q1 = q1;
    g.q2 = q2;
    g.e1 = g.e2 = 0;
    g.lo = g.hi = 1.0;
    return g;
}

// Does the step end in its own cell (false for a non-finite one)?
__device__ __forceinline__ bool stays(const Step &g) {
    return g.u1 >= 0.0 && g.u1 < 1.0 && g.u2 >= 0.0 && g.u2 < 1.0;
}

// Cell change and crossing parameters of a step that leaves its cell.
__device__ __forceinline__ void cross_step(Step &g, bool live, int &flags) {
    const double f1 = floor(g.u1), f2 = floor(g.u2);
    if (!(fabs(f1) <= 1.0 && fabs(f2) <= 1.0)) {   // a cell or more, or not finite
        if (live) flags |= isfinite(g.s1 + g.s2) ? FLAG_CFL : FLAG_NONFINITE;
    } else {
        g.e1 = (int)f1;
        g.e2 = (int)f2;
    }
    const double bA = g.e1 ? ((g.e1 > 0 ? 1.0 : 0.0) - g.t1) * copysign(leg_rcp(g.s1), g.s1) : 1.0;
    const double bB = g.e2 ? ((g.e2 > 0 ? 1.0 : 0.0) - g.t2) * copysign(leg_rcp(g.s2), g.s2) : 1.0;
    g.lo = fmin(bA, bB);
    g.hi = fmax(bA, bB);
}

// One piece of the path inside the cell (k1, k2) relative to the start cell, from
// parameter sa over length len, for the component of degrees (DA, DB) with the
// patches F (mean field) and J (current): the mean field is accumulated into E
// and jw times the path integrals of the V1 basis are added to the current.
template <int P, int DA, int DB>
__device__ __forceinline__ void piece_of(const Step &g, bool live, double sa, double len, int k1, int k2,
                                         const Patch<P> &t, const double *F, double *J, double jw, double &E) {
    constexpr int PC = Patch<P>::PC;
    double W[DA + 1][DB + 1];
    piece_integrals<P, DA, DB>(g.t1 - k1, g.t2 - k2, g.s1, g.s2, sa, len, W);
    const int o = (P + 1 - DA + k1) * PC + g.c2 - t.C0 + k2 - DB;   // W[0][0] in the patch
#pragma unroll
    for (int u = 0; u <= DA; ++u)
#pragma unroll
        for (int v = 0; v <= DB; ++v) E += W[u][v] * F[o + u * PC + v];
    asm volatile("" : "+v"(E));   // summed before the deposit, not at the push (see legs_of)
    if (live) {
#pragma unroll
        for (int u = 0; u <= DA; ++u)
#pragma unroll
            for (int v = 0; v <= DB; ++v) atomicAdd(&J[o + u * PC + v], jw * W[u][v]);
    }
}

// Both components of one piece.
template <int P>
__device__ __forceinline__ void piece(const Step &g, bool live, double sa, double len, int k1, int k2,
                                      const Patch<P> &t, double w, double &E1, double &E2) {
    piece_of<P, P - 1, P>(g, live, sa, len, k1, k2, t, t.E1, t.J1, w * g.D1, E1);
    __builtin_amdgcn_sched_barrier(0);   // the second component's integrals reuse the first one's registers
    piece_of<P, P, P - 1>(g, live, sa, len, k1, k2, t, t.E2, t.J2, w * g.D2, E2);
}

// The pieces of a crossing path ([0, lo], [lo, hi], [hi, 1]); those no lane of the
// wave needs are skipped.
template <int P>
__device__ __forceinline__ void pieces(const Step &g, bool live, const Patch<P> &t, double w, double &E1, double &E2) {
    const int n1 = min(g.e1, 0), n2 = min(g.e2, 0);
#pragma unroll 1
    for (int q = 0; q < 3; ++q) {
        const double sa = q == 0 ? 0.0 : (q == 1 ? g.lo : g.hi);
        const double sb = q == 0 ? g.lo : (q == 1 ? g.hi : 1.0);
        const double len = live ? sb - sa : 0.0;
        if (!__builtin_amdgcn_ballot_w64(len > 0.0)) continue;
        const double sm = 0.5 * (sa + sb);
        const int k1 = min(max((int)floor(g.t1 + sm * g.s1), n1), n1 + 1);
        const int k2 = min(max((int)floor(g.t2 + sm * g.s2), n2), n2 + 1);
        piece<P>(g, len > 0.0, sa, len, k1, k2, t, w, E1, E2);
    }
}

// A_z at a start point (t1, t2) of the tile's row, cell column c2, from the patch.
template <int P>
__device__ __forceinline__ double start_A(const Patch<P> &t, double t1, double t2, int c2) {
    double b1[P + 1], b2[P + 1];
    basis_values<P>(t1, b1);
    basis_values<P>(t2, b2);
    double A = 0.0;
#pragma unroll
    for (int m1 = 0; m1 <= P; ++m1) {
        double ta = 0.0;
#pragma unroll
        for (int m2 = 0; m2 <= P; ++m2) ta += b2[m2] * t.A[(P + 1 - m1) * Patch<P>::PC + c2 - m2 - t.C0];
        A += b1[m1] * ta;
    }
    return A;
}

// gamma(x, p) from A_z(x) = A and p = (q1, q2).
__device__ __forceinline__ double gamma_of(double q1, double q2, double A) {
    return fsqrt(1.0 + q1 * q1 + q2 * q2 + A * A);
}

// What the push needs from the two legs of a step: the means of dA_z/dx2 along
// the vertical leg (Dv, at x1^n) and of dA_z/dx1 along the horizontal leg (Dh, at
// x2^{n+1}), and the spin force over hbar (F1, F2).
struct Legs {
    double Dv, Dh, F1, F2;
};

// All patch reads of the push: taken before the path integrals deposit, because
// LDS operations of a wave complete in order and reads behind the deposit's
// atomics would wait for them.  CROSS: the legs may enter a neighbour cell
// (otherwise they stay, and P of their P + 2 weights are nonzero).
template <int P, bool SPIN, bool CROSS>
__device__ __forceinline__ Legs legs_of(const Step &g, int i, const Patch<P> &t, const SweepArgs &a) {
    constexpr int PC = Patch<P>::PC, R = P + 1;            // R: the tile's row in the patch
    constexpr int KA = CROSS ? 0 : 1, KB = CROSS ? P + 1 : P;   // leg entries that can be nonzero
    const int c = g.c2 - t.C0;                             // column of the start cell in the patch
    const int cb = CROSS ? c + g.e2 : c;                   // of the end cell
    double ba1[P + 1], bb2[P + 1];
    basis_values<P>(g.t1, ba1);
    basis_values<P>(CROSS ? g.u2 - g.e2 : g.u2, bb2);
    double rl2 = 0.0, rl1 = 0.0, lm2[P + 2], lm1[P + 2];   // index (start cell) - P + k
    if constexpr (CROSS) {
        rl2 = leg_rcp(g.s2);
        rl1 = leg_rcp(g.s1);
        leg_mean_v1<P>(g.t2, g.u2, g.e2, rl2, lm2);
        leg_mean_v1<P>(g.t1, g.u1, g.e1, rl1, lm1);
    } else {
        leg_mean_cell<P>(g.t2, g.u2, lm2);
        leg_mean_cell<P>(g.t1, g.u1, lm1);
    }
    double Dv = 0.0, Dh = 0.0;
#pragma unroll
    for (int m1 = 0; m1 <= P; ++m1) {
        double s = 0.0;
#pragma unroll
        for (int k = KA; k <= KB; ++k) s += lm2[k] * t.G2[(R - m1) * PC + c - P + k];
        Dv += ba1[m1] * s;
    }
#pragma unroll
    for (int k = KA; k <= KB; ++k) {
        double s = 0.0;
#pragma unroll
        for (int m2 = 0; m2 <= P; ++m2) s += bb2[m2] * t.G1[(R - P + k) * PC + cb - m2];
        Dh += lm1[k] * s;
    }
    // formed here: the compiler would otherwise sink the arithmetic to the push and
    // keep every patch value read alive across the path integrals
    asm volatile("" : "+v"(Dv), "+v"(Dh));
    double F1 = 0.0, F2 = 0.0;   // spin force / hbar
    if constexpr (SPIN) {
        __builtin_amdgcn_sched_barrier(0);
        // Means along the same two legs of the derivatives of dA_z/dx2 (coefficients
        // G2 = (G a)_2, degrees (P, P-1)), dA_z/dx1 (G1, (P-1, P)) and B_z ((P-1, P-1)):
        // each derivative's coefficients are backward differences of the field's.
        double lq2[P + 1], lq1[P + 1], bm1[P], bmb2[P];   // legs of degree P-2, index (start cell) - P + 1 + k
        if constexpr (CROSS) {
            leg_mean_v1<P - 1>(g.t2, g.u2, g.e2, rl2, lq2);
            leg_mean_v1<P - 1>(g.t1, g.u1, g.e1, rl1, lq1);
        } else {
            leg_mean_cell<P - 1>(g.t2, g.u2, lq2);
            leg_mean_cell<P - 1>(g.t1, g.u1, lq1);
        }
        basis_values<P - 1>(g.t1, bm1);
        basis_values<P - 1>(CROSS ? g.u2 - g.e2 : g.u2, bmb2);
        const double i1 = a.inv_dx1, i2 = a.inv_dx2;
        // Summation by parts: sum_k m_k (F_k - F_{k-1}) = sum_j F_j (m_j - m_{j+1}), so
        // every patch value is read once, with difference weights formed once.  Entry j
        // of a weight vector belongs to index (start cell) - P - 1 + j; those of lm are
        // nonzero for j in [KA, KB + 1], those of lq for j in [KA + 1, KB + 1].
        double wa[P + 3], wb[P + 3];   // weights of lm2 (degree P-1) and lq2 (degree P-2)
#pragma unroll
        for (int j = 0; j <= P + 2; ++j) {
            const double m0 = j >= 1 ? lm2[j - 1] : 0.0, m1 = j <= P + 1 ? lm2[j] : 0.0;
            const double q0 = j >= 2 ? lq2[j - 2] : 0.0, q1 = (j >= 1 && j <= P + 1) ? lq2[j - 1] : 0.0;
            wa[j] = m0 - m1;
            wb[j] = q0 - q1;
        }
        double Sy2 = 0.0, Sx2 = 0.0, Sb2 = 0.0;
#pragma unroll
        for (int m1 = 0; m1 <= P; ++m1) {
            const int row = (R - m1) * PC + c - P - 1;
            double ty = 0.0, tx = 0.0, tb = 0.0;
#pragma unroll
            for (int j = KA; j <= KB + 1; ++j) {
                if (j > KA) ty += wb[j] * t.G2[row + j];
                tx += wa[j] * t.G1[row + j];
                if (j > KA) tb += wb[j] * t.Bz[row + j];
            }
            Sy2 += ba1[m1] * ty;
            if (m1 < P) {
                Sx2 += bm1[m1] * tx;
                Sb2 += bm1[m1] * tb;
            }
        }
        asm volatile("" : "+v"(Sy2), "+v"(Sx2), "+v"(Sb2));
        __builtin_amdgcn_sched_barrier(0);
        // x1 leg at x2^{n+1}: per row the x2 sums first.
        double Sy1 = 0.0, Sx1 = 0.0, Sb1 = 0.0;
#pragma unroll
        for (int j = KA; j <= KB + 1; ++j) {
            const double m0 = j >= 1 ? lm1[j - 1] : 0.0, m1 = j <= P + 1 ? lm1[j] : 0.0;
            const double q0 = j >= 2 ? lq1[j - 2] : 0.0, q1 = (j >= 1 && j <= P + 1) ? lq1[j - 1] : 0.0;
            const int row = (R - P - 1 + j) * PC;
            double ty = 0.0, tx = 0.0, tb = 0.0;
#pragma unroll
            for (int m2 = 0; m2 <= P; ++m2) {
                const int k = row + cb - m2;
                if (j > KA) tx += bb2[m2] * t.G1[k];
                if (m2 < P) {
                    ty += bmb2[m2] * t.G2[k];
                    if (j > KA) tb += bmb2[m2] * t.Bz[k];
                }
            }
            Sy1 += (m0 - m1) * ty;
            if (j > KA) {
                Sx1 += (q0 - q1) * tx;
                Sb1 += (q0 - q1) * tb;
            }
        }
        const double sx = a.sx[i], sy = a.sy[i], sz = a.sz[i];
        F1 = (sx * Sy1 - sy * Sx1 + sz * Sb1) * i1;
        F2 = (sx * Sy2 - sy * Sx2 + sz * Sb2) * i2;
    }
    if constexpr (SPIN) asm volatile("" : "+v"(F1), "+v"(F2));
    return Legs{Dv, Dh, F1, F2};
}

// The push of the Subsystem I scheme and the stores of particle i.  Aa = A_z(x^n)
// and gA = gamma(x^n, p^n) are fixed over the iteration; A_z at the end point is Aa
// plus the two legs' increments (the leg means are exact divided differences): 2
// operations instead of a gather, and (Aa + Ab)(D1 Dh + D2 Dv) = Ab^2 - Aa^2 then
// holds to rounding.
template <bool SPIN>
__device__ __forceinline__ void push(const Step &g, bool live, int i, double E1, double E2, double Aa, double gA,
                                     const Legs &l, const SweepArgs &a, double &rmax, int &flags) {
    const double Ab = Aa + (g.D1 * l.Dh + g.D2 * l.Dv);
    const double q1 = g.q1, q2 = g.q2;
    const double gB = gamma_of(q1, q2, Ab);
    const double f = -(Aa + Ab) * frcp(gA + gB);
    double n1, n2;
    if constexpr (SPIN) {
        n1 = q1 + a.dt * (E1 + f * l.Dh - a.hbar * l.F1);
        n2 = q2 + a.dt * (E2 + f * l.Dv - a.hbar * l.F2);
    } else {
        n1 = q1 + a.dt * (E1 + f * l.Dh);
        n2 = q2 + a.dt * (E2 + f * l.Dv);
    }
    const double gC = gamma_of(n1, n2, Ab);
    const double sc = a.dt * frcp(gB + gC);
    const double e1 = (q1 + n1) * sc, e2 = (q2 + n2) * sc;
    if (live) {
        if (!isfinite(e1 + e2 + n1 + n2)) flags |= FLAG_NONFINITE;
        a.dn1[i] = e1;
        a.dn2[i] = e2;
        if (a.keep_p) {
            a.pk1[i] = n1;
            a.pk2[i] = n2;
        }
        rmax = fmax(rmax, fmax(fabs(e1 - g.D1), fabs(e2 - g.D2)));
    }
}

// One sweep over a tile.  A step that stays in its cell (about nine in ten) is
// done inline: one path piece in the cell's own frame, and leg means whose P
// nonzero weights come from one piece.  A step that crosses a grid line has
// two or three pieces and legs of two; the indices of such particles wait in a
// per-wave LDS queue and are done with every term 64 at a time, so that the waves
// do not run the extra terms for lanes that have none.  The re-sort stores the
// particles expected to cross behind the others of their tile, so the rows here
// are nearly all of one kind: the queue fills a row at once, whose lines are
// still in cache when it is read again, and stores cover whole lines.
//
// Bound by HBM and by the latency of its dependent chains at two or three waves
// per SIMD (registers); at 512 x 512 cells, 2^24 particles, degree 3: 80 B per
// particle (96 when it stores its momentum), about 590 vector and 61 LDS
// instructions per row of 64 (917 and 87 with the general terms run for every
// lane), 460 us per launch against 660 us with crossing particles inline in any
// order, the general terms and every momentum stored (events).  Counters: vector
// units 62 %, LDS 73 % busy, 1.43 GB moved.
// Taking the 24 LDS atomics out would give 50 us.  More waves do not help when
// their registers spill: 629 us at four waves per SIMD (degree 3).
constexpr int QCAP = 2 * WAVE;   // fewer than 64 wait when a row starts

// FIRST (sweep 0): the increment is the explicit start d^(0) = dt p^n /
// gamma(x^n, p^n), formed from A_z on the patch and stored with A_z(x^n) and
// gamma(x^n, p^n), which the later sweeps read instead.
//
// Waves per SIMD: what the registers allow without spills.  With spin two at
// degree 3 (199 registers): 191 us per launch at 256 x 256 cells and 2^22
// particles, 243 us at three (168, 112 B per lane spilled).
template <int P, bool FIRST, bool SPIN>
__global__ __launch_bounds__(BLOCK) __attribute__((amdgpu_waves_per_eu(P <= 3 ? (SPIN ? 2 : 3) : 2))) void k2_sweep_I(SweepArgs a) {
    if (*a.gate) return;   // uniform over the grid
    using PT = Patch<P>;
    constexpr int PS = PT::SIZE, PC = PT::PC;
    __shared__ double sE1[PS], sE2[PS], sA[PS], sG1[PS], sG2[PS], sJ1[PS], sJ2[PS], sBz[SPIN ? PS : 1];
    __shared__ int qI[BLOCK / WAVE][QCAP];
    const int nseg = a.M2 / a.TW;
    int part;
    const int tile = tile_of_block(a.split, part);
    const int r = tile / nseg, c0 = (tile - r * nseg) * a.TW;
    const int width = a.TW + P + 2;   // columns of the patch in use
    const PT t{sE1, sE2, sA, sG1, sG2, sJ1, sJ2, sBz, r - P - 1, c0 - P - 1, r};
    for (int k = threadIdx.x; k < PS; k += blockDim.x) {
        const int i = k / PC, j = k - i * PC;
        if (j >= width) continue;
        const int g = wrapi(t.R0 + i, a.M1) * a.M2 + wrapi(t.C0 + j, a.M2);
        sE1[k] = a.eb1[g];
        sE2[k] = a.eb2[g];
        sA[k] = a.az[g];
        sG1[k] = a.g1a[g];
        sG2[k] = a.g2a[g];
        sJ1[k] = 0.0;
        sJ2[k] = 0.0;
        if constexpr (SPIN) sBz[k] = a.bz[g];
    }
    const int begin = a.start[tile], end = a.start[tile + 1];
    const int wid = threadIdx.x / WAVE, lane = lane_id();
    int *const qi = qI[wid];
    double rmax = 0.0;
    int flags = 0;
    int qn = 0;   // particles waiting in this wave's queue (uniform)
    auto wave_fence = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    const int passes = (end - begin + WAVE - 1) / WAVE;   // none for an empty tile
    const int w0 = part * (BLOCK / WAVE) + wid, nw = a.split * (BLOCK / WAVE);
    // the row after the current one, loaded ahead (indices clamped to the tile); the
    // spin sweep has no registers left for it and would wait for the loads to spill them
    constexpr bool AHEAD = !SPIN;
    double nx1 = 0.0, nx2 = 0.0, nq1 = 0.0, nq2 = 0.0, nd1 = 0.0, nd2 = 0.0, nA = 0.0, ng = 0.0;
    auto load_row = [&](int jr) {
        const int i = min(begin + jr * WAVE + lane, end - 1);
        nx1 = a.xi1[i];
        nx2 = a.xi2[i];
        nq1 = a.p1[i];
        nq2 = a.p2[i];
        if constexpr (!FIRST) {
            nd1 = a.d1[i];
            nd2 = a.d2[i];
            nA = a.azn[i];
            ng = a.gamn[i];
        }
    };
    if (AHEAD && w0 < passes) load_row(w0);
    __syncthreads();
    for (int jr = w0;; jr += nw) {
        const bool last = jr >= passes;   // only the waiting particles are left
        if (!last) {
            const int i = begin + jr * WAVE + lane;
            const bool live = i < end;
            if (!AHEAD) load_row(jr);
            const double x1 = nx1, x2 = nx2, q1 = nq1, q2 = nq2;
            double D1 = nd1, D2 = nd2, An = nA, gn = ng;
            if (AHEAD && jr + nw < passes) load_row(jr + nw);
            if constexpr (FIRST) {
                const int c2 = (int)x2;
                An = start_A<P>(t, x1 - r, x2 - c2, c2);
                gn = gamma_of(q1, q2, An);
                const double sc = a.dt * frcp(gn);
                D1 = q1 * sc;
                D2 = q2 * sc;
                if (live) {
                    a.d1[i] = D1;
                    a.d2[i] = D2;
                    a.azn[i] = An;
                    a.gamn[i] = gn;
                }
            }
            const Step g = make_step(a, x1, x2, q1, q2, D1, D2, r);
            const bool in = stays(g);
            const unsigned long long cm = __builtin_amdgcn_ballot_w64(live && !in);
            if (live && !in) qi[qn + rank_in(cm)] = i;
            qn += __builtin_popcountll(cm);
            if (live && in) {
                const Legs l = legs_of<P, SPIN, false>(g, i, t, a);
                __builtin_amdgcn_sched_barrier(0);   // each part keeps to its own registers
                double E1 = 0.0, E2 = 0.0;
                piece<P>(g, true, 0.0, 1.0, 0, 0, t, a.w, E1, E2);
                __builtin_amdgcn_sched_barrier(0);
                push<SPIN>(g, true, i, E1, E2, An, gn, l, a, rmax, flags);
            }
        }
        if (qn >= WAVE || (last && qn > 0)) {
            // do the first n waiting particles, one per lane, and move the rest up
            wave_fence();
            const int n = min(qn, WAVE);
            const bool valid = lane < n;
            const int i = qi[valid ? lane : 0];
            const double x1 = a.xi1[i], x2 = a.xi2[i], q1 = a.p1[i], q2 = a.p2[i];
            const int c2 = (int)x2;
            const double An = start_A<P>(t, x1 - r, x2 - c2, c2);
            double gn = gamma_of(q1, q2, An);
            asm volatile("" : "+v"(gn));   // formed here, as the legs below
            double D1, D2;
            if constexpr (FIRST) {   // as above
                const double sc = a.dt * frcp(gn);
                D1 = q1 * sc;
                D2 = q2 * sc;
            } else {
                D1 = a.d1[i];
                D2 = a.d2[i];
            }
            Step g = make_step(a, x1, x2, q1, q2, D1, D2, r);
            cross_step(g, valid, flags);
            const Legs l = legs_of<P, SPIN, true>(g, i, t, a);
            __builtin_amdgcn_sched_barrier(0);
            double E1 = 0.0, E2 = 0.0;
            pieces<P>(g, valid, t, a.w, E1, E2);
            __builtin_amdgcn_sched_barrier(0);
            push<SPIN>(g, valid, i, E1, E2, An, gn, l, a, rmax, flags);
            qn -= n;
            const int mi = qi[WAVE + lane];
            wave_fence();
            if (lane < qn) qi[lane] = mi;
        }
        if (last) break;
    }
    if (flags) atomicOr(a.flags, flags);
    block_max_to(rmax, a.res);
    __syncthreads();
    for (int k = threadIdx.x; k < PS; k += blockDim.x) {
        const int i = k / PC, j = k - i * PC;
        if (j >= width) continue;
        const int g = wrapi(t.R0 + i, a.M1) * a.M2 + wrapi(t.C0 + j, a.M2);
        if (sJ1[k] != 0.0) atomicAdd(&a.J1[g], sJ1[k]);
        if (sJ2[k] != 0.0) atomicAdd(&a.J2[g], sJ2[k]);
    }
}

// Tile starts from cell starts (after the full cell sort of set_particles): the
// first cell of tile T is (T / nseg) M2 + (T % nseg) TW.
__global__ void k2_tiles_from_cells(const int32_t *__restrict__ start, int32_t *__restrict__ tstart, int ntiles,
                                    int nseg, int M2, int TW, int Nc) {
    for (int T = blockIdx.x * blockDim.x + threadIdx.x; T <= ntiles; T += gridDim.x * blockDim.x)
        tstart[T] = T == ntiles ? start[Nc] : start[(T / nseg) * M2 + (T - (T / nseg) * nseg) * TW];
}

// New cell coordinate of a particle from its committed increment, wrapped into
// [0, M); the commit and the re-sort form it with the same operations.
__device__ __forceinline__ double new_coord(double u, double d, double inv_dx, int M) {
    double v = fma(d, inv_dx, u);
    if (v < 0.0) v += (double)M;
    if (v >= (double)M) v -= (double)M;
    if (!(v < (double)M) || v < 0.0) v = 0.0;   // -tiny + M rounded to M
    return v;
}

// A particle's packed place after the commit: the new tile, whether its next step
// is expected to leave its cell, and its column in the tile.
__device__ __forceinline__ int pack_place(int Tn, bool leaves, int col) { return (Tn << 7) | (leaves ? 64 : 0) | col; }
__device__ __forceinline__ int place_tile(int w) { return w >> 7; }
__device__ __forceinline__ int place_key(int w) { return w & 127; }   // sort key inside the tile

// Subsystem I commit, first half (one block per tile): every particle's place (the
// next step is expected to move it by the committed increment again, which is off
// by the step's change of velocity only); per tile the particles that stay and (by
// atomics) those that arrive, and the tile's leavers listed with the slot each has
// among its new tile's arrivals.  The new positions and momenta are written by the
// re-sort.
__global__ __launch_bounds__(BLOCK) void k2_commit_tiles(const double *__restrict__ xi1,
                                                         const double *__restrict__ xi2,
                                                         const double *__restrict__ d1, const double *__restrict__ d2,
                                                         int32_t *__restrict__ word, int2 *__restrict__ leavers,
                                                         const int32_t *__restrict__ tstart, int32_t *__restrict__ tstay,
                                                         int32_t *__restrict__ tarr, int M1, int M2, int TW,
                                                         double inv_dx1, double inv_dx2) {
    __shared__ int nleave;
    const int T = blockIdx.x, nseg = M2 / TW;
    const int begin = tstart[T], end = tstart[T + 1];
    if (threadIdx.x == 0) nleave = 0;
    __syncthreads();
    for (int i = begin + threadIdx.x; i < end; i += blockDim.x) {
        const double e1 = d1[i], e2 = d2[i];
        const double u1 = new_coord(xi1[i], e1, inv_dx1, M1), u2 = new_coord(xi2[i], e2, inv_dx2, M2);
        const int c1 = (int)u1, c2 = (int)u2, sg = c2 / TW;
        const int Tn = c1 * nseg + sg;
        const double v1 = fma(e1, inv_dx1, u1) - c1, v2 = fma(e2, inv_dx2, u2) - c2;
        word[i] = pack_place(Tn, !(v1 >= 0.0 && v1 < 1.0 && v2 >= 0.0 && v2 < 1.0), c2 - sg * TW);
        const bool go = Tn != T;
        const int slot = wave_claim(tarr, Tn, go);
        const unsigned long long m = __builtin_amdgcn_ballot_w64(go);
        if (m) {   // one counter update per wave
            const int leader = __builtin_ctzll(m);
            int at = 0;
            if (lane_id() == leader) at = atomicAdd(&nleave, __builtin_popcountll(m));
            at = __shfl(at, leader, WAVE);
            if (go) leavers[begin + at + rank_in(m)] = make_int2(i, slot);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) tstay[T] = end - begin - nleave;
}

// Tile starts of the new order: the exclusive scan of stay + arrivals over the
// tiles (at most SCAN_TILE: one block); the arrival counts start at zero again.
__global__ __launch_bounds__(SCAN_THREADS) void k2_scan_tiles(const int32_t *__restrict__ tstay,
                                                              int32_t *__restrict__ tarr,
                                                              int32_t *__restrict__ tstart, int ntiles) {
    const int T0 = threadIdx.x * SCAN_PER;
    int k[SCAN_PER], v = 0;
#pragma unroll
    for (int q = 0; q < SCAN_PER; ++q) {
        k[q] = T0 + q < ntiles ? tstay[T0 + q] + tarr[T0 + q] : 0;
        v += k[q];
    }
    int tot;
    int off = block_exscan1024(v, &tot);
#pragma unroll
    for (int q = 0; q < SCAN_PER; ++q)
        if (T0 + q < ntiles) {
            tstart[T0 + q] = off;
            off += k[q];
            tarr[T0 + q] = 0;
        }
    if (threadIdx.x == 0) tstart[ntiles] = tot;
}
static_assert((MAXM / TWMAX) * MAXM <= SCAN_TILE && MAXM <= SCAN_TILE, "one block scans the tiles of any grid");

// Arrivals listed per new tile: a leaver of old tile T puts its index at
// mig[tnew[Tn] + tstay[Tn] + slot] (the places after Tn's stayers in the new order).
__global__ __launch_bounds__(WAVE) void k2_list_arrivals(const int32_t *__restrict__ word,
                                                         const int2 *__restrict__ leavers,
                                                         const int32_t *__restrict__ told,
                                                         const int32_t *__restrict__ tnew,
                                                         const int32_t *__restrict__ tstay, int32_t *__restrict__ mig) {
    const int T = blockIdx.x, begin = told[T], n = told[T + 1] - begin - tstay[T];
    for (int k = threadIdx.x; k < n; k += blockDim.x) {
        const int2 l = leavers[begin + k];
        const int Tn = place_tile(word[l.x]);
        mig[tnew[Tn] + tstay[Tn] + l.y] = l.x;
    }
}

// Subsystem I commit, second half, and the re-sort in one pass (one block per
// new tile): the tile's particles are the stayers of its old range and its
// listed arrivals.  They are ordered by the sort key: those expected to stay in
// their cell by column, then those expected to leave it by column, each of the two
// parts in the transposed layout (tile_pos), so that a coalesced read hands the
// lanes of a wave particles of different cells and (for the sweep) of one kind.
// An LDS counter per key gives each particle its rank (in any order), the prefix
// over the keys its place.  Each particle is written with its new position
// (formed again from x^n and the increment), its momentum p^(k+1) and its id.
// When the tile's sources and particles fit INVCAP, every output array passes
// through LDS (sources read in order, values placed at their new positions, the
// tile written in order), the next array's values being loaded into registers
// while one is written; a fuller tile writes each particle to its position
// directly.  Latency-bound on its barriers: with the scans and the arrival lists
// 366 us at 2^24 particles for 1024 threads of 6 sources (106 registers, one
// block per CU), 570 us for 512 of 12 (spilling at two blocks per CU); stable
// ranks by wave ballots in the old order, with the values loaded between the
// barriers, took 700 us.
constexpr int SORT_THREADS = 1024;
constexpr int SORT_PER = 6;   // sources per thread
constexpr int INVCAP = SORT_THREADS * SORT_PER;
constexpr int NKEY = 128;

struct Resort {
    const double *xi1, *xi2, *d1, *d2, *pk1, *pk2;
    const int32_t *sid, *word, *mig, *told, *tnew, *tstay;
    double *o1, *o2, *r1, *r2;
    int32_t *did;
    int M1, M2;
    double inv_dx1, inv_dx2;
    const double *ss[3];   // spins (null without spin)
    double *os[3];
    // output array f of the sources i[k] >= 0, all loads issued before any is used
    template <int N>
    __device__ __forceinline__ void values(int f, const int (&i)[N], double (&v)[N]) const {
        auto from = [&](const double *x) {
#pragma unroll
            for (int k = 0; k < N; ++k) v[k] = i[k] >= 0 ? x[i[k]] : 0.0;
        };
        auto coord = [&](const double *x, const double *d, double inv_dx, int M) {
            double e[N];
            from(x);
#pragma unroll
            for (int k = 0; k < N; ++k) e[k] = i[k] >= 0 ? d[i[k]] : 0.0;
#pragma unroll
            for (int k = 0; k < N; ++k) v[k] = new_coord(v[k], e[k], inv_dx, M);
        };
        switch (f) {
            case 0: coord(xi1, d1, inv_dx1, M1); break;
            case 1: coord(xi2, d2, inv_dx2, M2); break;
            case 2: from(pk1); break;
            case 3: from(pk2); break;
            case 4:
#pragma unroll
                for (int k = 0; k < N; ++k) v[k] = i[k] >= 0 ? (double)sid[i[k]] : 0.0;
                break;
            default: from(ss[f - 5]); break;
        }
    }
    __device__ __forceinline__ void put(int j, int i) const {
        o1[j] = new_coord(xi1[i], d1[i], inv_dx1, M1);
        o2[j] = new_coord(xi2[i], d2[i], inv_dx2, M2);
        r1[j] = pk1[i];
        r2[j] = pk2[i];
        did[j] = sid[i];
        if (ss[0])
            for (int q = 0; q < 3; ++q) os[q][j] = ss[q][i];
    }
};

__global__ __launch_bounds__(SORT_THREADS) __attribute__((amdgpu_waves_per_eu(4))) void k2_tile_resort(Resort a) {
    __shared__ int hist[NKEY], first[NKEY];   // particles of a key; their first rank
    __shared__ int nstay;                     // particles expected to stay in their cell
    __shared__ double val[INVCAP];            // one output array of the tile, by new position
    const int T = tile_of_block();
    const int ob = a.told[T], nold = a.told[T + 1] - ob;
    const int base = a.tnew[T], cnt = a.tnew[T + 1] - base, arr0 = base + a.tstay[T];
    const int nsrc = nold + cnt - a.tstay[T];
    const int nt = SORT_THREADS, t0 = threadIdx.x;
    // source q < nold: old position q of the tile; q >= nold: listed arrival
    auto source = [&](int q) { return q < nold ? ob + q : a.mig[arr0 + q - nold]; };
    for (int k = t0; k < NKEY; k += nt) hist[k] = 0;
    __syncthreads();
    const bool direct = cnt > INVCAP || nsrc > INVCAP;   // uniform over the block
    int src[SORT_PER], pos[SORT_PER];   // source index (-1: none, or it left) and rank, later position
    if (!direct) {
#pragma unroll
        for (int k = 0; k < SORT_PER; ++k) {
            const int q = t0 + k * nt;
            src[k] = q < nsrc ? source(q) : -1;
        }
        int w[SORT_PER];
#pragma unroll
        for (int k = 0; k < SORT_PER; ++k) w[k] = src[k] >= 0 ? a.word[src[k]] : -1;
#pragma unroll
        for (int k = 0; k < SORT_PER; ++k) {
            pos[k] = 0;
            if (w[k] >= 0 && place_tile(w[k]) == T)
                pos[k] = (place_key(w[k]) << 16) | atomicAdd(&hist[place_key(w[k])], 1);
            else
                src[k] = -1;
        }
    } else {
        for (int q = t0; q < nsrc; q += nt) {
            const int w = a.word[source(q)];
            if (place_tile(w) == T) atomicAdd(&hist[place_key(w)], 1);
        }
    }
    __syncthreads();
    if (t0 < WAVE) {   // exclusive prefix over the keys, two per lane
        const int v0 = hist[2 * t0], v1 = hist[2 * t0 + 1];
        int inc = v0 + v1;
#pragma unroll
        for (int o = 1; o < WAVE; o <<= 1) {
            const int u = __shfl_up(inc, o, WAVE);
            if (t0 >= o) inc += u;
        }
        first[2 * t0] = inc - v0 - v1;
        first[2 * t0 + 1] = inc - v1;
        if (2 * t0 == NKEY / 2) nstay = inc - v0 - v1;
    }
    __syncthreads();
    const int nin = nstay;   // (first[] holds the direct path's cursors from here on)
    auto place = [&](int rank) { return rank < nin ? tile_pos(rank, nin) : nin + tile_pos(rank - nin, cnt - nin); };
    if (direct) {
        for (int q = t0; q < nsrc; q += nt) {
            const int i = source(q), w = a.word[i];
            if (place_tile(w) == T) a.put(base + place(atomicAdd(&first[place_key(w)], 1)), i);
        }
        return;
    }
    {
        // place() without its integer divisions: t / Q as (t + 1/2) times the float
        // 1 / Q, exact for t < INVCAP (the error stays below half of 1 / Q)
        const int Qi = nin / WAVE, Qo = (cnt - nin) / WAVE;
        const float ri = Qi ? 1.0f / (float)Qi : 0.0f, ro = Qo ? 1.0f / (float)Qo : 0.0f;
#pragma unroll
        for (int k = 0; k < SORT_PER; ++k) {
            const int rank = first[pos[k] >> 16] + (pos[k] & 0xffff);
            const bool in = rank < nin;
            const int t = in ? rank : rank - nin, Q = in ? Qi : Qo;
            const int l = (int)(((float)t + 0.5f) * (in ? ri : ro));
            pos[k] = (in ? 0 : nin) + (t < WAVE * Q ? (t - l * Q) * WAVE + l : t);
        }
    }
    const int nf = a.ss[0] ? 8 : 5;   // with spin: s_x, s_y, s_z as well
    double v[SORT_PER];
    a.values(0, src, v);
    for (int f = 0; f < nf; ++f) {
        if (f > 0) __syncthreads();   // the previous array is written
#pragma unroll
        for (int k = 0; k < SORT_PER; ++k)
            if (src[k] >= 0) val[pos[k]] = v[k];
        if (f + 1 < nf) a.values(f + 1, src, v);
        __syncthreads();
        double *out = f == 0 ? a.o1 : f == 1 ? a.o2 : f == 2 ? a.r1 : f == 3 ? a.r2 : f == 4 ? nullptr : a.os[f - 5];
        for (int p = t0; p < cnt; p += nt) {
            if (f != 4) out[base + p] = val[p];
            else a.did[base + p] = (int32_t)val[p];
        }
    }
}

// ---------------------------------------------------------------------------
// Subsystem III particle term and the charge deposit (tiles, no motion)
// ---------------------------------------------------------------------------
struct DepArgs {
    const double *xi1, *xi2, *p1, *p2;
    const int32_t *start;   // first particle of each tile (ntiles + 1)
    const double *an;    // a_z^n                     (III)
    const double *ezn;   // e_z^n                     (III)
    const double *ezk;   // e_z^(k)                   (III)
    double *S;           // deposit target (zero on entry)
    double *anp;         // A^n at each particle (III): written on the first iteration, read after
    int M1, M2, TW;
    double dt, w;
    int mode;            // 0: charge w Lambda0; 1: Subsystem III source
    int first;           // III: first iteration of the substep
    const int *gate;     // III: nonzero once an earlier iteration converged (nothing to do)
    int split;           // blocks per tile
};

// mode 1: S += w (A^n + A^(k)) / (gamma(p, A^n) + gamma(p, A^(k))) Lambda0(x_a),
// with A^(k) the field of a^(k) = a^n - dt (e^n + e^(k)) / 2.
// Bound by the LDS pipe: (P+1)^2 reads and (P+1)^2 atomics of 15 cycles a row, 115 us of
// 512 x 512 cells with 2^24 cubic particles, and by its 40 bytes a particle (145 us).  The
// patch's stride is a constant, so that the nodes are immediate offsets, and a row's loads
// are issued a row ahead: 187 -> 167 us.
template <int P>
__global__ __launch_bounds__(BLOCK) void k2_deposit0(DepArgs a) {
    if (a.gate && *a.gate) return;   // uniform over the grid
    constexpr int PR = P + 1, PCM = TWMAX + P, PS = PR * PCM;
    __shared__ double sAn[PS], sAk[PS], sS[PS];
    const int nseg = a.M2 / a.TW;
    int part;
    const int tile = tile_of_block(a.split, part);
    const int r = tile / nseg, c0 = (tile - r * nseg) * a.TW;
    const int PC = a.TW + P;
    const int R0 = r - P, C0 = c0 - P;
    const int begin = a.start[tile], end = a.start[tile + 1];
    const int passes = (end - begin + WAVE - 1) / WAVE;   // none for an empty tile
    const int nw = a.split * (BLOCK / WAVE);
    int jr = part * (BLOCK / WAVE) + threadIdx.x / WAVE;
    // a row's loads are issued a row ahead
    double nu1 = 0.0, nu2 = 0.0, nq1 = 0.0, nq2 = 0.0, nA = 0.0;
    auto load = [&](int row) {
        if (row >= passes) return;
        const int i = min(begin + row * WAVE + lane_id(), end - 1);
        nu1 = a.xi1[i];
        nu2 = a.xi2[i];
        if (a.mode == 1) {
            nq1 = a.p1[i];
            nq2 = a.p2[i];
            if (!a.first) nA = a.anp[i];
        }
    };
    load(jr);
    for (int t = threadIdx.x; t < PR * PC; t += blockDim.x) {
        const int i = t / PC, j = t - i * PC;
        const int g = wrapi(R0 + i, a.M1) * a.M2 + wrapi(C0 + j, a.M2);
        if (a.mode == 1) {
            const double an = a.an[g];
            if (a.first) sAn[i * PCM + j] = an;
            sAk[i * PCM + j] = an - 0.5 * a.dt * (a.ezn[g] + a.ezk[g]);
        }
        sS[i * PCM + j] = 0.0;
    }
    __syncthreads();
    for (; jr < passes; jr += nw) {
        const int i = begin + jr * WAVE + lane_id();
        const bool live = i < end;
        const double u1 = nu1, u2 = nu2, q1 = nq1, q2 = nq2;
        double An = nA;
        load(jr + nw);
        const int c2 = (int)u2;
        double b1[P + 1], b2[P + 1];
        basis_values<P>(u1 - r, b1);
        basis_values<P>(u2 - c2, b2);
        const int s0 = P * PCM + c2 - C0;   // node (r, c2) of the patch; (m1, m2) back from it
        double q = a.w;
        if (a.mode == 1) {
            double An0 = 0.0, Ak = 0.0;
#pragma unroll
            for (int m1 = 0; m1 <= P; ++m1) {
                double tn = 0.0, tk = 0.0;
#pragma unroll
                for (int m2 = 0; m2 <= P; ++m2) {
                    const int s = s0 - m1 * PCM - m2;
                    if (a.first) tn += b2[m2] * sAn[s];
                    tk += b2[m2] * sAk[s];
                }
                An0 += b1[m1] * tn;
                Ak += b1[m1] * tk;
            }
            if (a.first) {
                An = An0;
                if (live) a.anp[i] = An;
            }
            const double pp = 1.0 + q1 * q1 + q2 * q2;
            q = a.w * (An + Ak) * frcp(fsqrt(pp + An * An) + fsqrt(pp + Ak * Ak));
        }
        if (live) {
#pragma unroll
            for (int m1 = 0; m1 <= P; ++m1) {
                const double qb = q * b1[m1];
#pragma unroll
                for (int m2 = 0; m2 <= P; ++m2) atomicAdd(&sS[s0 - m1 * PCM - m2], qb * b2[m2]);
            }
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < PR * PC; t += blockDim.x) {
        const int i = t / PC, j = t - i * PC;
        const int g = wrapi(R0 + i, a.M1) * a.M2 + wrapi(C0 + j, a.M2);
        if (sS[i * PCM + j] != 0.0) atomicAdd(&a.S[g], sS[i * PCM + j]);
    }
}

// Subsystem II over tiles: B_z (V2) and A_z (V0) gathered from the tile's LDS
// patch, every momentum turned by the angle B_z dt / gamma.  SPIN: every spin
// also turns about B_h = (dA_z/dx2, -dA_z/dx1, B_z) by the angle -|B_h| dt
// (ds/dt = s x B_h, Rodrigues' formula), with G a_z staged as well.
struct RotArgs {
    const double *xi1, *xi2;
    double *p1, *p2, *sx, *sy, *sz;
    const int32_t *start;
    const double *bz, *az, *g1, *g2;
    int M1, M2, TW;
    double dt;
    int split;   // blocks per tile
};

template <int P, bool SPIN>
__global__ __launch_bounds__(BLOCK) void k2_rotate_tiles(RotArgs a) {
    constexpr int PR = P + 1, PCM = TWMAX + P, PS = PR * PCM;
    __shared__ double sA[PS], sB[PS], sG1[SPIN ? PS : 1], sG2[SPIN ? PS : 1];
    const int nseg = a.M2 / a.TW;
    int part;
    const int tile = tile_of_block(a.split, part);
    const int r = tile / nseg, c0 = (tile - r * nseg) * a.TW;
    const int PC = a.TW + P;
    const int R0 = r - P, C0 = c0 - P;
    for (int t = threadIdx.x; t < PR * PC; t += blockDim.x) {
        const int i = t / PC, j = t - i * PC;
        const int g = wrapi(R0 + i, a.M1) * a.M2 + wrapi(C0 + j, a.M2);
        sA[t] = a.az[g];
        sB[t] = a.bz[g];
        if constexpr (SPIN) {
            sG1[t] = a.g1[g];
            sG2[t] = a.g2[g];
        }
    }
    __syncthreads();
    const int begin = a.start[tile], end = a.start[tile + 1];
    for (int i = begin + part * BLOCK + threadIdx.x; i < end; i += a.split * BLOCK) {
        const double u1 = a.xi1[i], u2 = a.xi2[i];
        const int c2 = (int)u2;
        const double t1 = u1 - r, t2 = u2 - c2;
        double a1[P + 1], a2[P + 1], b1[P], b2[P];
        basis_values<P>(t1, a1);
        basis_values<P>(t2, a2);
        basis_values<P - 1>(t1, b1);
        basis_values<P - 1>(t2, b2);
        double A = 0.0, B = 0.0, Bx = 0.0, By = 0.0;
#pragma unroll
        for (int m1 = 0; m1 <= P; ++m1) {
            double ta = 0.0, tb = 0.0, tx = 0.0, ty = 0.0;
#pragma unroll
            for (int m2 = 0; m2 <= P; ++m2) {
                const int s = (r - m1 - R0) * PC + c2 - m2 - C0;
                ta += a2[m2] * sA[s];
                if (m1 < P && m2 < P) tb += b2[m2] * sB[s];
                if constexpr (SPIN) {
                    if (m2 < P) tx += b2[m2] * sG2[s];   // dA_z/dx2: degrees (P, P-1)
                    if (m1 < P) ty += a2[m2] * sG1[s];   // dA_z/dx1: degrees (P-1, P)
                }
            }
            A += a1[m1] * ta;
            if (m1 < P) B += b1[m1] * tb;
            if constexpr (SPIN) {
                Bx += a1[m1] * tx;
                if (m1 < P) By -= b1[m1] * ty;
            }
        }
        const double q1 = a.p1[i], q2 = a.p2[i];
        const double th = B * a.dt / sqrt(1.0 + q1 * q1 + q2 * q2 + A * A);
        double sn, cs;
        sincos(th, &sn, &cs);
        a.p1[i] = q1 * cs + q2 * sn;
        a.p2[i] = -q1 * sn + q2 * cs;
        if constexpr (SPIN) {
            const double nb = sqrt(Bx * Bx + By * By + B * B);
            if (nb > 0.0) {
                const double k0 = Bx / nb, k1 = By / nb, k2 = B / nb;
                const double s0 = a.sx[i], s1 = a.sy[i], s2 = a.sz[i];
                const double x0 = k1 * s2 - k2 * s1, x1 = k2 * s0 - k0 * s2, x2 = k0 * s1 - k1 * s0;
                const double ks = k0 * s0 + k1 * s1 + k2 * s2;
                double sb, cb;
                sincos(nb * a.dt, &sb, &cb);
                a.sx[i] = s0 * cb - x0 * sb + k0 * ks * (1.0 - cb);
                a.sy[i] = s1 * cb - x1 * sb + k1 * ks * (1.0 - cb);
                a.sz[i] = s2 * cb - x2 * sb + k2 * ks * (1.0 - cb);
            }
        }
    }
}

// a^{n+1} = a^n - dt (e^n + e^{n+1}) / 2, e_z = e^{n+1}.
__global__ void k2_finish_III(double *__restrict__ az, double *__restrict__ ez, const double *__restrict__ ezn,
                              const double *__restrict__ ezk, int N, double dt) {
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < N; i += gridDim.x * blockDim.x) {
        az[i] -= 0.5 * dt * (ezn[i] + ezk[i]);
        ez[i] = ezk[i];
    }
}

// ---------------------------------------------------------------------------
// Diagnostics: kinetic energy, quadratic forms, Gauss residual
// ---------------------------------------------------------------------------
template <int P>
__global__ __launch_bounds__(BLOCK) void k2_kinetic(const double *__restrict__ xi1, const double *__restrict__ xi2,
                           const double *__restrict__ p1, const double *__restrict__ p2,
                           const double *__restrict__ az, int64_t n, int M1, int M2, double w,
                           double *__restrict__ partial) {
    double s = 0.0;
    for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double u1 = xi1[i], u2 = xi2[i];
        const int c1 = (int)u1, c2 = (int)u2;
        const double A = gather00<P>(az, M1, M2, c1, c2, u1 - c1, u2 - c2);
        const double q1 = p1[i], q2 = p2[i];
        const double pp = q1 * q1 + q2 * q2 + A * A;
        s += w * pp / (sqrt(1.0 + pp) + 1.0);   // gamma - 1 without cancellation
    }
    block_sum_to(s, &partial[blockIdx.x]);
}

struct MassRows {
    double r1[11], r2[11];   // rows of the 1D mass matrices (dimensionless), 2d+1 entries
    int d1, d2;
    double scale;            // dx1 dx2
};

// y = (Mass_{d1} (x) Mass_{d2}) x on the periodic grid.
__global__ __launch_bounds__(BLOCK) void k2_mass(const double *__restrict__ x, double *__restrict__ y, int M1, int M2, MassRows m) {
    const int N = M1 * M2;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < N; i += gridDim.x * blockDim.x) {
        const int i1 = i / M2, i2 = i - i1 * M2;
        double s = 0.0;
        for (int k1 = -m.d1; k1 <= m.d1; ++k1) {
            const double *row = x + wrapi(i1 + k1, M1) * M2;
            double t = 0.0;
            for (int k2 = -m.d2; k2 <= m.d2; ++k2) t += m.r2[k2 + m.d2] * row[wrapi(i2 + k2, M2)];
            s += m.r1[k1 + m.d1] * t;
        }
        y[i] = m.scale * s;
    }
}

// partial[block] = sum of x_i y_i over the block's nodes.
__global__ void k2_dot(const double *__restrict__ x, const double *__restrict__ y, int N, double *partial) {
    double s = 0.0;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < N; i += gridDim.x * blockDim.x) s += x[i] * y[i];
    block_sum_to(s, &partial[blockIdx.x]);
}

// out = sum of partial[0..n) in order (one block).
__global__ void k2_sum(const double *__restrict__ partial, int n, double *out) {
    double s = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) s += partial[i];
    block_sum_to(s, out);
}

// r = G^T u + rho - dx1 dx2 with u = M1 e (two components); max |r| into *res.
__global__ __launch_bounds__(BLOCK) void k2_gauss(const double *__restrict__ u1, const double *__restrict__ u2,
                         const double *__restrict__ rho, double *__restrict__ r, int M1, int M2, double inv_dx1,
                         double inv_dx2, double cell_area, unsigned long long *res) {
    const int N = M1 * M2;
    double m = 0.0;
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < N; i += gridDim.x * blockDim.x) {
        const int i1 = i / M2, i2 = i - i1 * M2;
        const double v = (u1[i] - u1[wrapi(i1 + 1, M1) * M2 + i2]) * inv_dx1 +
                         (u2[i] - u2[i1 * M2 + wrapi(i2 + 1, M2)]) * inv_dx2 + rho[i] - cell_area;
        r[i] = v;
        m = fmax(m, fabs(v));
    }
    block_max_to(m, res);
}

// End of one fixed-point iteration, run by the last block of its solve: the
// larger of the residuals ra, rb (rb may be null; +inf if one is not finite), or
// -2 - flags if a status flag is set (flags may be null), goes to the iteration's
// word of the host mirror, and the gate closes when a flag is set, a residual is
// not finite, or the larger one is at most tol: the conditions on which the host
// stops at this iteration.
struct IterEnd {
    const unsigned long long *ra, *rb;
    const int *flags;
    double tol;
    int *gate;
    double *h;        // null: the solve ends no iteration
    unsigned *done;   // blocks finished (zero between solves)
};

// Called by thread 0 of every block once it has recorded the block's residual by an
// atomic.  Only atomics are exchanged here, so waiting for them is enough: a fence
// would write every block's field values back from L2 (3 to 4 us per solve), which
// the next kernel's start does anyway.
__device__ __forceinline__ void end_iteration(const IterEnd &e) {
    wait_memory();
    if (atomicAdd(e.done, 1u) != gridDim.x - 1) return;
    wait_memory();
    auto load = [](const unsigned long long *p) {
        return __longlong_as_double((long long)__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    };
    const double a = load(e.ra), b = e.rb ? load(e.rb) : 0.0;
    const int f = e.flags ? __hip_atomic_load(e.flags, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0;
    const double r = isfinite(a) && isfinite(b) ? fmax(a, b) : HUGE_VAL;
    *e.done = 0u;
    if (f || !(r > e.tol) || !isfinite(r)) *e.gate = 1;
    *const_cast<volatile double *>(e.h) = f ? -2.0 - f : r;
}

// ---------------------------------------------------------------------------
// Spectral solves: 2D FFT (rows, then columns with the spectral step fused)
// ---------------------------------------------------------------------------
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

template <bool INV>
__device__ __forceinline__ double2 mul_i(double2 a) {   // a exp(-+ i pi / 2): -i a forward, +i a inverse
    return INV ? make_double2(-a.y, a.x) : make_double2(a.y, -a.x);
}

// DFT of R = 2, 4 or 8 points in registers: X_q = sum_r v_r exp(-+ 2 pi i r q / R)
// (the + sign for INV).
template <int R, bool INV>
__device__ __forceinline__ void dft_reg(double2 (&v)[R]) {
    if constexpr (R == 2) {
        const double2 a = v[0], b = v[1];
        v[0] = make_double2(a.x + b.x, a.y + b.y);
        v[1] = make_double2(a.x - b.x, a.y - b.y);
    } else if constexpr (R == 4) {
        const double2 s02 = make_double2(v[0].x + v[2].x, v[0].y + v[2].y);
        const double2 d02 = make_double2(v[0].x - v[2].x, v[0].y - v[2].y);
        const double2 s13 = make_double2(v[1].x + v[3].x, v[1].y + v[3].y);
        const double2 d13 = mul_i<INV>(make_double2(v[1].x - v[3].x, v[1].y - v[3].y));
        v[0] = make_double2(s02.x + s13.x, s02.y + s13.y);
        v[2] = make_double2(s02.x - s13.x, s02.y - s13.y);
        v[1] = make_double2(d02.x + d13.x, d02.y + d13.y);
        v[3] = make_double2(d02.x - d13.x, d02.y - d13.y);
    } else {
        double2 e[4] = {v[0], v[2], v[4], v[6]}, o[4] = {v[1], v[3], v[5], v[7]};
        dft_reg<4, INV>(e);
        dft_reg<4, INV>(o);
        constexpr double c = 0.70710678118654752440;
        o[1] = cmul(o[1], make_double2(c, INV ? c : -c));
        o[2] = mul_i<INV>(o[2]);
        o[3] = cmul(o[3], make_double2(-c, INV ? c : -c));
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            v[q] = make_double2(e[q].x + o[q].x, e[q].y + o[q].y);
            v[q + 4] = make_double2(e[q].x - o[q].x, e[q].y - o[q].y);
        }
    }
}

// FFT of n = 2^k points (8 <= n <= MAXM), Stockham autosort with radix-8
// stages and one final radix-2 or radix-4 stage when k is not a multiple of 3.
// A transform is spread over T = n / 8 threads; thread t holds the 8 values at
// positions t + m T (m < 8) in x, before and after.  In a stage of radix R
// after Ns points have been combined, butterfly j = t + q T (q < 8 / R) takes
// the inputs j + r n / R (x[q + r 8/R]), multiplies input r by
// w^(r (j mod Ns) n / (Ns R)) with w = exp(-+ 2 pi i / n), and sends output r
// to (j - j mod Ns) R + j mod Ns + r Ns.  Between stages the values pass
// through LDS (position p of this transform at lds[base + p sp]); the last
// stage's outputs are this thread's own positions, so they stay in registers.
// stw holds w^m for m < n / 2.  Every thread of the block takes part (the
// stages synchronise the block).
template <int R, bool INV>
__device__ __forceinline__ void fft_stage(double2 (&x)[8], int t, int T, int n, int Ns, bool last, double2 *lds,
                                          int sp, int base, const double2 *stw) {
    constexpr int Q = 8 / R;
    const int step = n / (Ns * R), h = n >> 1;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        const int j = t + q * T, k = j & (Ns - 1);
        double2 v[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            double2 a = x[q + r * Q];
            if (r > 0) {
                const int m = r * k * step;
                double2 w = m < h ? stw[m] : make_double2(-stw[m - h].x, -stw[m - h].y);
                if (INV) w.y = -w.y;
                a = cmul(a, w);
            }
            v[r] = a;
        }
        dft_reg<R, INV>(v);
        const int o = (j - k) * R + k;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            if (last)
                x[q + r * Q] = v[r];
            else
                lds[base + (o + r * Ns) * sp] = v[r];
        }
    }
    if (!last) {
        __syncthreads();
#pragma unroll
        for (int m = 0; m < 8; ++m) x[m] = lds[base + (t + m * T) * sp];
        __syncthreads();
    }
}

template <bool INV>
__device__ void fft8(double2 (&x)[8], int t, int n, double2 *lds, int sp, int base, const double2 *stw) {
    const int T = n >> 3;
    const int e = 31 - __clz(n), n8 = e / 3, rem = e % 3;
    int Ns = 1;
    for (int s = 0; s < n8; ++s) {
        fft_stage<8, INV>(x, t, T, n, Ns, s == n8 - 1 && rem == 0, lds, sp, base, stw);
        Ns <<= 3;
    }
    if (rem == 1) fft_stage<2, INV>(x, t, T, n, Ns, true, lds, sp, base, stw);
    if (rem == 2) fft_stage<4, INV>(x, t, T, n, Ns, true, lds, sp, base, stw);
}

template <int NB>
struct Ptrs {
    double *p[NB];
};

// The five fields into one block of host memory (pinned, written over the link): one launch
// and one wait instead of five copies through the runtime's staging buffer (256 nodes: 90 us
// so, 20 this way).
constexpr int FIELDS_NODES = 65536;   // larger grids are copied (2.6 MB of pinned memory at most)
__global__ void __launch_bounds__(BLOCK) k2_fields_out(Ptrs<5> f, double *out, int Nc) {
    const int i = blockIdx.x * BLOCK + threadIdx.x;
    if (i < Nc) out[(size_t)blockIdx.y * Nc + i] = f.p[blockIdx.y][i];
}

// Forward transform along x2 of NB real grids, one transform per (grid, row)
// over M2 / 8 threads; bit b of zero_mask zeroes grid b after it is read (the
// accumulators of the next deposit).
template <int NB>
__global__ __launch_bounds__(BLOCK) void k2_fft_rows_fwd(Ptrs<NB> src, int zero_mask, double2 *__restrict__ Z,
                                                         int M1, int M2, const double2 *__restrict__ tw2,
                                                         const int *gate) {
    if (gate && *gate) return;   // uniform over the grid
    __shared__ double2 lds[8 * BLOCK], stw[MAXM / 2];
    const int n = M2, T = n >> 3, per = BLOCK / T;
    const int fl = threadIdx.x / T, t = threadIdx.x - fl * T, f = blockIdx.x * per + fl;
    const bool act = f < NB * M1;
    const int b = act ? f / M1 : 0, row = act ? f - b * M1 : 0;
    for (int i = threadIdx.x; i < (n >> 1); i += blockDim.x) stw[i] = tw2[i];
    double *s = src.p[0];
#pragma unroll
    for (int q = 1; q < NB; ++q)
        if (b == q) s = src.p[q];
    s += (size_t)row * M2;
    const bool zero = (zero_mask >> b) & 1;
    double2 x[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) x[m] = make_double2(act ? s[t + m * T] : 0.0, 0.0);
    if (act && zero) {
#pragma unroll
        for (int m = 0; m < 8; ++m) s[t + m * T] = 0.0;
    }
    __syncthreads();
    fft8<false>(x, t, n, lds, 1, fl * n, stw);
    if (act) {
        double2 *z = Z + (size_t)b * M1 * M2 + (size_t)row * M2;
#pragma unroll
        for (int m = 0; m < 8; ++m) z[t + m * T] = x[m];
    }
}

// 1D symbols of the spectral step, per direction (length M1 and M2): the mass
// matrices' eigenvalues m0, m1 (dx included) and the backward difference
// (1 - exp(-i theta)) / dx as (cr, ci).
struct Sym {
    const double *m0a, *m1a, *cra, *cia;
    const double *m0b, *m1b, *crb, *cib;
};

// Along x1 for NB grids: forward transform of each grid's column, the spectral
// step op(k1, k2, v) on every frequency (all NB grids at once, in registers),
// then (if op.INVERSE) the inverse transforms, written back to Z.  The block's
// BLOCK / (M1 / 8) columns are adjacent and consecutive threads take
// consecutive columns, so every row access is contiguous; adjacent column
// groups go to blocks on the same XCD.
template <int NB, class Op>
__global__ __launch_bounds__(BLOCK) void k2_fft_cols(double2 *__restrict__ Z, int M1, int M2,
                                                     const double2 *__restrict__ tw1, Op op, const int *gate) {
    if (gate && *gate) return;   // uniform over the grid
    __shared__ double2 lds[8 * BLOCK], stw[MAXM / 2];
    const int n = M1, T = n >> 3, per = BLOCK / T;
    const int c = threadIdx.x % per, t = threadIdx.x / per;
    const int col = tile_of_block() * per + c;
    const bool act = col < M2;
    const size_t N = (size_t)M1 * M2;
    for (int i = threadIdx.x; i < (n >> 1); i += blockDim.x) stw[i] = tw1[i];
    double2 x[NB][8];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int m = 0; m < 8; ++m)
            x[b][m] = act ? Z[b * N + (size_t)(t + m * T) * M2 + col] : make_double2(0.0, 0.0);
    __syncthreads();
#pragma unroll
    for (int b = 0; b < NB; ++b) fft8<false>(x[b], t, n, lds, per, c, stw);
    if (act) {
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            double2 v[NB];
#pragma unroll
            for (int b = 0; b < NB; ++b) v[b] = x[b][m];
            op(t + m * T, col, v);
#pragma unroll
            for (int b = 0; b < NB; ++b) x[b][m] = v[b];
        }
    }
    if constexpr (Op::INVERSE) {
#pragma unroll
        for (int b = 0; b < NB; ++b) fft8<true>(x[b], t, n, lds, per, c, stw);
        if (act) {
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int m = 0; m < 8; ++m) Z[b * N + (size_t)(t + m * T) * M2 + col] = x[b][m];
        }
    }
}

// Inverse transform along x2 of NB grids, scaled by 1/(M1 M2); the real part of
// entry g of grid b goes to epi(b, g, v), whose return values are max-reduced
// into epi.res (if set).
template <int NB, class Epi>
__global__ __launch_bounds__(BLOCK) void k2_fft_rows_inv(const double2 *__restrict__ Z, int M1, int M2,
                                                         const double2 *__restrict__ tw2, double invN, Epi epi,
                                                         const int *gate, IterEnd end) {
    if (gate && *gate) return;   // uniform over the grid
    __shared__ double2 lds[8 * BLOCK], stw[MAXM / 2];
    const int n = M2, T = n >> 3, per = BLOCK / T;
    const int fl = threadIdx.x / T, t = threadIdx.x - fl * T, f = blockIdx.x * per + fl;
    const bool act = f < NB * M1;
    const int b = act ? f / M1 : 0, row = act ? f - b * M1 : 0;
    for (int i = threadIdx.x; i < (n >> 1); i += blockDim.x) stw[i] = tw2[i];
    const double2 *z = Z + (size_t)b * M1 * M2 + (size_t)row * M2;
    double2 x[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) x[m] = act ? z[t + m * T] : make_double2(0.0, 0.0);
    __syncthreads();
    fft8<true>(x, t, n, lds, 1, fl * n, stw);
    double mx = 0.0;
    if (act) {
        typename Epi::In in[8];   // every load issued before the first store
#pragma unroll
        for (int m = 0; m < 8; ++m) in[m] = epi.load(b, row * M2 + t + m * T);
#pragma unroll
        for (int m = 0; m < 8; ++m) mx = fmax(mx, epi(b, row * M2 + t + m * T, x[m].x * invN, in[m]));
    }
    if (epi.res) block_max_to(mx, epi.res);
    if (end.h && threadIdx.x == 0) end_iteration(end);
}

// The whole solve of one grid in one block, for grids of at most SMALL_SOLVE
// nodes and operators that act on each grid by itself (op.one): the transform
// along x2, along x1, the spectral step, and both back, the values in registers (8
// per thread) and exchanged through LDS, one block per grid.  Against the three
// kernels (events): 16 x 16 nodes 14.0 and 18.9 us, 32 x 64 17.3 and 20.2, 64 x 64
// 22.5 and 21.3.
constexpr int SMALL_SOLVE = 2048;

inline size_t small_solve_lds(int M1, int M2) {
    return sizeof(double2) * ((size_t)std::max(M1 * M2, 8 * WAVE) + M1 / 2 + M2 / 2);
}

template <int NB, class Op, class Epi>
__global__ __launch_bounds__(SMALL_SOLVE / 8) void k2_solve_small(Ptrs<NB> src, int M1, int M2,
                                                                  const double2 *__restrict__ tw1,
                                                                  const double2 *__restrict__ tw2, double invN, Op op,
                                                                  Epi epi, const int *gate, IterEnd end) {
    if (gate && *gate) return;   // uniform over the grid
    extern __shared__ double2 small_lds[];
    const int N = M1 * M2, b = blockIdx.x, tid = threadIdx.x;
    double2 *lds = small_lds, *st1 = lds + max(N, 8 * WAVE), *st2 = st1 + M1 / 2;
    double *s = src.p[0];
#pragma unroll
    for (int q = 1; q < NB; ++q)
        if (b == q) s = src.p[q];
    for (int i = tid; i < M1 / 2; i += blockDim.x) st1[i] = tw1[i];
    for (int i = tid; i < M2 / 2; i += blockDim.x) st2[i] = tw2[i];
    const bool act = tid < N / 8;   // a block has at least one wave; idle threads have LDS of their own
    const int T2 = M2 >> 3, row = tid / T2, t2 = tid - row * T2;
    const int T1 = M1 >> 3, t1 = tid / M2, col = tid - t1 * M2;
    const int base2 = row * M2, o2 = base2 + t2;
    double2 x[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) x[m] = make_double2(act ? s[o2 + m * T2] : 0.0, 0.0);
    if (act) {   // the accumulator of the next deposit
#pragma unroll
        for (int m = 0; m < 8; ++m) s[o2 + m * T2] = 0.0;
    }
    __syncthreads();
    fft8<false>(x, t2, M2, lds, 1, base2, st2);
#pragma unroll
    for (int m = 0; m < 8; ++m) lds[o2 + m * T2] = x[m];
    __syncthreads();
    // idle threads (grids under 512 nodes) read and write behind the grid's columns
    const int c1 = act ? col : N + tid, sp = act ? M2 : 0;
#pragma unroll
    for (int m = 0; m < 8; ++m) x[m] = lds[c1 + (t1 + m * T1) * sp];
    __syncthreads();
    fft8<false>(x, t1, M1, lds, sp, c1, st1);
    if (act) {
#pragma unroll
        for (int m = 0; m < 8; ++m) x[m] = op.one(b, t1 + m * T1, col, x[m]);
    }
    fft8<true>(x, t1, M1, lds, sp, c1, st1);
    if (act) {
#pragma unroll
        for (int m = 0; m < 8; ++m) lds[c1 + (t1 + m * T1) * sp] = x[m];
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < 8; ++m) x[m] = lds[o2 + m * T2];
    __syncthreads();
    fft8<true>(x, t2, M2, lds, 1, base2, st2);
    double mx = 0.0;
    if (act) {
        typename Epi::In in[8];
#pragma unroll
        for (int m = 0; m < 8; ++m) in[m] = epi.load(b, o2 + m * T2);
#pragma unroll
        for (int m = 0; m < 8; ++m) mx = fmax(mx, epi(b, o2 + m * T2, x[m].x * invN, in[m]));
    }
    block_max_to(mx, epi.res);
    if (tid == 0) end_iteration(end);
}

// ---- spectral steps -------------------------------------------------------
// M1 is a tensor product on each component, so its inverse is one circulant
// convolution along x2 and one along x1, with the first rows of the 1D inverses.
// Those decay geometrically (down to 1e-18 in 101 entries for the quadratic mass matrix,
// 135 for the cubic, 205 for the quintic) and wrap around a grid that is shorter.
// A thread forms 8 neighbouring outputs from a sliding window: 64 FMAs per 8 LDS
// reads, the weights in scalar registers.
struct ConvTaps {           // one direction, per component
    const double *rt[2];    // the row's entries in reverse, zeros on both sides
    int nt[2], hi[2];       // entries; offset of the first one
};

__host__ __device__ constexpr int conv_steps(int nt) { return (nt + 14) & ~7; }

// acc[j] = sum_q rt[q] x(q + j), q = 0 .. nt - 1, j < 8: output 8 t + j of the
// convolution when x(s) is the input at 8 t - hi + s.
template <class X>
__device__ __forceinline__ void conv8(double (&acc)[8], const double *__restrict__ rt, int nt, X x) {
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0.0;
    for (int s0 = 0; s0 < conv_steps(nt); s0 += 8) {
        double v[8], w[15];
#pragma unroll
        for (int r = 0; r < 8; ++r) v[r] = x(s0 + r);
#pragma unroll
        for (int k = 0; k < 15; ++k) w[k] = rt[s0 - 7 + k];
#pragma unroll
        for (int r = 0; r < 8; ++r)
#pragma unroll
            for (int j = 0; j < 8; ++j) acc[j] = fma(w[7 + r - j], v[r], acc[j]);
    }
}

// LDS place of position i of a row: consecutive threads are 8 positions apart, the
// padding spreads them over the banks.
__device__ __forceinline__ int conv_pad(int i) { return i + (i >> 3); }

// Along x2: T = (1D inverse) J row by row, M2 / 8 threads each; J is zeroed (the
// accumulators of the next deposit).
__global__ __launch_bounds__(BLOCK) void k2_conv_rows(Ptrs<2> src, double *__restrict__ T, int M1, int M2, ConvTaps tp,
                                                      const int *gate) {
    if (gate && *gate) return;   // uniform over the grid
    __shared__ double lds[9 * BLOCK];
    const int T2 = M2 >> 3, per = BLOCK / T2;
    const int fl = threadIdx.x / T2, t = threadIdx.x - fl * T2;
    const int blocks = (M1 + per - 1) / per, b = blockIdx.x / blocks;   // component
    const int row = (blockIdx.x - b * blocks) * per + fl;
    const bool act = row < M1;
    double *s = (b ? src.p[1] : src.p[0]) + (size_t)row * M2;
    double *x = lds + fl * 9 * T2;
    double in[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) in[m] = act ? s[t + m * T2] : 0.0;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        x[conv_pad(t + m * T2)] = in[m];
        if (act) s[t + m * T2] = 0.0;
    }
    __syncthreads();
    const double *rt = b ? tp.rt[1] : tp.rt[0];
    const int nt = b ? tp.nt[1] : tp.nt[0], first = 8 * t - (b ? tp.hi[1] : tp.hi[0]), mask = M2 - 1;
    double acc[8];
    conv8(acc, rt, nt, [&](int q) { return x[conv_pad((first + q) & mask)]; });
    if (act) {
        double2 *o = reinterpret_cast<double2 *>(T + (size_t)b * M1 * M2 + (size_t)row * M2 + 8 * t);
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = make_double2(acc[2 * j], acc[2 * j + 1]);
    }
}

// Along x1: a block forms TR rows (64, or M1 if it is less) of BLOCK 8 / TR columns,
// its input rows in LDS (lanes of a wave on consecutive columns); entry g of
// component b goes to epi(b, g, v).
template <class Epi>
__global__ __launch_bounds__(BLOCK) void k2_conv_cols(const double *__restrict__ T, int M1, int M2, int TR, ConvTaps tp,
                                                      Epi epi, const int *gate, IterEnd end) {
    if (gate && *gate) return;   // uniform over the grid
    extern __shared__ double conv_lds[];
    const int CB = 8 * BLOCK / TR, cblocks = (M2 + CB - 1) / CB, rblocks = M1 / TR;
    const int b = blockIdx.x / (cblocks * rblocks), q = blockIdx.x - b * cblocks * rblocks;
    const int r0 = (q / cblocks) * TR, c0 = (q % cblocks) * CB;
    const double *rt = b ? tp.rt[1] : tp.rt[0];
    const int nt = b ? tp.nt[1] : tp.nt[0], hi = b ? tp.hi[1] : tp.hi[0];
    const int H = TR - 8 + conv_steps(nt);   // input rows r0 - hi .. r0 - hi + H - 1
    const int col = threadIdx.x % CB, t = threadIdx.x / CB;
    const bool act = c0 + col < M2;
    const double *src = T + (size_t)b * M1 * M2 + min(c0 + col, M2 - 1);
    const int step = BLOCK / CB;
    for (int h0 = t; h0 < H; h0 += 8 * step) {   // 8 loads in flight
        double v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = src[(size_t)((r0 - hi + min(h0 + k * step, H - 1)) & (M1 - 1)) * M2];
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (h0 + k * step < H) conv_lds[(h0 + k * step) * CB + col] = v[k];
    }
    __syncthreads();
    double acc[8];
    typename Epi::In in[8];   // in flight during the sums
    const int g0 = (r0 + 8 * t) * M2 + min(c0 + col, M2 - 1);
#pragma unroll
    for (int j = 0; j < 8; ++j) in[j] = epi.load(b, g0 + j * M2);
    const double *x = conv_lds + 8 * t * CB + col;
    conv8(acc, rt, nt, [&](int s) { return x[s * CB]; });
    double mx = 0.0;
    if (act) {
#pragma unroll
        for (int j = 0; j < 8; ++j) mx = fmax(mx, epi(b, g0 + j * M2, acc[j], in[j]));
    }
    block_max_to(mx, epi.res);
    if (threadIdx.x == 0) end_iteration(end);
}

// Both directions in one block per component, for grids of at most CONV_SMALL nodes
// (two FFT solves took 15.7 us at 16 x 16 nodes, this takes 8.6; 64 x 64 in 18 us, the
// two kernels above 23 us at 128 x 128; 512 x 512: 34 us, by FFTs 48).
constexpr int CONV_SMALL = 4096;

template <class Epi>
__global__ __launch_bounds__(CONV_SMALL / 8) void k2_conv_small(Ptrs<2> src, int M1, int M2, ConvTaps rows,
                                                                ConvTaps cols, Epi epi, const int *gate, IterEnd end) {
    if (gate && *gate) return;   // uniform over the grid
    __shared__ double lds[CONV_SMALL / 8 * 9];
    const int N = M1 * M2, b = blockIdx.x, tid = threadIdx.x;
    const bool act = tid < N / 8;   // a block has at least one wave
    double *s = b ? src.p[1] : src.p[0];
    double acc[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) acc[m] = act ? s[tid + m * (N / 8)] : 0.0;
    if (act) {
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            lds[conv_pad(tid + m * (N / 8))] = acc[m];
            s[tid + m * (N / 8)] = 0.0;
        }
    }
    __syncthreads();
    {
        const int T2 = M2 >> 3, row = tid / T2, t = tid - row * T2;
        const double *x = lds + (act ? 9 * T2 * row : 0);
        const int first = 8 * t - (b ? rows.hi[1] : rows.hi[0]), mask = M2 - 1;
        conv8(acc, b ? rows.rt[1] : rows.rt[0], b ? rows.nt[1] : rows.nt[0],
              [&](int q) { return x[conv_pad((first + q) & mask)]; });
    }
    __syncthreads();   // every input is read
    if (act) {
#pragma unroll
        for (int j = 0; j < 8; ++j) lds[conv_pad(8 * tid + j)] = acc[j];
    }
    __syncthreads();
    const int t = tid / M2, col = tid - t * M2;
    {
        const int first = 8 * t - (b ? cols.hi[1] : cols.hi[0]), mask = M1 - 1;
        conv8(acc, b ? cols.rt[1] : cols.rt[0], b ? cols.nt[1] : cols.nt[0],
              [&](int q) { return lds[conv_pad(((first + q) & mask) * M2 + col)]; });
    }
    double mx = 0.0;
    if (act) {
        typename Epi::In in[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) in[j] = epi.load(b, (8 * t + j) * M2 + col);
#pragma unroll
        for (int j = 0; j < 8; ++j) mx = fmax(mx, epi(b, (8 * t + j) * M2 + col, acc[j], in[j]));
    }
    block_max_to(mx, epi.res);
    if (tid == 0) end_iteration(end);
}

// e^{(k+1)} = e^n - M1^{-1} J; residual |e^{(k+1)} - e^{(k)}|; ebar = (e^n + e^{(k+1)})/2.
// An epilogue's In holds the values it reads at an entry.
struct EpiI {
    const double *en1, *en2;
    double *ek1, *ek2, *eb1, *eb2;
    unsigned long long *res;
    struct In {
        double en, ek;
    };
    __device__ In load(int b, int g) const { return b ? In{en2[g], ek2[g]} : In{en1[g], ek1[g]}; }
    __device__ double operator()(int b, int g, double v, const In &in) const {
        double *ek = b ? ek2 : ek1;
        double *eb = b ? eb2 : eb1;
        const double e = in.en - v;
        const double d = fabs(e - in.ek);
        ek[g] = e;
        eb[g] = 0.5 * (in.en + e);
        return isfinite(d) ? d : HUGE_VAL;   // a non-finite field shows in the residual
    }
};

__device__ __forceinline__ double kappa(const Sym &s, int k1, int k2) {   // symbol of K = G^T M1 G
    const double c1 = s.cra[k1] * s.cra[k1] + s.cia[k1] * s.cia[k1];
    const double c2 = s.crb[k2] * s.crb[k2] + s.cib[k2] * s.cib[k2];
    return c1 * s.m1a[k1] * s.m0b[k2] + c2 * s.m0a[k1] * s.m1b[k2];
}

// Subsystem III constant part: R = (M0 - q K) e^n + dt K a^n (q = dt^2/4), kept in Fourier space.
struct OpIIIrhs {
    static constexpr bool INVERSE = false;
    Sym s;
    double2 *R;
    int M2;
    double dt;
    __device__ void operator()(int k1, int k2, double2 (&v)[2]) const {
        const double kp = kappa(s, k1, k2), m0 = s.m0a[k1] * s.m0b[k2];
        const double ce = m0 - 0.25 * dt * dt * kp, ca = dt * kp;
        R[(size_t)k1 * M2 + k2] = make_double2(ce * v[0].x + ca * v[1].x, ce * v[0].y + ca * v[1].y);
    }
};

// With spin (v[2] = G*^T Lambda1*^T W S_xy): R gains dt hbar v[2].
struct OpIIIrhsS {
    static constexpr bool INVERSE = false;
    Sym s;
    double2 *R;
    int M2;
    double dt, hbar;
    __device__ void operator()(int k1, int k2, double2 (&v)[3]) const {
        const double kp = kappa(s, k1, k2), m0 = s.m0a[k1] * s.m0b[k2];
        const double ce = m0 - 0.25 * dt * dt * kp, ca = dt * kp, cs = dt * hbar;
        R[(size_t)k1 * M2 + k2] = make_double2(ce * v[0].x + ca * v[1].x + cs * v[2].x,
                                               ce * v[0].y + ca * v[1].y + cs * v[2].y);
    }
};

// Subsystem III solve: e = (R + dt S) / (M0 + q K).
struct OpIII {
    static constexpr bool INVERSE = true;
    Sym s;
    const double2 *R;
    int M2;
    double dt;
    __device__ double2 one(int, int k1, int k2, double2 v) const {
        const double lam = s.m0a[k1] * s.m0b[k2] + 0.25 * dt * dt * kappa(s, k1, k2);
        const double2 r = R[(size_t)k1 * M2 + k2];
        return make_double2((r.x + dt * v.x) / lam, (r.y + dt * v.y) / lam);
    }
    __device__ void operator()(int k1, int k2, double2 (&v)[1]) const { v[0] = one(0, k1, k2, v[0]); }
};

struct EpiIII {
    double *ezk;
    unsigned long long *res;
    struct In {
        double ek;
    };
    __device__ In load(int, int g) const { return In{ezk[g]}; }
    __device__ double operator()(int, int g, double v, const In &in) const {
        const double d = fabs(v - in.ek);
        ezk[g] = v;
        return isfinite(d) ? d : HUGE_VAL;   // a non-finite field shows in the residual
    }
};

// Subsystem IV in Fourier space (v = e1, e2, b): with c_k = (1 - exp(-i t_k))/dx_k and
// sigma = |c1|^2 m1a/m0a + |c2|^2 m1b/m0b the symbol of C M1^{-1} C^T M2,
//   b' = ((1 - q sigma) b - dt (c1 e2 - c2 e1)) / (1 + q sigma),
//   e1' = e1 - dt conj(c2) (m1b/m0b) (b + b')/2,  e2' = e2 + dt conj(c1) (m1a/m0a) (b + b')/2,
// the implicit midpoint step of the Maxwell subsystem eliminated for b.
// One Fourier mode of the Maxwell step (e1, e2, b in place).
__device__ __forceinline__ void maxwell_mode(const Sym &s, double dt, int k1, int k2, double2 &e1, double2 &e2,
                                             double2 &b) {
    const double2 c1 = make_double2(s.cra[k1], s.cia[k1]), c2 = make_double2(s.crb[k2], s.cib[k2]);
    const double ra = s.m1a[k1] / s.m0a[k1], rb = s.m1b[k2] / s.m0b[k2];
    const double sig = (c1.x * c1.x + c1.y * c1.y) * ra + (c2.x * c2.x + c2.y * c2.y) * rb;
    const double q = 0.25 * dt * dt;
    const double2 t1 = cmul(c1, e2), t2 = cmul(c2, e1);
    const double2 ce = make_double2(t1.x - t2.x, t1.y - t2.y);
    const double den = 1.0 / (1.0 + q * sig), num = 1.0 - q * sig;
    const double2 bn = make_double2((num * b.x - dt * ce.x) * den, (num * b.y - dt * ce.y) * den);
    const double2 bm = make_double2(0.5 * (b.x + bn.x), 0.5 * (b.y + bn.y));
    const double2 u1 = cmul(make_double2(c2.x, -c2.y), bm), u2 = cmul(make_double2(c1.x, -c1.y), bm);
    e1 = make_double2(e1.x - dt * rb * u1.x, e1.y - dt * rb * u1.y);
    e2 = make_double2(e2.x + dt * ra * u2.x, e2.y + dt * ra * u2.y);
    b = bn;
}

struct OpIV {
    static constexpr bool INVERSE = true;
    Sym s;
    double dt;
    __device__ void operator()(int k1, int k2, double2 (&v)[3]) const { maxwell_mode(s, dt, k1, k2, v[0], v[1], v[2]); }
};

// With spin the b_z equation carries hbar Lambda2^T W S_z (v[3], constant): with
// b~ = b + hbar M2^{-1} D_z the scheme is the one without spin, so b~ is stepped
// and the shift taken off again.
struct OpIVs {
    static constexpr bool INVERSE = true;
    Sym s;
    double dt, hbar;
    __device__ void operator()(int k1, int k2, double2 (&v)[4]) const {
        const double sh = hbar / (s.m1a[k1] * s.m1b[k2]);
        double2 b = make_double2(v[2].x + sh * v[3].x, v[2].y + sh * v[3].y);
        maxwell_mode(s, dt, k1, k2, v[0], v[1], b);
        v[2] = make_double2(b.x - sh * v[3].x, b.y - sh * v[3].y);
    }
};

// Gauss-law correction (v = e1, e2, rho): r = G^T M1 e + rho (the constant part
// lives in the mean, which phi does not see), phi = r / kappa, e -= G phi.
struct OpPoisson {
    static constexpr bool INVERSE = true;
    Sym s;
    __device__ void operator()(int k1, int k2, double2 (&v)[3]) const {
        if (k1 == 0 && k2 == 0) return;
        const double2 c1 = make_double2(s.cra[k1], s.cia[k1]), c2 = make_double2(s.crb[k2], s.cib[k2]);
        const double w1 = s.m1a[k1] * s.m0b[k2], w2 = s.m0a[k1] * s.m1b[k2];
        const double2 a = cmul(make_double2(c1.x, -c1.y), v[0]), b = cmul(make_double2(c2.x, -c2.y), v[1]);
        const double kp = kappa(s, k1, k2);
        const double2 phi = make_double2((w1 * a.x + w2 * b.x + v[2].x) / kp, (w1 * a.y + w2 * b.y + v[2].y) / kp);
        const double2 g1 = cmul(c1, phi), g2 = cmul(c2, phi);
        v[0] = make_double2(v[0].x - g1.x, v[0].y - g1.y);
        v[1] = make_double2(v[1].x - g2.x, v[1].y - g2.y);
    }
};

template <int NB>
struct EpiStore {
    Ptrs<NB> out;
    unsigned long long *res;
    struct In {};
    __device__ In load(int, int) const { return In{}; }
    __device__ double operator()(int b, int g, double v, const In &) const {
#pragma unroll
        for (int q = 0; q < NB; ++q)
            if (b == q && out.p[q]) out.p[q][g] = v;
        return 0.0;
    }
};

}  // namespace ecpic2d

// ===========================================================================
// Host side
// ===========================================================================
using namespace ecpic2d;

namespace {

int64_t eulerian2(int n, int k) {   // A(n, k) = sum_j (-1)^j C(n+1, j) (k+1-j)^n
    int64_t s = 0;
    for (int j = 0; j <= k; ++j) {
        int64_t b = 1;
        for (int q = 1; q <= j; ++q) b = b * (n + 1 - j + q) / q;
        int64_t pw = 1;
        for (int q = 0; q < n; ++q) pw *= (k + 1 - j);
        s += (j % 2 == 0) ? b * pw : -b * pw;
    }
    return s;
}

// Row of the degree-d B-spline mass matrix with dx = 1: the cardinal B-spline of
// degree 2d+1 at the integers, A(2d+1, k) / (2d+1)!.
std::vector<double> mass_row2(int d) {
    const int n = 2 * d + 1;
    double f = 1.0;
    for (int q = 2; q <= n; ++q) f *= q;
    std::vector<double> r(n);
    for (int k = 0; k < n; ++k) r[k] = (double)eulerian2(n, k) / f;
    return r;
}

struct Prof2 {
    bool on = false;
    std::map<std::string, std::pair<double, int64_t>> acc;
    std::vector<std::pair<std::string, std::pair<hipEvent_t, hipEvent_t>>> pending;
};

constexpr int RED_BLOCKS = 1024;

}  // namespace

struct ecpic2d_ctx {
    ecpic2d_config cfg{};
    int P = 3, M1 = 0, M2 = 0, Nc = 0, TW = 16, kmax = 50, device = 0;
    int64_t N = 0;
    double dx1 = 0, dx2 = 0, w = 0, tol = 0;
    hipStream_t stream = nullptr;
    int cur = 0;
    double *xi1[2] = {}, *xi2[2] = {}, *p1[2] = {}, *p2[2] = {};
    int32_t *id[2] = {};
    double *d1[2] = {}, *d2[2] = {}, *pk1 = nullptr, *pk2 = nullptr;
    double *azn = nullptr, *gamn = nullptr;   // A_z(x^n), gamma^n during Subsystem I (sweep order)
    int32_t *cell = nullptr /* new cell (set_particles) or packed new tile and column (commit) */, *count = nullptr,
            *start = nullptr, *bsum = nullptr;
    int32_t *mig = nullptr;   // arrivals per new tile, after the stayers' slots
    int32_t *tstart[2] = {}, *tstay = nullptr, *tarr = nullptr;
    int ts = 0, ntiles = 0;   // tstart[ts]: first particle of each tile
    double *e1 = nullptr, *e2 = nullptr, *bz = nullptr, *ez = nullptr, *az = nullptr;
    double *ek1 = nullptr, *ek2 = nullptr, *eb1[2] = {}, *eb2[2] = {};   // iterate; mean field by parity
    double *J1 = nullptr, *J2 = nullptr, *g1a = nullptr, *g2a = nullptr, *ezn = nullptr, *ezk = nullptr,
           *S = nullptr, *tmp = nullptr;
    double2 *Z = nullptr, *R = nullptr, *tw1 = nullptr, *tw2 = nullptr;
    ConvTaps conv_a{}, conv_b{};  // M1^{-1} along x1 and x2
    double *sym = nullptr;        // m0a m1a cra cia (M1 each) m0b m1b crb cib (M2 each)
    double *partial = nullptr;    // RED_BLOCKS + 8
    unsigned long long *res = nullptr;   // 3 * MAXK + 4 slots
    int *flags = nullptr;
    int *gate = nullptr;                 // [0] set once an iteration has converged (or failed), [1] never
    int spin = 0;                        // particles carry spins (hbar terms on)
    double hbar = 0.0;
    double *sx[2] = {}, *sy[2] = {}, *sz[2] = {};   // spins, in the particle buffers' order
    double *Dx = nullptr, *Dy = nullptr, *Dz = nullptr, *ssrc = nullptr;   // spin deposits and G*^T source
    double *hres = nullptr, *hres_dev = nullptr;   // pinned mirror: a word per iteration (I, then III)
    unsigned *done = nullptr;            // blocks finished of the solve that ends an iteration
    int keep_from = 0, last_k = 0;       // first sweep that stores its momentum; last sweep of the last substep
    bool have_particles = false;
    std::vector<double> m0row, m1row;
    ecpic::HostCopy host_copy;   // large arrays to the caller's memory
    double *hfields = nullptr, *hfields_dev = nullptr;   // behind it: the five fields read out (grids up to FIELDS_NODES)
    Prof2 prof;
    std::vector<void *> allocs;
};

namespace {

template <typename T>
int dalloc(ecpic2d_ctx *c, T **p, size_t n) {
    *p = nullptr;
    if (n == 0) n = 1;
    if (hipMalloc((void **)p, n * sizeof(T)) != hipSuccess) { *p = nullptr; return ECPIC_ENOMEM; }
    c->allocs.push_back((void *)*p);
    return ECPIC_OK;
}

int sync2(ecpic2d_ctx *c) {
    if (hipStreamSynchronize(c->stream) != hipSuccess) return ECPIC_EDEVICE;
    if (c->prof.on) {
        for (auto &pe : c->prof.pending) {
            float ms = 0.f;
            hipEventElapsedTime(&ms, pe.second.first, pe.second.second);
            auto &a = c->prof.acc[pe.first];
            a.first += ms;
            a.second += 1;
            hipEventDestroy(pe.second.first);
            hipEventDestroy(pe.second.second);
        }
        c->prof.pending.clear();
    }
    return hipGetLastError() == hipSuccess ? ECPIC_OK : ECPIC_EDEVICE;
}

// Launch with HIP events around it when profiling.
template <class F>
void timed(ecpic2d_ctx *c, const char *name, F launch) {
    if (!c->prof.on) { launch(); return; }
    hipEvent_t a, b;
    hipEventCreate(&a);
    hipEventCreate(&b);
    hipEventRecord(a, c->stream);
    launch();
    hipEventRecord(b, c->stream);
    c->prof.pending.push_back({name, {a, b}});
}

int grid_for(int64_t n) {
    int64_t g = (n + BLOCK - 1) / BLOCK;
    return (int)std::max<int64_t>(1, std::min<int64_t>(g, 8192));
}

Sym sym_of(ecpic2d_ctx *c) {
    const double *s = c->sym;
    const int M1 = c->M1, M2 = c->M2;
    return Sym{s, s + M1, s + 2 * M1, s + 3 * M1, s + 4 * M1, s + 4 * M1 + M2, s + 4 * M1 + 2 * M2,
               s + 4 * M1 + 3 * M2};
}

int n_tiles(ecpic2d_ctx *c) { return c->M1 * (c->M2 / c->TW); }

// Blocks per tile of the particle passes: enough that the launch has 512 blocks, the
// number that the sweeps of high degree or with spin keep resident (two a CU), as long
// as every wave keeps a row of 64 particles on average.  Each block stages its own
// patch, finishes its own crossing particles and adds its own deposits to the grid, so a
// second round of blocks costs: 128 tiles (128 x 64 cells, 5e5 quintic particles) sweep
// 71 us with 2 blocks a tile, 66 with 4, 81 with 8; 256 tiles (64 x 256, 3.6e5 quintic
// with spin) 75 us with 1, 67 with 2, 101 with 4, cubic without spin 25.2, 24.9 and 36;
// 1024 tiles (256 x 256, 2^22 with spin) 180 us with one block, 194 with two.
int blocks_per_tile(ecpic2d_ctx *c) {
    const int64_t nt = n_tiles(c), rows = c->N / nt / BLOCK;   // rows of a tile per wave of one block
    return (int)std::max<int64_t>(1, std::min<int64_t>(512 / nt, rows));
}

// Full cell sort (set_particles): counts in c->count, cells in c->cell; each tile
// is stored transposed (tile_pos), and the tile starts are taken from the cell starts.
void sort_particles(ecpic2d_ctx *c) {
    const int A = c->cur, B = 1 - c->cur;
    timed(c, "sort", [&] {
        const int nb = (c->Nc + SCAN_TILE - 1) / SCAN_TILE;
        k2_scan_sums<<<nb, SCAN_THREADS, 0, c->stream>>>(c->count, c->bsum, c->Nc);
        k2_scan_top<<<1, SCAN_THREADS, 0, c->stream>>>(c->bsum, nb, c->start + c->Nc);
        k2_scan_apply<<<nb, SCAN_THREADS, 0, c->stream>>>(c->count, c->start, c->bsum, c->Nc);
        k2_scatter<<<grid_for(c->N), BLOCK, 0, c->stream>>>(c->xi1[A], c->xi2[A], c->p1[A], c->p2[A], c->id[A],
                                                           c->xi1[B], c->xi2[B], c->p1[B], c->p2[B], c->id[B],
                                                           c->cell, c->start, c->count, c->N, c->M2, c->TW);
        k2_fill_i32<<<grid_for(c->Nc), BLOCK, 0, c->stream>>>(c->count, c->Nc);
        k2_tiles_from_cells<<<grid_for(c->ntiles + 1), BLOCK, 0, c->stream>>>(
            c->start, c->tstart[c->ts], c->ntiles, c->M2 / c->TW, c->M2, c->TW, c->Nc);
    });
    c->cur = B;
}

// The commit's list of leavers takes the increment buffer that is not committed.
int2 *leavers_of(ecpic2d_ctx *c, int di) { return reinterpret_cast<int2 *>(c->d1[1 - di]); }

// Re-sort after the first half of a Subsystem I commit (places in c->cell, stay and arrival counts per tile; increment in buffer di):
// new tile starts, the arrival lists, then each new tile formed and sorted by
// cell into the transposed layout in the other particle buffer.
void sort_tiles(ecpic2d_ctx *c, int di) {
    const int A = c->cur, B = 1 - c->cur, T0 = c->ts, T1 = 1 - c->ts;
    timed(c, "sort", [&] {
        const int nt = c->ntiles;
        k2_scan_tiles<<<1, SCAN_THREADS, 0, c->stream>>>(c->tstay, c->tarr, c->tstart[T1], nt);
        k2_list_arrivals<<<nt, WAVE, 0, c->stream>>>(c->cell, leavers_of(c, di), c->tstart[T0], c->tstart[T1],
                                                    c->tstay, c->mig);
        const Resort r{c->xi1[A], c->xi2[A], c->d1[di], c->d2[di], c->pk1, c->pk2, c->id[A], c->cell, c->mig,
                       c->tstart[T0], c->tstart[T1], c->tstay, c->xi1[B], c->xi2[B], c->p1[B], c->p2[B], c->id[B],
                       c->M1, c->M2, 1.0 / c->dx1, 1.0 / c->dx2, {c->sx[A], c->sy[A], c->sz[A]},
                       {c->sx[B], c->sy[B], c->sz[B]}};
        k2_tile_resort<<<nt, SORT_THREADS, 0, c->stream>>>(r);
    });
    c->cur = B;
    c->ts = T1;
}

// Forward rows -> columns with op -> inverse rows with epi, over NB grids; with
// `end` the solve ends an iteration.
template <int NB, class Op, class Epi>
void spectral(ecpic2d_ctx *c, const char *name, Ptrs<NB> src, int zero_mask, Op op, Epi epi,
              const int *gate = nullptr, IterEnd end = {}) {
    timed(c, name, [&] {
        // transforms per block: BLOCK / (n / 8) for n points
        const int rows = NB * c->M1, per_row = BLOCK / (c->M2 / 8), per_col = BLOCK / (c->M1 / 8);
        const int grow = (rows + per_row - 1) / per_row, gcol = (c->M2 + per_col - 1) / per_col;
        k2_fft_rows_fwd<NB><<<grow, BLOCK, 0, c->stream>>>(src, zero_mask, c->Z, c->M1, c->M2, c->tw2, gate);
        k2_fft_cols<NB, Op><<<gcol, BLOCK, 0, c->stream>>>(c->Z, c->M1, c->M2, c->tw1, op, gate);
        if (Op::INVERSE)
            k2_fft_rows_inv<NB, Epi><<<grow, BLOCK, 0, c->stream>>>(c->Z, c->M1, c->M2, c->tw2, 1.0 / (double)c->Nc,
                                                                  epi, gate, end);
    });
}

// The Subsystem III solve that ends an iteration (S is zeroed after it is read): one
// block where the grid fits, else the three kernels.
template <class Op, class Epi>
void solve_iteration(ecpic2d_ctx *c, const char *name, double *S, Op op, Epi epi, IterEnd end) {
    if (c->Nc > SMALL_SOLVE) {
        spectral<1>(c, name, Ptrs<1>{{S}}, 1, op, epi, c->gate, end);
        return;
    }
    timed(c, name, [&] {
        k2_solve_small<1, Op, Epi><<<1, std::max(WAVE, c->Nc / 8), small_solve_lds(c->M1, c->M2), c->stream>>>(
            Ptrs<1>{{S}}, c->M1, c->M2, c->tw1, c->tw2, 1.0 / (double)c->Nc, op, epi, c->gate, end);
    });
}

// M1^{-1} of the current with epi: the convolutions in one kernel where the grid fits,
// else one per direction.
template <class Epi>
void solve_M1(ecpic2d_ctx *c, const char *name, Epi epi, IterEnd end) {
    const Ptrs<2> J{{c->J1, c->J2}};
    timed(c, name, [&] {
        if (c->Nc <= CONV_SMALL) {
            k2_conv_small<Epi><<<2, std::max(WAVE, c->Nc / 8), 0, c->stream>>>(J, c->M1, c->M2, c->conv_b, c->conv_a, epi,
                                                                            c->gate, end);
            return;
        }
        const int per = BLOCK / (c->M2 / 8), TR = std::min(64, c->M1), CB = 8 * BLOCK / TR;
        double *T = reinterpret_cast<double *>(c->Z);
        k2_conv_rows<<<2 * ((c->M1 + per - 1) / per), BLOCK, 0, c->stream>>>(J, T, c->M1, c->M2, c->conv_b, c->gate);
        const int nt = std::max(c->conv_a.nt[0], c->conv_a.nt[1]);
        const size_t lds = sizeof(double) * (size_t)CB * (TR - 8 + conv_steps(nt));
        k2_conv_cols<Epi><<<2 * (c->M1 / TR) * ((c->M2 + CB - 1) / CB), BLOCK, lds, c->stream>>>(
            T, c->M1, c->M2, TR, c->conv_a, epi, c->gate, end);
    });
}

// Wait until the iteration with the mirror word h is done: the last block of its
// solve writes it (it is set to MIRROR_WAIT when the iteration is queued).  Ends
// also if the stream runs dry or fails without it.  r gets the residual.
constexpr double MIRROR_WAIT = -1.0;

int wait_mirror(ecpic2d_ctx *c, const double *h, double &r) {
    const volatile double *flag = h;
    for (unsigned n = 1;; ++n) {
        if (*flag != MIRROR_WAIT) break;
        // Other threads (of other contexts or ranks) get the processor while this one waits,
        // and the polls leave the link to the GPU's write: a step of 16 x 16 cells 380 us
        // without the pause and the yield, 338 with them; two contexts on one processor
        // 764 and 354.
        if (n % 32 == 0) std::this_thread::yield();
        else __builtin_ia32_pause();
        if (n % 4096 == 0) {
            // an error that a launch has left for the end of the call is not queried over
            const hipError_t left = hipPeekAtLastError();
            const bool query = left == hipSuccess || left == hipErrorNotReady;
            const hipError_t e = query ? hipStreamQuery(c->stream) : hipStreamSynchronize(c->stream);
            if (hipPeekAtLastError() == hipErrorNotReady) (void)hipGetLastError();   // no error
            if (e == hipErrorNotReady) continue;
            if (e != hipSuccess || *flag == MIRROR_WAIT) return ECPIC_EDEVICE;
        }
    }
    r = *flag;
    if (r < 0.0) {
        const int f = (int)(-2.0 - r);
        return (f & FLAG_NONFINITE) ? ECPIC_ENONFINITE : ECPIC_ECFL;
    }
    return std::isfinite(r) ? ECPIC_OK : ECPIC_ENONFINITE;
}

int flags_status(ecpic2d_ctx *c) {
    int f = 0;
    if (hipMemcpyAsync(&f, c->flags, sizeof(int), hipMemcpyDeviceToHost, c->stream) != hipSuccess) return ECPIC_EDEVICE;
    int rc = sync2(c);
    if (rc) return rc;
    if (f & FLAG_NONFINITE) return ECPIC_ENONFINITE;
    if (f & FLAG_CFL) return ECPIC_ECFL;
    return ECPIC_OK;
}

double read_res(ecpic2d_ctx *c, int slot, int *rc) {
    unsigned long long b = 0;
    if (hipMemcpyAsync(&b, c->res + slot, sizeof(b), hipMemcpyDeviceToHost, c->stream) != hipSuccess) {
        *rc = ECPIC_EDEVICE;
        return 0.0;
    }
    *rc = sync2(c);
    double v;
    std::memcpy(&v, &b, sizeof(v));
    return v;
}

#define LAUNCH_P(P, ...)                                      \
    switch (P) {                                              \
        case 2: { constexpr int PP = 2; __VA_ARGS__; } break; \
        case 3: { constexpr int PP = 3; __VA_ARGS__; } break; \
        case 4: { constexpr int PP = 4; __VA_ARGS__; } break; \
        case 5: { constexpr int PP = 5; __VA_ARGS__; } break; \
    }

int substep_I(ecpic2d_ctx *c, double dt, ecpic2d_iter_stats *st) {
    const int A = c->cur, Nc = c->Nc;
    hipStream_t s = c->stream;
    k2_begin_I<<<grid_for(Nc), BLOCK, 0, s>>>(BeginI{c->az, c->e1, c->e2, c->g1a, c->g2a, c->ek1, c->ek2, c->eb1[0],
                                                     c->eb2[0], c->J1, c->J2, c->res, 2 * MAXK, c->flags, c->gate,
                                                     c->M1, c->M2, 1.0 / c->dx1, 1.0 / c->dx2});
    const int split = blocks_per_tile(c);
    // Sweep k reads d^(k) and the mean field from buffers k & 1 and writes d^(k+1)
    // to the other.
    auto sweep = [&](int k, bool keep_p, const int *gate) {
        const int di = k & 1;
        SweepArgs a{c->xi1[A], c->xi2[A], c->p1[A], c->p2[A], c->d1[di], c->d2[di], c->d1[1 - di], c->d2[1 - di],
                    c->pk1, c->pk2, c->tstart[c->ts], c->eb1[di], c->eb2[di], c->az, c->g1a, c->g2a, c->J1, c->J2,
                    c->res + k, c->flags, gate, c->M1, c->M2, c->TW, 1.0 / c->dx1, 1.0 / c->dx2, dt, c->w,
                    c->sx[A], c->sy[A], c->sz[A], c->bz, c->hbar, c->azn, c->gamn, keep_p ? 1 : 0, split};
        timed(c, "sweep_I", [&] {
            if (c->spin) {
                if (k == 0) {
                    LAUNCH_P(c->P, k2_sweep_I<PP, true, true><<<n_tiles(c) * split, BLOCK, 0, s>>>(a));
                } else {
                    LAUNCH_P(c->P, k2_sweep_I<PP, false, true><<<n_tiles(c) * split, BLOCK, 0, s>>>(a));
                }
            } else if (k == 0) {
                LAUNCH_P(c->P, k2_sweep_I<PP, true, false><<<n_tiles(c) * split, BLOCK, 0, s>>>(a));
            } else {
                LAUNCH_P(c->P, k2_sweep_I<PP, false, false><<<n_tiles(c) * split, BLOCK, 0, s>>>(a));
            }
        });
    };
    // Only the committed sweep's momentum is wanted, so sweeps store theirs from the
    // index on at which the last two substeps ended (16 of a sweep's 96 B per
    // particle); a substep that ends earlier repeats its last sweep with the store.
    auto iterate = [&](int k) {
        const int di = k & 1;
        c->hres[k] = MIRROR_WAIT;
        sweep(k, k >= c->keep_from, c->gate);
        solve_M1(c, "solve_I",
                 EpiI{c->e1, c->e2, c->ek1, c->ek2, c->eb1[1 - di], c->eb2[1 - di], c->res + MAXK + k},
                 IterEnd{c->res + k, c->res + MAXK + k, c->flags, c->tol, c->gate, c->hres_dev + k, c->done});
    };
    // Iteration k + 1 is queued before iteration k is read back, so the GPU
    // does not wait for the host; it does nothing if iteration k closed the gate.
    // With kernel timing on, iterations are queued one at a time (every timed
    // launch does its work).
    const bool ahead = !c->prof.on;
    double r = 0.0;
    int k, rc = ECPIC_OK;
    iterate(0);
    for (k = 0; k < c->kmax; ++k) {
        if (ahead && k + 1 < c->kmax) iterate(k + 1);
        rc = wait_mirror(c, c->hres + k, r);
        if (rc) break;
        if (r <= c->tol) break;
        if (!ahead && k + 1 < c->kmax) iterate(k + 1);
    }
    if (rc) {
        sync2(c);
        return rc;
    }
    const int di = k & 1;
    if (st) { st->sweeps = std::min(k + 1, c->kmax); st->residual = r; st->reserved = 0; }
    if (k == c->kmax) return ECPIC_ENOTCONV;
    if (k < c->keep_from) sweep(k, true, c->gate + 1);   // a gate that never closes
    c->keep_from = std::min(k, c->last_k);
    c->last_k = k;
    // commit x^n + d^(k) (buffer di), p^(k+1), e^(k+1): places and counts, the
    // fields, then the re-sort writes the particles in their new order
    timed(c, "commit_I", [&] {
        k2_commit_tiles<<<c->ntiles, BLOCK, 0, s>>>(c->xi1[A], c->xi2[A], c->d1[di], c->d2[di], c->cell,
                                                    leavers_of(c, di), c->tstart[c->ts], c->tstay, c->tarr, c->M1,
                                                    c->M2, c->TW, 1.0 / c->dx1, 1.0 / c->dx2);
    });
    std::swap(c->e1, c->ek1);
    std::swap(c->e2, c->ek2);
    sort_tiles(c, di);
    return hipGetLastError() == hipSuccess ? ECPIC_OK : ECPIC_EDEVICE;
}

int substep_II(ecpic2d_ctx *c, double dt) {
    const int A = c->cur;
    if (c->spin)
        k2_grad<<<grid_for(c->Nc), BLOCK, 0, c->stream>>>(c->az, c->g1a, c->g2a, c->M1, c->M2, 1.0 / c->dx1,
                                                          1.0 / c->dx2);
    const RotArgs a{c->xi1[A], c->xi2[A], c->p1[A], c->p2[A], c->sx[A], c->sy[A], c->sz[A], c->tstart[c->ts],
                    c->bz, c->az, c->g1a, c->g2a, c->M1, c->M2, c->TW, dt, blocks_per_tile(c)};
    timed(c, "rotate_II", [&] {
        if (c->spin) {
            LAUNCH_P(c->P, k2_rotate_tiles<PP, true><<<n_tiles(c) * a.split, BLOCK, 0, c->stream>>>(a));
        } else {
            LAUNCH_P(c->P, k2_rotate_tiles<PP, false><<<n_tiles(c) * a.split, BLOCK, 0, c->stream>>>(a));
        }
    });
    return ECPIC_OK;
}

int substep_III(ecpic2d_ctx *c, double dt, ecpic2d_iter_stats *st) {
    const int A = c->cur, Nc = c->Nc, gC = grid_for(Nc);
    hipStream_t s = c->stream;
    k2_begin_III<<<gC, BLOCK, 0, s>>>(c->ez, c->ezn, c->ezk, c->S, Nc, c->res + 2 * MAXK, MAXK, c->gate);
    const Sym sy = sym_of(c);
    const int split = blocks_per_tile(c);
    // constant part in Fourier space (with spin: plus dt hbar G*^T Lambda1*^T W S_xy)
    if (c->spin) {
        k2_fill<<<gC, BLOCK, 0, s>>>(c->Dx, Nc, 0.0);
        k2_fill<<<gC, BLOCK, 0, s>>>(c->Dy, Nc, 0.0);
        LAUNCH_P(c->P, k2_deposit_spin<PP><<<n_tiles(c) * split, BLOCK, 0, s>>>(c->xi1[A], c->xi2[A], c->sx[A], c->sy[A],
                                                                         c->sz[A], c->tstart[c->ts], c->Dx, c->Dy,
                                                                         nullptr, c->M1, c->M2, c->TW, c->w, 0, split));
        k2_spin_src<<<gC, BLOCK, 0, s>>>(c->Dx, c->Dy, c->ssrc, c->M1, c->M2, 1.0 / c->dx1, 1.0 / c->dx2);
        spectral<3>(c, "solve_III", Ptrs<3>{{c->ezn, c->az, c->ssrc}}, 0, OpIIIrhsS{sy, c->R, c->M2, dt, c->hbar},
                    EpiStore<3>{Ptrs<3>{{nullptr, nullptr, nullptr}}, nullptr});
    } else {
        spectral<2>(c, "solve_III", Ptrs<2>{{c->ezn, c->az}}, 0, OpIIIrhs{sy, c->R, c->M2, dt},
                    EpiStore<2>{Ptrs<2>{{nullptr, nullptr}}, nullptr});
    }
    auto iterate = [&](int k) {   // as in Subsystem I
        DepArgs a{c->xi1[A], c->xi2[A], c->p1[A], c->p2[A], c->tstart[c->ts], c->az, c->ezn, c->ezk, c->S,
                  c->pk1, c->M1, c->M2, c->TW, dt, c->w, 1, k == 0, c->gate, split};
        c->hres[MAXK + k] = MIRROR_WAIT;
        timed(c, "deposit_III", [&] { LAUNCH_P(c->P, k2_deposit0<PP><<<n_tiles(c) * split, BLOCK, 0, s>>>(a)); });
        solve_iteration(c, "solve_III", c->S, OpIII{sy, c->R, c->M2, dt}, EpiIII{c->ezk, c->res + 2 * MAXK + k},
                        IterEnd{c->res + 2 * MAXK + k, nullptr, nullptr, c->tol, c->gate, c->hres_dev + MAXK + k,
                                c->done});
    };
    const bool ahead = !c->prof.on;
    double r = 0.0;
    int k, rc = ECPIC_OK;
    iterate(0);
    for (k = 0; k < c->kmax; ++k) {
        if (ahead && k + 1 < c->kmax) iterate(k + 1);
        rc = wait_mirror(c, c->hres + MAXK + k, r);
        if (rc) break;
        if (r <= c->tol) break;
        if (!ahead && k + 1 < c->kmax) iterate(k + 1);
    }
    if (rc) {
        sync2(c);
        return rc;
    }
    if (st) { st->sweeps = std::min(k + 1, c->kmax); st->residual = r; st->reserved = 0; }
    if (k == c->kmax) return ECPIC_ENOTCONV;
    k2_finish_III<<<gC, BLOCK, 0, s>>>(c->az, c->ez, c->ezn, c->ezk, Nc, dt);
    return ECPIC_OK;
}

int substep_IV(ecpic2d_ctx *c, double dt) {
    if (c->spin) {   // with the constant source hbar C^T Lambda2^T W S_z
        const int A = c->cur;
        k2_fill<<<grid_for(c->Nc), BLOCK, 0, c->stream>>>(c->Dz, c->Nc, 0.0);
        const int split = blocks_per_tile(c);
        LAUNCH_P(c->P, k2_deposit_spin<PP><<<n_tiles(c) * split, BLOCK, 0, c->stream>>>(
                           c->xi1[A], c->xi2[A], c->sx[A], c->sy[A], c->sz[A], c->tstart[c->ts], nullptr, nullptr,
                           c->Dz, c->M1, c->M2, c->TW, c->w, 1, split));
        spectral<4>(c, "maxwell_IV", Ptrs<4>{{c->e1, c->e2, c->bz, c->Dz}}, 0, OpIVs{sym_of(c), dt, c->hbar},
                    EpiStore<4>{Ptrs<4>{{c->e1, c->e2, c->bz, nullptr}}, nullptr});
        return ECPIC_OK;
    }
    spectral<3>(c, "maxwell_IV", Ptrs<3>{{c->e1, c->e2, c->bz}}, 0, OpIV{sym_of(c), dt},
                EpiStore<3>{Ptrs<3>{{c->e1, c->e2, c->bz}}, nullptr});
    return ECPIC_OK;
}

void deposit_rho(ecpic2d_ctx *c, double *rho) {
    const int A = c->cur;
    k2_fill<<<grid_for(c->Nc), BLOCK, 0, c->stream>>>(rho, c->Nc, 0.0);
    DepArgs a{c->xi1[A], c->xi2[A], c->p1[A], c->p2[A], c->tstart[c->ts], nullptr, nullptr, nullptr, rho,
              nullptr, c->M1, c->M2, c->TW, 0.0, c->w, 0, 0, nullptr, blocks_per_tile(c)};
    LAUNCH_P(c->P, k2_deposit0<PP><<<n_tiles(c) * a.split, BLOCK, 0, c->stream>>>(a));
}

MassRows rows_of(ecpic2d_ctx *c, int d1, int d2) {
    MassRows m{};
    const std::vector<double> &a = d1 == c->P ? c->m0row : c->m1row, &b = d2 == c->P ? c->m0row : c->m1row;
    for (size_t i = 0; i < a.size(); ++i) m.r1[i] = a[i];
    for (size_t i = 0; i < b.size(); ++i) m.r2[i] = b[i];
    m.d1 = d1;
    m.d2 = d2;
    m.scale = c->dx1 * c->dx2;
    return m;
}

// x^T Mass x for a grid (result left in partial[RED_BLOCKS + slot]).
void quad(ecpic2d_ctx *c, const double *x, int d1, int d2, int slot) {
    const int gC = std::min(grid_for(c->Nc), RED_BLOCKS);
    k2_mass<<<grid_for(c->Nc), BLOCK, 0, c->stream>>>(x, c->tmp, c->M1, c->M2, rows_of(c, d1, d2));
    k2_dot<<<gC, BLOCK, 0, c->stream>>>(x, c->tmp, c->Nc, c->partial);
    k2_sum<<<1, BLOCK, 0, c->stream>>>(c->partial, gC, c->partial + RED_BLOCKS + slot);
}

}  // namespace

extern "C" {

int ecpic2d_create(const ecpic2d_config *cfg, ecpic2d_ctx **out) {
    if (!cfg || !out) return ECPIC_EINVAL;
    *out = nullptr;
    const ecpic2d_config g = *cfg;
    auto pow2 = [](int m) { return m >= 8 && m <= MAXM && (m & (m - 1)) == 0; };
    const double dx1 = g.L1 / g.M1, dx2 = g.L2 / g.M2;
    if (!(g.L1 > 0) || !(g.L2 > 0) || !pow2(g.M1) || !pow2(g.M2) || g.degree < 2 || g.degree > 5 ||
        g.n_particles < 0 || g.n_particles > INT32_MAX || !(g.picard_tol > 0) || g.picard_max_iter < 0 ||
        g.picard_max_iter > MAXK || !(g.dt > 0) || !(g.dt < std::min(dx1, dx2)) || g.weight < 0 ||
        !std::isfinite(g.weight) || (g.spin != 0 && g.spin != 1) || !std::isfinite(g.hbar) ||
        (!g.spin && g.hbar != 0.0))
        return ECPIC_EINVAL;
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || g.device < 0 || g.device >= ndev) return ECPIC_EDEVICE;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, g.device) != hipSuccess) return ECPIC_EDEVICE;
    if (std::strncmp(prop.gcnArchName, "gfx950", 6) != 0) return ECPIC_EDEVICE;
    if (hipSetDevice(g.device) != hipSuccess) return ECPIC_EDEVICE;
    ecpic2d_ctx *c = new ecpic2d_ctx();
    c->cfg = g;
    c->device = g.device;
    c->P = g.degree;
    c->M1 = g.M1;
    c->M2 = g.M2;
    c->Nc = g.M1 * g.M2;
    c->TW = std::min(TWMAX, g.M2);
    c->kmax = g.picard_max_iter ? g.picard_max_iter : 50;
    c->N = g.n_particles;
    c->dx1 = dx1;
    c->dx2 = dx2;
    c->w = g.weight > 0 ? g.weight : (c->N > 0 ? g.L1 * g.L2 / (double)c->N : 0.0);
    c->tol = g.picard_tol;
    c->spin = g.spin;
    c->hbar = g.hbar;
    c->m0row = mass_row2(c->P);
    c->m1row = mass_row2(c->P - 1);
    if (hipStreamCreate(&c->stream) != hipSuccess) { delete c; return ECPIC_EDEVICE; }
    const size_t N = (size_t)c->N, Nc = (size_t)c->Nc;
    int rc = 0;
    for (int b = 0; b < 2; ++b) {
        rc |= dalloc(c, &c->xi1[b], N) | dalloc(c, &c->xi2[b], N) | dalloc(c, &c->p1[b], N) |
              dalloc(c, &c->p2[b], N) | dalloc(c, &c->id[b], N) | dalloc(c, &c->d1[b], N) |
              dalloc(c, &c->d2[b], N);
    }
    rc |= dalloc(c, &c->pk1, N) | dalloc(c, &c->pk2, N) | dalloc(c, &c->azn, N) | dalloc(c, &c->gamn, N) |
          dalloc(c, &c->cell, N) | dalloc(c, &c->mig, N) |
          dalloc(c, &c->count, Nc) | dalloc(c, &c->start, Nc + 1) | dalloc(c, &c->bsum, Nc / SCAN_TILE + 2);
    c->ntiles = c->M1 * (c->M2 / c->TW);
    rc |= dalloc(c, &c->tstart[0], (size_t)c->ntiles + 1) | dalloc(c, &c->tstart[1], (size_t)c->ntiles + 1) |
          dalloc(c, &c->tstay, (size_t)c->ntiles) | dalloc(c, &c->tarr, (size_t)c->ntiles);
    double **grids[] = {&c->e1, &c->e2, &c->bz, &c->ez, &c->az, &c->ek1, &c->ek2, &c->eb1[0],
                        &c->eb1[1], &c->eb2[0], &c->eb2[1], &c->J1, &c->J2, &c->g1a, &c->g2a, &c->ezn, &c->ezk, &c->S, &c->tmp};
    for (double **gp : grids) rc |= dalloc(c, gp, Nc);
    if (c->spin) {
        for (int b = 0; b < 2; ++b) rc |= dalloc(c, &c->sx[b], N) | dalloc(c, &c->sy[b], N) | dalloc(c, &c->sz[b], N);
        rc |= dalloc(c, &c->Dx, Nc) | dalloc(c, &c->Dy, Nc) | dalloc(c, &c->Dz, Nc) | dalloc(c, &c->ssrc, Nc);
    }
    rc |= dalloc(c, &c->Z, 4 * Nc) | dalloc(c, &c->R, Nc) | dalloc(c, &c->partial, RED_BLOCKS + 16) |
          dalloc(c, &c->res, 3 * MAXK + 4) | dalloc(c, &c->flags, 1) | dalloc(c, &c->gate, 2) |
          dalloc(c, &c->done, 1);
    const size_t pinned = 2 * MAXK + (Nc <= (size_t)FIELDS_NODES ? 5 * Nc : 0);   // the mirror, then the fields
    if (rc || hipHostMalloc((void **)&c->hres, sizeof(double) * pinned, hipHostMallocMapped) != hipSuccess) {
        ecpic2d_destroy(c);
        return ECPIC_ENOMEM;
    }
    if (hipHostGetDevicePointer((void **)&c->hres_dev, c->hres, 0) != hipSuccess) {
        ecpic2d_destroy(c);
        return ECPIC_EDEVICE;
    }
    if (Nc <= (size_t)FIELDS_NODES) {
        c->hfields = c->hres + 2 * MAXK;
        c->hfields_dev = c->hres_dev + 2 * MAXK;
    }
    // twiddles and 1D symbols (host, long double)
    const long double PI = 3.14159265358979323846264338327950288L;
    std::vector<double2> t1(c->M1 / 2), t2(c->M2 / 2);
    for (int j = 0; j < c->M1 / 2; ++j)
        t1[j] = make_double2((double)cosl(2 * PI * j / c->M1), (double)-sinl(2 * PI * j / c->M1));
    for (int j = 0; j < c->M2 / 2; ++j)
        t2[j] = make_double2((double)cosl(2 * PI * j / c->M2), (double)-sinl(2 * PI * j / c->M2));
    std::vector<double> sy(4 * (size_t)(c->M1 + c->M2));
    auto fill_dir = [&](int M, double dx, double *m0, double *m1, double *cr, double *ci) {
        const int p = c->P;
        for (int k = 0; k < M; ++k) {
            const long double th = 2 * PI * k / M;
            long double s0 = 0, s1 = 0;
            for (int q = -p; q <= p; ++q) s0 += (long double)c->m0row[q + p] * cosl(q * th);
            for (int q = -(p - 1); q <= p - 1; ++q) s1 += (long double)c->m1row[q + p - 1] * cosl(q * th);
            m0[k] = (double)(s0 * dx);
            m1[k] = (double)(s1 * dx);
            cr[k] = (double)((1 - cosl(th)) / dx);
            ci[k] = (double)(sinl(th) / dx);
        }
    };
    const int M1 = c->M1, M2 = c->M2;
    fill_dir(M1, dx1, &sy[0], &sy[M1], &sy[2 * M1], &sy[3 * M1]);
    fill_dir(M2, dx2, &sy[4 * M1], &sy[4 * M1 + M2], &sy[4 * M1 + 2 * M2], &sy[4 * M1 + 3 * M2]);
    // The twiddles, the symbols and the rows of M1^{-1} (component 1: m1(x1) m0(x2),
    // component 2: m0(x1) m1(x2)) go up in one block.
    std::vector<double> tab;
    auto append = [&](const double *v, size_t n) {
        tab.insert(tab.end(), v, v + n);
        return tab.size() - n;
    };
    const size_t at1 = append(&t1[0].x, M1), at2 = append(&t2[0].x, M2), at_sym = append(sy.data(), sy.size());
    size_t at_row[4];
    for (int q = 0; q < 4; ++q) {   // the rows along x1, then along x2
        ConvTaps &t = q < 2 ? c->conv_a : c->conv_b;
        const int b = q & 1;
        const std::vector<double> row =
            inverse_row(q < 2 ? M1 : M2, (b == 0) == (q < 2) ? c->m1row : c->m0row, q < 2 ? dx1 : dx2, t.hi[b]);
        t.nt[b] = (int)row.size();
        std::vector<double> pad(8 + conv_steps(t.nt[b]) + 16, 0.0);
        std::copy(row.begin(), row.end(), pad.begin() + 8);
        at_row[q] = append(pad.data(), pad.size()) + 8;
    }
    double *d = nullptr;
    rc = dalloc(c, &d, tab.size());
    if (!rc && hipMemcpy(d, tab.data(), sizeof(double) * tab.size(), hipMemcpyHostToDevice) != hipSuccess)
        rc = ECPIC_EDEVICE;
    if (rc) { ecpic2d_destroy(c); return rc; }
    c->tw1 = reinterpret_cast<double2 *>(d + at1);
    c->tw2 = reinterpret_cast<double2 *>(d + at2);
    c->sym = d + at_sym;
    for (int q = 0; q < 4; ++q) (q < 2 ? c->conv_a : c->conv_b).rt[q & 1] = d + at_row[q];
    for (double **gp : grids) k2_fill<<<grid_for(c->Nc), BLOCK, 0, c->stream>>>(*gp, c->Nc, 0.0);
    k2_fill_i32<<<grid_for(c->Nc), BLOCK, 0, c->stream>>>(c->count, c->Nc);
    // the commit accumulates arrivals per tile: every tile counter starts at zero
    for (int32_t *tp : {c->tstay, c->tarr})
        k2_fill_i32<<<grid_for(c->ntiles), BLOCK, 0, c->stream>>>(tp, c->ntiles);
    k2_fill_i32<<<1, 1, 0, c->stream>>>(c->flags, 1);
    k2_fill_i32<<<1, 2, 0, c->stream>>>(c->gate, 2);   // gate[1] stays open
    k2_fill_i32<<<1, 1, 0, c->stream>>>(reinterpret_cast<int32_t *>(c->done), 1);
    if (sync2(c)) { ecpic2d_destroy(c); return ECPIC_EDEVICE; }
    *out = c;
    return ECPIC_OK;
}

int ecpic2d_destroy(ecpic2d_ctx *c) {
    if (!c) return ECPIC_OK;
    hipSetDevice(c->device);
    if (c->stream) hipStreamSynchronize(c->stream);
    for (auto &pe : c->prof.pending) { hipEventDestroy(pe.second.first); hipEventDestroy(pe.second.second); }
    c->host_copy.release();
    for (void *p : c->allocs) hipFree(p);
    if (c->hres) hipHostFree(c->hres);
    if (c->stream) hipStreamDestroy(c->stream);
    delete c;
    return ECPIC_OK;
}

int ecpic2d_set_particles(ecpic2d_ctx *c, const double *x1, const double *x2, const double *p1, const double *p2,
                          int64_t n) {
    if (!c || n != c->N || (n > 0 && (!x1 || !x2 || !p1 || !p2))) return ECPIC_EINVAL;
    for (int64_t i = 0; i < n; ++i)
        if (!std::isfinite(x1[i]) || !std::isfinite(x2[i]) || !std::isfinite(p1[i]) || !std::isfinite(p2[i]))
            return ECPIC_EINVAL;
    hipSetDevice(c->device);
    const int B = 1 - c->cur, A = c->cur;
    const size_t bytes = sizeof(double) * (size_t)n;
    hipStream_t s = c->stream;
    // raw positions into the B buffers, momenta into A (scatter moves A -> B)
    if (n > 0) {
        if (hipMemcpyAsync(c->d1[0], x1, bytes, hipMemcpyHostToDevice, s) != hipSuccess ||
            hipMemcpyAsync(c->d2[0], x2, bytes, hipMemcpyHostToDevice, s) != hipSuccess ||
            hipMemcpyAsync(c->p1[A], p1, bytes, hipMemcpyHostToDevice, s) != hipSuccess ||
            hipMemcpyAsync(c->p2[A], p2, bytes, hipMemcpyHostToDevice, s) != hipSuccess)
            return ECPIC_EDEVICE;
    }
    (void)B;
    k2_fill_i32<<<1, 1, 0, s>>>(c->flags, 1);
    k2_fill_i32<<<grid_for(c->Nc), BLOCK, 0, s>>>(c->count, c->Nc);
    for (int32_t *tp : {c->tstay, c->tarr})
        k2_fill_i32<<<grid_for(c->ntiles), BLOCK, 0, s>>>(tp, c->ntiles);
    k2_iota<<<grid_for(n), BLOCK, 0, s>>>(c->id[A], n);
    k2_bin_new<<<grid_for(n), BLOCK, 0, s>>>(c->d1[0], c->d2[0], c->xi1[A], c->xi2[A], c->cell, c->count, n,
                                             c->M1, c->M2, 1.0 / c->dx1, 1.0 / c->dx2, c->flags);
    sort_particles(c);
    if (c->spin)   // the spins start at zero; ecpic2d_set_spins gives them
        for (double *sp : {c->sx[c->cur], c->sy[c->cur], c->sz[c->cur]})
            k2_fill<<<grid_for(n), BLOCK, 0, s>>>(sp, n, 0.0);
    int rc = flags_status(c);
    if (rc) return rc == ECPIC_ENONFINITE ? ECPIC_EINVAL : rc;
    c->have_particles = true;
    return ECPIC_OK;
}

int ecpic2d_set_spins(ecpic2d_ctx *c, const double *sx, const double *sy, const double *sz, int64_t n) {
    if (!c || !c->spin || n != c->N || (n > 0 && (!sx || !sy || !sz))) return ECPIC_EINVAL;
    for (int64_t i = 0; i < n; ++i)
        if (!std::isfinite(sx[i]) || !std::isfinite(sy[i]) || !std::isfinite(sz[i])) return ECPIC_EINVAL;
    if (!c->have_particles) return ECPIC_ESTATE;
    hipSetDevice(c->device);
    const int A = c->cur;
    const size_t bytes = sizeof(double) * (size_t)n;
    const double *in[3] = {sx, sy, sz};
    double *dst[3] = {c->sx[A], c->sy[A], c->sz[A]};
    for (int q = 0; q < 3 && n > 0; ++q) {
        // staging buffer: pk1 (free between substeps), in the caller's order
        if (hipMemcpyAsync(c->pk1, in[q], bytes, hipMemcpyHostToDevice, c->stream) != hipSuccess)
            return ECPIC_EDEVICE;
        k2_gather_id<<<grid_for(n), BLOCK, 0, c->stream>>>(c->pk1, c->id[A], dst[q], n);
    }
    return sync2(c);
}

int ecpic2d_get_spins(ecpic2d_ctx *c, double *sx, double *sy, double *sz, int64_t n) {
    if (!c || !c->spin || n != c->N || (n > 0 && (!sx || !sy || !sz))) return ECPIC_EINVAL;
    if (!c->have_particles) return ECPIC_ESTATE;
    hipSetDevice(c->device);
    const int A = c->cur;
    const size_t bytes = sizeof(double) * (size_t)n;
    double *outs[3] = {sx, sy, sz};
    const double *srcs[3] = {c->sx[A], c->sy[A], c->sz[A]};
    for (int q = 0; q < 3 && n > 0; ++q) {
        k2_unsort<<<grid_for(n), BLOCK, 0, c->stream>>>(srcs[q], c->id[A], c->pk1, n, 1.0);
        if (c->host_copy.to_host(outs[q], c->pk1, bytes, c->stream, c->device) != hipSuccess) return ECPIC_EDEVICE;
    }
    return sync2(c);
}

int ecpic2d_get_particles(ecpic2d_ctx *c, double *x1, double *x2, double *p1, double *p2, int64_t n) {
    if (!c || n != c->N || (n > 0 && (!x1 || !x2 || !p1 || !p2))) return ECPIC_EINVAL;
    if (!c->have_particles) return ECPIC_ESTATE;
    hipSetDevice(c->device);
    const int A = c->cur;
    const size_t bytes = sizeof(double) * (size_t)n;
    double *outs[4] = {x1, x2, p1, p2};
    const double *srcs[4] = {c->xi1[A], c->xi2[A], c->p1[A], c->p2[A]};
    const double scales[4] = {c->dx1, c->dx2, 1.0, 1.0};
    for (int q = 0; q < 4; ++q) {
        if (n == 0) break;
        k2_unsort<<<grid_for(n), BLOCK, 0, c->stream>>>(srcs[q], c->id[A], c->pk1, n, scales[q]);
        if (c->host_copy.to_host(outs[q], c->pk1, bytes, c->stream, c->device) != hipSuccess) return ECPIC_EDEVICE;
    }
    return sync2(c);
}

int ecpic2d_set_fields(ecpic2d_ctx *c, const double *e1, const double *e2, const double *bz, const double *ez,
                       const double *az) {
    if (!c) return ECPIC_EINVAL;
    hipSetDevice(c->device);
    const double *src[5] = {e1, e2, bz, ez, az};
    double *dst[5] = {c->e1, c->e2, c->bz, c->ez, c->az};
    for (int q = 0; q < 5; ++q) {
        if (src[q]) {
            if (hipMemcpyAsync(dst[q], src[q], sizeof(double) * c->Nc, hipMemcpyHostToDevice, c->stream) !=
                hipSuccess)
                return ECPIC_EDEVICE;
        } else {
            k2_fill<<<grid_for(c->Nc), BLOCK, 0, c->stream>>>(dst[q], c->Nc, 0.0);
        }
    }
    return sync2(c);
}

int ecpic2d_get_fields(ecpic2d_ctx *c, double *e1, double *e2, double *bz, double *ez, double *az) {
    if (!c) return ECPIC_EINVAL;
    hipSetDevice(c->device);
    double *dst[5] = {e1, e2, bz, ez, az};
    const double *src[5] = {c->e1, c->e2, c->bz, c->ez, c->az};
    if (c->hfields) {
        k2_fields_out<<<dim3(grid_for(c->Nc), 5), BLOCK, 0, c->stream>>>(
            Ptrs<5>{{c->e1, c->e2, c->bz, c->ez, c->az}}, c->hfields_dev, c->Nc);
        const int rc = sync2(c);
        for (int q = 0; q < 5 && !rc; ++q)
            if (dst[q] && ecpic::HostCopy::from_pinned(dst[q], c->hfields + (size_t)q * c->Nc,
                                                       sizeof(double) * c->Nc, c->stream) != hipSuccess)
                return ECPIC_EDEVICE;
        return rc;
    }
    for (int q = 0; q < 5; ++q)
        if (dst[q] &&
            hipMemcpyAsync(dst[q], src[q], sizeof(double) * c->Nc, hipMemcpyDeviceToHost, c->stream) != hipSuccess)
            return ECPIC_EDEVICE;
    return sync2(c);
}

int ecpic2d_solve_gauss(ecpic2d_ctx *c) {
    if (!c) return ECPIC_EINVAL;
    if (!c->have_particles) return ECPIC_ESTATE;
    hipSetDevice(c->device);
    deposit_rho(c, c->S);
    spectral<3>(c, "poisson", Ptrs<3>{{c->e1, c->e2, c->S}}, 4, OpPoisson{sym_of(c)},
                EpiStore<3>{Ptrs<3>{{c->e1, c->e2, c->S}}, nullptr});
    k2_fill<<<grid_for(c->Nc), BLOCK, 0, c->stream>>>(c->S, c->Nc, 0.0);
    return sync2(c);
}

int ecpic2d_substep_I(ecpic2d_ctx *c, double dt, ecpic2d_iter_stats *st) {
    if (!c || !(dt > 0) || !(dt < std::min(c->dx1, c->dx2))) return ECPIC_EINVAL;
    if (!c->have_particles) return ECPIC_ESTATE;
    hipSetDevice(c->device);
    const int rc = substep_I(c, dt, st);
    return rc ? rc : sync2(c);
}

int ecpic2d_substep_II(ecpic2d_ctx *c, double dt) {
    if (!c || !std::isfinite(dt)) return ECPIC_EINVAL;
    if (!c->have_particles) return ECPIC_ESTATE;
    hipSetDevice(c->device);
    substep_II(c, dt);
    return sync2(c);
}

int ecpic2d_substep_III(ecpic2d_ctx *c, double dt, ecpic2d_iter_stats *st) {
    if (!c || !(dt > 0) || !std::isfinite(dt)) return ECPIC_EINVAL;
    if (!c->have_particles) return ECPIC_ESTATE;
    hipSetDevice(c->device);
    int rc = substep_III(c, dt, st);
    if (rc) return rc;
    return sync2(c);
}

int ecpic2d_substep_IV(ecpic2d_ctx *c, double dt) {
    if (!c || !std::isfinite(dt)) return ECPIC_EINVAL;
    hipSetDevice(c->device);
    substep_IV(c, dt);
    return sync2(c);
}

int ecpic2d_step(ecpic2d_ctx *c, int32_t nsteps, int32_t *sweeps_I, int32_t *iters_III) {
    if (!c || nsteps < 0) return ECPIC_EINVAL;
    if (!c->have_particles) return ECPIC_ESTATE;
    hipSetDevice(c->device);
    const double dt = c->cfg.dt;
    for (int s = 0; s < nsteps; ++s) {
        ecpic2d_iter_stats a{}, b{};
        int rc = substep_I(c, dt, &a);
        if (sweeps_I) sweeps_I[s] = a.sweeps;
        if (rc) return rc;
        substep_II(c, dt);
        rc = substep_III(c, dt, &b);
        if (iters_III) iters_III[s] = b.sweeps;
        if (rc) return rc;
        substep_IV(c, dt);
    }
    return sync2(c);
}

int ecpic2d_energy(ecpic2d_ctx *c, ecpic2d_energy_parts *out) {
    if (!c || !out) return ECPIC_EINVAL;
    if (!c->have_particles) return ECPIC_ESTATE;
    hipSetDevice(c->device);
    const int A = c->cur, P = c->P;
    hipStream_t s = c->stream;
    const int gN = std::min(grid_for(c->N), RED_BLOCKS);
    k2_fill<<<1, BLOCK, 0, s>>>(c->partial, RED_BLOCKS + 16, 0.0);
    LAUNCH_P(P, k2_kinetic<PP><<<gN, BLOCK, 0, s>>>(c->xi1[A], c->xi2[A], c->p1[A], c->p2[A], c->az, c->N, c->M1,
                                                     c->M2, c->w, c->partial));
    k2_sum<<<1, BLOCK, 0, s>>>(c->partial, gN, c->partial + RED_BLOCKS + 0);
    quad(c, c->e1, P - 1, P, 1);
    quad(c, c->e2, P, P - 1, 2);
    quad(c, c->bz, P - 1, P - 1, 3);
    quad(c, c->ez, P, P, 4);
    k2_grad<<<grid_for(c->Nc), BLOCK, 0, s>>>(c->az, c->g1a, c->g2a, c->M1, c->M2, 1.0 / c->dx1, 1.0 / c->dx2);
    quad(c, c->g1a, P - 1, P, 5);
    quad(c, c->g2a, P, P - 1, 6);
    if (c->spin) {
        k2_fill<<<1, BLOCK, 0, s>>>(c->partial, RED_BLOCKS, 0.0);
        LAUNCH_P(P, k2_zeeman<PP><<<gN, BLOCK, 0, s>>>(c->xi1[A], c->xi2[A], c->sx[A], c->sy[A], c->sz[A], c->g1a,
                                                        c->g2a, c->bz, c->N, c->M1, c->M2, c->w, c->partial));
        k2_sum<<<1, BLOCK, 0, s>>>(c->partial, gN, c->partial + RED_BLOCKS + 7);
    }
    double v[8];
    if (hipMemcpyAsync(v, c->partial + RED_BLOCKS, sizeof(v), hipMemcpyDeviceToHost, s) != hipSuccess)
        return ECPIC_EDEVICE;
    int rc = sync2(c);
    if (rc) return rc;
    out->kinetic = v[0];
    out->e_xy = 0.5 * (v[1] + v[2]);
    out->b_z = 0.5 * v[3];
    out->e_z = 0.5 * v[4];
    out->a_z = 0.5 * (v[5] + v[6]);
    out->zeeman = c->spin ? c->hbar * v[7] : 0.0;
    out->total = out->kinetic + out->e_xy + out->b_z + out->e_z + out->a_z + out->zeeman;
    return ECPIC_OK;
}

int ecpic2d_deposit_charge(ecpic2d_ctx *c, double *rho) {
    if (!c || !rho) return ECPIC_EINVAL;
    if (!c->have_particles) return ECPIC_ESTATE;
    hipSetDevice(c->device);
    deposit_rho(c, c->S);
    if (hipMemcpyAsync(rho, c->S, sizeof(double) * c->Nc, hipMemcpyDeviceToHost, c->stream) != hipSuccess)
        return ECPIC_EDEVICE;
    int rc = sync2(c);
    k2_fill<<<grid_for(c->Nc), BLOCK, 0, c->stream>>>(c->S, c->Nc, 0.0);
    return rc ? rc : sync2(c);
}

int ecpic2d_gauss_residual(ecpic2d_ctx *c, double *linf, double *vec) {
    if (!c || !linf) return ECPIC_EINVAL;
    if (!c->have_particles) return ECPIC_ESTATE;
    hipSetDevice(c->device);
    hipStream_t s = c->stream;
    const int P = c->P;
    deposit_rho(c, c->S);
    k2_mass<<<grid_for(c->Nc), BLOCK, 0, s>>>(c->e1, c->J1, c->M1, c->M2, rows_of(c, P - 1, P));
    k2_mass<<<grid_for(c->Nc), BLOCK, 0, s>>>(c->e2, c->J2, c->M1, c->M2, rows_of(c, P, P - 1));
    k2_fill_u64<<<1, 1, 0, s>>>(c->res + 3 * MAXK, 1);
    k2_gauss<<<std::min(grid_for(c->Nc), RED_BLOCKS), BLOCK, 0, s>>>(c->J1, c->J2, c->S, c->tmp, c->M1, c->M2,
                                                                     1.0 / c->dx1, 1.0 / c->dx2, c->dx1 * c->dx2,
                                                                     c->res + 3 * MAXK);
    int rc = 0;
    *linf = read_res(c, 3 * MAXK, &rc);
    if (!rc && vec &&
        hipMemcpyAsync(vec, c->tmp, sizeof(double) * c->Nc, hipMemcpyDeviceToHost, s) != hipSuccess)
        rc = ECPIC_EDEVICE;
    k2_fill<<<grid_for(c->Nc), BLOCK, 0, s>>>(c->S, c->Nc, 0.0);
    k2_fill<<<grid_for(c->Nc), BLOCK, 0, s>>>(c->J1, c->Nc, 0.0);
    k2_fill<<<grid_for(c->Nc), BLOCK, 0, s>>>(c->J2, c->Nc, 0.0);
    int rc2 = sync2(c);
    return rc ? rc : rc2;
}

int ecpic2d_profile_enable(ecpic2d_ctx *c, int32_t enable) {
    if (!c) return ECPIC_EINVAL;
    sync2(c);
    c->prof.on = enable != 0;
    if (c->prof.on) c->prof.acc.clear();
    return ECPIC_OK;
}

int ecpic2d_kernel_time(ecpic2d_ctx *c, const char *name, double *ms, int64_t *launches) {
    if (!c || !name || !ms || !launches) return ECPIC_EINVAL;
    sync2(c);
    auto it = c->prof.acc.find(name);
    *ms = it == c->prof.acc.end() ? 0.0 : it->second.first;
    *launches = it == c->prof.acc.end() ? 0 : it->second.second;
    return ECPIC_OK;
}

}  // extern "C"
