// Device kernels of the time march (gfx950).  FP64 grids are row-major n x n,
// V[i * n + j], i the axis-1 index (slow), j the axis-2 index (fast).
//
// The FFT correlation (B v)_m = sum_d K_d v_{m+d} (Sec. 3.2.2 with the
// half-cell interpolation folded into K) is three passes over an
// intermediate X stored transposed, X[k2 * ldx + i1] (column k2 of the
// row-transformed grid is contiguous):
//   rows_fwd : pairs of real rows -> one complex length-L FFT -> split into
//              the two half spectra k2 = 0..L/2 (zero padding n -> L);
//   cols     : per column k2: forward FFT over i1 (zero padded), multiply by
//              the stored spectrum conj(K^)/L^2, inverse FFT, keep n rows;
//   rows_inv : per pair of rows: Hermitian completion of the two half
//              spectra into one complex sequence, inverse FFT, real part ->
//              row a, imaginary part -> row b, keep n columns, then a fused
//              epilogue (plain store, or the affine stencil form below).
#pragma once

#include <hip/hip_runtime.h>

#include "fft.hpp"
#include "gmem.hpp"

namespace lpide {

// Coefficients of the log-grid diffusion operator D (Sec. 3.2.1):
// D u = 1/2 a11 [i interior](d11 - d1) u + a12 d~1 d~2 u + 1/2 a22 [j interior](d22 - d2) u.
struct StencilArgs {
    int    n;
    double h, a11, a12, a22;
};

// Bijective block -> work-item remap that gives each of the 8 XCDs (which
// receive blocks round-robin) a contiguous range of work items.
__device__ __forceinline__ int xcd_remap(int b, int nb) {
    const int x = b & 7, i = b >> 3, q = nb >> 3, rem = nb & 7;
    return x * q + (x < rem ? x : rem) + i;
}

// D applied to U at (i, j).  Second differences only on interior indices of
// their own axis (the log form of the boundary rule "v linear in x"); the
// mixed term uses d~ = central inside, forward at 0, backward at n-1.
__device__ __forceinline__ double apply_D(GP<double> U, const StencilArgs& s, int i, int j, double u) {
    const int n = s.n;
    const double ih2 = 1.0 / (s.h * s.h), i2h = 0.5 / s.h;
    double d = 0.0;
    if (i > 0 && i < n - 1) {
        const double um = U[(i - 1) * n + j], up = U[(i + 1) * n + j];
        d += 0.5 * s.a11 * ((up - 2.0 * u + um) * ih2 - (up - um) * i2h);
    }
    if (j > 0 && j < n - 1) {
        const double um = U[i * n + j - 1], up = U[i * n + j + 1];
        d += 0.5 * s.a22 * ((up - 2.0 * u + um) * ih2 - (up - um) * i2h);
    }
    if (s.a12 != 0.0) {
        int i0, i1, j0, j1;
        double gi, gj;
        if (i == 0) { i0 = 0; i1 = 1; gi = 1.0 / s.h; }
        else if (i == n - 1) { i0 = n - 2; i1 = n - 1; gi = 1.0 / s.h; }
        else { i0 = i - 1; i1 = i + 1; gi = i2h; }
        if (j == 0) { j0 = 0; j1 = 1; gj = 1.0 / s.h; }
        else if (j == n - 1) { j0 = n - 2; j1 = n - 1; gj = 1.0 / s.h; }
        else { j0 = j - 1; j1 = j + 1; gj = i2h; }
        const double u00 = U[i0 * n + j0], u01 = U[i0 * n + j1];
        const double u10 = U[i1 * n + j0], u11 = U[i1 * n + j1];
        d += s.a12 * gi * gj * ((u11 - u10) - (u01 - u00));
    }
    return d;
}

// D at (i, j) from the node's value u and its eight neighbours, read at indices
// clamped into the grid (the mixed term's nodes are those neighbours): u1m, u1p
// along axis 1, u2m, u2p along axis 2, u00 .. u11 the corners (first index axis
// 1).  The interior tests select the arithmetic only (a zero a12 adds a zero
// mixed term), so that none of a node's reads is conditional.  The row c2r
// kernel's forms whose stencil follows the transform (the explicit part, and the
// mixed form above L = 1536) unroll many elements and keep apply_D, whose branches
// throttle the reads in flight.
__device__ __forceinline__ double D_of(const StencilArgs& s, int i, int j, double u, double u1m, double u1p, double u2m,
                                       double u2p, double u00, double u01, double u10, double u11) {
    const int n = s.n;
    const double ih2 = 1.0 / (s.h * s.h), i2h = 0.5 / s.h;
    const bool iin = i > 0 && i < n - 1, jin = j > 0 && j < n - 1;
    double d = 0.0;
    if (iin) d += 0.5 * s.a11 * ((u1p - 2.0 * u + u1m) * ih2 - (u1p - u1m) * i2h);
    if (jin) d += 0.5 * s.a22 * ((u2p - 2.0 * u + u2m) * ih2 - (u2p - u2m) * i2h);
    const double gi = iin ? i2h : 1.0 / s.h, gj = jin ? i2h : 1.0 / s.h;
    d += s.a12 * gi * gj * ((u11 - u10) - (u01 - u00));
    return d;
}

// The three unit-coefficient parts of D at (i, j): D u = a11 d11 + a12 d12 + a22 d22
// (the derivative of D u with respect to each coefficient).
__device__ __forceinline__ void apply_D_parts(GP<double> U, int n, double h, int i, int j, double u, double& d11,
                                              double& d12, double& d22) {
    const double ih2 = 1.0 / (h * h), i2h = 0.5 / h;
    d11 = d12 = d22 = 0.0;
    if (i > 0 && i < n - 1) {
        const double um = U[(i - 1) * n + j], up = U[(i + 1) * n + j];
        d11 = 0.5 * ((up - 2.0 * u + um) * ih2 - (up - um) * i2h);
    }
    if (j > 0 && j < n - 1) {
        const double um = U[i * n + j - 1], up = U[i * n + j + 1];
        d22 = 0.5 * ((up - 2.0 * u + um) * ih2 - (up - um) * i2h);
    }
    int i0, i1, j0, j1;
    double gi, gj;
    if (i == 0) { i0 = 0; i1 = 1; gi = 1.0 / h; }
    else if (i == n - 1) { i0 = n - 2; i1 = n - 1; gi = 1.0 / h; }
    else { i0 = i - 1; i1 = i + 1; gi = i2h; }
    if (j == 0) { j0 = 0; j1 = 1; gj = 1.0 / h; }
    else if (j == n - 1) { j0 = n - 2; j1 = n - 1; gj = 1.0 / h; }
    else { j0 = j - 1; j1 = j + 1; gj = i2h; }
    const double u00 = U[i0 * n + j0], u01 = U[i0 * n + j1];
    const double u10 = U[i1 * n + j0], u11 = U[i1 * n + j1];
    d12 = gi * gj * ((u11 - u10) - (u01 - u00));
}

// D^T u at (i, j), the transposed log-grid stencil with the boundary rows' terms:
// arguments as D_of (neighbours clamped into the grid).  Every node takes the same
// reads and arithmetic, the edges by their weights: row r of a second difference
// exists for interior r only, and the rows of the first-difference matrix of the
// mixed term are central inside, forward at 0 and backward at n - 1.
__device__ __forceinline__ double DT_of(const StencilArgs& s, int i, int j, double u, double u1m, double u1p, double u2m,
                                        double u2p, double u00, double u01, double u10, double u11) {
    const int n = s.n;
    const double ih2 = 1.0 / (s.h * s.h), i2h = 0.5 / s.h, ih = 1.0 / s.h;
    const double cu = 0.5 * (ih2 - i2h);   // coefficient of v_{r+1} in row r
    const double cl = 0.5 * (ih2 + i2h);   // coefficient of v_{r-1} in row r
    auto second = [&](int p, double v, double vm, double vp) {
        return (p >= 2 ? cu : 0.0) * vm + (p <= n - 3 ? cl : 0.0) * vp - (p > 0 && p < n - 1 ? ih2 : 0.0) * v;
    };
    // entries of column p in the rows max(p - 1, 0) and min(p + 1, n - 1)
    auto lo = [&](int p) { return p == 0 ? -ih : (p == 1 ? ih : i2h); };
    auto hi = [&](int p) { return p == n - 1 ? ih : (p == n - 2 ? -ih : -i2h); };
    return s.a11 * second(i, u, u1m, u1p) + s.a22 * second(j, u, u2m, u2p) +
           s.a12 * (lo(i) * (lo(j) * u00 + hi(j) * u01) + hi(i) * (lo(j) * u10 + hi(j) * u11));
}

}  // namespace lpide
