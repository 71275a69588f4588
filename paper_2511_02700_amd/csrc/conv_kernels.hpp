// Stand-alone FFT correlation kernels (FP64) for lpide_apply_B, the plan-time
// spectrum and the adjoint's kernel-gradient transforms, and a plain copy kernel.
//
// Rows bound these passes by the 32 contiguous bytes that a frequency's two rows
// have in the transposed intermediate: with a lane pair moving them together, each
// wave's store or load is half as many lines (forward rows at n = 2000, L = 3072:
// 30.0 -> 24.6 us, n = 1400, L = 2048: 14.5 -> 11.5; inverse rows 29.6 -> 25.5 and
// 14.9 -> 12.9).  Below a side (pair_fwd, pair_inv) a pass is one block's latency
// instead, and one thread with both rows' values in flight is the shorter chain
// (inverse rows at L = 512: 3.4 us against 5.1, L = 1024: 4.7 against 5.2; forward
// rows at L = 512: 3.6 against 3.9, but L = 768: 5.1 against 4.7).
// In the same way the two real columns 0 and L/2 share one transform only where the
// column pass is several waves of blocks (pair_cols): at L = 512 that block's longer
// chain makes the pass 5.0 us against 4.2.  B v: 33.8 -> 33.1 us at n = 1001,
// 49.2 -> 43.4 at n = 1200 in L = 2048, 118 -> 81 at n = 1400 in L = 3072, 139 -> 97
// at n = 2000.
// The plan-time spectrum keeps conv_e(L) elements so that the mixed form's results
// stay bit for bit what they were; a change of its rounding would move them by 1e-9,
// within their error of about 1e-8.
#pragma once

#include <hip/hip_runtime.h>

#include "fft.hpp"
#include "kernels.hpp"

namespace lpide {
namespace detail {

// Elements per thread of the row and the column transforms of lpide_apply_B, by the
// time of the three passes together: at L = 512 8 over 4 (12.1 against 13.9 us),
// 1536 and 2048 8 over 4 (34.1 / 34.4 and 43.5 / 47.1), 1024 and 3072 4 over 8
// (20.3 / 22.9 and 95 / 133).
constexpr int rows_e(int L) { return L == 512 || L == 1536 || L == 2048 || L == 4096 ? 8 : 4; }
constexpr int cols_e(int L) { return L == 4096 ? 16 : rows_e(L); }
constexpr bool pair_fwd(int L) { return L >= 768; }
constexpr bool pair_inv(int L) { return L >= 1536; }
constexpr bool pair_cols(int L) { return L >= 1024; }

// Forward real FFT of pairs of rows (2p, 2p+1) of Y (n_rows x n_cols used,
// zero padded to L) into the transposed half spectra X[k2 * ldx + row].
template <int L, int KE>
__global__ __launch_bounds__(L / KE) void k_rows_fwd(const double* __restrict__ Y, int ldy, int n_rows,
                                                   int n_cols, double2* __restrict__ X, int ldx,
                                                   const double2* __restrict__ tw) {
    constexpr int T = L / KE;
    __shared__ double2 lds[lds_slots(L)];
    __shared__ double2 tw4[tw_slots<L, KE>()];
    load_twiddles<L, KE>(tw, tw4);
    const int np = (n_rows + 1) >> 1;
    const int p = xcd_remap(blockIdx.x, np);
    const int ra = 2 * p, rb = 2 * p + 1;
    const bool hasb = rb < n_rows;
    const double* ya = Y + (size_t)ra * ldy;
    const double* yb = Y + (size_t)(hasb ? rb : ra) * ldy;
    const int tid = threadIdx.x;
    double2 reg[KE];
#pragma unroll
    for (int e = 0; e < KE; ++e) {
        const int idx = tid + e * T;
        double a = 0.0, b = 0.0;
        if (idx < n_cols) {
            a = ya[idx];
            b = hasb ? yb[idx] : 0.0;
        }
        reg[e] = make_double2(a, b);
    }
    fft_block<L, KE, false>(reg, lds, tw4);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < KE; ++e) lds[tid + e * T] = reg[e];
    __syncthreads();
    // Z = FFT(a + i b): A_k = (Z_k + conj Z_{L-k}) / 2, B_k = (Z_k - conj Z_{L-k}) / (2i).
    if constexpr (pair_fwd(L)) {
        // item idx is frequency idx / 2 of row ra + idx mod 2
        constexpr int NI = (L + 2 + T - 1) / T;
#pragma unroll
        for (int it = 0; it < NI; ++it) {
            const int idx = tid + it * T;
            const int kk = idx >> 1, r = idx & 1;
            if (kk > L / 2 || (r == 1 && !hasb)) continue;
            const double2 z = lds[kk], w = lds[kk == 0 ? 0 : L - kk];
            X[(size_t)kk * ldx + ra + r] = r == 0 ? make_double2(0.5 * (z.x + w.x), 0.5 * (z.y - w.y))
                                                  : make_double2(0.5 * (z.y + w.y), -0.5 * (z.x - w.x));
        }
    } else {
#pragma unroll
        for (int e = 0; e < KE / 2 + 1; ++e) {
            const int kk = tid + e * T;
            if (kk > L / 2) continue;
            const double2 z = lds[kk], w = lds[kk == 0 ? 0 : L - kk];
            X[(size_t)kk * ldx + ra] = make_double2(0.5 * (z.x + w.x), 0.5 * (z.y - w.y));
            if (hasb) X[(size_t)kk * ldx + rb] = make_double2(0.5 * (z.y + w.y), -0.5 * (z.x - w.x));
        }
    }
}

// Column pass of lpide_apply_B: X[col] <- first n of IFFT(FFT(X[col]) * spec[col]);
// apply_col_blocks(L) blocks; with pair_cols block 0 takes the two real columns 0 and
// L/2 (mul_real_pair).
constexpr int apply_col_blocks(int L) { return L / 2 + (pair_cols(L) ? 0 : 1); }
template <int L, int KE>
__global__ __launch_bounds__(L / KE) void k_cols_apply(double2* __restrict__ X, int n, const double2* __restrict__ spec,
                                                      const double2* __restrict__ tw) {
    constexpr int T = L / KE;
    __shared__ double2 lds[lds_slots(L)];
    __shared__ double2 tw4[tw_slots<L, KE>()];
    load_twiddles<L, KE>(tw, tw4);
    const int col = blockIdx.x, tid = threadIdx.x;
    const bool pair = pair_cols(L) && col == 0;
    double2* xc = X + (size_t)col * n;
    double2* xh = X + (size_t)(L / 2) * n;
    const double2* sc = spec + (size_t)col * L;
    double2 reg[KE];
#pragma unroll
    for (int e = 0; e < KE; ++e) {
        const int idx = tid + e * T;
        if (idx < n) reg[e] = pair ? make_double2(xc[idx].x, xh[idx].x) : xc[idx];
        else reg[e] = make_double2(0.0, 0.0);
    }
    fft_block<L, KE, false>(reg, lds, tw4);
    if (pair) {
        mul_real_pair<L, KE, false>(reg, lds, sc, spec + (size_t)(L / 2) * L);
    } else {
#pragma unroll
        for (int e = 0; e < KE; ++e) reg[e] = cmul(reg[e], sc[tid + e * T]);
    }
    fft_block<L, KE, true>(reg, lds, tw4);
#pragma unroll
    for (int e = 0; e < KE; ++e) {
        const int idx = tid + e * T;
        if (idx >= n) continue;
        if (pair) {
            xc[idx] = make_double2(reg[e].x, 0.0);
            xh[idx] = make_double2(reg[e].y, 0.0);
        } else {
            xc[idx] = reg[e];
        }
    }
}

// Column pass.  MODE 1 (plan time): spec_out[col] = conj(FFT(X[col])) * scale.
// MODE 2: X[col] <- first n_out of IFFT(X[col], zero padded from n_in).
template <int L, int MODE>
__global__ __launch_bounds__(L / conv_e(L)) void k_cols(double2* __restrict__ X, int ldx, int n_in, int n_out,
                                               double2* __restrict__ spec_out, double scale,
                                               const double2* __restrict__ tw) {
    constexpr int KE = conv_e(L), T = L / KE;
    __shared__ double2 lds[lds_slots(L)];
    __shared__ double2 tw4[tw_slots<L, KE>()];
    load_twiddles<L, KE>(tw, tw4);
    const int col = blockIdx.x;
    const int tid = threadIdx.x;
    double2* xc = X + (size_t)col * ldx;
    double2 reg[KE];
#pragma unroll
    for (int e = 0; e < KE; ++e) {
        const int idx = tid + e * T;
        reg[e] = idx < n_in ? xc[idx] : make_double2(0.0, 0.0);
    }
    if constexpr (MODE == 2) {
        fft_block<L, KE, true>(reg, lds, tw4);
#pragma unroll
        for (int e = 0; e < KE; ++e) {
            const int idx = tid + e * T;
            if (idx < n_out) xc[idx] = reg[e];
        }
    } else {
        fft_block<L, KE, false>(reg, lds, tw4);
        double2* so = spec_out + (size_t)col * L;
#pragma unroll
        for (int e = 0; e < KE; ++e) so[tid + e * T] = make_double2(reg[e].x * scale, -reg[e].y * scale);
    }
}

// Inverse real FFT of row pairs from the transposed half spectra; keeps the
// first n columns: row a <- real part, row b <- imaginary part.
template <int L, int KE>
__global__ __launch_bounds__(L / KE) void k_rows_inv(const double2* __restrict__ X, int ldx, int n,
                                                    double* __restrict__ out, const double2* __restrict__ tw) {
    constexpr int T = L / KE;
    __shared__ double2 lds[lds_slots(L)];
    __shared__ double2 tw4[tw_slots<L, KE>()];
    load_twiddles<L, KE>(tw, tw4);
    const int np = (n + 1) >> 1;
    const int p = xcd_remap(blockIdx.x, np);
    const int ra = 2 * p, rb = 2 * p + 1;
    const bool hasb = rb < n;
    const int tid = threadIdx.x;
    double2 reg[KE];
    // Z_k = A_k + i B_k, with A_{L-k} = conj A_k, B_{L-k} = conj B_k, imaginary parts dropped
    // at DC and Nyquist
    if constexpr (pair_inv(L)) {
        // item idx is frequency idx / 2 of row ra + idx mod 2; the lanes of a pair swap their
        // values, the even one forms Z_k and the odd one Z_{L-k}
        constexpr int NI = (L + 2 + T - 1) / T;
#pragma unroll
        for (int it = 0; it < NI; ++it) {
            const int idx = tid + it * T;
            const int kk = idx >> 1, r = idx & 1;
            const bool in = kk <= L / 2;
            const double2 v = (in && (r == 0 || hasb)) ? X[(size_t)kk * ldx + ra + r] : make_double2(0.0, 0.0);
            const double2 u = make_double2(__shfl_xor(v.x, 1), __shfl_xor(v.y, 1));
            const bool real_bin = kk == 0 || kk == L / 2;
            const double2 ta = r == 0 ? v : u, tb = r == 0 ? u : v;
            const double2 ha = make_double2(ta.x, real_bin ? 0.0 : ta.y);
            const double2 hb = make_double2(tb.x, real_bin ? 0.0 : tb.y);
            if (in && r == 0) lds[lds_slot(kk)] = make_double2(ha.x - hb.y, ha.y + hb.x);
            if (in && r == 1 && kk > 0 && kk < L / 2) lds[lds_slot(L - kk)] = make_double2(ha.x + hb.y, hb.x - ha.y);
        }
        __syncthreads();
#pragma unroll
        for (int e = 0; e < KE; ++e) reg[e] = lds[lds_slot(tid + e * T)];
    } else {
        // a frequency's values are read twice, for Z_k and for Z_{L-k}, and need no exchange
#pragma unroll
        for (int e = 0; e < KE; ++e) {
            const int idx = tid + e * T;
            const bool lo = idx <= L / 2;
            const int kk = lo ? idx : L - idx;
            const bool real_bin = kk == 0 || kk == L / 2;
            const double2 ta = X[(size_t)kk * ldx + ra];
            const double2 tb = hasb ? X[(size_t)kk * ldx + rb] : make_double2(0.0, 0.0);
            const double2 ha = make_double2(ta.x, real_bin ? 0.0 : ta.y);
            const double2 hb = make_double2(tb.x, real_bin ? 0.0 : tb.y);
            reg[e] = lo ? make_double2(ha.x - hb.y, ha.y + hb.x) : make_double2(ha.x + hb.y, hb.x - ha.y);
        }
    }
    fft_block<L, KE, true>(reg, lds, tw4);
#pragma unroll
    for (int e = 0; e < KE; ++e) {
        const int j = tid + e * T;
        if (j >= n) continue;
        out[(size_t)ra * n + j] = reg[e].x;
        if (hasb) out[(size_t)rb * n + j] = reg[e].y;
    }
}


static __global__ void k_copy(const double* __restrict__ a, double* __restrict__ b, size_t cnt) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < cnt) b[i] = a[i];
}

}  // namespace detail
}  // namespace lpide
