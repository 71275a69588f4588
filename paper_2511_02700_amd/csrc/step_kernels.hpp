// Device-controlled time steps (Sec. 3.3, Algorithm 1) for gfx950.
//
// The host enqueues whole time steps without waiting: every step is
//   [explicit part: cols + rows_inv(explicit)]        (theta < 1 only)
//   sl        W = T^SL E, Y^0, and the row FFT of Y^0 (begin_lin instead once
//             B Y^0 comes by linearity: E, W, Y^0 and iteration 1's R in one)
//   kmax x {  cols          column pass of B Y (spectrum multiply)
//             rows_inv      R = W + dt theta ((D - r_omega) Y + B Y) - Y
//             line_cols     R <- T_1^{-1} R                 (axis 1)
//             line_rows     delta = T_2^{-1} R; Y += delta; err_k; row FFT of Y }
//   step_end  first k with err_k < tol; rotate the history; set up the next step
// Iteration k's kernels return at once when err_{k-1} < tol (the step has
// converged) or when a step failed to converge within its kmax iterations
// (then everything after it is a no-op until the host has added iterations).
// All buffers are addressed through a control block updated only by step_end,
// so the same launch sequence serves every step, whatever its kind (the
// explicit-part kernels return at once in theta = 1 steps of the FP64 form).
//
// Every kernel serves a group of independent plans with the same transform
// size: blockIdx.y selects the plan (its MarchArgs in device memory), and each
// plan has its own control block, so plans advance, converge and stop
// independently inside one launch.
//
// Mixed form (FP32 correlation, FP64 everything else): each step first applies
// B to V^{n-1} in FP64 (BV, and the explicit part), then the iteration
// correlations run in FP32 on increments only: B Y^0 = BV + B32(Y^0 - V^{n-1})
// and B Y^k = B Y^{k-1} + B32(delta^k), accumulated in FP64.  FP32 rounding is
// thus relative to the increments, which shrink geometrically, and does not
// accumulate across steps.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "fft.hpp"
#include "kernels.hpp"
#include "linesolve.hpp"

namespace lpide {

constexpr int KSLOTS = 136;          // err[.][0] (sentinel) + up to 128 iterations per step
constexpr int NX = 8;                 // stopping-rule partial maxima per iteration (one per XCD)
constexpr int MAX_ITER_CAP = 128;
constexpr int POOL = 6;               // grid buffers: history (4) + start state + iterate

struct StepDesc {
    double theta, dt;
    const double *fl1, *bu1, *bc1;    // axis-1 line factors of I - dt theta A_1
    const double *fl2, *bu2, *bc2;    // axis-2 line factors
    const int *s1, *s2;               // semi-Lagrangian stencil starts per axis
    const double *w1, *w2;            // semi-Lagrangian weights per axis
    // adjoint march only (null otherwise): transposed SL matrices per axis
    // (source rows and weights, padded to widths wt1, wt2) and the weight
    // derivatives with respect to the drift coefficient kappa_omega^(i)
    const int *t1i, *t2i;
    const double *t1w, *t2w;
    int wt1, wt2;
    const double *w1d, *w2d;
};

// What the kernels of one step need, resolved from the step list and the pool
// bookkeeping by the kernel that starts the step (ks_init, ks_step_end,
// ks_adj_begin), so that every kernel reads it in one go instead of following
// step -> set -> pointer through memory.
struct StepNow {
    int lin;                          // B Y^0 by linearity: every source of the start value has its product stored
    int expl;                         // explicit part E: EXPL_NONE, EXPL_IDENTITY, EXPL_CORR
    int anchor;                       // mixed form: B V^{n-1} afresh by the FP64 correlation
    int set;                          // index of the step's set
    double cth, cex, rho;             // dt theta, dt (1 - theta), rho of the identity
    const double* V;                  // state the step starts from
    double *Y, *W, *Wp;               // iterate, SL output, SL output of the step before (takes E where E is formed apart)
    double* B;                        // store of B applied to the iterate (or null)
    const double *H[4], *Hb[4];       // sources of the start value and their stored products
    double coef[4];                   // Y^0 = sum_q coef[q] H[q]; past the count of sources H[0] at weight 0
                                      // (so a loop over all four terms gives the same sums)
    const double *fl1, *bu1, *bc1, *fl2, *bu2, *bc2;
    const int *s1, *s2;
    const double *w1, *w2;
};
constexpr int EXPL_NONE = 0, EXPL_IDENTITY = 1, EXPL_CORR = 2;

struct Ctl {
    int step;                         // completed entries of the step list
    int fail;                         // current step not converged within its launched iterations
    int fail_step;
    int hold;                         // set by the host while another plan of the group is being completed
    StepNow now;                      // the current step (valid while step < nsteps)
    int cur;                          // pool index of the state the current step starts from
    int y;                            // pool index of the iterate
    int hc;                           // history length (main steps)
    int nsrc;                         // terms of the starting-value combination
    int hist[4];                      // pool indices, newest first
    int bvalid;                       // bit b: bpool[b] holds B applied to pool[b] (this march)
    int w;                            // SL buffer of this step (the step before wrote the other one)
    int recent[4];                    // iteration counts of the last four steps, at step mod 4
    // stopping-rule value after iteration k: the maximum over x of err[x][k]
    // (bit patterns of non-negative doubles).  The row blocks of the line-solve
    // kernel reduce into the partial of their XCD, so the atomics of one launch
    // go to eight cache lines instead of one (they are serialised per line).
    unsigned long long err[NX][KSLOTS];
};

struct MarchArgs {
    double* pool[POOL];
    const StepDesc* sets;
    const int* step_set;
    int n, n_sub, damping, P_cols;
    double* Wb[2];                    // SL outputs W of a step and of the one before it, in turn
    double* R;
    double2* X;
    const double2* spec;
    const double2* tw;
    int* counts;
    double* incs;
    double tol, r_omega;
    StencilArgs st;
    int mixed;                        // FP32 iteration correlations on increments
    float2* X32;                      // FP32 intermediate (mixed form)
    const float2* spec32;             // FP32 spectrum (mixed form)
    double* BV;                       // B V^{n-1}, FP64 (mixed form)
    double* BY;                       // B Y^k accumulated in FP64 (mixed form)
    int nsteps;                       // step-list entries to march (the plan stops after them)
    int step0;                        // step-list index of the state in pool[0] at the start
    double* seg;                      // recorded states: V^s to seg[(s - seg_base) / seg_every] (or null)
    double* segE;                     // recorded explicit parts E_s = M_E V^s to segE[s - seg_base] (theta < 1)
    int seg_base, seg_every;
    int anchor_every;                 // mixed form: B V^{n-1} afresh in FP64 every this many steps
    const double* cn_rho;             // per step: rho of the explicit part from the previous step's
                                      // implicit equation (0: by the correlation); null: never
    double* bpool[POOL];              // B applied to the pool grids (FP64 form; bpool[0] null: off)
};

using Args = const LPIDE_CONST MarchArgs;      // the plan's arguments and its control block, as every
using CtlK = const LPIDE_CONST Ctl;            // kernel but the controlling ones reads them (KRef)

__device__ __forceinline__ double bits_to_d(unsigned long long b) { return __longlong_as_double((long long)b); }

// Stopping-rule value after iteration k (maximum of the partials).
template <typename C>
__device__ __forceinline__ double err_max(C& c, int k) {
    unsigned long long m = c.err[0][k];
#pragma unroll
    for (int x = 1; x < NX; ++x) m = c.err[x][k] > m ? c.err[x][k] : m;
    return bits_to_d(m);
}

// Reset the stopping-rule partials (err[.][0] = +inf sentinel); by all threads of a block.
__device__ __forceinline__ void err_reset(Ctl* c) {
    for (int q = threadIdx.x; q < NX * KSLOTS; q += blockDim.x)
        c->err[q / KSLOTS][q % KSLOTS] = (q % KSLOTS) == 0 ? 0x7FF0000000000000ull : 0ull;
}

// The same for slots 0..kmax only: a step that ran iterations 1..kmax wrote
// no other slot, and every other slot is still zero from an earlier reset.
__device__ __forceinline__ void err_reset_upto(Ctl* c, int kmax) {
    const int w = kmax + 1;
    for (int q = threadIdx.x; q < NX * w; q += blockDim.x)
        c->err[q / w][q % w] = (q % w) == 0 ? 0x7FF0000000000000ull : 0ull;
}

// Uniform early-exit test of iteration k (k = 0: parts that run once per step).
// No read waits for another's test (the partial maxima are compared one by one,
// as bit patterns: a NaN lies above every tol), so all are in flight together.
__device__ __forceinline__ bool halted(Args& a, CtlK& c, int k) {
    const int kp = k > 0 ? k - 1 : 0;            // err[.][0] is the sentinel: never below tol
    unsigned long long e[NX];
#pragma unroll
    for (int x = 0; x < NX; ++x) e[x] = c.err[x][kp];
    const int off = c.fail | c.hold, left = a.nsteps - c.step;
    const unsigned long long tol = (unsigned long long)__double_as_longlong(a.tol);
    int open = 0;                                // partials that have not met tol
#pragma unroll
    for (int x = 0; x < NX; ++x) open |= e[x] >= tol ? 1 : 0;
    return off != 0 || left <= 0 || open == 0;
}

// The plan and the control block of this thread block.
__device__ __forceinline__ Args& plan_args(const MarchArgs* A) { return kref(A + blockIdx.y); }
__device__ __forceinline__ CtlK& plan_ctl(const Ctl* C) { return kref(C + blockIdx.y); }

__device__ __forceinline__ StencilArgs stencil(Args& a) {
    return StencilArgs{a.st.n, a.st.h, a.st.a11, a.st.a12, a.st.a22};
}

template <typename C> __device__ __forceinline__ GP<C> xbuf(Args& a);
template <> __device__ __forceinline__ GP<double2> xbuf<double2>(Args& a) { return GP<double2>(a.X); }
template <> __device__ __forceinline__ GP<float2> xbuf<float2>(Args& a) { return GP<float2>(a.X32); }
template <typename C> __device__ __forceinline__ GP<C> specbuf(Args& a);
template <> __device__ __forceinline__ GP<double2> specbuf<double2>(Args& a) { return GP<double2>(a.spec); }
template <> __device__ __forceinline__ GP<float2> specbuf<float2>(Args& a) { return GP<float2>(a.spec32); }

// Explicit part of a step from the implicit equation of the step before it
// (EXPL_IDENTITY).  That step solved (I - c A) V^{n-1} = W (c = dt theta of that
// step, W still in now.Wp), so A V^{n-1} = (V^{n-1} - W) / c and
//   E = V^{n-1} + dt (1 - theta) A V^{n-1} = V^{n-1} + rho (V^{n-1} - W),
// rho = dt (1 - theta) / c: the same explicit part without applying B, exact
// at the fixed point (the converged iterate leaves the stopping-rule residual).
// Used from the second step of a march on, when the previous step had
// theta > 0 (cn_rho > 0, set by the host; null with every product by the
// correlation and in the adjoint march); in the mixed form outside its anchor
// steps, whose FP64 correlation forms the explicit part.
//
// B Y^0 of the first iteration by linearity (lin): Y^0 = sum_q coef_q V^{src_q}, so
// B Y^0 = sum_q coef_q B V^{src_q}, with B V^{src_q} stored by the row kernel of
// the step that produced V^{src_q} (B applied to its last iterate before the
// final update, so B V^{src_q} is off by B of an increment below the stopping
// tolerance; the first iteration only sets where the iteration starts, its
// fixed point is unchanged).  Needs every source grid from this march.
//
// Mixed form: the steps whose B V^{n-1} is computed afresh by the FP64
// correlation (anchor: every anchor_every-th step of the march, its first step
// included).  In the others B V^{n-1} is carried from the previous step: its
// last accumulated B Y, still in BY when the step's first iteration adds to it.

// The pool bookkeeping of a step, in registers of the kernel that starts it.
struct Book {
    int step, cur, y, w, nsrc, bvalid;
    int src[4];
    double coef[4];
};

// Fill c->now for step k.step (below nsteps) from the pool bookkeeping k and the
// step's set sd (index id); cn: cn_rho of the step.  One thread.
template <typename SD>
__device__ __forceinline__ void step_setup(Args& a, Ctl* c, const Book& k, SD& sd, int id, double cn) {
    StepNow& w = c->now;
    const double rho = a.cn_rho && k.step > a.step0 ? cn : 0.0, theta = sd.theta, dt = sd.dt;
    w.set = id;
    w.cth = dt * theta;
    w.cex = dt * (1.0 - theta);
    w.rho = rho;
    w.expl = theta >= 1.0 ? EXPL_NONE : (rho > 0.0 ? EXPL_IDENTITY : EXPL_CORR);
    w.anchor = a.mixed && (k.step - a.step0) % a.anchor_every == 0;
    w.V = a.pool[k.cur];
    w.Y = a.pool[k.y];
    w.W = a.Wb[k.w];
    w.Wp = a.Wb[k.w ^ 1];
    w.B = a.bpool[k.y];
    bool lin = a.bpool[0] != nullptr;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int b = k.src[q < k.nsrc ? q : 0];
        if (q < k.nsrc) lin = lin && ((k.bvalid >> b) & 1);
        w.coef[q] = q < k.nsrc ? k.coef[q] : 0.0;
        w.H[q] = a.pool[b];
        w.Hb[q] = a.bpool[b];
    }
    w.lin = lin;
    w.fl1 = sd.fl1; w.bu1 = sd.bu1; w.bc1 = sd.bc1;
    w.fl2 = sd.fl2; w.bu2 = sd.bu2; w.bc2 = sd.bc2;
    w.s1 = sd.s1; w.s2 = sd.s2; w.w1 = sd.w1; w.w2 = sd.w2;
}

// Whether the step runs the FP64 correlation of V^{n-1}: for the explicit part
// (theta < 1, unless it comes from the previous step's equation), or to anchor
// B V^{n-1} in the mixed form.
__device__ __forceinline__ bool needs_explicit_fft(Args& a, CtlK& c) {
    return a.mixed ? c.now.anchor != 0 : c.now.expl == EXPL_CORR;
}

// Column pass of the correlation on the intermediate X (transposed half
// spectra); L/2 blocks for the L/2 + 1 columns.  Columns 0 (DC) and L/2 (Nyquist)
// hold real values (the row transforms of real rows; the row c2r kernels read
// only their real parts), so block 0 filters both as one complex column
// (mul_real_pair): a launch of L/2 + 1 blocks would end with one block running
// alone after the last full set of resident blocks had finished.
//
// FP64: the spectrum is read after the forward transform; held in registers
// from the start it costs the 3072-point pass (E = 4) its second block per CU
// (45 -> 60 us at 2048^2).  FP32, half the registers: fetched up front.
// CONJ (adjoint march): multiply by the conjugate spectrum, which applies B^T
// (the correlation with the reflected kernel).
template <int L, int E, typename C, bool CONJ = false>
__global__ __launch_bounds__(L / E) void ks_cols(const MarchArgs* __restrict__ A, const Ctl* __restrict__ Cs, int k) {
    Args& a = plan_args(A);
    CtlK& c = plan_ctl(Cs);
    if (halted(a, c, k) || (k == 0 && !needs_explicit_fft(a, c)) || (k == 1 && c.now.lin)) return;
    constexpr int T = L / E;
    __shared__ C lds[lds_slots(L)];
    __shared__ double2 tw4[tw_slots<L, E>()];
    load_twiddles<L, E>(GP<double2>(a.tw), tw4);
    const int n = a.n, col = blockIdx.x, tid = threadIdx.x;
    C reg[E];
    if (col == 0) {
        const GP<C> x0 = xbuf<C>(a), xh(x0, (size_t)(L / 2) * n);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int idx = tid + e * T;
            reg[e] = idx < n ? CplxOps<C>::make(x0[idx].x, xh[idx].x) : CplxOps<C>::make(0, 0);
        }
        fft_block<L, E, false>(reg, lds, tw4);
        const GP<C> s0 = specbuf<C>(a);
        mul_real_pair<L, E, CONJ>(reg, lds, s0, GP<C>(s0, (size_t)(L / 2) * L));
        fft_block<L, E, true>(reg, lds, tw4);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int idx = tid + e * T;
            if (idx < n) {
                x0.put(idx, CplxOps<C>::make(reg[e].x, 0));
                xh.put(idx, CplxOps<C>::make(reg[e].y, 0));
            }
        }
        return;
    }
    const GP<C> xc(xbuf<C>(a), (size_t)col * n), sc(specbuf<C>(a), (size_t)col * L);
    if constexpr (sizeof(C) == sizeof(float2)) {
        C sp[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int idx = tid + e * T;
            reg[e] = idx < n ? xc[idx] : CplxOps<C>::make(0, 0);
            sp[e] = sc[idx];              // spectrum fetched up front, used after the forward FFT
        }
        fft_block<L, E, false>(reg, lds, tw4);
#pragma unroll
        for (int e = 0; e < E; ++e) reg[e] = CONJ ? cmulc(reg[e], sp[e]) : cmul(reg[e], sp[e]);
    } else {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int idx = tid + e * T;
            reg[e] = idx < n ? xc[idx] : CplxOps<C>::make(0, 0);
        }
        fft_block<L, E, false>(reg, lds, tw4);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const C sv = sc[tid + e * T];
            reg[e] = CONJ ? cmulc(reg[e], sv) : cmul(reg[e], sv);
        }
    }
    fft_block<L, E, true>(reg, lds, tw4);
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int idx = tid + e * T;
        if (idx < n) xc.put(idx, reg[e]);
    }
}

// The FP64 pass of the mixed form's anchor steps, its spectrum fetched up front.
// Apart from ks_cols for reproducibility only, neither faster nor more exact: with
// it the mixed form keeps its results bit for bit, while a change of the rounding
// here moves them by 2e-9 of the deltas (its error is about 1e-8, its bound 1e-6).
template <int L, int E>
__global__ __launch_bounds__(L / E) void ks_cols_anchor(const MarchArgs* __restrict__ A, const Ctl* __restrict__ Cs) {
    using C = double2;
    Args& a = plan_args(A);
    CtlK& c = plan_ctl(Cs);
    if (halted(a, c, 0) || !c.now.anchor) return;
    constexpr int T = L / E;
    __shared__ C lds[lds_slots(L)];
    __shared__ double2 tw4[tw_slots<L, E>()];
    load_twiddles<L, E>(GP<double2>(a.tw), tw4);
    const int n = a.n, col = blockIdx.x, tid = threadIdx.x;
    C reg[E];
    if (col == 0) {
        const GP<C> x0 = xbuf<C>(a), xh(x0, (size_t)(L / 2) * n);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int idx = tid + e * T;
            reg[e] = idx < n ? CplxOps<C>::make(x0[idx].x, xh[idx].x) : CplxOps<C>::make(0, 0);
        }
        fft_block<L, E, false>(reg, lds, tw4);
        const GP<C> s0 = specbuf<C>(a);
        mul_real_pair<L, E, false>(reg, lds, s0, GP<C>(s0, (size_t)(L / 2) * L));
        fft_block<L, E, true>(reg, lds, tw4);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int idx = tid + e * T;
            if (idx < n) {
                x0.put(idx, CplxOps<C>::make(reg[e].x, 0));
                xh.put(idx, CplxOps<C>::make(reg[e].y, 0));
            }
        }
        return;
    }
    const GP<C> xc(xbuf<C>(a), (size_t)col * n), sc(specbuf<C>(a), (size_t)col * L);
    C sp[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int idx = tid + e * T;
        reg[e] = idx < n ? xc[idx] : CplxOps<C>::make(0, 0);
        sp[e] = sc[idx];                  // spectrum fetched up front, used after the forward FFT
    }
    fft_block<L, E, false>(reg, lds, tw4);
#pragma unroll
    for (int e = 0; e < E; ++e) reg[e] = cmul(reg[e], sp[e]);
    fft_block<L, E, true>(reg, lds, tw4);
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int idx = tid + e * T;
        if (idx < n) xc.put(idx, reg[e]);
    }
}

// Forward FFT of the row pair (ra, ra+1) of the FP64 grid U at the step start
// (mixed form: the FP64 correlation of V^{n-1}).
template <int L, int E>
__global__ __launch_bounds__(L / E) void ks_rows_fwd(const MarchArgs* __restrict__ A, const Ctl* __restrict__ Cs);

// The packed spectrum of the row pair (ra, ra+1) from the transposed half
// spectra, into the canonical registers: z[k] = X_a[k] + i X_b[k] for k <= L/2
// and z[L-k] = conj(X_a[k]) + i conj(X_b[k]) (imaginary parts dropped at DC and
// Nyquist).  Item idx is frequency (idx >> 1) of row ra + (idx & 1), so a lane
// pair reads the 32 contiguous bytes of one frequency once; the pair swaps its
// values, the even lane forms z[k], the odd one z[L-k], and both go through LDS
// to the canonical layout.
constexpr int rows_inv_items(int L, int E) { return (L + 2 + L / E - 1) / (L / E); }

// The gather's reads: item it of a thread.
template <int L, int E, typename C, int NI>
__device__ __forceinline__ void rows_inv_read(C (&v)[NI], GP<C> X, int n, int ra, bool hasb) {
    constexpr int T = L / E;
#pragma unroll
    for (int it = 0; it < NI; ++it) {
        const int idx = threadIdx.x + it * T;
        const int kk = idx >> 1, r = idx & 1;
        const bool in = kk <= L / 2;
        v[it] = (in && (r == 0 || hasb)) ? X[kk * n + ra + r] : CplxOps<C>::make(0, 0);
    }
}

// The exchange of what rows_inv_read read.
template <int L, int E, typename C, int NI>
__device__ __forceinline__ void rows_inv_exchange(C (&reg)[E], C* lds, const C (&v)[NI]) {
    constexpr int T = L / E;
    const int tid = threadIdx.x;
#pragma unroll
    for (int it = 0; it < NI; ++it) {
        const int idx = tid + it * T;
        const int kk = idx >> 1, r = idx & 1;
        const bool in = kk <= L / 2;
        // every lane of the wave takes part in the swap (pairs never straddle the range end)
        const C u = CplxOps<C>::make(__shfl_xor(v[it].x, 1), __shfl_xor(v[it].y, 1));
        const bool real_bin = kk == 0 || kk == L / 2;
        const C ta = r == 0 ? v[it] : u, tb = r == 0 ? u : v[it];
        const C ha = CplxOps<C>::make(ta.x, real_bin ? 0 : ta.y);
        const C hb = CplxOps<C>::make(tb.x, real_bin ? 0 : tb.y);
        if (in && r == 0) lds[lds_slot(kk)] = CplxOps<C>::make(ha.x - hb.y, ha.y + hb.x);
        if (in && r == 1 && kk > 0 && kk < L / 2)
            lds[lds_slot(L - kk)] = CplxOps<C>::make(ha.x + hb.y, hb.x - ha.y);
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) reg[e] = lds[lds_slot(tid + e * T)];
}

template <int L, int E, typename C>
__device__ __forceinline__ void rows_inv_gather(C (&reg)[E], C* lds, GP<C> X, int n, int ra, bool hasb) {
    C v[rows_inv_items(L, E)];
    rows_inv_read<L, E>(v, X, n, ra, hasb);
    rows_inv_exchange<L, E>(reg, lds, v);
}

// Row inverse FFT of the pairs (2p, 2p+1) with a fused epilogue.
// MODE 0 (once per step, FP64): E = V + dt(1-theta)((D - r_omega) V + B V) into wprev
//         (theta < 1), and B V into BV (mixed form);
// MODE 1 (FP64 iteration):  R = W + dt theta((D - r_omega) Y + B Y) - Y;
// MODE 2 (mixed iteration): B Y = (k == 1 in an anchor step ? BV : B Y) + B32(increment)
//         into BY, then R as in MODE 1 with that B Y (k == 1 elsewhere: BY still holds
//         the previous step's last B Y, the carried B V^{n-1}).
// Adjoint march (B^T from a CONJ column pass, D^T the transposed stencil):
// MODE 3 (iteration): R = Ybar + dt theta ((D^T - r_omega) lam + B^T lam) - lam,
//         with Ybar in W and lam the iterate;
// MODE 4 (once per step, theta < 1): W = mu + dt (1 - theta)((D^T - r_omega) mu + B^T mu),
//         mu in pool[cur]: the cotangent of V^{n-1}.
template <int L, int E, int MODE>
__global__ __launch_bounds__(L / E) void ks_rows_inv(const MarchArgs* __restrict__ A,
                                                     const Ctl* __restrict__ Cs, int k) {
    Args& a = plan_args(A);
    CtlK& c = plan_ctl(Cs);
    if (halted(a, c, k) || ((MODE == 0 || MODE == 4) && !needs_explicit_fft(a, c)) ||
        (MODE == 1 && k == 1 && c.now.lin))               // ks_begin_lin ran instead
        return;
    using C = typename std::conditional<MODE == 2, float2, double2>::type;
    constexpr int T = L / E;
    const int n = a.n, np = (n + 1) >> 1;
    const int p = xcd_remap(blockIdx.x, gridDim.x);
    if (p >= np) return;
    __shared__ C lds[lds_slots(L)];
    __shared__ double2 tw4[tw_slots<L, E>()];
    load_twiddles<L, E>(GP<double2>(a.tw), tw4);
    const int ra = 2 * p, rb = 2 * p + 1;
    const bool hasb = rb < n;
    const int tid = threadIdx.x;
    C reg[E];
    if constexpr (MODE == 1 || MODE >= 3) {
        // everything but the correlation's term first: its reads need no transform and are in
        // flight with the gather's, and only stores follow the transform.  The two
        // rows share their stencils' reads (twelve nodes for both).  Per launch at
        // 2048^2 56 -> 47 us, at 512^2 9.9 -> 8.5, at 64^2 8.0 -> 6.7; the adjoint's,
        // with the edges as weights instead of a path of their own, at 512^2 13.1 -> 9.0.
        const GP<double> U(MODE == 4 ? c.now.V : c.now.Y), W(MODE == 4 ? c.now.V : c.now.W),
            R(MODE == 4 ? c.now.W : a.R), Bout(c.now.B);
        const double cf = MODE == 4 ? c.now.cex : c.now.cth, r_omega = a.r_omega;
        const StencilArgs st = stencil(a);
        const int o0 = max(ra - 1, 0) * n, o1 = ra * n, o2 = min(rb, n - 1) * n, o3 = min(rb + 1, n - 1) * n;
        // up to 1024 the gather's reads go first and are in flight with the stencil's (64^2
        // 6.8 -> 6.0, 128^2 6.3 -> 4.9, 512^2 8.5 -> 7.6); above, their registers would cost
        // blocks in flight
        constexpr bool AHEAD = L <= 1024;
        C xv[rows_inv_items(L, E)];
        if constexpr (AHEAD) rows_inv_read<L, E>(xv, xbuf<C>(a), n, ra, hasb);
        double g[E][2];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int j = min(tid + e * T, n - 1), jm = max(j - 1, 0), jp = min(j + 1, n - 1);
            const double a0 = U[o0 + jm], a1 = U[o0 + j], a2 = U[o0 + jp], b0 = U[o1 + jm], b1 = U[o1 + j], b2 = U[o1 + jp];
            const double c0 = U[o2 + jm], c1 = U[o2 + j], c2 = U[o2 + jp], d0 = U[o3 + jm], d1 = U[o3 + j], d2 = U[o3 + jp];
            if constexpr (MODE == 1) {
                g[e][0] = W[o1 + j] + cf * (D_of(st, ra, j, b1, a1, c1, b0, b2, a0, a2, c0, c2) - r_omega * b1) - b1;
                g[e][1] = W[o2 + j] + cf * (D_of(st, rb, j, c1, b1, d1, c0, c2, b0, b2, d0, d2) - r_omega * c1) - c1;
            } else {
                const double ga = cf * (DT_of(st, ra, j, b1, a1, c1, b0, b2, a0, a2, c0, c2) - r_omega * b1);
                const double gb = cf * (DT_of(st, rb, j, c1, b1, d1, c0, c2, b0, b2, d0, d2) - r_omega * c1);
                g[e][0] = MODE == 4 ? b1 + ga : W[o1 + j] + ga - b1;
                g[e][1] = MODE == 4 ? c1 + gb : W[o2 + j] + gb - c1;
            }
            if constexpr (L > 1024) asm volatile("" : "+v"(g[e][0]), "+v"(g[e][1])::"memory");
        }
        // formed here: left to the compiler, the arithmetic moves behind the transform
        // and the 14 values read per element stay in registers instead of g's two.  Up
        // to 1024 all elements' reads are in flight together, above one element's.
#pragma unroll
        for (int e = 0; e < E; ++e) asm volatile("" : "+v"(g[e][0]), "+v"(g[e][1]));
        if constexpr (AHEAD) rows_inv_exchange<L, E>(reg, lds, xv);
        else rows_inv_gather<L, E>(reg, lds, xbuf<C>(a), n, ra, hasb);
        fft_block<L, E, true>(reg, lds, tw4);
        const bool keepB = MODE == 1 && c.now.B != nullptr;       // B Y of the iterate, for the start of later steps
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int j = tid + e * T;
            if (j >= n) continue;
            if (keepB) Bout.put(o1 + j, reg[e].x);
            R.put(o1 + j, g[e][0] + cf * reg[e].x);
            if (hasb) {
                if (keepB) Bout.put(o2 + j, reg[e].y);
                R.put(o2 + j, g[e][1] + cf * reg[e].y);
            }
        }
        return;
    }
    if constexpr (MODE == 2 && L <= 1536) {
        // the mixed form likewise: the epilogue's sums in the same order as below, from values
        // held across the transform (march at 300^2 15.4 -> 14.4 ms, 512^2 29.4 -> 28.4,
        // 1000^2 84.4 -> 82.4).  Up to 1024 the gather's reads go first; at 1536 that takes
        // 131 registers and 47.9 ms at 700^2 against 44.8, above 1536 the held values alone
        // cost blocks in flight.
        const GP<double> U(c.now.Y), W(c.now.W), R(a.R), BY(a.BY), base((k == 1 && c.now.anchor) ? a.BV : a.BY);
        const double cf = c.now.cth, r_omega = a.r_omega, c0 = -1.0;
        const StencilArgs st = stencil(a);
        const int o0 = max(ra - 1, 0) * n, o1 = ra * n, o2 = min(rb, n - 1) * n, o3 = min(rb + 1, n - 1) * n;
        constexpr bool AHEAD = L <= 1024;
        C xv[rows_inv_items(L, E)];
        if constexpr (AHEAD) rows_inv_read<L, E>(xv, xbuf<C>(a), n, ra, hasb);
        double d[E][2], u[E][2], w[E][2], b[E][2];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int j = min(tid + e * T, n - 1), jm = max(j - 1, 0), jp = min(j + 1, n - 1);
            const double a0 = U[o0 + jm], a1 = U[o0 + j], a2 = U[o0 + jp], b0 = U[o1 + jm], b1 = U[o1 + j], b2 = U[o1 + jp];
            const double c0_ = U[o2 + jm], c1 = U[o2 + j], c2 = U[o2 + jp], d0 = U[o3 + jm], d1 = U[o3 + j], d2 = U[o3 + jp];
            d[e][0] = D_of(st, ra, j, b1, a1, c1, b0, b2, a0, a2, c0_, c2);
            d[e][1] = D_of(st, rb, j, c1, b1, d1, c0_, c2, b0, b2, d0, d2);
            u[e][0] = b1;
            u[e][1] = c1;
            w[e][0] = W[o1 + j];
            w[e][1] = W[o2 + j];
            b[e][0] = base[o1 + j];
            b[e][1] = base[o2 + j];
            if constexpr (!AHEAD) asm volatile("" : "+v"(d[e][0]), "+v"(d[e][1])::"memory");
        }
#pragma unroll
        for (int e = 0; e < E; ++e)
            asm volatile("" : "+v"(d[e][0]), "+v"(d[e][1]), "+v"(u[e][0]), "+v"(u[e][1]), "+v"(w[e][0]), "+v"(w[e][1]),
                         "+v"(b[e][0]), "+v"(b[e][1]));
        if constexpr (AHEAD) rows_inv_exchange<L, E>(reg, lds, xv);
        else rows_inv_gather<L, E>(reg, lds, xbuf<C>(a), n, ra, hasb);
        fft_block<L, E, true>(reg, lds, tw4);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int j = tid + e * T;
            if (j >= n) continue;
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                if (r == 1 && !hasb) break;
                const int o = (ra + r) * n + j;
                double bu = r == 0 ? (double)reg[e].x : (double)reg[e].y;
                bu += b[e][r];
                BY.put(o, bu);
                R.put(o, w[e][r] + cf * (d[e][r] + bu - r_omega * u[e][r]) + c0 * u[e][r]);
            }
        }
        return;
    }
    rows_inv_gather<L, E>(reg, lds, xbuf<C>(a), n, ra, hasb);
    fft_block<L, E, true>(reg, lds, tw4);
    constexpr bool EXPL = MODE == 0;
    const GP<double> U(EXPL ? c.now.V : c.now.Y), P0(EXPL ? c.now.V : c.now.W);
    const GP<double> out(MODE == 0 ? c.now.Wp : a.R);
    const double cf = EXPL ? c.now.cex : c.now.cth, c0 = EXPL ? 0.0 : -1.0;
    const bool want_r = MODE != 0 || c.now.expl != EXPL_NONE;
    const GP<double> base((MODE == 2 && k == 1 && c.now.anchor) ? a.BV : a.BY), BY(a.BY), BV(a.BV);
    const bool mixed = a.mixed != 0;
    const StencilArgs st = stencil(a);
    const double r_omega = a.r_omega;
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int j = tid + e * T;
        if (j >= n) continue;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            if (r == 1 && !hasb) break;
            const int i = ra + r, o = i * n + j;
            double bu = r == 0 ? (double)reg[e].x : (double)reg[e].y;
            if constexpr (MODE == 2) {
                bu += base[o];
                BY.put(o, bu);
            }
            if constexpr (MODE == 0) {
                if (mixed) BV.put(o, bu);
            }
            if (want_r) {
                const double u = U[o];
                out.put(o, P0[o] + cf * (apply_D(U, st, i, j, u) + bu - r_omega * u) + c0 * u);
            }
        }
    }
}

// The same affine forms without the correlation (zero Levy measure); one
// block per grid row.
template <bool EXPLICIT>
__global__ __launch_bounds__(256) void ks_affine_noB(const MarchArgs* __restrict__ A,
                                                     const Ctl* __restrict__ Cs, int k) {
    Args& a = plan_args(A);
    CtlK& c = plan_ctl(Cs);
    if (halted(a, c, k) || (EXPLICIT && c.now.expl == EXPL_NONE)) return;
    const int n = a.n;
    const int i = xcd_remap(blockIdx.x, gridDim.x);   // neighbouring rows on one XCD (stencil reads share L2)
    if (i >= n) return;
    const GP<double> U(EXPLICIT ? c.now.V : c.now.Y), P0(EXPLICIT ? c.now.V : c.now.W), out(EXPLICIT ? c.now.Wp : a.R);
    const double cf = EXPLICIT ? c.now.cex : c.now.cth, c0 = EXPLICIT ? 0.0 : -1.0, r_omega = a.r_omega;
    const StencilArgs st = stencil(a);
    for (int j = threadIdx.x; j < n; j += blockDim.x) {
        const int o = i * n + j;
        const double u = U[o];
        const double d = apply_D(U, st, i, j, u);
        out.put(o, P0[o] + cf * (d - r_omega * u) + c0 * u);
    }
}

// Mixed form, steps between anchors whose explicit part does not come from the
// previous step's equation (explicit_by_identity): B V^{n-1} is carried from
// the previous step, whose last iteration left B Y in BY (FP64 sums of FP32
// correlations of the increments; it misses B applied to the final increment,
// which is below the stopping tolerance), and the explicit part
// E = V + dt (1 - theta)((D - r_omega) V + B V) (theta < 1) is formed without
// a correlation.  One block per grid row.
static __global__ __launch_bounds__(256) void ks_carry(const MarchArgs* __restrict__ A, const Ctl* __restrict__ Cs) {
    Args& a = plan_args(A);
    CtlK& c = plan_ctl(Cs);
    if (halted(a, c, 0) || !a.mixed || c.now.anchor || c.now.expl != EXPL_CORR) return;
    const int n = a.n;
    const int i = xcd_remap(blockIdx.x, gridDim.x);   // neighbouring rows on one XCD (stencil reads share L2)
    if (i >= n) return;
    const GP<double> U(c.now.V), E(c.now.Wp), BY(a.BY);
    const double cf = c.now.cex, r_omega = a.r_omega;
    const StencilArgs st = stencil(a);
    for (int j = threadIdx.x; j < n; j += blockDim.x) {
        const int o = i * n + j;
        const double u = U[o];
        E.put(o, u + cf * (apply_D(U, st, i, j, u) + BY[o] - r_omega * u));
    }
}

// Explicit part from the previous step's implicit equation (EXPL_IDENTITY), over
// the W it comes from: E = V + rho (V - W); one block per grid row.  Mixed form:
// not in anchor steps.  Steps that ks_begin_lin takes form it there.
static __global__ __launch_bounds__(256) void ks_expl_identity(const MarchArgs* __restrict__ A,
                                                               const Ctl* __restrict__ Cs) {
    Args& a = plan_args(A);
    CtlK& c = plan_ctl(Cs);
    if (halted(a, c, 0) || c.now.expl != EXPL_IDENTITY || c.now.anchor || c.now.lin) return;
    const int n = a.n, i = blockIdx.x;
    if (i >= n) return;
    const double rho = c.now.rho;
    const GP<double> V(c.now.V), W(c.now.Wp);
    for (int j = threadIdx.x; j < n; j += blockDim.x) {
        const double v = V[i * n + j];
        W.put(i * n + j, v + rho * (v - W[i * n + j]));
    }
}

// Threads of ks_begin_lin, and the columns of its tiles for a grid side n: at
// most BEGIN_T - 4, so that one thread per column covers the start value with its
// stencil's neighbours (two more) and the gather's source columns (P more);
// rounded to whole cache lines where that fits.
constexpr int BEGIN_T = 256;
__host__ __device__ __forceinline__ int begin_cols(int n) {
    const int t = (n + BEGIN_T - 5) / (BEGIN_T - 4), c = (n + t - 1) / t, r = (c + 15) & ~15;
    return r <= BEGIN_T - 4 ? r : c;
}
// Tiles of TR rows that cover an n x n grid.
__host__ __device__ __forceinline__ int begin_tiles(int n, int TR) {
    const int c = begin_cols(n);
    return ((n + TR - 1) / TR) * ((n + c - 1) / c);
}

// The start of an FP64 step whose B Y^0 comes by linearity (StepNow::lin),
// without any transform, on a tile of TR rows:
//   E = V + rho (V - W_prev) (EXPL_IDENTITY; V when theta = 1; W_prev where the
//       correlation left E there),
//   W = T^SL E, the row weights first, then the column taps from LDS,
//   Y^0 = sum_q coef_q V^{src_q},  B Y^0 = sum_q coef_q B V^{src_q} (stored products),
//   R = W + dt theta ((D - r_omega) Y^0 + B Y^0) - Y^0, the residual of iteration 1.
// One streaming pass (13 n^2 reads and writes of FP64) in place of three kernels
// of 3, 7 and 8 that passed E, W and Y^0 through memory: 92 us instead of 17 + 62
// + 66 at 2048^2, 9.1 instead of 4.8 + 7.8 + 7.0 at 512^2.  A tile's start value is
// formed once per node and halo row and its stencil reads LDS, so the history is
// read (TR + 2) / TR times; the terms past the count of stored grids repeat the
// first at weight zero (StepNow), so that one loop serves every count.
template <int P, int TR>
__global__ __launch_bounds__(BEGIN_T) void ks_begin_lin(const MarchArgs* __restrict__ A, const Ctl* __restrict__ Cs) {
    Args& a = plan_args(A);
    CtlK& c = plan_ctl(Cs);
    if (halted(a, c, 0) || !c.now.lin) return;
    constexpr int T = BEGIN_T, NS = 4;
    __shared__ double ys[TR + 2][T];              // Y^0, rows r0 - 1 .., columns c0 - 1 ..
    __shared__ double ec[TR][T];                  // row-combined E, columns k0 ..
    const int n = a.n, tcw = begin_cols(n), tc = (n + tcw - 1) / tcw, nt = ((n + TR - 1) / TR) * tc;
    if ((int)blockIdx.x >= nt) return;
    const int tile = xcd_remap(blockIdx.x, nt);   // neighbouring tiles on one XCD (halo rows share L2)
    const int r0 = (tile / tc) * TR, c0 = (tile % tc) * tcw, c1 = min(n, c0 + tcw), t = threadIdx.x;
    const GP<double> V(c.now.V), Wp(c.now.Wp), W(c.now.W), Y(c.now.Y), R(a.R), Bout(c.now.B), w1(c.now.w1), w2t(c.now.w2);
    const GP<int> s1(c.now.s1), s2(c.now.s2);
    const GP<double> H[NS] = {GP<double>(c.now.H[0]), GP<double>(c.now.H[1]), GP<double>(c.now.H[2]),
                              GP<double>(c.now.H[3])};
    const GP<double> Hb[NS] = {GP<double>(c.now.Hb[0]), GP<double>(c.now.Hb[1]), GP<double>(c.now.Hb[2]),
                               GP<double>(c.now.Hb[3])};
    double cf[NS];
#pragma unroll
    for (int q = 0; q < NS; ++q) cf[q] = c.now.coef[q];
    const double cth = c.now.cth, r_omega = a.r_omega, rho = c.now.rho;
    const int expl = c.now.expl;
    const StencilArgs st = stencil(a);
    auto e_at = [&](int o) -> double {
        if (expl == EXPL_CORR) return Wp[o];
        const double v = V[o];
        return expl == EXPL_IDENTITY ? v + rho * (v - Wp[o]) : v;
    };
    // start value of this thread's column, its rows and the two around them
    double y[TR + 2];
    {
        const int j = min(max(c0 - 1 + t, 0), n - 1);
#pragma unroll
        for (int q = 0; q < TR + 2; ++q) {
            const int o = min(max(r0 - 1 + q, 0), n - 1) * n + j;
            double v = cf[0] * H[0][o];
#pragma unroll
            for (int h = 1; h < NS; ++h) v += cf[h] * H[h][o];
            y[q] = v;
            ys[q][t] = v;
        }
    }
    // E's source rows combined by the row weights.  Away from the grid's ends the
    // source rows of consecutive rows are consecutive (one set of reads per tile).
    const int k0 = s2[c0], k = k0 + t;
    if (k <= s2[c1 - 1] + P) {
        const int rl = min(TR, n - r0), a0 = s1[r0];
        bool run = true;
#pragma unroll
        for (int r = 1; r < TR; ++r) run = run && (r >= rl || s1[r0 + r] == a0 + r);
        if (run) {
            double e[TR + P];
#pragma unroll
            for (int q = 0; q < TR + P; ++q) e[q] = e_at(min(a0 + q, n - 1) * n + k);
#pragma unroll
            for (int r = 0; r < TR; ++r) {
                double v = 0.0;
#pragma unroll
                for (int q = 0; q <= P; ++q) v += w1[min(r0 + r, n - 1) * (P + 1) + q] * e[r + q];
                ec[r][t] = v;
            }
        } else {
            for (int r = 0; r < rl; ++r) {
                double v = 0.0;
                for (int q = 0; q <= P; ++q) v += w1[(r0 + r) * (P + 1) + q] * e_at((s1[r0 + r] + q) * n + k);
                ec[r][t] = v;
            }
        }
    }
    __syncthreads();
    const int j = c0 - 1 + t;
    if (t == 0 || j >= c1) return;
    const int b0 = s2[j] - k0;
    double w2[P + 1];
#pragma unroll
    for (int b = 0; b <= P; ++b) w2[b] = w2t[j * (P + 1) + b];
    const bool rec = a.segE && expl != EXPL_NONE;
    const GP<double> segE(GP<double>(a.segE), rec ? (size_t)(c.step - a.seg_base) * n * n : 0);
#pragma unroll
    for (int r = 0; r < TR; ++r) {
        const int i = r0 + r;
        if (i >= n) break;
        const int o = i * n + j;
        double bu = 0.0, w = 0.0;
#pragma unroll
        for (int q = 0; q < NS; ++q) bu += cf[q] * Hb[q][o];
#pragma unroll
        for (int b = 0; b <= P; ++b) w += w2[b] * ec[r][b0 + b];
        const double u = y[r + 1];
        const double d = D_of(st, i, j, u, y[r], y[r + 2], ys[r + 1][t - 1], ys[r + 1][t + 1], ys[r][t - 1],
                              ys[r][t + 1], ys[r + 2][t - 1], ys[r + 2][t + 1]);
        W.put(o, w);
        Y.put(o, u);
        Bout.put(o, bu);
        R.put(o, w + cth * (d + bu - r_omega * u) - u);
        if (rec) segE.put(o, e_at(o));
    }
}

// Forward FFT of the row pair held in reg (canonical layout) into the
// transposed half spectra X[k2 * n + row].
// X2, if not null, receives a second copy.
template <int L, int E, typename C>
__device__ __forceinline__ void rows_fwd_store(C (&reg)[E], C* lds, const double2* tw4, GP<C> X, int n, int ra,
                                               bool hasb, const C* X2 = nullptr) {
    constexpr int T = L / E;
    using Rl = typename CplxOps<C>::real;
    const int tid = threadIdx.x;
    __syncthreads();
    fft_block<L, E, false>(reg, lds, tw4);
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; ++e) lds[tid + e * T] = reg[e];
    __syncthreads();
    // item idx = frequency (idx >> 1) of row ra + (idx & 1): the two rows of a
    // frequency are adjacent in X, so a lane pair stores them as one 32-byte piece
    constexpr int NI = (L + 2 + T - 1) / T;
#pragma unroll
    for (int it = 0; it < NI; ++it) {
        const int idx = tid + it * T;
        const int kk = idx >> 1, r = idx & 1;
        if (kk > L / 2 || (r == 1 && !hasb)) continue;
        const C z = lds[kk], w = lds[kk == 0 ? 0 : L - kk];
        const C v = r == 0 ? CplxOps<C>::make(Rl(0.5) * (z.x + w.x), Rl(0.5) * (z.y - w.y))
                           : CplxOps<C>::make(Rl(0.5) * (z.y + w.y), Rl(-0.5) * (z.x - w.x));
        X.put(kk * n + ra + r, v);
        if (X2) GP<C>(X2).put(kk * n + ra + r, v);
    }
}

template <int L, int E>
__global__ __launch_bounds__(L / E) void ks_rows_fwd(const MarchArgs* __restrict__ A, const Ctl* __restrict__ Cs) {
    Args& a = plan_args(A);
    CtlK& c = plan_ctl(Cs);
    if (halted(a, c, 0) || !c.now.anchor) return;
    constexpr int T = L / E;
    const int n = a.n, np = (n + 1) >> 1;
    const int p = xcd_remap(blockIdx.x, gridDim.x);
    if (p >= np) return;
    __shared__ double2 lds[lds_slots(L)];
    __shared__ double2 tw4[tw_slots<L, E>()];
    load_twiddles<L, E>(GP<double2>(a.tw), tw4);
    const int ra = 2 * p, rb = 2 * p + 1;
    const bool hasb = rb < n;
    const GP<double> U(c.now.V);
    double2 reg[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int j = threadIdx.x + e * T;
        reg[e] = j < n ? make_double2(U[ra * n + j], hasb ? U[rb * n + j] : 0.0) : make_double2(0.0, 0.0);
    }
    rows_fwd_store<L, E>(reg, lds, tw4, xbuf<double2>(a), n, ra, hasb);
}

// Semi-Lagrangian gather W = (T_1 (x) T_2) E (order P), starting value Y^0 into
// the iterate buffer, and (FFT) the row transform of Y^0 (FP64) or, in the
// mixed form, of Y^0 - V^{n-1} (FP32); one row pair per block.
template <int L, int E, int P, bool FFT, bool MIXED>
__global__ __launch_bounds__(L / E) void ks_sl(const MarchArgs* __restrict__ A, const Ctl* __restrict__ Cs) {
    Args& a = plan_args(A);
    CtlK& c = plan_ctl(Cs);
    // FP64 steps whose B Y^0 comes by linearity need no row transform of Y^0:
    // ks_begin_lin does their gather and start value
    if (halted(a, c, 0) || (FFT && !MIXED && c.now.lin)) return;
    constexpr int T = L / E;
    using C = typename std::conditional<MIXED, float2, double2>::type;
    const int n = a.n, np = (n + 1) >> 1;
    const int p = xcd_remap(blockIdx.x, gridDim.x);
    if (p >= np) return;
    __shared__ C lds[FFT ? lds_slots(L) : 1];
    __shared__ double2 tw4[FFT ? tw_slots<L, E>() : 1];
    if constexpr (FFT) load_twiddles<L, E>(GP<double2>(a.tw), tw4);
    const int ra = 2 * p, rb = 2 * p + 1;
    const bool hasb = rb < n;
    const int tid = threadIdx.x;
    const GP<double> Ex(c.now.expl != EXPL_NONE ? c.now.Wp : c.now.V);   // explicit part E_s
    const GP<double> W(c.now.W), Y(c.now.Y), V(c.now.V), w1t(c.now.w1), w2t(c.now.w2);
    const GP<int> s1(c.now.s1), s2(c.now.s2);
    const int nsrc = c.nsrc;
    const GP<double> H[4] = {GP<double>(c.now.H[0]), GP<double>(c.now.H[1]), GP<double>(c.now.H[2]), GP<double>(c.now.H[3])};
    double cf[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) cf[q] = c.now.coef[q];
    // Two phases: the gathers and the history reads of every element first,
    // then the writes (the compiler cannot tell that W and Y alias none of the
    // read grids, so reads after writes would wait for each element in turn).
    double wv[E][2], yv[E][2], yf[E][2];   // W, Y^0, and the row-transform input
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int j = tid + e * T;
        wv[e][0] = wv[e][1] = yv[e][0] = yv[e][1] = yf[e][0] = yf[e][1] = 0.0;
        if (j < n) {
            const int b0 = s2[j];
            double w2[P + 1];
#pragma unroll
            for (int b = 0; b <= P; ++b) w2[b] = w2t[j * (P + 1) + b];
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                const int i = ra + r;
                if (r == 1 && !hasb) break;
                const int a0 = s1[i];
                double acc = 0.0;
#pragma unroll
                for (int aa = 0; aa <= P; ++aa) {
                    const int eo = (a0 + aa) * n + b0;
                    double s = 0.0;
#pragma unroll
                    for (int b = 0; b <= P; ++b) s += w2[b] * Ex[eo + b];
                    acc += w1t[i * (P + 1) + aa] * s;
                }
                const int o = i * n + j;
                wv[e][r] = acc;
                // unrolled with a predicate, so the history reads are all in flight together
                double y = 0.0;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (q < nsrc) y += cf[q] * H[q][o];
                yv[e][r] = y;
                yf[e][r] = MIXED ? y - V[o] : y;      // the mixed form transforms Y^0 - V^{n-1}
            }
        }
    }
    C reg[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int j = tid + e * T;
        double y0[2] = {0.0, 0.0};
        if (j < n) {
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                if (r == 1 && !hasb) break;
                const int o = (ra + r) * n + j;
                W.put(o, wv[e][r]);
                Y.put(o, yv[e][r]);
                y0[r] = yf[e][r];
            }
        }
        reg[e] = CplxOps<C>::make(y0[0], y0[1]);
    }
    if constexpr (FFT) rows_fwd_store<L, E>(reg, lds, tw4, xbuf<C>(a), n, ra, hasb);
}

// Axis-1 line solves R <- T_1^{-1} R: CPB adjacent columns x P chunks per block
// (thread = column + CPB * chunk); launched with CPB * P <= MAXT threads.
// MM: chunk capacity (at least ceil(n / P_cols)).
template <int CPB, int MAXT, int MM>
__global__ __launch_bounds__(MAXT) void ks_line_cols(const MarchArgs* __restrict__ A,
                                                     const Ctl* __restrict__ Cs, int k) {
    Args& a = plan_args(A);
    CtlK& c = plan_ctl(Cs);
    if (halted(a, c, k)) return;
    extern __shared__ double2 sbuf[];
    const int n = a.n, P = a.P_cols;
    const int cc = threadIdx.x % CPB, t = threadIdx.x / CPB;
    const int g = xcd_remap(blockIdx.x, gridDim.x);
    if (CPB * g >= n) return;
    const int col = g * CPB + cc;
    const int m = (n + P - 1) / P;
    const int s = t * m;
    const int cnt = col < n ? max(0, min(m, n - s)) : 0;
    const GP<double> R(a.R);
    double x[MM];
#pragma unroll
    for (int q = 0; q < MM; ++q) x[q] = q < cnt ? R[(s + q) * n + col] : 0.0;
    chunk_solve<MM>(x, s, cnt, cc, t, P, CPB, c.now.fl1, c.now.bu1, c.now.bc1, sbuf);
#pragma unroll
    for (int q = 0; q < MM; ++q)
        if (q < cnt) R.put((s + q) * n + col, x[q]);
}

// Axis-2 line solves of a row pair, the update Y += delta, the stopping-rule
// maximum err_k = max |delta| / max(1, |Y|), and (FFT) the row transform of the
// updated Y (FP64) or, in the mixed form, of delta (FP32) for the next iteration.
// MM: the chunk capacity, at least the longest chunk ceil(n / PR) of the
// launch's plans (at most 2E, since n <= L = 2 E PR); the line-solve sweeps run
// over all MM slots, so the host takes the smallest of E, 3E/2 and 2E that
// holds the chunks (24 instead of 32 at n = 2048, L = 3072: 65 -> 55 us alone).
template <int L, int E, bool FFT, bool MIXED, int MM = 2 * E>
__global__ __launch_bounds__(L / E) void ks_line_rows(const MarchArgs* __restrict__ A,
                                                     const Ctl* __restrict__ Cs, int k) {
    static_assert(MM <= 2 * E && MM % 2 == 0, "chunk capacity: even, at most 2E");
    Args& a = plan_args(A);
    CtlK& c = plan_ctl(Cs);
    if (halted(a, c, k)) return;
    constexpr int T = L / E, PR = T / 2;
    using C = typename std::conditional<MIXED, float2, double2>::type;
    const int n = a.n, np = (n + 1) >> 1;
    const int p = xcd_remap(blockIdx.x, gridDim.x);
    if (p >= np) return;
    // union: row buffer 2 (n + PR + 1) doubles (n <= L) | scan totals | FFT exchange buffer
    __shared__ double2 lds[L + (PR > L / 16 ? PR : L / 16) + 2];
    __shared__ double2 tw4[FFT ? tw_slots<L, E>() : 1];
    if constexpr (FFT) load_twiddles<L, E>(GP<double2>(a.tw), tw4);
    double* rows = reinterpret_cast<double*>(lds);
    const int ra = 2 * p, rb = 2 * p + 1;
    const bool hasb = rb < n;
    const int tid = threadIdx.x;
    const int m = (n + PR - 1) / PR;
    const int stride = n + PR + 1;
    const GP<double> Y(c.now.Y);
    // each thread reads its chunk of the residual row straight from memory: the
    // chunks of consecutive lanes are adjacent, so the reads stay coalesced
    const int r = tid / PR, ch = tid % PR;
    const int s = ch * m;
    const int cnt = (r == 1 && !hasb) ? 0 : max(0, min(m, n - s));
    double x[MM];
    {
        const int o = (r == 0 ? ra : rb) * n + s;
        if (((n | m) & 1) == 0) {
            // 16-byte loads: the chunk starts at an even element of a row of
            // even length, so every pair is aligned (half the load
            // instructions and addresses of element-wise reads)
            const GP<double2> R2(reinterpret_cast<const double2*>(a.R));
#pragma unroll
            for (int q = 0; q < MM / 2; ++q) {
                const double2 v = 2 * q < cnt ? R2[(o >> 1) + q] : make_double2(0.0, 0.0);
                x[2 * q] = v.x;
                x[2 * q + 1] = v.y;
            }
        } else {
            const GP<double> Rr(a.R);
#pragma unroll
            for (int q = 0; q < MM; ++q) x[q] = q < cnt ? Rr[o + q] : 0.0;
        }
    }
    // the iterate, every element read before any write of the update (reads
    // after those writes would wait element by element: the compiler cannot
    // separate them): at E = 4 with the residual, its latency behind the line solve;
    // above, and at L = 3072, after the solve, so that it is not held in registers across
    // it (at E = 4 of L = 3072 82 registers leave one block per CU: 45.3 -> 61.7 us).
    constexpr bool EARLY_Y = E <= 4 && L < 3072;
    double yoa[E], yob[E];
    auto read_iterate = [&] {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int j = tid + e * T;
            yoa[e] = j < n ? Y[ra * n + j] : 0.0;
            yob[e] = (j < n && hasb) ? Y[rb * n + j] : 0.0;
        }
    };
    if constexpr (EARLY_Y) read_iterate();
    chunk_solve<MM, (MM <= 4)>(x, s, cnt, r, ch, PR, 1, c.now.fl2, c.now.bu2, c.now.bc2, lds);
#pragma unroll
    for (int q = 0; q < MM; ++q)
        if (q < cnt) rows[r * stride + s + q + ch] = x[q];
    __syncthreads();
    if constexpr (!EARLY_Y) read_iterate();
    const unsigned inv_m = 0xFFFFFFFFu / (unsigned)m + 1;      // j / m = mulhi(j, inv_m) for j < 2^16, m > 1
    auto chunk_of = [&](int j) { return m > 1 ? (int)__umulhi((unsigned)j, inv_m) : j; };
    double emax = 0.0;
    C reg[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int j = tid + e * T;
        double ya = 0.0, yb = 0.0, da = 0.0, db = 0.0;
        if (j < n) {
            const int at = j + chunk_of(j);
            da = rows[at];
            ya = yoa[e] + da;
            Y.put(ra * n + j, ya);
            double ev = fabs(da) / fmax(1.0, fabs(ya));
            emax = (ev > emax || ev != ev) ? ev : emax;
            if (hasb) {
                db = rows[stride + at];
                yb = yob[e] + db;
                Y.put(rb * n + j, yb);
                ev = fabs(db) / fmax(1.0, fabs(yb));
                emax = (ev > emax || ev != ev) ? ev : emax;
            }
        }
        reg[e] = MIXED ? CplxOps<C>::make(da, db) : CplxOps<C>::make(ya, yb);
    }
    // block maximum: a wave reduction over the active lanes (T may be below
    // 64), the wave maxima through LDS, then one atomic per block
    // (non-negative doubles order like their bit patterns; NaN sorts above
    // +inf).  Same-address atomics serialise in the L2, so one per block
    // instead of one per wave shortens the tail of the kernel.
    constexpr int WL = T < 64 ? T : 64, NWV = (T + 63) / 64;
#pragma unroll
    for (int off = WL / 2; off > 0; off >>= 1) {
        const double o = __shfl_xor(emax, off, WL);
        emax = (o > emax || o != o) ? o : emax;
    }
    __shared__ double wmax[NWV];
    if ((tid & 63) == 0) wmax[tid >> 6] = emax;
    __syncthreads();
    if (tid == 0) {                       // issued before the row transform, which hides its latency
        double b = wmax[0];
#pragma unroll
        for (int w = 1; w < NWV; ++w) b = (wmax[w] > b || wmax[w] != wmax[w]) ? wmax[w] : b;
        atomicMax(&const_cast<Ctl*>(Cs + blockIdx.y)->err[(blockIdx.x + blockIdx.y * gridDim.x) & (NX - 1)][k],
                  (unsigned long long)__double_as_longlong(b));
    }
    if constexpr (FFT) rows_fwd_store<L, E>(reg, reinterpret_cast<C*>(lds), tw4, xbuf<C>(a), n, ra, hasb);
}

// Threads of ks_step_end: one wave, so that the verdict is a ballot.
constexpr int END_T = 64;

// End of a step: convergence verdict, history rotation, next starting value.
// One block per plan.  A chain of reads bounds it (control block, step list, set, pool
// pointers): each is one set of scalar reads, the bookkeeping stays in registers and is
// written once (reading and writing it in memory word by word: 5.0 us
// behind a step of the 512^2 march, now 4.5).
static __global__ __launch_bounds__(END_T) void ks_step_end(const MarchArgs* __restrict__ A, Ctl* __restrict__ Cs,
                                                            int kmax) {
    Args& a = plan_args(A);
    Ctl* c = Cs + blockIdx.y;
    CtlK& r = plan_ctl(Cs);
    int s = r.step, hold = r.hold, fail = r.fail, y = r.y, hc = r.hc, w = r.w, bv = r.bvalid;
    int h0 = r.hist[0], h1 = r.hist[1], h2 = r.hist[2], h3 = r.hist[3];
    // read here: none of these reads may move behind the writes below
    asm volatile("" : "+s"(s), "+s"(y), "+s"(hc), "+s"(w), "+s"(bv), "+s"(h0), "+s"(h1), "+s"(h2), "+s"(h3)::"memory");
    if (hold || s >= a.nsteps) return;
    // the next step's set, read ahead of the verdict
    const int s2 = s + 1, sn = s2 < a.nsteps ? s2 : s;
    const int id = kref(a.step_set + sn);
    const double cn = a.cn_rho ? (double)kref(a.cn_rho + sn) : 0.0;
    KRef<StepDesc> sd = kref(a.sets + id);
    if (fail) return;
    int kk = 0;
    double inc = 0.0;
    for (int q0 = 0; q0 <= kmax && kk == 0; q0 += END_T) {
        const int q = q0 + (int)threadIdx.x;
        const double e = q <= kmax ? err_max(r, q) : 0.0;
        const unsigned long long met = __ballot(q >= 1 && q <= kmax && e < a.tol);
        if (met) {
            const int lane = __ffsll(met) - 1;
            kk = q0 + lane;
            inc = __shfl(e, lane);
        }
    }
    if (kk == 0) {
        if (threadIdx.x == 0) {
            c->fail = 1;
            c->fail_step = s;
        }
        return;
    }
    Book k;
    const bool sub = a.damping && s < a.n_sub - 1;    // the next damped sub-step starts here
    const int hist[4] = {sub ? h0 : y, sub ? h1 : h0, sub ? h2 : h1, sub ? h3 : h2};
    const int hn = sub ? hc : (hc < 4 ? hc + 1 : 4);
    k.cur = y;
    int fr = -1;
#pragma unroll
    for (int b = POOL - 1; b >= 0; --b) {
        bool used = b == k.cur;
#pragma unroll
        for (int q = 0; q < 4; ++q) used = used || (q < hn && b == hist[q]);
        if (!used) fr = b;
    }
    k.y = fr;
    k.bvalid = (bv | (1 << k.cur)) & ~(1 << fr);      // B of the state was stored by the row kernel; the free
                                                      // grid takes the next iterate
    k.w = w ^ 1;
    k.step = s2;
    const bool damped = a.damping && s2 < a.n_sub;
    k.nsrc = damped ? 1 : hn;
#pragma unroll
    for (int q = 0; q < 4; ++q) k.src[q] = hist[q];
    if (damped) k.src[0] = k.cur;
    // extrapolation from nsrc states
    k.coef[0] = k.nsrc;
    k.coef[1] = k.nsrc == 2 ? -1.0 : (k.nsrc == 3 ? -3.0 : -6.0);
    k.coef[2] = k.nsrc == 3 ? 1.0 : 4.0;
    k.coef[3] = -1.0;
    if (threadIdx.x == 0) {
        a.counts[s] = kk;
        a.incs[s] = inc;
        c->recent[s & 3] = kk;
        c->cur = k.cur;
        c->y = k.y;
        c->w = k.w;
        c->hc = hn;
        c->bvalid = k.bvalid;
        c->nsrc = k.nsrc;
        c->step = s2;
#pragma unroll
        for (int q = 0; q < 4; ++q) c->hist[q] = hist[q];
        if (s2 < a.nsteps) step_setup(a, c, k, sd, id, cn);
    }
    err_reset_upto(c, kmax);
}

// Recording for the adjoint march.  After sl (once per step): E_s, held in now.Wp
// when theta < 1, to segE (ks_begin_lin records it itself).  After step_end: the current state to seg when its
// step index is on the recording stride (idempotent: a slot whose step did not
// advance writes the same state again).
static __global__ void ks_store_E(const MarchArgs* __restrict__ A, const Ctl* __restrict__ Cs) {
    Args& a = plan_args(A);
    CtlK& c = plan_ctl(Cs);
    if (halted(a, c, 0) || !a.segE || c.now.expl == EXPL_NONE || c.now.lin) return;
    const size_t N = (size_t)a.n * a.n;
    const GP<double> src(c.now.Wp), dst(GP<double>(a.segE), (size_t)(c.step - a.seg_base) * N);
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (size_t)gridDim.x * blockDim.x)
        dst.put(i, src[i]);
}

static __global__ void ks_store_V(const MarchArgs* __restrict__ A, const Ctl* __restrict__ Cs) {
    Args& a = plan_args(A);
    CtlK& c = plan_ctl(Cs);
    if (!a.seg || c.hold) return;
    const int rel = c.step - a.seg_base;
    if (rel < 0 || rel % a.seg_every != 0) return;
    const size_t N = (size_t)a.n * a.n;
    const GP<double> src(a.pool[c.cur]), dst(GP<double>(a.seg), (size_t)(rel / a.seg_every) * N);
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < N; i += (size_t)gridDim.x * blockDim.x)
        dst.put(i, src[i]);
}

// ---- adjoint march (reverse time steps) ----
// Per reverse step s (forward V^s -> V^{s+1} = Y): lam solves
// (I - dt theta A)^T lam = Ybar by the transposed preconditioned iteration
// (the forward iteration kernels with B^T, D^T and the transposed line factors),
// mu = (T^SL)^T lam, and the cotangent of V^s is (I + dt (1 - theta) A)^T mu.
// Buffers of the adjoint MarchArgs: pool[1] = lam, pool[0] = mu, Wb = Ybar.

// Control block for reverse step s: iterate in pool[1], no failure, stopping values reset.
static __global__ void ks_adj_begin(const MarchArgs* __restrict__ A, Ctl* __restrict__ Cs, int s) {
    Ctl* c = Cs;
    err_reset(c);
    if (threadIdx.x == 0) {
        Args& a = kref(A);
        const int id = a.step_set[s];
        c->step = s;
        c->fail = 0;
        c->fail_step = -1;
        c->hold = 0;
        c->cur = 0;
        c->y = 1;
        c->w = 0;
        c->nsrc = 0;
        c->bvalid = 0;
        const Book k = {s, 0, 1, 0, 0, 0, {0, 0, 0, 0}, {0.0, 0.0, 0.0, 0.0}};
        step_setup(a, c, k, kref(a.sets + id), id, 0.0);
    }
}

// Starting value lam^0 = Ybar + w1 c1 + w2 c2 + w3 c3 + w4 c4 and its row
// transform, where c1..c4 = lam - Ybar of the previous reverse steps, newest
// first (lam - Ybar = dt theta A^T lam), weighted by the host: the correction
// extrapolated over the previous steps of the same kind and rescaled to this
// step's dt theta; unused c are null.
template <int L, int E>
__global__ __launch_bounds__(L / E) void ks_adj_start(const MarchArgs* __restrict__ A, const Ctl* __restrict__ Cs,
                                                     const double* __restrict__ c1, double w1,
                                                     const double* __restrict__ c2, double w2,
                                                     const double* __restrict__ c3, double w3,
                                                     const double* __restrict__ c4, double w4) {
    Args& a = plan_args(A);
    CtlK& c = plan_ctl(Cs);
    if (halted(a, c, 0)) return;
    constexpr int T = L / E;
    const int n = a.n, np = (n + 1) >> 1;
    const int p = xcd_remap(blockIdx.x, gridDim.x);
    if (p >= np) return;
    __shared__ double2 lds[lds_slots(L)];
    __shared__ double2 tw4[tw_slots<L, E>()];
    load_twiddles<L, E>(GP<double2>(a.tw), tw4);
    const int ra = 2 * p, rb = 2 * p + 1;
    const bool hasb = rb < n;
    const GP<double> lam(c.now.Y), Yb(c.now.W);
    const GP<double> g1(c1), g2(c2), g3(c3), g4(c4);
    auto start = [&](int o) {
        return Yb[o] + (c1 ? w1 * g1[o] : 0.0) + (c2 ? w2 * g2[o] : 0.0) + (c3 ? w3 * g3[o] : 0.0) +
               (c4 ? w4 * g4[o] : 0.0);
    };
    double2 reg[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int j = threadIdx.x + e * T;
        const double va = j < n ? start(ra * n + j) : 0.0, vb = j < n && hasb ? start(rb * n + j) : 0.0;
        reg[e] = make_double2(va, vb);
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int j = threadIdx.x + e * T;
        if (j < n) lam.put(ra * n + j, reg[e].x);
        if (j < n && hasb) lam.put(rb * n + j, reg[e].y);
    }
    rows_fwd_store<L, E>(reg, lds, tw4, xbuf<double2>(a), n, ra, hasb);
}

// Verdict of the adjoint fixed point of the current reverse step: iteration
// count (first k with err_k < tol) or the failure flag.
static __global__ void ks_adj_end(const MarchArgs* __restrict__ A, Ctl* __restrict__ Cs, int kmax) {
    Args& a = kref(A);
    Ctl* c = Cs;
    if (c->fail) return;
    __shared__ double ek[KSLOTS];
    for (int q = threadIdx.x; q <= kmax; q += blockDim.x) ek[q] = err_max(*c, q);
    __syncthreads();
    if (threadIdx.x != 0) return;
    int kk = 0;
    for (int q = 1; q <= kmax; ++q)
        if (ek[q] < a.tol) { kk = q; break; }
    if (kk == 0) {
        c->fail = 1;
        c->fail_step = c->step;
    } else {
        a.counts[c->step] = kk;
        a.incs[c->step] = ek[kk];
    }
}

// mu = (T_1^T (x) T_2^T) lam (the transposed semi-Lagrangian gather) into pool[0]
// and corr = lam - Ybar (start of later reverse steps); when theta < 1 also mu's row
// transform for B^T mu, into X and into X2 (the spectral gradient term of the next
// reverse step reads it), otherwise mu is the cotangent of V^s and goes to Ybar as well.
// One axis after the other: the rows' combination of axis 1 by coalesced reads into
// LDS, the columns' of axis 2 from there (W1 + W2 terms per node; all W1 W2 of them
// gathered from memory, and corr by a kernel of its own, took 18.3 + 4 us at 512^2; now 14.1).
// WM > 0: the transposed tables are at most WM wide (the host checks): fixed bounds,
// terms past the width are the last one's with weight 0; WM = 0: any width.
template <int L, int E, int WM>
__global__ __launch_bounds__(L / E) void ks_adj_sl(const MarchArgs* __restrict__ A, const Ctl* __restrict__ Cs,
                                                  double2* __restrict__ X2, double* __restrict__ corr) {
    Args& a = plan_args(A);
    CtlK& c = plan_ctl(Cs);
    if (halted(a, c, 0)) return;
    constexpr int T = L / E;
    const int n = a.n, np = (n + 1) >> 1;
    const int p = xcd_remap(blockIdx.x, gridDim.x);
    if (p >= np) return;
    __shared__ double2 lds[lds_slots(L)];
    __shared__ double2 tw4[tw_slots<L, E>()];
    KRef<StepDesc> sd = kref(a.sets + c.now.set);
    const bool fft = sd.theta < 1.0;
    if (fft) load_twiddles<L, E>(GP<double2>(a.tw), tw4);
    const int ra = 2 * p, rb = 2 * p + 1;
    const bool hasb = rb < n;
    const int rs = hasb ? rb : ra;
    const GP<double> lam(c.now.Y), mu(c.now.V), Yb(c.now.W), t1w(sd.t1w), t2w(sd.t2w), cr(corr);
    const GP<int> t1i(sd.t1i), t2i(sd.t2i);
    const int W1 = sd.wt1, W2 = sd.wt2;
    if constexpr (WM > 0) {
        int ia[WM], ib[WM];
        double wa[WM], wb[WM];
#pragma unroll
        for (int q = 0; q < WM; ++q) {
            const int t = min(q, W1 - 1);
            ia[q] = t1i[ra * W1 + t] * n;
            ib[q] = t1i[rs * W1 + t] * n;
            wa[q] = q < W1 ? t1w[ra * W1 + t] : 0.0;
            wb[q] = q < W1 ? t1w[rs * W1 + t] : 0.0;
        }
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const int j = min((int)threadIdx.x + e * T, n - 1);
            double sa = 0.0, sb = 0.0;
#pragma unroll
            for (int q = 0; q < WM; ++q) {
                sa += wa[q] * lam[ia[q] + j];
                sb += wb[q] * lam[ib[q] + j];
            }
            if ((int)threadIdx.x + e * T < n) lds[j] = make_double2(sa, sb);
        }
    } else {
        for (int j = threadIdx.x; j < n; j += T) {
            double sa = 0.0, sb = 0.0;
            for (int q = 0; q < W1; ++q) {
                sa += t1w[ra * W1 + q] * lam[t1i[ra * W1 + q] * n + j];
                sb += t1w[rs * W1 + q] * lam[t1i[rs * W1 + q] * n + j];
            }
            lds[j] = make_double2(sa, sb);
        }
    }
    __syncthreads();
    double2 reg[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int j = threadIdx.x + e * T;
        double sa = 0.0, sb = 0.0;
        if (j < n) {
            if constexpr (WM > 0) {
#pragma unroll
                for (int q = 0; q < WM; ++q) {
                    const int t = min(q, W2 - 1);
                    const double w = q < W2 ? t2w[j * W2 + t] : 0.0;
                    const double2 v = lds[t2i[j * W2 + t]];
                    sa += w * v.x;
                    sb += w * v.y;
                }
            } else {
                for (int q = 0; q < W2; ++q) {
                    const double w = t2w[j * W2 + q];
                    const double2 v = lds[t2i[j * W2 + q]];
                    sa += w * v.x;
                    sb += w * v.y;
                }
            }
        }
        reg[e] = make_double2(sa, hasb ? sb : 0.0);
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int j = threadIdx.x + e * T;
        if (j >= n) continue;
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            if (r == 1 && !hasb) break;
            const int o = (ra + r) * n + j;
            const double m = r == 0 ? reg[e].x : reg[e].y;
            cr.put(o, lam[o] - Yb[o]);
            mu.put(o, m);
            if (!fft) Yb.put(o, m);
        }
    }
    if (fft) rows_fwd_store<L, E>(reg, lds, tw4, xbuf<double2>(a), n, ra, hasb, X2);
}

// Per-step gradient terms of the reverse step (one block per row pair,
// deterministic per-block accumulators acc[block * 8 + q]):
//   q = 0, 1, 2: dt theta lam . D_c Y + dt (1 - theta) mu . D_c V    (c = 11, 12, 22)
//   q = 3:       -(dt theta lam . Y + dt (1 - theta) mu . V)         (r_omega)
//   q = 4, 5:    lam . ((dT_1 (x) T_2) E), lam . ((T_1 (x) dT_2) E)   (kappa_omega^(1,2))
// with Y = V^{s+1}, V = V^s and E = E_s (V^s when theta = 1).
template <int P>
__global__ __launch_bounds__(256) void ks_adj_accum(const MarchArgs* __restrict__ A, const Ctl* __restrict__ Cs,
                                                    const double* __restrict__ Yg,
                                                    const double* __restrict__ Vg, const double* __restrict__ Eg,
                                                    double* __restrict__ acc) {
    Args& a = plan_args(A);
    CtlK& c = plan_ctl(Cs);
    if (halted(a, c, 0)) return;
    const int n = a.n;
    const int i = xcd_remap(blockIdx.x, gridDim.x);   // neighbouring rows on one XCD (stencil reads share L2)
    if (i >= n) return;
    KRef<StepDesc> sd = kref(a.sets + c.now.set);
    const GP<double> lam(c.now.Y), mu(c.now.V), Yp(Yg), Vp(Vg), Ep(Eg), w1t(sd.w1), w1dt(sd.w1d), w2t(sd.w2), w2dt(sd.w2d);
    const GP<int> s2(sd.s2);
    const double ci = c.now.cth, ce = c.now.cex, h = a.st.h;
    double t[6] = {0, 0, 0, 0, 0, 0};
    const int a0 = GP<int>(sd.s1)[i];
    double w1[P + 1], w1d[P + 1];
#pragma unroll
    for (int q = 0; q <= P; ++q) {
        w1[q] = w1t[i * (P + 1) + q];
        w1d[q] = w1dt[i * (P + 1) + q];
    }
    for (int j = threadIdx.x; j < n; j += blockDim.x) {
        const int o = i * n + j;
        const double l = lam[o], m = mu[o], y = Yp[o], v = Vp[o];
        double y11, y12, y22, v11 = 0.0, v12 = 0.0, v22 = 0.0;
        apply_D_parts(Yp, n, h, i, j, y, y11, y12, y22);
        if (ce != 0.0) apply_D_parts(Vp, n, h, i, j, v, v11, v12, v22);
        t[0] += ci * l * y11 + ce * m * v11;
        t[1] += ci * l * y12 + ce * m * v12;
        t[2] += ci * l * y22 + ce * m * v22;
        t[3] -= ci * l * y + ce * m * v;
        const int b0 = s2[j];
        double w2[P + 1], w2d[P + 1];
#pragma unroll
        for (int b = 0; b <= P; ++b) {
            w2[b] = w2t[j * (P + 1) + b];
            w2d[b] = w2dt[j * (P + 1) + b];
        }
        double g1 = 0.0, g2 = 0.0;
#pragma unroll
        for (int aa = 0; aa <= P; ++aa) {
            const int eo = (a0 + aa) * n + b0;
            double s0 = 0.0, sdd = 0.0;
#pragma unroll
            for (int b = 0; b <= P; ++b) {
                const double ev = Ep[eo + b];
                s0 += w2[b] * ev;
                sdd += w2d[b] * ev;
            }
            g1 += w1d[aa] * s0;
            g2 += w1[aa] * sdd;
        }
        t[4] += l * g1;
        t[5] += l * g2;
    }
    __shared__ double red[6][256];
    for (int q = 0; q < 6; ++q) red[q][threadIdx.x] = t[q];
    __syncthreads();
    for (int w = blockDim.x / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w)
            for (int q = 0; q < 6; ++q) red[q][threadIdx.x] += red[q][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0)
        for (int q = 0; q < 6; ++q) acc[(size_t)i * 8 + q] += red[q][0];
}

// Spectral accumulation of the kernel gradient.  V^{s+1} meets lam of reverse step s
// (weight c1) and mu of the step before it, s + 1 (weight c2): per column k2 of the
// row transforms (transposed half spectra, n rows each) one column FFT of their sum and
// one of V^{s+1}'s, S[k2][k1] += conj(FFT(c1 XL + c2 XM)) FFT XV; a weight of 0 leaves its
// term out.  After the march, the inverse 2D transform of S / L^2 is sum_m lam_m Y_{m+d}
// summed over the steps with their weights: the gradient of the loss with respect to the
// folded kernel K_d.  (Four FFTs a step, with both terms' pairs transformed by
// themselves, and a copy of XL kept for them: 14.7 + 5 us at 512^2; now 10.9.)
template <int L, int E>
__global__ __launch_bounds__(L / E) void ks_adj_spec(const MarchArgs* __restrict__ A, const Ctl* __restrict__ Cs,
                                                     const double2* __restrict__ XM, const double2* __restrict__ XV,
                                                     double c1, double c2, double2* __restrict__ S) {
    Args& a = plan_args(A);
    CtlK& c = plan_ctl(Cs);
    if (halted(a, c, 0)) return;
    constexpr int T = L / E;
    __shared__ double2 lds[lds_slots(L)];
    __shared__ double2 tw4[tw_slots<L, E>()];
    load_twiddles<L, E>(GP<double2>(a.tw), tw4);
    const int n = a.n, col = blockIdx.x, tid = threadIdx.x;
    const GP<double2> xl(GP<double2>(a.X), (size_t)col * n), xm(GP<double2>(XM), (size_t)col * n),
        xv(GP<double2>(XV), (size_t)col * n), sc(GP<double2>(S), (size_t)col * L);
    double2 ru[E], rv[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int idx = tid + e * T, at = min(idx, n - 1);
        double2 l = make_double2(0.0, 0.0), m = make_double2(0.0, 0.0);
        if (c1 != 0.0) l = xl[at];
        if (c2 != 0.0) m = xm[at];
        const double2 v = xv[at];
        const bool in = idx < n;
        ru[e] = in ? make_double2(c1 * l.x + c2 * m.x, c1 * l.y + c2 * m.y) : make_double2(0.0, 0.0);
        rv[e] = in ? v : make_double2(0.0, 0.0);
    }
    fft_block<L, E, false>(ru, lds, tw4);
    __syncthreads();
    fft_block<L, E, false>(rv, lds, tw4);
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const double2 pr = cmulc(rv[e], ru[e]), t = sc[tid + e * T];    // conj(U) V
        sc.put(tid + e * T, make_double2(t.x + pr.x, t.y + pr.y));
    }
}

// Control block at the start of a march: the state of step-list entry step0
// in pool[0], the iterate in pool[1], no history before it.  One block per plan.
static __global__ void ks_init(const MarchArgs* __restrict__ A, Ctl* __restrict__ Cs) {
    Args& a = plan_args(A);
    Ctl* c = Cs + blockIdx.y;
    err_reset(c);
    if (threadIdx.x == 0) {
        c->step = a.step0;
        c->fail = 0;
        c->fail_step = -1;
        c->hold = 0;
        c->cur = 0;
        c->y = 1;
        c->w = 0;
        c->hc = 1;
        c->nsrc = 1;
        c->bvalid = 0;
        for (int q = 0; q < 4; ++q) { c->hist[q] = 0; c->recent[q] = 0; }
        const Book k = {a.step0, 0, 1, 0, 1, 0, {0, 0, 0, 0}, {1.0, 0.0, 0.0, 0.0}};
        if (a.step0 < a.nsteps) {
            const int id = a.step_set[a.step0];
            step_setup(a, c, k, kref(a.sets + id), id, a.cn_rho ? a.cn_rho[a.step0] : 0.0);
        }
    }
}

static __global__ void ks_clear_fail(Ctl* __restrict__ Cs, int plan) {
    if (threadIdx.x == 0) Cs[plan].fail = 0;
}

// hold = 1 on every plan of the group except `keep` (keep < 0: release all).
static __global__ void ks_hold(Ctl* __restrict__ Cs, int np, int keep) {
    for (int q = threadIdx.x; q < np; q += blockDim.x) Cs[q].hold = (keep >= 0 && q != keep) ? 1 : 0;
}

}  // namespace lpide
