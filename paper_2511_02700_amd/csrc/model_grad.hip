// Gradient with respect to the subordination parameters, from the native gradient of
// the adjoint march: the model's quantities a_11, a_12, a_22 (artificial diffusion),
// omega, and through omega r_omega = r + sum omega and kappa_omega = r - sum omega
// (e^z - 1), differentiated by central differences at the plan's structure.
//
// Fourteen evaluations of the quadrature weights and of the small-jump covariance,
// about 2 million densities at n = 96, on the host's threads were the largest part of
// a calibration point (90 of 118 ms there).  Here a thread takes one density (or one
// pair of a central difference), and what a weight contributes to the gradient is
// summed at once: only the sums leave the device.  The whole gradient takes
// 0.8 ms at n = 96 (N_z = 63), 2.1 at 512 (253), 6.1 at 1024 (505); a calibration point
// at n = 96 (plan, march, adjoint, gradient) went from 118 to 32 ms.
//
// K_nu by the trapezoidal rule on K_nu(x) = int_0^inf exp(-x cosh t) cosh(nu t) dt
// (the even, analytic integrand makes its error e^(-pi^2 / h) and e^(-2 pi^2 / (x h^2));
// Trefethen and Weideman, SIAM Review 56 (2014)): positive terms only, with cosh t - 1
// and cosh(nu t) tabulated by the host once per order.  The step halves as x grows
// fourfold; from 512 on the asymptotic series that the host's density takes too.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "plan.hpp"

namespace lpide {
namespace detail {

namespace {

constexpr int NT0 = 800, NT1 = 48, NTAB = NT0 + 3 * NT1;   // nodes of the coarse level and of each finer one
constexpr int NEVAL = 14;                                  // parameter q up: 2 q, down: 2 q + 1
constexpr int MG_T = 256;

struct NtsEval {
    double ri[3], ri_eta[2], c1, nu, logpref;
    int tab;            // which cosh(nu t) table
    int pad;
};

__device__ double log_bessel_k_dev(double nu, double x, const double* __restrict__ ch1, const double* __restrict__ cn) {
    if (x >= 512.0) {
        const double mu = 4.0 * nu * nu;
        double term = 1.0, sum = 1.0;
        for (int k = 1; k < 12; ++k) {
            term *= (mu - (2.0 * k - 1) * (2.0 * k - 1)) / (8.0 * k * x);
            sum += term;
        }
        return -x + 0.5 * log(3.14159265358979323846 / (2.0 * x)) + log(sum);
    }
    const int lv = x < 8.0 ? 0 : (x < 32.0 ? 1 : (x < 128.0 ? 2 : 3));
    const double h = lv == 0 ? 0.2 : (lv == 1 ? 0.1 : (lv == 2 ? 0.05 : 0.025));
    const int off = lv == 0 ? 0 : NT0 + (lv - 1) * NT1, cap = lv == 0 ? NT0 : NT1;
    // the integrand peaks at asinh(nu / x), falls like e^(nu t) before it (left out past
    // e^-40) and like exp(-x cosh t) behind it
    const double r = nu / x, tp = log(r + sqrt(1.0 + r * r));
    const int k0 = min(cap - 1, max(0, (int)((tp - 40.0 / nu) / h)));
    double s = 0.0;
    for (int k = k0; k < cap; ++k) {
        const double arg = x * ch1[off + k];
        if (arg > 60.0) break;
        const double t = cn[off + k] * exp(-arg);
        s += k == 0 ? 0.5 * t : t;
    }
    return log(s * h) - x;
}

__device__ double log_density_dev(const NtsEval& p, double z1, double z2, const double* __restrict__ tab) {
    const double q = sqrt(p.ri[0] * z1 * z1 + 2.0 * p.ri[1] * z1 * z2 + p.ri[2] * z2 * z2);
    return p.logpref + log_bessel_k_dev(p.nu, p.c1 * q, tab, tab + NTAB * (1 + p.tab)) - p.nu * log(q) +
           p.ri_eta[0] * z1 + p.ri_eta[1] * z2;
}

// Sum over a block of MG_T threads (all take part), the same order every time.
__device__ double block_sum(double v, double* red) {
    red[threadIdx.x] = v;
    __syncthreads();
    for (int w = MG_T / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
        __syncthreads();
    }
    return red[0];
}

struct OmegaArgs {
    int N, M1, M2, ng;
    double h, n3, n4, n5;      // mesh width; native gradient of r_omega, kappa_1, kappa_2
    const double* nat;         // native gradient of omega, (2N)^2
    const double *gx, *gw;     // quadrature of a cell
    const double* tab;         // cosh t - 1, then the tables of cosh(nu t)
    const NtsEval* ev;
    const double* ih;          // 1 / (2 step) per parameter
};

// What d J / d omega_l is with omega's way through r_omega and kappa_omega.
__device__ double total_weight(const OmegaArgs& o, int l1, int l2) {
    return o.nat[(size_t)(l1 + o.N) * (2 * o.N) + (l2 + o.N)] + o.n3 - o.n4 * expm1((l1 + 0.5) * o.h) -
           o.n5 * expm1((l2 + 0.5) * o.h);
}

// Outer cells (midpoint rule), parameter blockIdx.y: partial sums of
// (omega_l(up) - omega_l(down)) / (2 step) times the total weight.
__global__ __launch_bounds__(MG_T) void k_grad_outer(OmegaArgs o, double* __restrict__ part) {
    __shared__ double red[MG_T];
    const int W2 = 2 * o.N, q = blockIdx.y;
    const NtsEval up = o.ev[2 * q], dn = o.ev[2 * q + 1];
    double acc = 0.0;
    for (int c = blockIdx.x * MG_T + threadIdx.x; c < W2 * W2; c += gridDim.x * MG_T) {
        const int l1 = c / W2 - o.N, l2 = c % W2 - o.N;
        const double c1 = (l1 + 0.5) * o.h, c2 = (l2 + 0.5) * o.h;
        if (fmax(fabs(l1 + 0.5), fabs(l2 + 0.5)) <= max(o.M1, o.M2)) continue;
        const double d = exp(log_density_dev(up, c1, c2, o.tab)) - exp(log_density_dev(dn, c1, c2, o.tab));
        acc += d * o.h * o.h * o.ih[q] * total_weight(o, l1, l2);
    }
    const double s = block_sum(acc, red);
    if (threadIdx.x == 0) part[(size_t)q * gridDim.x + blockIdx.x] = s;
}

// Cells of the middle region (||z_l||^-2 int ||z||^2 l over the cell, ng x ng nodes):
// one wave per cell of the square of side 2 M2, its lanes over the nodes.
__global__ __launch_bounds__(MG_T) void k_grad_inner(OmegaArgs o, double* __restrict__ part) {
    __shared__ double red[MG_T];
    const int W = 2 * o.M2, q = blockIdx.y, lane = threadIdx.x & 63;
    const int nodes = o.ng * o.ng;
    const NtsEval up = o.ev[2 * q], dn = o.ev[2 * q + 1];
    double acc = 0.0;
    for (int c = blockIdx.x * (MG_T / 64) + (int)(threadIdx.x >> 6); c < W * W; c += gridDim.x * (MG_T / 64)) {
        const int l1 = c / W - o.M2, l2 = c % W - o.M2;
        if (fmax(fabs(l1 + 0.5), fabs(l2 + 0.5)) <= o.M1) continue;
        const double c1 = (l1 + 0.5) * o.h, c2 = (l2 + 0.5) * o.h;
        double s = 0.0;
        for (int t = lane; t < nodes; t += 64) {
            const int i = t / o.ng, j = t % o.ng;
            const double z1 = c1 + 0.5 * o.h * o.gx[i], z2 = c2 + 0.5 * o.h * o.gx[j];
            s += o.gw[i] * o.gw[j] * (z1 * z1 + z2 * z2) *
                 (exp(log_density_dev(up, z1, z2, o.tab)) - exp(log_density_dev(dn, z1, z2, o.tab)));
        }
        acc += s * (0.25 * o.h * o.h / (c1 * c1 + c2 * c2)) * o.ih[q] * total_weight(o, l1, l2);
    }
    const double s = block_sum(acc, red);
    if (threadIdx.x == 0) part[(size_t)q * gridDim.x + blockIdx.x] = s;
}

// Radial integrals of the small-jump covariance: angle blockIdx.x of evaluation
// blockIdx.y, int_0^R r^3 l(r u) dr by the nodes tx, tw on [0, 1].
__global__ __launch_bounds__(MG_T) void k_grad_cov(const NtsEval* __restrict__ ev, const double* __restrict__ tab,
                                                   const double* __restrict__ u1, const double* __restrict__ u2,
                                                   const double* __restrict__ R, const double* __restrict__ tx,
                                                   const double* __restrict__ tw, int nt, double* __restrict__ out) {
    __shared__ double red[MG_T];
    const int a = blockIdx.x;
    const NtsEval p = ev[blockIdx.y];
    double acc = 0.0;
    for (int k = threadIdx.x; k < nt; k += MG_T) {
        const double r = R[a] * tx[k];
        acc += tw[k] * R[a] * exp(3.0 * log(r) + log_density_dev(p, r * u1[a], r * u2[a], tab));
    }
    const double s = block_sum(acc, red);
    if (threadIdx.x == 0) out[(size_t)blockIdx.y * gridDim.x + a] = s;
}

// dJ/d omega_l = sum_j s_j1 s_j2 dJ/dK_{l + jlo + j} (K = omega folded with the half-cell
// taps s), from the inverse transform G of the spectral accumulator (L^2 x dJ/dK).
struct Taps { double s[4]; };
__global__ __launch_bounds__(MG_T) void k_native_omega(const double* __restrict__ G, int L, int Nz, int P, Taps taps,
                                                       double scale, double* __restrict__ out) {
    const int W2 = 2 * Nz, jlo = -(P - 1) / 2;
    const int c = blockIdx.x * MG_T + threadIdx.x;
    if (c >= W2 * W2) return;
    const int l1 = c / W2 - Nz + jlo, l2 = c % W2 - Nz + jlo;
    double t = 0.0;
    for (int j1 = 0; j1 <= P; ++j1) {
        const double* row = G + (size_t)((l1 + j1 + 2 * L) % L) * L;
        for (int j2 = 0; j2 <= P; ++j2) t += taps.s[j1] * taps.s[j2] * (row[(l2 + j2 + 2 * L) % L] * scale);
    }
    out[c] = t;
}

}  // namespace

int native_omega(Plan* p, const double* G, double* out, hipStream_t s) {
    const int Pin = p->hp.in_order, jlo = -(Pin - 1) / 2, W2 = 2 * p->hp.N_z;
    Taps taps{};
    for (int i = 0; i <= Pin; ++i) {
        double v = 1.0;
        for (int j = 0; j <= Pin; ++j)
            if (j != i) v *= (0.5 - (jlo + j)) / double(i - j);
        taps.s[i] = v;
    }
    hipLaunchKernelGGL(k_native_omega, dim3((W2 * W2 + MG_T - 1) / MG_T), dim3(MG_T), 0, s, G, p->L, p->hp.N_z, Pin, taps,
                       1.0 / (double(p->L) * double(p->L)), out);
    HIP_TRY(hipGetLastError());
    return LPIDE_OK;
}

int model_gradient(Plan* p, const double* x, const double* nat, double* grad) {
    const HostPlan& hp = p->hp;
    const int N = hp.N_z, W2 = 2 * N, ng = p->grid.gl_nodes;
    NtsEval ev[NEVAL];
    double ih[7];
    std::vector<double> orders;
    for (int q = 0; q < 7; ++q) {
        const double hq = 1e-4 * std::max(std::fabs(x[q]), 0.1);
        ih[q] = 1.0 / (2.0 * hq);
        for (int side = 0; side < 2; ++side) {
            double y[8];
            std::copy(x, x + 8, y);
            y[q] += side == 0 ? hq : -hq;
            lpide_levy lv;
            int rc = lpide_levy_from_std(y[0], y[1], y[2], y[3], y[4], y[5], y[6], y[7], &lv);
            if (rc) return rc;
            Nts m;
            std::string err;
            if (!make_nts(lv, m, err)) return fail(LPIDE_E_PARAM, "model quantities: " + err);
            NtsEval& e = ev[2 * q + side];
            std::copy(m.ri, m.ri + 3, e.ri);
            std::copy(m.ri_eta, m.ri_eta + 2, e.ri_eta);
            e.c1 = m.c1;
            e.nu = m.nu;
            e.logpref = m.logpref;
            e.pad = 0;
            size_t t = std::find(orders.begin(), orders.end(), m.nu) - orders.begin();
            if (t == orders.size()) orders.push_back(m.nu);
            e.tab = int(t);
        }
    }
    // one packed upload: evaluations, 1 / (2 step), tables, cell quadrature, angles, radial nodes
    std::vector<double> gx, gw, ax, aw, tx, tw;
    gauss_legendre(ng, gx, gw);
    gauss_legendre(48, ax, aw);
    radial_nodes(tx, tw);
    const int na = 8 * int(ax.size()), nt = int(tx.size());
    std::vector<double> buf;
    auto put = [&](const double* v, size_t cnt) {
        const size_t at = buf.size();
        buf.insert(buf.end(), v, v + cnt);
        return at;
    };
    static_assert(sizeof(NtsEval) % sizeof(double) == 0, "packed with doubles");
    std::vector<double> evd(NEVAL * sizeof(NtsEval) / sizeof(double));
    std::memcpy(evd.data(), ev, sizeof ev);
    const size_t o_ev = put(evd.data(), evd.size()), o_ih = put(ih, 7);
    std::vector<double> tab((size_t)NTAB * (1 + orders.size()));
    for (int k = 0; k < NTAB; ++k) {
        const int lv = k < NT0 ? 0 : 1 + (k - NT0) / NT1, i = k < NT0 ? k : (k - NT0) % NT1;
        const long double t = 0.2L * i / (1 << lv), sh = sinhl(0.5L * t);
        tab[k] = double(2.0L * sh * sh);
        for (size_t m = 0; m < orders.size(); ++m) tab[NTAB * (1 + m) + k] = double(coshl((long double)orders[m] * t));
    }
    const size_t o_tab = put(tab.data(), tab.size()), o_gx = put(gx.data(), ng), o_gw = put(gw.data(), ng);
    std::vector<double> U1(na), U2(na), R(na), Wp(na);
    for (int q = 0; q < na; ++q) {
        const int oct = q / (na / 8), i = q % (na / 8);
        const double pi = 3.14159265358979323846, a = oct * pi / 4.0, b = (oct + 1) * pi / 4.0;
        const double phi = 0.5 * (b - a) * ax[i] + 0.5 * (a + b);
        Wp[q] = 0.5 * (b - a) * aw[i];
        U1[q] = std::cos(phi);
        U2[q] = std::sin(phi);
        R[q] = hp.M1 * hp.h / std::max(std::fabs(U1[q]), std::fabs(U2[q]));
    }
    const size_t o_u1 = put(U1.data(), na), o_u2 = put(U2.data(), na), o_R = put(R.data(), na);
    const size_t o_tx = put(tx.data(), nt), o_tw = put(tw.data(), nt);
    const int nb_o = std::min(1024, (W2 * W2 + MG_T - 1) / MG_T), wi = 2 * hp.M2;
    const int nb_i = std::max(1, std::min(2048, (wi * wi + MG_T / 64 - 1) / (MG_T / 64)));
    const size_t n_out = (size_t)7 * nb_o + (size_t)7 * nb_i + (size_t)NEVAL * na;
    const size_t o_out = buf.size();
    Adjoint* a = p->adj;
    if (a->mg_n < o_out + n_out) {            // grows with the order tables only: once or twice per plan
        double* d = nullptr;
        int rc = dalloc_into(a->allocs, nullptr, &d, o_out + n_out);
        if (rc) return rc;
        a->mg = d;
        a->mg_n = o_out + n_out;
    }
    double* d = a->mg;
    hipStream_t s = p->stream;
    HIP_TRY(hipMemcpyAsync(d, buf.data(), sizeof(double) * o_out, hipMemcpyHostToDevice, s));
    OmegaArgs o{};
    o.N = N;
    o.M1 = hp.M1;
    o.M2 = hp.M2;
    o.ng = ng;
    o.h = hp.h;
    o.n3 = nat[3];
    o.n4 = nat[4];
    o.n5 = nat[5];
    o.nat = a->nat;
    o.gx = d + o_gx;
    o.gw = d + o_gw;
    o.tab = d + o_tab;
    o.ev = reinterpret_cast<const NtsEval*>(d + o_ev);
    o.ih = d + o_ih;
    double *p_o = d + o_out, *p_i = p_o + (size_t)7 * nb_o, *p_c = p_i + (size_t)7 * nb_i;
    hipLaunchKernelGGL(k_grad_cov, dim3(na, NEVAL), dim3(MG_T), 0, s, o.ev, o.tab, d + o_u1, d + o_u2, d + o_R, d + o_tx,
                       d + o_tw, nt, p_c);
    hipLaunchKernelGGL(k_grad_inner, dim3(nb_i, 7), dim3(MG_T), 0, s, o, p_i);
    hipLaunchKernelGGL(k_grad_outer, dim3(nb_o, 7), dim3(MG_T), 0, s, o, p_o);
    HIP_TRY(hipGetLastError());
    std::vector<double> out(n_out);
    HIP_TRY(hipMemcpyAsync(out.data(), p_o, sizeof(double) * n_out, hipMemcpyDeviceToHost, s));
    HIP_TRY(hipStreamSynchronize(s));
    const double *h_o = out.data(), *h_i = h_o + (size_t)7 * nb_o, *h_c = h_i + (size_t)7 * nb_i;
    for (int q = 0; q < 7; ++q) {
        double t = 0.0;
        for (int b = 0; b < nb_o; ++b) t += h_o[(size_t)q * nb_o + b];
        for (int b = 0; b < nb_i; ++b) t += h_i[(size_t)q * nb_i + b];
        double s11 = 0.0, s12 = 0.0, s22 = 0.0;
        for (int k = 0; k < na; ++k) {
            const double dI = (h_c[(size_t)(2 * q) * na + k] - h_c[(size_t)(2 * q + 1) * na + k]) * Wp[k];
            s11 += U1[k] * U1[k] * dI;
            s12 += U1[k] * U2[k] * dI;
            s22 += U2[k] * U2[k] * dI;
        }
        grad[q] = t + (nat[0] * s11 + nat[1] * s12 + nat[2] * s22) * ih[q];
    }
    grad[7] = nat[3] + nat[4] + nat[5];      // r_omega = r + ..., kappa_omega = r - ...
    return LPIDE_OK;
}

}  // namespace detail
}  // namespace lpide
