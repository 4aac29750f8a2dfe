// Derivatives of S = sum_f Re(chi_f^H D[mu] psi_f) with respect to psi and to
// the links, for D[mu] with the rational sign function
//   eps(K) = K sum_l omega_l X_l,  X_l = (K^2 + sigma_l)^{-1}
// (Sec. 1 eqs. 1, 2, 4 and Sec. 3 eq. 7; the exactly treated low modes are not
// differentiated, so the context must hold none).  Gradients are d/dRe + i d/dIm,
// each link entry an independent complex variable:
//   dS/dpsi = gamma_5 D gamma_5 chi
//   dS/dU_mu(y) = -(1 - mu)/4 sum_l omega_l [T(chi', a_l) - T(b_l, K a_l) - T(K b_l, a_l)]
// with chi' = gamma_5 chi, a_l = X_l psi, b_l = X_l K chi' (from
// dX_l = -X_l (dK K + K dK) X_l and dK = -gamma_5 dH / 2), and for spinor fields
// (alpha, beta) the colour matrix on link (y, mu)
//   T(alpha, beta)_ab = sum_{t=0,1} [ (P+ alpha(y))_ta conj((P- beta(y+mu))_tb)
//                                   + (P+ beta(y))_ta conj((P- alpha(y+mu))_tb) ],
// where P-+ psi = psi_up -+ A_mu psi_down is the upper half of (1 -+ gamma_mu) psi.
// The lower half of (1 -+ gamma_mu) psi is a unitary image of the upper one,
// so the two-spin sum equals the four-spin contraction of the definition.
//
// Cost: one multi-shift solve over both sources (psi and K chi'), which keeps
// every shifted solution, 2 N_Z kernel applications and one pass of the force
// kernel below.  With both derivatives wanted, dS/dpsi comes from the same
// solutions, eps(K) chi' = sum_l omega_l b_l, so that its sign call (another
// multi-shift solve) falls away.  Both derivatives took 14.0 ms on 8^3 x 16 in
// FP64 and 335 ms on 32^3 x 64 in FP32 with three solves one after another
// (their shift vectors updated in every iteration), and take 3.4 and 123 ms.
#include <algorithm>
#include <cmath>
#include <vector>

#include "context.h"
#include "fields.h"
#include "kernels.h"
#include "mscg_state.h"
#include "ops.h"

namespace ovl {

struct ForceCoef {
    double w[NZMAX];   // -(1 - mu)/4 omega_l
};

// h = psi_up + A psi_down (PLUS) or psi_up - A psi_down
template <int MU, bool PLUS, typename R>
__device__ __forceinline__ void half_proj(const cplx<R> v[12], cplx<R> h[6])
{
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        cplx<R> a0, a1;
        apply_A<MU>(v[6 + c], v[9 + c], a0, a1);
        if constexpr (PLUS) {
            h[c] = v[c] + a0;
            h[3 + c] = v[3 + c] + a1;
        } else {
            h[c] = v[c] - a0;
            h[3 + c] = v[3 + c] - a1;
        }
    }
}

// acc_ab += w sum_t x_ta conj(y_tb)
template <typename R>
__device__ __forceinline__ void outer_acc(double w, const cplx<R> x[6], const cplx<R> y[6], cplx<double> acc[9])
{
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            const cplx<R> t = cmul_conj(y[b], x[a]) + cmul_conj(y[3 + b], x[3 + a]);
            acc[a * 3 + b].re += w * (double)t.re;
            acc[a * 3 + b].im += w * (double)t.im;
        }
}

template <int MU, typename ST>
__device__ __forceinline__ void force_dir(const ST *chip, const ST *a, const ST *b, const ST *ka, const ST *kb,
                                          int64_t lstride, const ForceCoef &k, int nz, int64_t V, int64_t s,
                                          int64_t sf, double2 *__restrict__ G, bool accumulate)
{
    using R = typename Planes<ST>::R;
    cplx<double> acc[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) acc[i] = {0.0, 0.0};
    cplx<R> v[12], cp[6], cm[6];
    ld_sp(chip, V, s, v);
    half_proj<MU, true>(v, cp);    // P+ chi'(y)
    ld_sp(chip, V, sf, v);
    half_proj<MU, false>(v, cm);   // P- chi'(y+mu)
    for (int l = 0; l < nz; ++l) {
        const double w = k.w[l];
        const int64_t o = l * lstride;
        cplx<R> ap[6], am[6], xp[6], xm[6];
        ld_sp(a + o, V, s, v);
        half_proj<MU, true>(v, ap);    // P+ a_l(y)
        ld_sp(a + o, V, sf, v);
        half_proj<MU, false>(v, am);   // P- a_l(y+mu)
        ld_sp(kb + o, V, s, v);
        half_proj<MU, true>(v, xp);    // P+ K b_l(y)
        ld_sp(kb + o, V, sf, v);
        half_proj<MU, false>(v, xm);   // P- K b_l(y+mu)
        // T(chi', a_l) - T(K b_l, a_l) = (P+ chi' - P+ K b_l) (x) P- a_l + P+ a_l (x) (P- chi' - P- K b_l)
#pragma unroll
        for (int c = 0; c < 6; ++c) {
            xp[c] = cp[c] - xp[c];
            xm[c] = cm[c] - xm[c];
        }
        outer_acc(w, xp, am, acc);
        outer_acc(w, ap, xm, acc);
        // - T(b_l, K a_l)
        ld_sp(b + o, V, s, v);
        half_proj<MU, true>(v, xp);    // P+ b_l(y)
        ld_sp(ka + o, V, sf, v);
        half_proj<MU, false>(v, am);   // P- K a_l(y+mu)
        outer_acc(-w, xp, am, acc);
        ld_sp(ka + o, V, s, v);
        half_proj<MU, true>(v, ap);    // P+ K a_l(y)
        ld_sp(b + o, V, sf, v);
        half_proj<MU, false>(v, xm);   // P- b_l(y+mu)
        outer_acc(-w, ap, xm, acc);
    }
    double2 *g = G + (s * 4 + MU) * 9;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        double2 o = make_double2(acc[i].re, acc[i].im);
        if (accumulate) {
            const double2 p = g[i];
            o.x += p.x;
            o.y += p.y;
        }
        g[i] = o;
    }
}

// 64 sites per block, one wave per link direction; G canonical [V][4][3][3].
// Field arguments point at the field of one right-hand side; shift l of
// a, b, ka, kb is lstride elements further on.  Bound by the loads: each pole
// brings four spinors of the site and four of each neighbour, and the waves of
// a block find the site's own in cache.  With one lane walking the four
// directions there were a quarter of the waves, one per SIMD: 436 against 86 us
// on 8^3 x 16 in FP64, 19.4 against 11.5 ms on 32^3 x 64 in FP32 (20 poles).
template <typename ST>
__global__ __launch_bounds__(256, 2) void k_link_force(const ST *__restrict__ chip, const ST *__restrict__ a,
                                                       const ST *__restrict__ b, const ST *__restrict__ ka,
                                                       const ST *__restrict__ kb, int64_t lstride, ForceCoef k, int nz,
                                                       Geom g, double2 *__restrict__ G, int accumulate)
{
    const int64_t V = g.V;
    unsigned tile, field;
    tile_of_block<true>(tile, field);
    const int64_t s = (int64_t)tile * 64 + (threadIdx.x & 63);
    if (s >= V) return;
    const int mu = threadIdx.x >> 6;
    const int64_t st = g.stride[mu];
    const int32_t Lm = g.L[mu], co = (int32_t)((s / st) % Lm);
    const int64_t sf = co + 1 == Lm ? s - (int64_t)(Lm - 1) * st : s + st;
    switch (mu) {
    case 0: force_dir<0>(chip, a, b, ka, kb, lstride, k, nz, V, s, sf, G, accumulate != 0); break;
    case 1: force_dir<1>(chip, a, b, ka, kb, lstride, k, nz, V, s, sf, G, accumulate != 0); break;
    case 2: force_dir<2>(chip, a, b, ka, kb, lstride, k, nz, V, s, sf, G, accumulate != 0); break;
    default: force_dir<3>(chip, a, b, ka, kb, lstride, k, nz, V, s, sf, G, accumulate != 0); break;
    }
}

// dpsi = (1 + mu)/2 chi + (1 - mu)/2 sum_l omega_l b_l, that is gamma_5 D chi'
// (gamma_5 chi' = chi): the sum in the solutions' precision, as the multi-shift
// CG forms its own sums, 16 bytes of a field per lane.
struct PoleCoef {
    double w[NZMAX];
};
template <typename ST>
__global__ __launch_bounds__(256) void k_psi_gradient(const ST *__restrict__ b, int64_t lstride, PoleCoef k, int nz,
                                                      const double2 *__restrict__ chip, double2 *__restrict__ dpsi,
                                                      double cc, double cs, int64_t V)
{
    using R = typename Planes<ST>::R;
    constexpr int PL = Planes<ST>::n, NC = 12 / PL;   // planes, complex numbers per plane
    const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (i >= PL * V) return;
    const int f = blockIdx.y;
    const int64_t s = i % V;
    const int q = (int)(i / V);   // plane
    const ST *bf = b + f * fstride<ST>(V) + i;
    R acc[2 * NC];
#pragma unroll
    for (int c = 0; c < 2 * NC; ++c) acc[c] = R(0);
    for (int l = 0; l < nz; ++l) {
        const ST t = bf[l * lstride];
        const R w = (R)k.w[l];
        const R *tr = reinterpret_cast<const R *>(&t);
#pragma unroll
        for (int c = 0; c < 2 * NC; ++c) acc[c] += w * tr[c];
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int64_t o = (int64_t)f * 12 * V + (q * NC + c) * V + s;
        const double g = q * NC + c < 6 ? cc : -cc;   // chi = gamma_5 chi'
        const double2 x = chip[o];
        dpsi[o] = make_double2(g * x.x + cs * (double)acc[2 * c], g * x.y + cs * (double)acc[2 * c + 1]);
    }
}

// The link gradient into dU and, with dpsi, dS/dpsi; src holds psi (nf fields)
// and room for as many sources K chi' after it.
template <typename ST>
static void link_force_t(Context &c, double rho, double mu, const ovl_zolo &z, ST *src, const void *chip,
                         const double2 *chip64, double2 *dpsi, double2 *dU, int nf, double eta, int prec, int maxiter,
                         ovl_stats *st)
{
    const Geom &g = c.g;
    const int nz = z.n_z;
    const size_t FB = field_bytes(g, prec);
    const int64_t fs = fstride<ST>(g.V);   // elements of ST per field
    const size_t half_bytes = FB * nf * nz;
    ST *x = (ST *)c.buf("adj_x", 2 * half_bytes);    // a_l and b_l
    ST *kx = (ST *)c.buf("adj_kx", 2 * half_bytes);  // K a_l and K b_l
    stencil(c, EPI_K, prec, chip, src + nf * fs, nf, rho, 0.0, nullptr, nullptr);   // K chi'
    // a_l = X_l psi and b_l = X_l K chi', each to |zeta_l| ||r|| <= eta ||source||.
    // Where sum_l omega_l b_l stands for the sign function its error has to
    // stay within eta ||chi'||: ||X_l|| <= 1/(sigma_l + a^2) on the interval
    // [a, b] of |K|, and ||K chi'|| <= (|4 - rho| + 4) ||chi'||, so eta is
    // scaled by the smallest (sigma_l + a^2)/(omega_l N_Z (|4 - rho| + 4)), as
    // if every pole erred by its N_Z-th part.
    double tight = 1.0;
    if (dpsi)
        for (int l = 0; l < nz; ++l)
            tight = std::min(tight, (z.sigma[l] + z.a * z.a) / (z.omega[l] * nz * (std::fabs(4.0 - rho) + 4.0)));
    std::vector<double> e(2 * nf, eta);
    for (int f = 0; f < nf; ++f) e[nf + f] = eta * tight;
    // Both sources in one multi-shift CG (one launch carries both, links read
    // once), its shift vectors [l][2 nf], while the device has room for twice
    // as many; else one after the other, [l][nf] each.
    // (22 more fields per right-hand side: those of the CG and its ring)
    const size_t want = 2 * half_bytes + 22 * FB * nf, have = c.idle_bytes();
    bool together = want <= have || want <= have + c.room() / 2;
    if (together) {
        try {
            shifts_mscg(c, rho, z, src, x, 2 * nf, e.data(), prec, maxiter, st);
        } catch (const Error &err) {
            if (err.code != OVL_ERR_NOMEM) throw;
            together = false;
        }
    }
    if (!together) {
        shifts_mscg(c, rho, z, src, x, nf, e.data(), prec, maxiter, st);
        shifts_mscg(c, rho, z, src + nf * fs, x + (int64_t)nf * nz * fs, nf, e.data() + nf, prec, maxiter, st);
    }
    const int half = nf * nz;
    for (int h = 0; h < 2; ++h)   // two launches: the launch shapes are timed on half the fields
        stencil(c, EPI_K, prec, x + (int64_t)h * half * fs, kx + (int64_t)h * half * fs, half, rho, 0.0, nullptr,
                nullptr);
    if (st) st->dslash_calls[prec] += nf * (1 + 2 * nz);
    const int64_t lstride = (int64_t)(together ? 2 : 1) * nf * fs;
    const int64_t to_b = (int64_t)(together ? nf : half) * fs;
    const ST *xb = x + to_b, *kb = kx + to_b;
    if (dpsi) {
        PoleCoef w{};
        for (int l = 0; l < nz; ++l) w.w[l] = z.omega[l];
        const int64_t n = (int64_t)Planes<ST>::n * g.V;
        k_psi_gradient<ST><<<dim3((unsigned)((n + 255) / 256), nf), 256, 0, c.stream>>>(
            xb, lstride, w, nz, chip64, dpsi, 0.5 * (1.0 + mu), 0.5 * (1.0 - mu), g.V);
        OVL_HIP(hipGetLastError());
        if (st) st->sign_calls[prec] += nf;   // eps(K) chi' of every field
    }
    ForceCoef k{};
    for (int l = 0; l < nz; ++l) k.w[l] = -0.25 * (1.0 - mu) * z.omega[l];
    for (int f = 0; f < nf; ++f) {
        const int64_t o = (int64_t)f * fs;
        k_link_force<ST><<<site_blocks(g, 64), 256, 0, c.stream>>>((const ST *)chip + o, x + o, xb + o, kx + o, kb + o,
                                                              lstride, k, nz, g, dU, f > 0);
        OVL_HIP(hipGetLastError());
    }
}

void overlap_adjoint(Context &c, double rho, double mu, const ovl_zolo &z, const double2 *psi, const double2 *chi,
                     double2 *dpsi, double2 *dU, int nf, double eta, int prec, int maxiter, ovl_stats *st)
{
    OVL_REQUIRE(c.n_low == 0, OVL_ERR_UNSUPPORTED,
                "the derivative of the exact low-mode part is not provided; remove the low modes first");
    OVL_REQUIRE(prec == OVL_F64 || prec == OVL_F32, OVL_ERR_UNSUPPORTED, "the adjoint runs in FP64 or FP32");
    const size_t FB64 = field_bytes(c.g, OVL_F64) * nf;
    double2 *chip = (double2 *)c.buf("adj_chip", FB64);
    copy_fields(c, chi, chip, nf, OVL_F64);
    gamma5_f64(c, chip, nf);   // chi' = gamma_5 chi
    if (!dU) {                 // D^dagger chi = gamma_5 D chi'
        overlap_f64(c, rho, mu, z, chip, dpsi, nf, eta, prec, maxiter, st);
        gamma5_f64(c, dpsi, nf);
        return;
    }
    const size_t FB = field_bytes(c.g, prec) * nf;
    void *src = c.buf("adj_src", 2 * FB);
    convert_spinor(c, psi, OVL_F64, src, prec, nf);
    if (prec == OVL_F64) {
        link_force_t<double2>(c, rho, mu, z, (double2 *)src, chip, chip, dpsi, dU, nf, eta, prec, maxiter, st);
    } else {
        void *c32 = c.buf("adj_chi32", FB);
        convert_spinor(c, chip, OVL_F64, c32, prec, nf);
        link_force_t<float4>(c, rho, mu, z, (float4 *)src, c32, chip, dpsi, dU, nf, eta, prec, maxiter, st);
    }
}

}  // namespace ovl
