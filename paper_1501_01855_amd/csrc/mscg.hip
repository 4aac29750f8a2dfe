// sign(K) by the Zolotarev partial fractions (paper Sec. 3, eq. 7) with the
// lowest kernel eigenvectors treated exactly (Sec. 1 after eq. 4), the
// shifted inversions of K^2 + sigma_l done by one multi-shift CG.
//
// One CG iteration is three launches on the context's stream; the recurrence
// scalars live in device memory (mscg_state.h) so the host never waits inside
// the loop:
//   1. t = K p                                  (stencil)
//   2. w = K t + s0 p, (p, w) per tile          (stencil + fused dots)
//   3. alpha = rr/(p, w), beta; r' = r - alpha w;  (every block reduces the
//      p = r' + beta p of the smallest shift        tile partials itself;
//      zeta_l', alpha_l, beta_l of every shift      block 0 writes the state)
// and, once per group of up to eight iterations, one pass over the shift
// vectors that applies the group's updates to each of them in turn:
//   4. y += sum_l omega_l alpha_l p_l,  p_l = zeta_l' r' + beta_l p_l
// Only the smallest shift's p enters the next iteration's K, so the others can
// wait: the group's residuals r' are kept (a ring of fields instead of one) and
// a shift vector is read and written once per group instead of once per
// iteration.  The sums over shifts and iterations are the same; only y's terms
// are added in another order, and with FP16 storage a shift vector is rounded
// once per group.
// Only y = sum_l omega_l x_l is stored, never the x_l themselves.  A shift is
// frozen once omega_l |zeta_l| ||r|| / (2 sqrt(sigma_l)) <= eta ||b|| / N_Z,
// which bounds the error of the rational function by eta ||b||.  The host
// polls a per-field stop iteration every few iterations.
#include <algorithm>
#include <cmath>

#include <cstring>
#include <initializer_list>
#include <string>
#include <type_traits>

#include "context.h"
#include "fields.h"
#include "kernels.h"
#include "mscg_state.h"
#include "ops.h"

namespace ovl {


struct MscgFinal {
    int iters, breakdown, act_total, pad;
};

// Host memory the device writes (pinned, mapped): each field's final counts
// and then its stop flag, once, when the field stops, so that polling needs no
// copy commands in the stream.  The host presets the flags to "running"
// before a call; every device store there is followed by a system-scope
// fence.  Data flows only device -> host here: the accuracies travel as a
// kernel argument and the constants by an ordinary copy.
constexpr int MS_MAXF = 64;   // fields of one multi-shift solve
struct MscgPinned {
    int stop[MS_MAXF];
    MscgFinal fin[MS_MAXF];
};
struct MscgEta {
    double e2[MS_MAXF];   // eta_f^2 (0: skip field f)
};

__global__ void k_mscg_init(MscgScal *S, int *stop, const double *partial, int nblk, MscgConst k,
                            MscgEta eta2, int *stop_h, MscgFinal *fin_h)
{
    __shared__ double lds[4];
    const int f = blockIdx.x;
    const double b2 = block_allsum(partial + (int64_t)f * nblk, nblk, lds);
    MscgScal &s = S[f];   // parity 0
    if ((int)threadIdx.x < k.nz) {
        const int l = threadIdx.x;
        s.zeta[l] = 1.0;
        s.zeta_old[l] = 1.0;
        s.act[l] = b2 > 0.0 ? 1 : 0;
    }
    if (threadIdx.x != 0) return;
    s.rr = b2;
    // the freezing test uses eta_f^2 ||b||^2; eta_f <= 0 marks a field to skip
    const double e2 = eta2.e2[f];
    s.b2 = e2 > 0.0 ? e2 * b2 : 0.0;
    s.alpha_old = 1.0;
    s.beta_old = 0.0;
    s.iters = 0;
    s.breakdown = 0;
    s.act_total = 0;
    const int st0 = (b2 > 0.0 && e2 > 0.0) ? 0x7fffffff : 0;
    stop[f] = st0;
    if (st0 == 0) {   // nothing to iterate: report the field stopped (the host preset "running")
        fin_h[f] = MscgFinal{0, 0, 0, 0};
        __threadfence_system();
        stop_h[f] = 0;
        __threadfence_system();   // the stores are complete before the kernel is
    }
}

template <typename ST>
__global__ __launch_bounds__(256) void k_norm2(const ST *__restrict__ x, int64_t V, double *partial)
{
    using R = typename Planes<ST>::R;
    const int64_t s = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    const int f = blockIdx.y;
    double d = 0.0;
    if (s < V) {
        cplx<R> v[12];
        ld_sp(x + f * fstride<ST>(V), V, s, v);
#pragma unroll
        for (int c = 0; c < 12; ++c) d += (double)v[c].re * (double)v[c].re + (double)v[c].im * (double)v[c].im;
    }
    __shared__ double lds[4];
    const double t = block_sum<256>(d, lds);
    if (threadIdx.x == 0) partial[(int64_t)f * gridDim.x + blockIdx.x] = t;
}

// Iterations whose shift-vector updates are applied together (their residuals
// cost 32 registers per lane, 40 in FP16 storage).
constexpr int GROUP = 8;

// One element of FP64 / FP32 storage (16 bytes: two or four reals); the
// coefficients of the multi-shift CG are real, so its vector updates act on
// elements whatever complex component they hold.
__device__ __forceinline__ double2 el_axpy(double a, double2 x, double2 y) { return {y.x + a * x.x, y.y + a * x.y}; }
__device__ __forceinline__ float4 el_axpy(float a, float4 x, float4 y)
{
    return {y.x + a * x.x, y.y + a * x.y, y.z + a * x.z, y.w + a * x.w};
}
__device__ __forceinline__ double2 el_comb(double a, double2 x, double b, double2 y)
{
    return {a * x.x + b * y.x, a * x.y + b * y.y};
}
__device__ __forceinline__ float4 el_comb(float a, float4 x, float b, float4 y)
{
    return {a * x.x + b * y.x, a * x.y + b * y.y, a * x.z + b * y.z, a * x.w + b * y.w};
}
__device__ __forceinline__ double el_norm2(double2 x) { return x.x * x.x + x.y * x.y; }
__device__ __forceinline__ double el_norm2(float4 x)
{
    return (double)x.x * (double)x.x + (double)x.y * (double)x.y + (double)x.z * (double)x.z +
           (double)x.w * (double)x.w;
}

// FP16 storage: a lane holds one 16-byte plane (four of the site's twelve
// components) of a site, three waves apart; the site's scale joins the planes
// through LDS.  Three times the lanes of a whole site per lane, a third of its
// registers, and the loads stay consecutive over the wave.
struct HPlane {
    uint4 q;
    float sc;
};
__device__ __forceinline__ HPlane ld_plane(const h8 *p, int64_t V, int k, int64_t s)
{
    return {p[k * V + s].v, reinterpret_cast<const float *>(p + 3 * V)[s]};
}
__device__ __forceinline__ void plane_values(const HPlane &h, float v[8])
{
    const uint32_t w[4] = {h.q.x, h.q.y, h.q.z, h.q.w};
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const float2 a = h2f2(w[c]);
        v[2 * c] = a.x * h.sc;
        v[2 * c + 1] = a.y * h.sc;
    }
}
// The site's largest component from the three planes' values (every thread of
// the block calls it; two buffers in turn, so one barrier per call).
template <int NS>
__device__ __forceinline__ float site_max(const float v[8], float (*mx)[3][NS], int &turn, int k, int j)
{
    float m = 0.f;
#pragma unroll
    for (int c = 0; c < 8; ++c) m = fmaxf(m, fabsf(v[c]));
    float (*b)[NS] = mx[turn];
    turn ^= 1;
    b[k][j] = m;
    __syncthreads();
    return fmaxf(b[0][j], fmaxf(b[1][j], b[2][j]));
}
// Store the plane with the site's scale m; v takes the values as stored.
__device__ __forceinline__ void st_plane(h8 *p, int64_t V, int k, int64_t s, float v[8], float m)
{
    const float inv = h8_inv_scale(m);
    uint32_t w[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        w[c] = f22h2(v[2 * c] * inv, v[2 * c + 1] * inv);
        const float2 a = h2f2(w[c]);
        v[2 * c] = a.x * m;
        v[2 * c + 1] = a.y * m;
    }
    p[k * V + s].v = make_uint4(w[0], w[1], w[2], w[3]);
    if (k == 0) reinterpret_cast<float *>(p + 3 * V)[s] = m;
}

// One multi-shift CG step after the two stencils of the iteration:
//   alpha = (r, r) / (p, w)      (p, w) from the stencil's tile partials;
//                                (r, r) exact, from the previous step's blocks
//   r' = r - alpha w             into the next slot of the ring of residuals;
//                                exact ||r'||^2 per block for the next step
//   beta = ||r'||^2 / (r, r)     with ||r'||^2 = (r, r) - 2 alpha Re (r, w)
//                                + alpha^2 (w, w) (the stencil's other partials),
//                                so that no step waits on a grid-wide sum of r'
//   p = r' + beta p              of the smallest shift, whose zeta stays 1
// Every block derives the scalars from the same partial sums in the same
// order; block 0 also advances the recurrences of the other shifts and writes
// the next state and the iteration's coefficients for k_mscg_flush.
struct MscgStep {
    MscgScal *S;
    MscgCoef *coef;
    int group;
    const MscgConst *kc;
    int *stop;
    const int *itb;   // device iteration base (graph replays), or null
    int itj;
    const double *part;
    int pw_n;
    double *rr_part;
    int rr_n;
    int *stop_h;
    MscgFinal *fin_h;
};

// The scalars of iteration it for field f; false when the field breaks down or
// has stopped (stop: its stopping iteration, tested only once the loads are on
// their way, as it is itself a load from memory).
template <int NT>
__device__ __forceinline__ bool step_scalars(const MscgStep &a, int f, int nf, int it, int stop, double &alpha,
                                             double &beta)
{
    // exact ||r||^2 partials by iteration parity: read this step's, write the next's
    const double *rf = a.rr_part + (size_t)(it & 1) * a.rr_n * nf + (int64_t)f * a.rr_n;
    const double *pf = a.part + (int64_t)f * 3 * a.pw_n;
    const MscgScal &sc = a.S[(it & 1) * nf + f];
    const int pw_n = a.pw_n, rr_n = a.rr_n, group = a.group;
    // block 0 also advances the shifts' recurrences: their state arrives during
    // the sums (one lane per shift; every entry exists, whatever nz)
    const MscgConst *kc = a.kc;
    const int l = threadIdx.x % NZMAX;
    double z = 1.0, zo = 1.0, sig = 0.0, om = 0.0, tol2 = 0.0, al_old = 1.0, be_old = 0.0, b2 = 0.0, s0 = 0.0;
    int was = 0, nz = 0, maxiter = 0, iters = 0, broken = 0, act_total = 0;
    if (blockIdx.x == 0) {
        z = sc.zeta[l];
        zo = sc.zeta_old[l];
        was = sc.act[l];
        sig = kc->sigma[l];
        om = kc->omega[l];
        tol2 = kc->tol2[l];
        al_old = sc.alpha_old;
        be_old = sc.beta_old;
        b2 = sc.b2;
        s0 = kc->s0;
        nz = kc->nz;
        maxiter = kc->maxiter;
        iters = sc.iters;
        broken = sc.breakdown;
        act_total = sc.act_total;
    }
    const double rr0 = sc.rr;
    // The four sums of partials.  Each thread adds its terms in index order;
    // the loads of PB consecutive terms of each sum are issued together (an
    // index past the end reads the last entry, and adds nothing).
    double v0 = 0.0, v1 = 0.0, v2 = 0.0, v3 = 0.0;
    const int nmax = pw_n > rr_n ? pw_n : rr_n;
    constexpr int PB = 4;
    for (int j0 = threadIdx.x; j0 < nmax; j0 += PB * NT) {
        double a0[PB], a1[PB], a2[PB], a3[PB];
#pragma unroll
        for (int q = 0; q < PB; ++q) {
            const int j = j0 + q * NT;
            const int jp = j < pw_n ? j : pw_n - 1, jr = j < rr_n ? j : rr_n - 1;
            a0[q] = pf[jp];
            a1[q] = pf[pw_n + jp];
            a2[q] = pf[2 * pw_n + jp];
            a3[q] = rf[jr];
        }
#pragma unroll
        for (int q = 0; q < PB; ++q) {
            const int j = j0 + q * NT;
            if (j < pw_n) {
                v0 += a0[q];
                v1 += a1[q];
                v2 += a2[q];
            }
            if (it != 0 && j < rr_n) v3 += a3[q];
        }
    }
    if (it >= stop) return false;
    double vv[4] = {v0, v1, v2, v3}, tot[4];
    block_bcast_sum4<NT>(vv, tot);
    const double pw = tot[0], rw = tot[1], ww = tot[2];
    const double rr = it == 0 ? rr0 : tot[3];
    alpha = rr / pw;
    const double rr_new = fmax(0.0, rr - 2.0 * alpha * rw + alpha * alpha * ww);
    const bool ok = pw > 0.0 && isfinite(alpha) && isfinite(rr_new);
    beta = rr_new / rr;
    if (blockIdx.x == 0) {   // the shifts' recurrences (the whole block takes this branch)
        __shared__ int s_act[NZMAX];
        __shared__ int s_keep_any;
        MscgScal &nx = a.S[((it + 1) & 1) * nf + f];
        if (threadIdx.x == 0) s_keep_any = 0;
        __syncthreads();
        if ((int)threadIdx.x < nz) {   // NT >= NZMAX >= nz
            const int act = was && ok;
            s_act[l] = act;
            double zn = z, cy = 0.0, bl = 0.0;
            if (act) {
                zn = (z * zo * al_old) / (alpha * be_old * (zo - z) + zo * al_old * (1.0 + (sig - s0) * alpha));
                const double q = zn / z;
                cy = om * (alpha * zn / z);
                bl = beta * q * q;
            }
            MscgCoef &cf = a.coef[(int64_t)f * group + it % group];
            cf.cy[l] = cy;
            cf.zn[l] = zn;
            cf.bl[l] = bl;
            cf.act[l] = act;
            nx.zeta_old[l] = act ? z : zo;
            nx.zeta[l] = zn;
            const int keep = act && !(zn * zn * rr_new <= tol2 * b2);
            nx.act[l] = keep;
            if (keep) atomicOr(&s_keep_any, 1);
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            int na = 0;
            if (it % group == 0)
                for (int q = 0; q < nz; ++q) na += s_act[q];
            broken = broken || !ok;
            iters += 1;
            act_total += na;
            nx.rr = rr_new;
            nx.b2 = b2;
            nx.alpha_old = alpha;
            nx.beta_old = beta;
            nx.iters = iters;
            nx.breakdown = broken;
            nx.act_total = act_total;
            if (!s_keep_any || broken || iters >= maxiter) {
                // host memory is written once per field and call, when it stops;
                // the counts reach the host before the flag
                a.fin_h[f] = MscgFinal{iters, broken, act_total, 0};
                __threadfence_system();
                a.stop[f] = it + 1;
                a.stop_h[f] = it + 1;
                __threadfence_system();   // complete before the kernel is
            }
        }
    }
    return ok;
}

// FP64 and FP32.  Memory-bound, five fields moved; 1024 threads per block on
// large lattices, because every block reads all partials (three sums over up
// to 5376 tiles on 24^3 x 48): larger blocks are fewer, and each thread's share
// of the sums is one or two batches of loads.  256 on small ones, where the
// reductions over a block are what takes the time.
template <typename ST, int NT>
__global__ __launch_bounds__(NT) void k_mscg_step(const ST *rin, ST *rout, const ST *__restrict__ w,
                                                       const ST *pin, ST *pb, MscgStep a, int64_t V)
{
    using R = typename Planes<ST>::R;
    const int f = blockIdx.y, nf = gridDim.y;
    const int it = a.itb ? *a.itb + a.itj : a.itj;
    const int stop = a.stop[f];   // tested once the first loads are on their way
    const int64_t fo = f * fstride<ST>(V);
    const int64_t n = Planes<ST>::n * V;
    int64_t i = blockIdx.x * (int64_t)NT + threadIdx.x;
    // Two elements per thread and pass.  The first pass's loads do not depend
    // on the step's scalars: they go out before the sums of partials, and
    // arrive during them.
    const int64_t step = (int64_t)gridDim.x * NT;
    ST rv[2]{}, wv[2]{}, pv[2]{};
    auto load = [&] {
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (i + q * step < n) {
                const int64_t o = fo + i + q * step;
                rv[q] = rin[o];
                wv[q] = w[o];
                pv[q] = pin[o];
            }
    };
    load();
    double alpha, beta;
    if (!step_scalars<NT>(a, f, nf, it, stop, alpha, beta)) return;
    const R ar = (R)alpha, br = (R)beta;
    double rn = 0.0;
    while (i < n) {
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (i + q * step < n) {
                const int64_t o = fo + i + q * step;
                rv[q] = el_axpy(-ar, wv[q], rv[q]);
                rout[o] = rv[q];
                rn += el_norm2(rv[q]);
                pb[o] = el_axpy(br, pv[q], rv[q]);
            }
        i += 2 * step;
        load();
    }
    __shared__ double lds[NT / 64];
    const double t = block_sum<NT>(rn, lds);
    if (threadIdx.x == 0)
        a.rr_part[(size_t)((it + 1) & 1) * a.rr_n * nf + (int64_t)f * gridDim.x + blockIdx.x] = t;
}

// FP16 storage, NS sites per block and pass, three lanes per site: 256 sites
// (few blocks, so few readings of the partials) where the lattice fills the
// chip with them, else 64.
template <int NS>
__global__ __launch_bounds__(3 * NS) void k_mscg_step_h(const h8 *rin, h8 *rout, const h8 *__restrict__ w,
                                                        const h8 *pin, h8 *pb, MscgStep a, int64_t V)
{
    const int f = blockIdx.y, nf = gridDim.y;
    const int it = a.itb ? *a.itb + a.itj : a.itj;
    const int stop = a.stop[f];   // tested once the first loads are on their way
    __shared__ float mx[2][3][NS];
    const int64_t fo = f * fstride<h8>(V);
    const int k = threadIdx.x / NS, j = threadIdx.x % NS;   // plane (the same for a wave) and site of the pass
    int64_t s0 = blockIdx.x * (int64_t)NS;
    HPlane rq{}, wq{}, pq{};
    auto load = [&] {
        if (s0 + j < V) {
            rq = ld_plane(rin + fo, V, k, s0 + j);
            wq = ld_plane(w + fo, V, k, s0 + j);
            pq = ld_plane(pin + fo, V, k, s0 + j);
        }
    };
    load();
    double alpha, beta;
    if (!step_scalars<3 * NS>(a, f, nf, it, stop, alpha, beta)) return;
    const float ar = (float)alpha, br = (float)beta;
    double rn = 0.0;
    int turn = 0;
    while (s0 < V) {   // the same passes for every thread of the block
        const int64_t s = s0 + j;
        const bool valid = s < V;
        float rv[8], pv[8];
        plane_values(rq, rv);
        plane_values(wq, pv);
#pragma unroll
        for (int c = 0; c < 8; ++c) rv[c] = rv[c] - ar * pv[c];
        float m = site_max<NS>(rv, mx, turn, k, j);
        if (valid) {
            st_plane(rout + fo, V, k, s, rv, m);   // continue with r' as stored
#pragma unroll
            for (int c = 0; c < 8; ++c) rn += (double)rv[c] * (double)rv[c];
        }
        plane_values(pq, pv);
#pragma unroll
        for (int c = 0; c < 8; ++c) pv[c] = rv[c] + br * pv[c];
        s0 += (int64_t)gridDim.x * NS;
        load();
        m = site_max<NS>(pv, mx, turn, k, j);
        if (valid) st_plane(pb + fo, V, k, s, pv, m);
    }
    __shared__ double lds[3 * NS / 64];
    const double t = block_sum<3 * NS>(rn, lds);
    if (threadIdx.x == 0)
        a.rr_part[(size_t)((it + 1) & 1) * a.rr_n * nf + (int64_t)f * gridDim.x + blockIdx.x] = t;
}

// The shift vectors brought up to date by the group of iterations that starts
// at it0 (a multiple of group): for the group's iterations k that the field
// ran, in order, y += cy_l p_l and p_l = zn_l r_{k+1} + bl_l p_l over the
// shifts active in them, each p_l held in registers through the group.  In the
// first group every p_l starts as the source and y at zero (also for a field
// that ran no iteration).  A p_l that no later iteration needs is not written
// back.
// Memory-bound: per group (cnt + 2 + 2 n_active) fields, against (2 +
// 2 n_active) fields in every iteration when the shift vectors follow at once.
// Measured per iteration, step and an eighth of a flush against one update of
// everything in every iteration: 24^3 x 48, one FP64 field, sign call to 1e-10
// with 20 poles, 105 + 74 against 485 us (the step at 6.1 TB/s); twelve FP32
// fields of 16^3 x 32 to 1e-5, 167 + 81 against 523 us; one FP16 field of
// 24^3 x 48 in a relaxed solve (3 to 6 poles), 29 + 10 against 43 us.
struct MscgFlush {
    const MscgScal *S;
    const MscgCoef *coef;
    int group;
    const MscgConst *kc;
    const int *stop;
    const int *itb;
    int itj;
};

// The group's work for field f: the coefficients in the arithmetic type, the
// list of shifts active in it and in how many of its iterations each is (a
// frozen shift stays frozen; negative where its p_l is needed no more).
// False when the field has nothing to do.
template <typename R>
struct GroupWork {
    R cy[GROUP][NZMAX], zn[GROUP][NZMAX], bl[GROUP][NZMAX];
    int l[NZMAX], n[NZMAX], na;
};
template <typename R>
__device__ __forceinline__ bool group_work(const MscgFlush &a, int f, int nf, GroupWork<R> &g, int &it0, int &cnt)
{
    it0 = a.itb ? *a.itb + a.itj : a.itj;
    const int st = a.stop[f];
    if (st <= it0 && it0 != 0) return false;
    cnt = st - it0 < a.group ? st - it0 : a.group;
    const int nz = a.kc->nz;
    const MscgScal &nx = a.S[((it0 + cnt) & 1) * nf + f];
    for (int q = threadIdx.x; q < cnt * nz; q += blockDim.x) {
        const int k = q / nz, l = q % nz;
        const MscgCoef &cf = a.coef[(int64_t)f * a.group + k];
        g.cy[k][l] = (R)cf.cy[l];
        g.zn[k][l] = (R)cf.zn[l];
        g.bl[k][l] = (R)cf.bl[l];
    }
    if (threadIdx.x < 64) {   // one wave: NZMAX = 64 shifts
        const int l = threadIdx.x;
        int na = 0;
        if (l < nz)
            for (int k = 0; k < cnt; ++k) na += a.coef[(int64_t)f * a.group + k].act[l] != 0;
        const unsigned long long m = __ballot(na > 0);
        if (na > 0) {
            const int at = __popcll(m & ((1ull << l) - 1));
            g.l[at] = l;
            g.n[at] = st > it0 + cnt && nx.act[l] ? na : -na;
        }
        if (l == 0) g.na = __popcll(m);
    }
    __syncthreads();
    return true;
}

// FP64 and FP32, element by element.  With ALL, y holds one solution per
// shift, shift-major like p, and x_l += cy_l p_l (the caller passes
// omega_l = 1).
template <typename ST, bool ALL>
__global__ __launch_bounds__(256) void k_mscg_flush(const ST *__restrict__ src, const ST *__restrict__ ring,
                                                    ST *__restrict__ y, ST *__restrict__ p, MscgFlush a, int64_t V)
{
    using R = typename Planes<ST>::R;
    const int f = blockIdx.y, nf = gridDim.y;
    __shared__ GroupWork<R> g;
    int it0, cnt;
    if (!group_work(a, f, nf, g, it0, cnt)) return;
    const bool first = it0 == 0;
    const int na = g.na;
    const int64_t fo = f * fstride<ST>(V);
    const int64_t fstep = (int64_t)nf * fstride<ST>(V);   // shift-major p[l][f]; ring slots likewise
    const int64_t n = Planes<ST>::n * V;
    const ST zero = el_comb(R(0), ST{}, R(0), ST{});
    for (int64_t i = blockIdx.x * (int64_t)256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        ST rk[GROUP];
#pragma unroll
        for (int k = 0; k < GROUP; ++k)
            if (k < cnt) rk[k] = ring[((k + 1) % a.group) * fstep + fo + i];
        ST yv = zero, sv = zero;
        if (first)
            sv = src[fo + i];
        else if constexpr (!ALL)
            yv = y[fo + i];
        constexpr int LB = 4;   // shift vectors whose loads are in flight together
        for (int a0 = 0; a0 < na; a0 += LB) {
            ST pv[LB], xv[LB];
#pragma unroll
            for (int b = 0; b < LB; ++b) {
                pv[b] = sv;
                xv[b] = zero;
                if (a0 + b < na && !first) {
                    const int64_t o = g.l[a0 + b] * fstep + fo + i;
                    pv[b] = p[o];
                    if constexpr (ALL) xv[b] = y[o];
                }
            }
#pragma unroll
            for (int b = 0; b < LB; ++b) {
                if (a0 + b >= na) continue;
                const int l = g.l[a0 + b], nl = g.n[a0 + b], kn = nl < 0 ? -nl : nl;
                ST xl = ALL ? xv[b] : yv;
#pragma unroll
                for (int k = 0; k < GROUP; ++k) {
                    if (k >= kn) continue;
                    xl = el_axpy(g.cy[k][l], pv[b], xl);
                    pv[b] = el_comb(g.zn[k][l], rk[k], g.bl[k][l], pv[b]);
                }
                const int64_t o = l * fstep + fo + i;
                if (nl > 0) p[o] = pv[b];
                if constexpr (ALL)
                    y[o] = xl;
                else
                    yv = xl;
            }
        }
        if constexpr (!ALL)
            y[fo + i] = yv;
        else if (cnt == 0)   // a field with no iteration: its solutions are zero
            for (int l = 0; l < a.kc->nz; ++l) y[l * fstep + fo + i] = zero;
    }
}

// FP16 storage: three lanes per site as in the step; a p_l and y are rounded
// to FP16 once per group.
template <int NS>
__global__ __launch_bounds__(3 * NS) void k_mscg_flush_h(const h8 *__restrict__ src, const h8 *__restrict__ ring,
                                                         h8 *__restrict__ y, h8 *__restrict__ p, MscgFlush a,
                                                         int64_t V)
{
    const int f = blockIdx.y, nf = gridDim.y;
    __shared__ GroupWork<float> g;
    __shared__ float mx[2][3][NS];
    int it0, cnt;
    if (!group_work(a, f, nf, g, it0, cnt)) return;
    const bool first = it0 == 0;
    const int na = g.na;
    const int64_t fo = f * fstride<h8>(V);
    const int64_t fstep = (int64_t)nf * fstride<h8>(V);
    const int k3 = threadIdx.x / NS, j = threadIdx.x % NS;
    int turn = 0;
    for (int64_t s0 = blockIdx.x * (int64_t)NS; s0 < V; s0 += (int64_t)gridDim.x * NS) {
        const int64_t s = s0 + j;
        const bool valid = s < V;
        HPlane rk[GROUP]{}, sq{}, yq{};
        float rv[GROUP][8], yv[8];
        if (valid) {
#pragma unroll
            for (int k = 0; k < GROUP; ++k)
                if (k < cnt) rk[k] = ld_plane(ring + ((k + 1) % a.group) * fstep + fo, V, k3, s);
            if (first)
                sq = ld_plane(src + fo, V, k3, s);
            else
                yq = ld_plane(y + fo, V, k3, s);
        }
        plane_values(yq, yv);   // zero in the first group
#pragma unroll
        for (int k = 0; k < GROUP; ++k) plane_values(rk[k], rv[k]);
        for (int b = 0; b < na; ++b) {
            const int l = g.l[b], nl = g.n[b], kn = nl < 0 ? -nl : nl;
            HPlane pq = sq;
            if (valid && !first) pq = ld_plane(p + l * fstep + fo, V, k3, s);
            float pv[8];
            plane_values(pq, pv);
#pragma unroll
            for (int k = 0; k < GROUP; ++k) {
                if (k >= kn) continue;
                const float cy = g.cy[k][l], zn = g.zn[k][l], bl = g.bl[k][l];
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    yv[c] = yv[c] + cy * pv[c];
                    pv[c] = zn * rv[k][c] + bl * pv[c];
                }
            }
            if (nl > 0) {   // the same for the whole block
                const float m = site_max<NS>(pv, mx, turn, k3, j);
                if (valid) st_plane(p + l * fstep + fo, V, k3, s, pv, m);
            }
        }
        const float m = site_max<NS>(yv, mx, turn, k3, j);
        if (valid) st_plane(y + fo, V, k3, s, yv, m);
    }
}

// Iteration base of graph replays: set, then advanced after each chunk.
__global__ void k_set_it(int *itb, int v)
{
    if (threadIdx.x == 0) *itb = v;
}
__global__ void k_advance(int *itb, int n)
{
    if (threadIdx.x == 0) *itb += n;
}

// ---- low-mode projection (basis [n] packed fields and the fields in the
// storage type ST of the call; sums in FP64)
template <typename ST>
__global__ __launch_bounds__(256) void k_low_dots(const ST *__restrict__ basis, int n,
                                                  const ST *__restrict__ x, int64_t V, double *partial)
{
    using R = typename Planes<ST>::R;
    constexpr int NB = 8;   // basis vectors per pass: their loads are issued together
    const int f = blockIdx.y;
    const int64_t s = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    __shared__ double lds[2 * NB][4];   // [value][wave]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    cplx<R> xv[12];
    if (s < V) ld_sp(x + f * fstride<ST>(V), V, s, xv);
    for (int j0 = 0; j0 < n; j0 += NB) {
        double d[2 * NB];
#pragma unroll
        for (int q = 0; q < 2 * NB; ++q) d[q] = 0.0;
#pragma unroll
        for (int q = 0; q < NB; ++q) {
            const int j = j0 + q;
            if (s < V && j < n) {
                cplx<R> b[12];
                ld_sp(basis + (int64_t)j * fstride<ST>(V), V, s, b);
                double dr = 0.0, di = 0.0;
#pragma unroll
                for (int c = 0; c < 12; ++c) {
                    const double xr = xv[c].re, xi = xv[c].im, br = b[c].re, bi = b[c].im;
                    dr += br * xr + bi * xi;
                    di += br * xi - bi * xr;
                }
                d[2 * q] = dr;
                d[2 * q + 1] = di;
            }
        }
        // block sums of the 2 NB values (fixed order, one LDS pass)
#pragma unroll
        for (int q = 0; q < 2 * NB; ++q)
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) d[q] += __shfl_xor(d[q], off, 64);
        __syncthreads();   // the previous pass has read lds
        if (lane == 0)
#pragma unroll
            for (int q = 0; q < 2 * NB; ++q) lds[q][wave] = d[q];
        __syncthreads();
        const int q = threadIdx.x;
        if (q < 2 * NB && j0 + q / 2 < n) {
            double t = 0.0;
#pragma unroll
            for (int w = 0; w < 4; ++w) t += lds[q][w];
            const int j = j0 + q / 2;
            partial[(((int64_t)f * n + j) * 2 + (q & 1)) * gridDim.x + blockIdx.x] = t;
        }
    }
}

__global__ void k_reduce_rows(const double *partial, int nblk, double *out)
{
    __shared__ double lds[4];
    const double v = block_allsum(partial + (int64_t)blockIdx.x * nblk, nblk, lds);
    if (threadIdx.x == 0) out[blockIdx.x] = v;
}

// x_perp = x - sum_j c_j v_j ; ex = sum_j sign(lambda_j) c_j v_j
template <typename ST>
__global__ __launch_bounds__(256) void k_low_project(const ST *__restrict__ basis, int n,
                                                     const double *__restrict__ coef, const double *__restrict__ sgn,
                                                     const ST *__restrict__ x, ST *__restrict__ xp,
                                                     ST *__restrict__ ex, int64_t V)
{
    using R = typename Planes<ST>::R;
    const int f = blockIdx.y;
    const int64_t s = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
    if (s >= V) return;
    cplx<R> xv[12];
    ld_sp(x + f * fstride<ST>(V), V, s, xv);
    cplx<double> a[12], e[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) {
        a[c] = {(double)xv[c].re, (double)xv[c].im};
        e[c] = {0.0, 0.0};
    }
    for (int j = 0; j < n; ++j) {
        const cplx<double> cj = {coef[((int64_t)f * n + j) * 2], coef[((int64_t)f * n + j) * 2 + 1]};
        const double sj = sgn[j];
        cplx<R> b[12];
        ld_sp(basis + (int64_t)j * fstride<ST>(V), V, s, b);
#pragma unroll
        for (int c = 0; c < 12; ++c) {
            const cplx<double> t = cj * cplx<double>{(double)b[c].re, (double)b[c].im};
            a[c] = a[c] - t;
            e[c] = e[c] + sj * t;
        }
    }
    cplx<R> o[12], oe[12];
#pragma unroll
    for (int c = 0; c < 12; ++c) {
        o[c] = {(R)a[c].re, (R)a[c].im};
        oe[c] = {(R)e[c].re, (R)e[c].im};
    }
    st_sp(xp + f * fstride<ST>(V), V, s, o);
    st_sp(ex + f * fstride<ST>(V), V, s, oe);
}

// --------------------------------------------------------------- host driver
// The graph of one chunk of multi-shift iterations (kernel nodes in launch
// order, then the advance of the iteration base), recorded once per launch
// configuration: buffers, constants that are passed by value, the stencil
// launch variants and the field count.  record(j) issues iteration j of the
// chunk through launch_k().
template <typename F>
static hipGraphExec_t chunk_graph(Context &c, int prec, int nf, bool all, int chunk, int *itb, F record,
                                  std::initializer_list<const void *> ptrs, std::initializer_list<double> vals)
{
    std::string key;
    auto put = [&](const void *d, size_t n) { key.append(reinterpret_cast<const char *>(d), n); };
    const int head[7] = {prec, nf, all ? 1 : 0, chunk, stencil_variant(c, EPI_K, prec, nf),
                         stencil_variant(c, EPI_K2DOT, prec, nf), c.g.two_row + 2 * c.g.two_row64};
    put(head, sizeof(head));
    put(&c.U64r, sizeof(c.U64r));
    for (const void *q : ptrs) put(&q, sizeof(q));
    for (double v : vals) put(&v, sizeof(v));
    put(&itb, sizeof(itb));
    auto found = c.graphs.find(key);
    if (found != c.graphs.end()) return found->second;
    GraphRec gr;
    OVL_HIP(hipGraphCreate(&gr.g, 0));
    c.rec = &gr;
    try {
        for (int j = 0; j < chunk; ++j) record(j);
        launch_k(c, nullptr, k_advance, dim3(1), dim3(64), 0, itb, chunk);
    } catch (...) {
        c.rec = nullptr;
        hipGraphDestroy(gr.g);
        throw;
    }
    c.rec = nullptr;
    hipGraphExec_t exec = nullptr;
    const hipError_t e = hipGraphInstantiate(&exec, gr.g, nullptr, nullptr, 0);
    hipGraphDestroy(gr.g);
    OVL_HIP(e);
    c.graphs[key] = exec;
    return exec;
}

// out = sign(K) in, or (xs != nullptr) every shifted solution
// xs[l][f] = (K^2 + sigma_l)^{-1} in_f, each to |zeta_l| ||r|| <= eta_f ||in_f||,
// with no low-mode split and no final K.
//
// The update kernels' grids are at most the number of their blocks resident on
// the device at once: they stride over a field, and a larger grid would leave a
// partial second round of blocks running after the first, with one more
// prologue each.  The step's blocks are shared among the fields of a launch
// (its prologue reads every tile's sums: 193 -> 168 us for 12 FP32 fields of
// 16^3 x 32); the flush, with its short prologue and one long chain of loads
// per element, is faster with that many blocks per field (649 against 882 us).
template <typename K>
static unsigned resident_blocks(Context &c, int &per_cu, K *kernel, int nt)
{
    if (per_cu == 0) {
        int b = 0;
        OVL_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, kernel, nt, 0));
        per_cu = b > 0 ? b : 1;
    }
    return (unsigned)(per_cu * c.num_cu);
}

// The ring of residuals: GROUP slots (iterations per group), halved while the
// ring would take more than a quarter of the memory to be had (one slot is the
// residual updated in place).
static void *residual_ring(Context &c, size_t field_set, int &group)
{
    const size_t held = c.pool["ms_ring"].bytes;
    if (held < field_set * group) {
        const size_t room = c.room() + held;
        while (group > 1 && field_set * group > room / 4) group /= 2;
    }
    for (; group > 1; group /= 2)
        if (void *p = c.opt_buf("ms_ring", field_set * group)) return p;
    return c.buf("ms_ring", field_set);
}

// The buffers of a multi-shift CG hold nothing once it has ended.
struct MscgScratch {
    Context &c;
    ~MscgScratch() { c.idle({"ms_src", "ms_pb", "ms_t", "ms_w", "ms_y", "ms_p", "ms_ring"}); }
};

template <typename ST>
static void sign_t(Context &c, double rho, const ovl_zolo &z, const void *in, void *out, int nf,
                   const double *eta, int prec, int maxiter, ovl_stats *st, void *xs = nullptr)
{
    const bool all = xs != nullptr;
    const Geom &g = c.g;
    const int64_t V = g.V;
    const size_t FB = field_bytes(g, prec);
    const unsigned nblk = site_blocks(g);
    const unsigned nblk_max = (unsigned)stencil_tiles_max(g);   // tiles of any stencil variant
    const dim3 grid(nblk, nf);
    // the update kernels and their grids: elements of 16 bytes, or in FP16
    // storage three lanes per site, with 64-site blocks in the step where
    // 256-site ones would be fewer than two per CU
    void (*step)(const ST *, ST *, const ST *, const ST *, ST *, MscgStep, int64_t) = nullptr;
    void (*flush)(const ST *, const ST *, ST *, ST *, MscgFlush, int64_t) = nullptr;
    unsigned step_nt, flush_nt = 256, nstep, nflush;
    int *const per_cu = c.upd_per_cu[prec];
    auto share = [&](unsigned blocks) { return (blocks + nf - 1) / (unsigned)nf; };
    if constexpr (std::is_same<ST, h8>::value) {
        const int ns = V >= (int64_t)512 * c.num_cu ? 256 : 64;
        step = ns == 256 ? k_mscg_step_h<256> : k_mscg_step_h<64>;
        flush = k_mscg_flush_h<64>;
        step_nt = 3 * ns;
        flush_nt = 3 * 64;
        nstep = std::min(share(resident_blocks(c, per_cu[0], step, 3 * ns)), (unsigned)((V + ns - 1) / ns));
        nflush = std::min(resident_blocks(c, per_cu[1], flush, 3 * 64), (unsigned)((V + 63) / 64));
    } else {
        flush = all ? k_mscg_flush<ST, true> : k_mscg_flush<ST, false>;
        const int64_t n = Planes<ST>::n * V;
        step_nt = n < (int64_t)1024 * c.num_cu ? 256 : 1024;
        step = step_nt == 256 ? k_mscg_step<ST, 256> : k_mscg_step<ST, 1024>;
        nstep = std::min(share(resident_blocks(c, per_cu[0], step, step_nt)), (unsigned)((n + step_nt - 1) / step_nt));
        nflush = std::min(resident_blocks(c, per_cu[all ? 2 : 1], flush, 256), (unsigned)((n + 255) / 256));
    }
    const int nz = z.n_z;
    OVL_REQUIRE(nz >= 1 && nz <= NZMAX, OVL_ERR_ARG, "n_z out of range");
    int nact = 0;
    std::vector<double> eta2(nf);
    for (int f = 0; f < nf; ++f) {
        eta2[f] = eta[f] > 0.0 ? eta[f] * eta[f] : 0.0;
        nact += eta[f] > 0.0;
    }
    for (int l = 0; l < nz; ++l)
        OVL_REQUIRE(z.sigma[l] > 0.0 && z.omega[l] > 0.0, OVL_ERR_ARG, "Zolotarev coefficients must be positive");

    const bool low = c.n_low > 0 && !all;
    const MscgScratch scratch{c};
    // the source: the input itself, or its part off the low modes (whose exact
    // part then waits in the output until the final K)
    const ST *src = low ? (const ST *)c.buf("ms_src", FB * nf) : (const ST *)in;
    ST *pb = (ST *)c.buf("ms_pb", FB * nf);   // the smallest shift's p, in step with the CG
    ST *t = (ST *)c.buf("ms_t", FB * nf);
    ST *w = (ST *)c.buf("ms_w", FB * nf);
    ST *y = all ? (ST *)xs : (ST *)c.buf("ms_y", FB * nf);
    ST *p = (ST *)c.buf("ms_p", FB * nf * nz);
    const int nl = c.n_low > 0 ? c.n_low : 1;
    double *part = (double *)c.buf("ms_part", sizeof(double) * (size_t)std::max(3 * nblk_max, nblk * 2 * nl) * nf);
    double *rr_part = (double *)c.buf("ms_part2", sizeof(double) * 2 * (size_t)nstep * nf);   // by step parity
    double *lcoef = (double *)c.buf("ms_coef", sizeof(double) * (size_t)nf * 2 * nl);
    MscgScal *S = (MscgScal *)c.buf("ms_scal", sizeof(MscgScal) * 2 * nf);
    int *stop = (int *)c.buf("ms_stop", sizeof(int) * nf);
    MscgConst *kdev = (MscgConst *)c.buf("ms_const", sizeof(MscgConst));
    MscgCoef *coef = (MscgCoef *)c.buf("ms_cring", sizeof(MscgCoef) * GROUP * nf);
    int group = GROUP;
    ST *ring = (ST *)residual_ring(c, FB * nf, group);

    // pinned staging: constants, accuracies, and two slots of polled flags
    OVL_REQUIRE(nf <= MS_MAXF, OVL_ERR_ARG, "too many fields in one multi-shift solve");
    if (!c.ms_pin) {
        OVL_HIP(hipHostMalloc(&c.ms_pin, sizeof(MscgPinned), hipHostMallocMapped | hipHostMallocCoherent));
        std::memset(c.ms_pin, 0, sizeof(MscgPinned));
        for (auto &e : c.ms_ev) OVL_HIP(hipEventCreate(&e));
    }
    volatile MscgPinned &hp = *(volatile MscgPinned *)c.ms_pin;
    MscgPinned *hpd = nullptr;   // the same memory, as the device addresses it
    OVL_HIP(hipHostGetDevicePointer((void **)&hpd, c.ms_pin, 0));

    // 1. low-mode split: src = (1 - P) in, ex = sum sign(lambda) P in, with the
    //    basis stored like the fields (its rounding is that of the call)
    if (low) {
        const ST *basis = (const ST *)c.low_basis(prec);
        const double *sgn = c.low_signs();
        k_low_dots<ST><<<grid, 256, 0, c.stream>>>(basis, c.n_low, (const ST *)in, V, part);
        k_reduce_rows<<<nf * c.n_low * 2, 256, 0, c.stream>>>(part, nblk, lcoef);
        k_low_project<ST><<<grid, 256, 0, c.stream>>>(basis, c.n_low, lcoef, sgn, (const ST *)in,
                                                         const_cast<ST *>(src), (ST *)out, V);
        OVL_HIP(hipGetLastError());
    }

    // 2. constants (uploaded when they change) and initial state
    MscgConst k{};
    k.nz = nz;
    k.maxiter = maxiter;
    int base = 0;
    for (int l = 1; l < nz; ++l)
        if (z.sigma[l] < z.sigma[base]) base = l;
    k.s0 = z.sigma[base];
    for (int l = 0; l < nz; ++l) {
        k.sigma[l] = z.sigma[l];
        k.omega[l] = all ? 1.0 : z.omega[l];
        const double tl = all ? 1.0 : 2.0 * std::sqrt(z.sigma[l]) / (nz * z.omega[l]);
        k.tol2[l] = tl * tl;
    }
    const char *kb = reinterpret_cast<const char *>(&k);
    if (c.ms_const_last.size() != sizeof(k) || std::memcmp(c.ms_const_last.data(), kb, sizeof(k)) != 0) {
        // from pageable memory: the runtime stages the copy before returning
        OVL_HIP(hipMemcpyAsync(kdev, &k, sizeof(MscgConst), hipMemcpyHostToDevice, c.stream));
        c.ms_const_last.assign(kb, kb + sizeof(k));
    }
    k_norm2<ST><<<grid, 256, 0, c.stream>>>(src, V, part);
    MscgEta ea{};
    for (int f = 0; f < nf; ++f) {
        ea.e2[f] = eta2[f];
        hp.stop[f] = 0x7fffffff;   // "running" until a kernel writes the field's stop
    }
    k_mscg_init<<<nf, 256, 0, c.stream>>>(S, stop, part, nblk, k, ea, hpd->stop, hpd->fin);
    OVL_HIP(hipGetLastError());

    // 3. iterations; poll the stop flags every CHUNK iterations, one chunk
    //    behind, so the queue never runs dry.  The first chunk is launched
    //    directly (it also settles the stencil launch variants); later chunks
    //    replay a graph of CHUNK iterations whose kernels read the iteration
    //    from *itb, unless profiling (per-launch events) is on.  A replayed
    //    chunk holds whole groups, so that its ring slots are the same.
    const bool replay = c.use_graphs && !c.prof;
    const int CHUNK = replay ? std::max(4, group) : 4;
    const size_t pst = (size_t)(FB / sizeof(ST)) * nf;   // elements between ring slots
    int *itb = (int *)c.buf("ms_itb", sizeof(int));
    // the group that starts at iteration *ib + j0; the source is read in the first
    // group only, which is never replayed, so a graph does not depend on it
    auto run_flush = [&](int j0, const int *ib) {
        PendingEvent pe;
        if (c.prof) c.prof_begin(pe, KERN_SHIFT, prec, 0.0);
        launch_k(c, c.prof ? &pe : nullptr, flush, dim3(nflush, nf), dim3(flush_nt), 0, ib ? pb : src, ring, y, p,
                 MscgFlush{S, coef, group, kdev, stop, ib, j0}, V);
        if (c.prof) c.prof_end(pe);
        OVL_HIP(hipGetLastError());
    };
    auto one_iter = [&](int j, const int *ib) {   // iteration *ib + j (ib null: iteration j)
        const bool zero = ib == nullptr && j == 0;
        const ST *pin = zero ? src : pb;
        const ST *rin = zero ? src : ring + (j % group) * pst;
        stencil(c, EPI_K, prec, pin, t, nf, rho, 0.0, nullptr, nullptr, stop, j, nullptr, ib);
        const int ntile = stencil_k2_dot(c, prec, t, w, nf, rho, k.s0, pin, rin, part, stop, j, ib);
        PendingEvent pe;
        if (c.prof) c.prof_begin(pe, KERN_SHIFT, prec, 0.0);
        launch_k(c, c.prof ? &pe : nullptr, step, dim3(nstep, nf), dim3(step_nt), 0, rin, ring + ((j + 1) % group) * pst,
                 w, pin, pb, MscgStep{S, coef, group, kdev, stop, ib, j, part, ntile, rr_part, (int)nstep, hpd->stop, hpd->fin},
                 V);
        if (c.prof) c.prof_end(pe);
        OVL_HIP(hipGetLastError());
        if ((j + 1) % group == 0) run_flush(j + 1 - group, ib);
    };
    hipGraphExec_t gexec = nullptr;
    int it = 0;
    int pending = -1;
    bool done = false;
    while (!done) {
        if (it == 0 || !replay) {
            for (int j = 0; j < CHUNK; ++j) one_iter(it + j, nullptr);
        } else {
            if (!gexec) gexec = chunk_graph(c, prec, nf, all, CHUNK, itb, [&](int j) { one_iter(j, itb); },
                                            {ring, t, w, y, p, pb, S, kdev, coef, stop, part, rr_part, hpd,
                                             (const void *)(intptr_t)group, (const void *)(intptr_t)nstep},
                                            {rho, k.s0});
            if (it == CHUNK) {
                k_set_it<<<1, 64, 0, c.stream>>>(itb, it);
                OVL_HIP(hipGetLastError());
            }
            OVL_HIP(hipGraphLaunch(gexec, c.stream));
        }
        it += CHUNK;
        const int slot = (it / CHUNK) & 1;
        OVL_HIP(hipEventRecord(c.ms_ev[slot], c.stream));
        if (pending >= 0) {
            // chunk `pending` has completed, so its flags are in host memory
            // (later chunks may have written newer ones: also valid)
            c.spin_wait(c.ms_ev[pending]);
            bool every = true;
            for (int f = 0; f < nf; ++f) every = every && hp.stop[f] != 0x7fffffff;
            if (every) done = true;
        }
        pending = slot;
        if (!done && it >= maxiter + 2 * CHUNK) {   // cannot happen: the kernels stop at maxiter
            OVL_HIP(hipEventSynchronize(c.ms_ev[slot]));
            done = true;
        }
    }
    if (it % group != 0) {   // the last, partial group, unless every field stopped before it
        int last = 0;
        for (int f = 0; f < nf; ++f) last = std::max(last, (int)hp.stop[f]);
        const int j0 = it - it % group;
        if (j0 == 0 || last > j0) run_flush(j0, nullptr);
    }

    // 4. s = K y + ex, the exact part in the output already
    if (all) {
    } else if (low) {
        stencil(c, EPI_KPLUS, prec, y, out, nf, rho, 0.0, out, nullptr);
    } else {
        stencil(c, EPI_K, prec, y, out, nf, rho, 0.0, nullptr, nullptr);
    }
    OVL_HIP(hipGetLastError());

    // every field has stopped: no kernel writes these any more
    std::vector<MscgFinal> hs(nf);
    std::vector<int> hstop_final(nf);
    for (int f = 0; f < nf; ++f) {
        hstop_final[f] = hp.stop[f];
        hs[f].iters = hp.fin[f].iters;
        hs[f].breakdown = hp.fin[f].breakdown;
        hs[f].act_total = hp.fin[f].act_total;
    }
    if (c.prof) c.prof_collect();
    int64_t iters = 0, act_total = 0, launches = 0, groups = 0;
    bool brk = false, capped = false;
    for (int f = 0; f < nf; ++f) {
        if (hstop_final[f] == 0) continue;   // zero source: no iteration ran
        iters += hs[f].iters;
        groups += (hs[f].iters + group - 1) / group;
        launches = std::max<int64_t>(launches, hs[f].iters);
        act_total += hs[f].act_total;
        brk = brk || hs[f].breakdown;
        capped = capped || hs[f].iters >= maxiter;
    }
    if (st) {
        st->mscg_iters += iters;
        st->dslash_calls[prec] += 2 * iters + (all ? 0 : nact);
        if (!all) st->sign_calls[prec] += nact;
    }
    c.last_mscg_iters = iters;
    c.last_field_iters.assign(nf, 0);
    for (int f = 0; f < nf; ++f)
        if (hstop_final[f] != 0) c.last_field_iters[f] = hs[f].iters;
    // algorithmic bytes of the updates: r, w, p in and r, p out per iteration;
    // the residuals once more, y in and out per group and 2 per shift active in
    // it (with every solution kept: p_l, x_l in and out, and no y)
    if (c.prof) {
        c.slots[KERN_SHIFT][prec].bytes +=
            all ? (double)FB * (6.0 * iters + 4.0 * act_total)
                : (double)FB * (6.0 * iters + 2.0 * groups + 2.0 * act_total);
        // the two stencils of each executed iteration (K, then K with the
        // shift, the dot and an extra read of p), the links read once per
        // launch however many fields it carries
        const double G = stencil_link_bytes(g, prec);
        c.slots[KERN_STENCIL][prec].bytes +=
            (double)iters * (stencil_bytes(g, prec, EPI_K) + stencil_bytes(g, prec, EPI_K2DOT) - 2.0 * G) +
            (double)launches * 2.0 * G;
    }
    OVL_REQUIRE(!brk, OVL_ERR_BREAKDOWN, "multi-shift CG breakdown (non-positive curvature or NaN)");
    OVL_REQUIRE(!capped, OVL_ERR_NOT_CONVERGED, "multi-shift CG hit its iteration limit");
}

// Right-hand sides of one multi-shift CG.  An iteration goes through five fields
// per right-hand side it works on (p, t, w and the residuals of two iterations)
// and the links; while they about fit the Infinity Cache (268e6 bytes) they come
// from there.  More of them are solved in as few equal batches as fit, if at
// least two fit at a time.  Fields that are skipped (eta <= 0: converged, or of
// another precision) cost no traffic and don't count.  Measured, twelve
// right-hand sides together and in batches: FP32 16^3 x 32 40.4 and 35.6 ms,
// 20^4 52.0 and 47.8 ms, 14^3 x 28 23.1 and 22.3 ms; FP64 12^3 x 24 48.6 and
// 46.6 ms.  The limit is the measured one and lies a little above the cache's
// size: batches of 277e6 bytes (four fields of 16^3 x 32) and six fields of the
// last two lattices are faster whole, the latter by 10 %, as part of the data
// still comes from the cache.  In FP16 the stencils are bound by their
// instructions and batches gain nothing.
static constexpr double CACHE_BYTES = 280e6;
static int fields_per_call(const Context &c, int prec, int nf, const double *eta)
{
    int active = 0;
    for (int f = 0; f < nf; ++f) active += eta[f] > 0.0;
    const double S = (double)field_bytes(c.g, prec), room = CACHE_BYTES - stencil_link_bytes(c.g, prec);
    const int fit = room > 0.0 ? (int)std::min(room / (5.0 * S), 1e6) : 0;
    if (prec == OVL_HALF || fit < 2 || fit >= active) return nf;
    const int calls = (active + fit - 1) / fit;
    return (nf + calls - 1) / calls;
}

void sign_mscg(Context &c, double rho, const ovl_zolo &z, const void *in, void *out, int nf,
               const double *eta, int prec, int maxiter, ovl_stats *st)
{
    const int per = fields_per_call(c, prec, nf, eta);
    const size_t FB = field_bytes(c.g, prec);
    std::vector<int64_t> iters;
    int64_t total = 0;
    for (int f = 0; f < nf; f += per) {
        const int n = std::min(per, nf - f);
        const void *i = (const char *)in + FB * f;
        void *o = (char *)out + FB * f;
        if (per < nf && std::none_of(eta + f, eta + f + n, [](double e) { return e > 0.0; })) {
            zero_fields(c, o, n, prec);
            iters.insert(iters.end(), n, 0);
            continue;
        }
        if (prec == OVL_F64)
            sign_t<double2>(c, rho, z, i, o, n, eta + f, prec, maxiter, st);
        else if (prec == OVL_F32)
            sign_t<float4>(c, rho, z, i, o, n, eta + f, prec, maxiter, st);
        else
            sign_t<h8>(c, rho, z, i, o, n, eta + f, prec, maxiter, st);
        if (per == nf) return;
        total += c.last_mscg_iters;
        iters.insert(iters.end(), c.last_field_iters.begin(), c.last_field_iters.end());
    }
    c.last_mscg_iters = total;
    c.last_field_iters = iters;
}

void shifts_mscg(Context &c, double rho, const ovl_zolo &z, const void *in, void *xs, int nf, const double *eta,
                 int prec, int maxiter, ovl_stats *st)
{
    OVL_REQUIRE(xs != nullptr, OVL_ERR_ARG, "no output for the shifted solutions");
    if (prec == OVL_F64)
        sign_t<double2>(c, rho, z, in, nullptr, nf, eta, prec, maxiter, st, xs);
    else if (prec == OVL_F32)
        sign_t<float4>(c, rho, z, in, nullptr, nf, eta, prec, maxiter, st, xs);
    else
        throw Error{OVL_ERR_UNSUPPORTED, "shifted solutions are kept in FP64 or FP32 only"};
}

void sign_mscg(Context &c, double rho, const ovl_zolo &z, const void *in, void *out, int nf,
               double eta, int prec, int maxiter, ovl_stats *st)
{
    OVL_REQUIRE(eta > 0.0, OVL_ERR_ARG, "eta must be positive");
    std::vector<double> e(nf, eta);
    sign_mscg(c, rho, z, in, out, nf, e.data(), prec, maxiter, st);
}

}  // namespace ovl
