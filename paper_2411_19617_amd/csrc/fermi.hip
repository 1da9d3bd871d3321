// Energy-space observables in FP64 (Sec. 3.4): the DOS from its partial
// sums (Eq. DOS.from.ldos), the Fermi level as the root of
// N_e = int f D (Eq. NumberElectrons_from_DOS), the band energy
// (Eq. band.energy), the electronic entropy and its free-energy term
// (Eqs. electronicentropyDOS, KSfreeenergy) and the Fermi weights that turn
// an LDOS into the density (Eq. density.from.ldos).
//
// D is taken piecewise linear between the energy grid points, and the
// integrals of f, f*e against each linear piece are exact: with
// x = (e - mu)/kT they are differences of the antiderivatives
//   x - ln(1+e^x),  x^2/2 - x ln(1+e^x) - Li2(-e^x),
//   x^3/3 - x^2 ln(1+e^x) - 2x Li2(-e^x) + 2 Li3(-e^x)
// (f written through the polylogarithm as in Eq. fermidiracspecial), used in
// the form that only needs Li_s(-y) with 0 < y <= 1.  Li_s(-y) is summed as
// its power series for y <= 1/2 and as the Taylor series in ln y about y = 1
// (coefficients -eta(s-n)/n!, computed on the host) otherwise.
//
// The root is bracketed like the paper's TOMS748 solver: Newton steps on
// N(mu) (dN/dmu = int D (-df/de) needs only f and the first antiderivative)
// from the zero-temperature root of the piecewise-linear D, kept inside a
// shrinking [lo, hi] and replaced by the midpoint whenever they leave it.
#include <math.h>

#include <mutex>

#include "mala_internal.h"

namespace mala {

constexpr double kPi = 3.14159265358979323846;

// Li_s(-y), s in {2, 3}, 0 <= y <= 1.  coef: [2][kLiTerms] Taylor
// coefficients at y = 1, then [2][kLiPow] inverse powers 1/k^s, in LDS: every
// lane reads the same one, and a global read per term had made each of the
// some fifty dependent terms wait for the cache.  The series runs four terms
// at a time until the last of them no longer counts.
__device__ double li_neg(int s, double y, const double* coef) {
    if (y <= 0.5) {
        static_assert(kLiPow % 4 == 1, "whole groups of four terms after k = 0");
        const double* ik = coef + 2 * kLiTerms + (s - 2) * kLiPow;
        double term = -y, sum = 0.0;
        for (int k = 1; k < kLiPow; k += 4) {
            const double c0 = ik[k], c1 = ik[k + 1], c2 = ik[k + 2], c3 = ik[k + 3];
            const double t1 = term * -y, t2 = t1 * -y, t3 = t2 * -y;
            sum += term * c0;
            sum += t1 * c1;
            sum += t2 * c2;
            const double t = t3 * c3;
            sum += t;
            if (fabs(t) <= 1e-18 * fabs(sum)) break;
            term = t3 * -y;
        }
        return sum;
    }
    const double t = log(y);                    // in (-ln 2, 0]
    const double* c = coef + (s - 2) * kLiTerms;
    double acc = c[kLiTerms - 1];
#pragma unroll 8
    for (int n = kLiTerms - 2; n >= 0; --n) acc = acc * t + c[n];
    return acc;
}

// G0, G1 (and, for the final pass, G2 and the entropy antiderivatives S0,
// S1) at x (see the file comment), and f(x) = 1/(1+e^x).  The entropy
// kernel -[f ln f + (1-f) ln(1-f)] = ln(1+e^x) - x (1-f) has
//   S0 = -2 Li2(-e^x) - x ln(1+e^x),  S1 = -x^2 ln(1+e^x) - 3x Li2(-e^x) + 3 Li3(-e^x);
// for x > 0 they are written through Li_s(-e^-x), with S0's constant pi^2/3
// left to the one interval that crosses x = 0.
__device__ void gfun(double x, const double* coef, bool final, double& g0, double& g1, double& g2, double& f,
                     double& s0, double& s1) {
    if (x <= 0.0) {
        const double y = exp(x), lg = log1p(y);
        const double l2 = li_neg(2, y, coef);
        g0 = x - lg;
        g1 = 0.5 * x * x - x * lg - l2;
        f = 1.0 / (1.0 + y);
        if (final) {
            const double l3 = li_neg(3, y, coef);
            g2 = x * x * x / 3.0 - x * x * lg - 2.0 * x * l2 + 2.0 * l3;
            s0 = -2.0 * l2 - x * lg;
            s1 = -x * x * lg - 3.0 * x * l2 + 3.0 * l3;
        }
    } else {
        const double y = exp(-x), lg = log1p(y);
        const double l2 = li_neg(2, y, coef);
        g0 = -lg;
        g1 = kPi * kPi / 6.0 - x * lg + l2;
        f = y / (1.0 + y);
        if (final) {
            const double l3 = li_neg(3, y, coef);
            g2 = -x * x * lg + 2.0 * x * l2 + 2.0 * l3;
            s0 = 2.0 * l2 - x * lg;
            s1 = -x * x * lg + 3.0 * x * l2 + 3.0 * l3;
        }
    }
    if (!final) g2 = s0 = s1 = 0.0;
}

// Fixed-shape sums of two values over each group of 256 threads: butterflies
// inside each wave, then the four wave sums in order.
__device__ void block_sum2(double& a, double& b, double* red) {
    for (int off = 32; off > 0; off >>= 1) {
        a += __shfl_xor(a, off, 64);
        b += __shfl_xor(b, off, 64);
    }
    if ((threadIdx.x & 63) == 0) {
        red[2 * ((threadIdx.x >> 6) & 3)] = a;
        red[2 * ((threadIdx.x >> 6) & 3) + 1] = b;
    }
    __syncthreads();
    a = (red[0] + red[2]) + (red[4] + red[6]);
    b = (red[1] + red[3]) + (red[5] + red[7]);
    __syncthreads();
}

// What one group of 256 threads holds of an evaluation at its Fermi level.
struct FermiEval {
    double red[8], g0[256], g1[256], g2[256], f[256], s0[256], s1[256];
};

struct FermiShared {
    double D[256], cum[4];
    double mu0;
    int first;
};

// Threads of k_fermi: the sum of the partial rows is 256 columns wide and waits
// on memory, so four groups of threads each take a quarter of the rows with
// sixteen reads in flight (one group with eight: 32 us for 256 rows, the
// latency of 32 dependent rounds; now about 6).  Three groups then evaluate the
// two ends of the energy grid and the start of the root search at once; the
// rest of the solve is the first group's.
constexpr int kFermiThreads = 1024;

// Antiderivatives and f at every grid point for Fermi level mu (one per thread).
__device__ void grid_g(FermiEval& ev, int n_e, double e0, double de, double mu, double kT, const double* coef,
                       bool final) {
    const int e = threadIdx.x & 255;
    if (e < n_e) {
        double g0, g1, g2, f, s0, s1;
        gfun((e0 + e * de - mu) / kT, coef, final, g0, g1, g2, f, s0, s1);
        ev.g0[e] = g0;
        ev.g1[e] = g1;
        ev.g2[e] = g2;
        ev.f[e] = f;
        ev.s0[e] = s0;
        ev.s1[e] = s1;
    }
    __syncthreads();
}

// Hat-piece integrals over interval i = [e_i, e_i + de] from the shared G's:
// wl = int f (1-t), wr = int f t; vl, vr the same with f*e.
__device__ void interval(const FermiEval& ev, int i, double e0, double de, double mu, double kT, double& wl,
                         double& wr, double& vl, double& vr) {
    const double xa = (e0 + i * de - mu) / kT, D = de / kT;
    const double d0 = ev.g0[i + 1] - ev.g0[i], d1 = ev.g1[i + 1] - ev.g1[i], d2 = ev.g2[i + 1] - ev.g2[i];
    const double I0 = d0 * kT;
    const double I1 = (d1 - xa * d0) * kT / D;
    const double K0 = d1 * kT;
    const double K1 = (d2 - xa * d1) * kT / D;
    wl = I0 - I1;
    wr = I1;
    vl = mu * (I0 - I1) + (K0 - K1) * kT;
    vr = mu * I1 + K1 * kT;
}

// N(mu) and dN/dmu.  On [a, b] with t = (e-a)/de, int (-df/de) = f(a) - f(b)
// and int t (-df/de) = (kT/de)(G0(xb) - G0(xa)) - f(b).
__device__ void electrons(const FermiShared& sh, FermiEval& ev, int n_e, double e0, double de, double mu, double kT,
                          const double* coef, double& n, double& dn) {
    grid_g(ev, n_e, e0, de, mu, kT, coef, false);
    const int e = threadIdx.x & 255;
    n = dn = 0.0;
    if (e < n_e - 1) {
        double wl, wr, vl, vr;
        interval(ev, e, e0, de, mu, kT, wl, wr, vl, vr);
        n = wl * sh.D[e] + wr * sh.D[e + 1];
        const double P = ev.f[e] - ev.f[e + 1];
        const double Q = kT / de * (ev.g0[e + 1] - ev.g0[e]) - ev.f[e + 1];
        dn = (P - Q) * sh.D[e] + Q * sh.D[e + 1];
    }
    block_sum2(n, dn, ev.red);
}

// Zero-temperature root of int_{e0}^{mu} D = n_target for the piecewise-linear
// D (a scan of the trapezoids, then the quadratic on the crossing interval);
// the midpoint of the grid if the count never crosses.
__device__ double zero_t_root(FermiShared& sh, int n_e, double e0, double de, double n_target) {
    const int e = threadIdx.x & 255;
    const double piece = e < n_e - 1 ? 0.5 * de * (sh.D[e] + sh.D[e + 1]) : 0.0;
    double scan = piece;                               // inclusive over the wave, then the waves before it
    for (int off = 1; off < 64; off <<= 1) {
        const double v = __shfl_up(scan, off, 64);
        if ((e & 63) >= off) scan += v;
    }
    if ((e & 63) == 63) sh.cum[e >> 6] = scan;
    if (e == 0) {
        sh.mu0 = e0 + 0.5 * (n_e - 1) * de;
        sh.first = n_e;
    }
    __syncthreads();
    for (int w = 0; w < (e >> 6); ++w) scan += sh.cum[w];
    const double after = scan, before = after - piece;
    const bool cross = e < n_e - 1 && before <= n_target && n_target < after;
    if (cross) atomicMin(&sh.first, e);               // lowest crossing interval
    __syncthreads();
    if (e == sh.first) {
        // de (D0 t + (D1 - D0) t^2 / 2) = n_target - before, t in [0, 1]
        const double r = (n_target - before) / de, D0 = sh.D[e], k = sh.D[e + 1] - sh.D[e];
        const double den = D0 + sqrt(fmax(D0 * D0 + 2.0 * k * r, 0.0));
        const double t = den > 0.0 ? fmin(fmax(2.0 * r / den, 0.0), 1.0) : 0.5;
        sh.mu0 = e0 + (e + t) * de;
    }
    __syncthreads();
    return sh.mu0;
}

// mode 0: exact solve (DOS, result, weights; window coverage if win != NULL)
// mode 1: estimate from a subsample -> energy window for the stored LDOS
__global__ __launch_bounds__(kFermiThreads) void k_fermi(const double* __restrict__ partials, int n_parts, int n_e,
                                               double dV, double e0, double de, double kT, double n_target,
                                               double* __restrict__ dos_out, double* __restrict__ w_out,
                                               ResultRec* __restrict__ res, WindowRec* __restrict__ win,
                                               const double* __restrict__ coef_g, int mode, int w_max,
                                               double margin, const int* __restrict__ cap_err) {
    __shared__ FermiShared sh;
    __shared__ double s_sum[kFermiThreads / 256][256];
    __shared__ double coef[kLiCoef];
    __shared__ FermiEval evs[3];
    __shared__ double s_ends[2];
    const int e = threadIdx.x & 255, group = threadIdx.x >> 8;
    constexpr int G = kFermiThreads / 256, U = 16;
    {
        // sixteen running sums per thread, combined in a fixed order
        double acc[U] = {};
        const int w_end = (int)((int64_t)n_parts * (group + 1) / G);
        int w = (int)((int64_t)n_parts * group / G);
        for (; w + U <= w_end; w += U) {
#pragma unroll
            for (int q = 0; q < U; ++q) acc[q] += partials[(size_t)(w + q) * kMlpMaxOut + e];
        }
        double v[U];
#pragma unroll
        for (int q = 0; q < U; ++q) v[q] = w + q < w_end ? partials[(size_t)(w + q) * kMlpMaxOut + e] : 0.0;
#pragma unroll
        for (int q = 0; q < U; ++q) acc[q] += v[q];
#pragma unroll
        for (int h = U / 2; h > 0; h >>= 1)
#pragma unroll
            for (int q = 0; q < h; ++q) acc[q] += acc[q + h];
        s_sum[group][e] = acc[0];
        for (int i = threadIdx.x; i < kLiCoef; i += kFermiThreads) coef[i] = coef_g[i];
    }
    __syncthreads();
    double d = 0.0;
    if (e < n_e) {
        d = ((s_sum[0][e] + s_sum[1][e]) + (s_sum[2][e] + s_sum[3][e])) * dV;
        if (mode == 0 && group == 0) dos_out[e] = d;
    }
    if (group == 0) sh.D[e] = d;
    __syncthreads();
    const double elast = e0 + (n_e - 1) * de;
    double mu = zero_t_root(sh, n_e, e0, de, n_target);
    double n, dn;
    FermiEval& ev = evs[group < 3 ? group : 0];
    {
        // the start of the search, the first and the last energy; the fourth
        // group repeats the first's values into the same places
        const double at = group == 1 ? e0 : group == 2 ? elast : mu;
        electrons(sh, ev, n_e, e0, de, at, kT, coef, n, dn);
    }
    if (e == 0 && (group == 1 || group == 2)) s_ends[group - 1] = n;
    __syncthreads();
    const double nlo = s_ends[0], nhi = s_ends[1];
    // the rest is the first group's: whole waves end here, and a barrier counts only
    // the waves that have not
    if (group > 0) return;
    const bool ok = nlo <= n_target && n_target <= nhi;
    if (!ok) {
        if (e == 0) {
            if (mode == 0) {
                res->e_fermi = NAN;
                res->e_band = NAN;
                res->n_found = NAN;
                res->entropy = NAN;
                res->e_entropy = NAN;
                res->n_target = n_target;
                res->iterations = 0;
                res->status = (cap_err && *cap_err) ? -7 : -4;     // MALA_E_CAPACITY first, else MALA_E_NO_ROOT
                res->density_from_window = 0;
                if (win) win->covered = 0;
            } else {
                win->lo = 0;
                win->hi = n_e - 1;
                win->valid = 0;
                win->covered = 0;
                win->e_fermi_est = NAN;
            }
        }
        if (mode == 0 && e < n_e) w_out[e] = 0.0;
        return;
    }
    const double tol = mode == 0 ? 1e-12 : 1e-6;
    double lo = e0, hi = elast;
    int it = 0;
    while (it < 200) {
        if (it > 0) electrons(sh, ev, n_e, e0, de, mu, kT, coef, n, dn);      // at the start: done above
        ++it;
        if (n == n_target) break;                       // mu is the root
        if (n < n_target) lo = mu;
        else hi = mu;
        double nx = dn > 0.0 ? mu - (n - n_target) / dn : lo;
        // a converged step is taken as it is (it may round onto mu, i.e. onto
        // the end of the bracket just moved there); any other step that
        // leaves the bracket becomes the midpoint
        if (dn > 0.0 && fabs(nx - mu) <= 0.1 * tol) {
            mu = nx;
            break;
        }
        if (!(nx > lo && nx < hi)) nx = 0.5 * (lo + hi);
        mu = nx;
        if (hi - lo < tol) break;
    }
    const double ef = mu;
    const double reach = 40.0 * kT;
    if (mode == 1) {
        if (e == 0) {
            int wl = (int)floor((ef - reach - margin - e0) / de), wh = (int)ceil((ef + reach + margin - e0) / de);
            wl = wl < 0 ? 0 : wl;
            wh = wh > n_e - 1 ? n_e - 1 : wh;
            win->lo = wl;
            win->hi = wh;
            win->valid = (wh - wl + 1) <= w_max ? 1 : 0;
            win->covered = 0;
            win->e_fermi_est = ef;
        }
        return;
    }
    grid_g(ev, n_e, e0, de, ef, kT, coef, true);
    double wl = 0, wr = 0, vl = 0, vr = 0, sc = 0;
    if (e < n_e - 1) {
        interval(ev, e, e0, de, ef, kT, wl, wr, vl, vr);
        // entropy (Eq. electronicentropyDOS) on the same hat pieces: int s,
        // int s t over the interval, t = (x - xa)/D
        const double xa = (e0 + e * de - ef) / kT, xb = (e0 + (e + 1) * de - ef) / kT, D = de / kT;
        double d0 = ev.s0[e + 1] - ev.s0[e];
        if (xa <= 0.0 && xb > 0.0) d0 += kPi * kPi / 3.0;
        const double J0 = d0 * kT, J1 = (ev.s1[e + 1] - ev.s1[e] - xa * d0) * kT / D;
        sc = (J0 - J1) * sh.D[e] + J1 * sh.D[e + 1];
    }
    __syncthreads();
    // reuse the g arrays for the per-interval pieces
    ev.g0[e] = wr;
    ev.g1[e] = vr;
    __syncthreads();
    double we = 0.0, ve = 0.0;
    if (e < n_e) {
        if (e < n_e - 1) { we += wl; ve += vl; }
        if (e >= 1) { we += ev.g0[e - 1]; ve += ev.g1[e - 1]; }
        w_out[e] = we;
    }
    double nf = we * sh.D[e], eb = ve * sh.D[e], s_kb = sc, unused = 0.0;
    block_sum2(nf, eb, ev.red);
    block_sum2(s_kb, unused, ev.red);
    if (e == 0) {
        res->e_fermi = ef;
        res->e_band = eb;
        res->n_found = nf;
        res->entropy = s_kb;
        res->e_entropy = -kT * s_kb;
        res->n_target = n_target;
        res->iterations = it;
        res->status = (cap_err && *cap_err) ? -7 : 0;     // MALA_E_CAPACITY: neighbour lists were truncated
        res->density_from_window = 0;
        if (win) {
            const bool lo_ok = win->lo == 0 || e0 + win->lo * de <= ef - reach;
            const bool hi_ok = win->hi == n_e - 1 || e0 + win->hi * de >= ef + reach;
            win->covered = (win->valid && lo_ok && hi_ok) ? 1 : 0;
            res->density_from_window = win->covered;
        }
    }
}

// n(p) = prefix(p) + sum over the stored window of w_e d_e(p), when the
// window covers E_F +- 40 kT (outside it the Fermi weights equal the full
// trapezoid weights or vanish to within e^-40).  A wave takes 64
// points at a time: their window rows are 64 W contiguous floats, read with
// consecutive lanes into LDS (row stride W: coalesced, where one lane per row
// strides W floats between the lanes of every load) and then summed by the
// row's lane in the fixed order of the energies (a tile's rows start on a
// 256 W-byte boundary, so the copy moves 16 bytes per lane).  The block's four waves
// move in step so that the staging area can be reused after a barrier.
// Windows wider than w_stage (the LDS the host gave, per point) are summed
// straight from memory.
__global__ __launch_bounds__(256) void k_density_window(const double* __restrict__ prefix,
                                                        const float* __restrict__ window, int64_t n_pts,
                                                        const WindowRec* __restrict__ win,
                                                        const ResultRec* __restrict__ res,
                                                        const double* __restrict__ w, double* __restrict__ dens,
                                                        int w_stage) {
    if (res->status != 0 || !win->covered) return;
    __shared__ double sw[kMlpMaxOut];
    extern __shared__ float srow[];                      // [4 waves][64 rows][w_stage]
    const int lo = win->lo, W = win->hi - win->lo + 1;
    for (int i = threadIdx.x; i < W; i += blockDim.x) sw[i] = w[lo + i];
    __syncthreads();
    if (W > w_stage) {
        for (int64_t p = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; p < n_pts;
             p += (int64_t)gridDim.x * blockDim.x) {
            double s = prefix[p];
            const float* row = window + p * W;
            for (int i = 0; i < W; ++i) s += sw[i] * (double)row[i];
            dens[p] = s;
        }
        return;
    }
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    float* rows = srow + wave * 64 * w_stage;
    for (int64_t t0 = (int64_t)blockIdx.x * 4; t0 * 64 < n_pts; t0 += (int64_t)gridDim.x * 4) {
        const int64_t p0 = (t0 + wave) * 64;
        const int np = p0 < n_pts ? (int)(n_pts - p0 < 64 ? n_pts - p0 : 64) : 0;
        // 64 W floats from 256 W-byte aligned rows: 16-byte loads, a few in flight
        const float* src = window + p0 * W;
        const int nf = np * W, n4 = nf >> 2;
        const float4* src4 = reinterpret_cast<const float4*>(src);
        float4* rows4 = reinterpret_cast<float4*>(rows);
#pragma unroll 4
        for (int i = lane; i < n4; i += 64) rows4[i] = src4[i];
        for (int i = (n4 << 2) + lane; i < nf; i += 64) rows[i] = src[i];
        __syncthreads();
        if (lane < np) {
            double s = prefix[p0 + lane];
            for (int i = 0; i < W; ++i) s += sw[i] * (double)rows[lane * W + i];
            dens[p0 + lane] = s;
        }
        __syncthreads();
    }
}

// Column sums of a stored LDOS [n][n_e] into FP64 partial rows, one per block
// over a fixed contiguous range of points.  Thread = (energy, row group): four
// groups take every fourth row with eight reads in flight each and are combined
// in a fixed order, so that few blocks (and few partial rows for the Fermi
// kernel, which one block sums) keep the memory busy.
constexpr int kColThreads = 1024;
__global__ __launch_bounds__(kColThreads) void k_ldos_colsum(const float* __restrict__ ldos, int64_t n_pts, int n_e,
                                                             double* __restrict__ partials, int n_blocks) {
    constexpr int G = kColThreads / 256, U = 8;
    __shared__ double s_sum[G][256];
    const int e = threadIdx.x & 255, group = threadIdx.x >> 8;
    const int64_t b = blockIdx.x;
    const int64_t p_begin = n_pts * b / n_blocks, p_end = n_pts * (b + 1) / n_blocks;
    double s = 0.0;
    if (e < n_e) {
        const float* col = ldos + e;
        int64_t p = p_begin + group;
        for (; p + (U - 1) * G < p_end; p += U * G) {
            float v[U];
#pragma unroll
            for (int q = 0; q < U; ++q) v[q] = col[(p + q * G) * n_e];
#pragma unroll
            for (int q = 0; q < U; ++q) s += (double)v[q];
        }
        for (; p < p_end; p += G) s += (double)col[p * n_e];
    }
    s_sum[group][e] = s;
    __syncthreads();
    if (group == 0) partials[b * kMlpMaxOut + e] = (s_sum[0][e] + s_sum[1][e]) + (s_sum[2][e] + s_sum[3][e]);
}

// n(p) = sum_e w_e d_e(p), one wave per four points at a time: sixteen reads in
// flight, and the four sums over the lanes share their butterfly (two steps that
// halve the values a lane holds, then four on one value).  The points run
// backwards: the column sums read the rows forwards just before, so the last
// ones are the ones still in the memory-side cache.
__global__ __launch_bounds__(256) void k_density_ldos(const float* __restrict__ ldos, int64_t n_pts, int n_e,
                                                      const double* __restrict__ w,
                                                      const ResultRec* __restrict__ res,
                                                      double* __restrict__ dens) {
    if (res->status != 0) return;
    const int lane = threadIdx.x & 63;
    double wr[4];
    int off[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int e = lane + 64 * q;
        wr[q] = e < n_e ? w[e] : 0.0;
        off[q] = e < n_e ? e : n_e - 1;        // in range; its weight is zero
    }
    const int64_t quads = (n_pts + 3) / 4;
    for (int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6); i < quads; i += (int64_t)gridDim.x * 4) {
        const int64_t p0 = (quads - 1 - i) * 4;
        float v[4][4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float* row = ldos + (p0 + r < n_pts ? p0 + r : n_pts - 1) * n_e;
#pragma unroll
            for (int q = 0; q < 4; ++q) v[r][q] = row[off[q]];
        }
        double s[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            s[r] = 0.0;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (lane + 64 * q < n_e) s[r] += wr[q] * (double)v[r][q];
        }
        // lanes with bit 5 keep points 2, 3; with bit 4 the odd one of their two
        const bool h5 = lane & 32, h4 = lane & 16;
        const double a0 = (h5 ? s[2] : s[0]) + __shfl_xor(h5 ? s[0] : s[2], 32, 64);
        const double a1 = (h5 ? s[3] : s[1]) + __shfl_xor(h5 ? s[1] : s[3], 32, 64);
        double t = (h4 ? a1 : a0) + __shfl_xor(h4 ? a0 : a1, 16, 64);
#pragma unroll
        for (int o = 8; o > 0; o >>= 1) t += __shfl_xor(t, o, 64);
        const int64_t p = p0 + (h5 ? 2 : 0) + (h4 ? 1 : 0);
        if ((lane & 15) == 0 && p < n_pts) dens[p] = t;
    }
}

hipError_t launch_fermi(hipStream_t s, const double* partials, int n_parts, int n_e, double dV, double e0,
                        double de, double kT, double n_target, double* dos_out, double* weights_out,
                        void* result, WindowRec* win, const double* li_coef, const int* cap_err) {
    hipLaunchKernelGGL(k_fermi, dim3(1), dim3(kFermiThreads), 0, s, partials, n_parts, n_e, dV, e0, de, kT, n_target,
                       dos_out, weights_out, static_cast<ResultRec*>(result), win, li_coef, 0, 0, 0.0, cap_err);
    return hipGetLastError();
}

hipError_t launch_fermi_estimate(hipStream_t s, const double* partials, int n_parts, int n_e, double dV,
                                 double e0, double de, double kT, double n_target, WindowRec* win,
                                 const double* li_coef, int w_max, double margin) {
    hipLaunchKernelGGL(k_fermi, dim3(1), dim3(kFermiThreads), 0, s, partials, n_parts, n_e, dV, e0, de, kT, n_target,
                       nullptr, nullptr, nullptr, win, li_coef, 1, w_max, margin, nullptr);
    return hipGetLastError();
}

hipError_t launch_density_window(hipStream_t s, const double* prefix, const float* window, int64_t n_pts,
                                 const WindowRec* win, const void* result, const double* weights,
                                 double* density, int w_max) {
    int64_t blocks = (n_pts + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    if (blocks < 1) return hipSuccess;
    // stage up to 96 energies per point (96 KB of LDS per block); wider
    // windows (high temperatures on fine energy grids) take the direct path
    const int w_stage = w_max <= kDensityStageMax ? (w_max > 0 ? w_max : 1) : 0;
    const size_t lds = sizeof(float) * 256 * (size_t)w_stage;
    static std::once_flag attr_once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(attr_once, [] {
        attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_density_window),
                                       hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)(sizeof(float) * 256 * kDensityStageMax));
    });
    if (attr_err != hipSuccess) return attr_err;
    hipLaunchKernelGGL(k_density_window, dim3((unsigned)blocks), dim3(256), lds, s, prefix, window, n_pts, win,
                       static_cast<const ResultRec*>(result), weights, density, w_stage);
    return hipGetLastError();
}

hipError_t launch_ldos_colsum(hipStream_t s, const float* ldos, int64_t n_pts, int n_e, double* partials,
                              int n_blocks) {
    hipLaunchKernelGGL(k_ldos_colsum, dim3(n_blocks), dim3(kColThreads), 0, s, ldos, n_pts, n_e, partials, n_blocks);
    return hipGetLastError();
}

hipError_t launch_density_from_ldos(hipStream_t s, const float* ldos, int64_t n_pts, int n_e,
                                    const double* weights, const void* result, double* density) {
    int64_t blocks = (n_pts + 15) / 16;          // four waves of four points
    if (blocks > 2048) blocks = 2048;
    if (blocks < 1) return hipSuccess;
    hipLaunchKernelGGL(k_density_ldos, dim3((unsigned)blocks), dim3(256), 0, s, ldos, n_pts, n_e, weights,
                       static_cast<const ResultRec*>(result), density);
    return hipGetLastError();
}

// Taylor coefficients of Li_s(-e^t) about t = 0 for s = 2, 3, then the
// inverse powers 1/k^s used by the power series:
// c_{s,n} = Li_{s-n}(-1)/n! = -eta(s-n)/n!, with eta(1) = ln 2,
// eta(2) = pi^2/12, eta(3) = 3 zeta(3)/4 and, for m >= 0,
// eta(-m) = (2^(m+1) - 1) B_{m+1}/(m+1) (B_1 = +1/2; B_{2k} from zeta(2k)).
void polylog_coefficients(double* coef) {
    for (int si = 0; si < 2; ++si)
        for (int k = 0; k < kLiPow; ++k)
            coef[2 * kLiTerms + si * kLiPow + k] = k == 0 ? 0.0 : pow((double)k, -(double)(2 + si));
    auto zeta_even = [](int n) {     // zeta(n), n >= 2 even: sum plus integral tail
        if (n == 2) return kPi * kPi / 6.0;
        const int K = 2000;
        double s = pow((double)K, 1.0 - n) / (n - 1) - 0.5 * pow((double)K, -(double)n);
        for (int k = K - 1; k >= 1; --k) s += pow((double)k, -(double)n);
        return s;
    };
    auto bernoulli = [&](int n) {    // B_n with B_1 = +1/2
        if (n == 0) return 1.0;
        if (n == 1) return 0.5;
        if (n & 1) return 0.0;
        double f = 1.0;
        for (int k = 2; k <= n; ++k) f *= k;
        const double sign = ((n / 2) & 1) ? 1.0 : -1.0;      // (-1)^(n/2+1)
        return sign * 2.0 * f * zeta_even(n) / pow(2.0 * kPi, n);
    };
    auto eta = [&](int s) {
        if (s == 1) return log(2.0);
        if (s == 2) return kPi * kPi / 12.0;
        if (s == 3) return 0.75 * 1.2020569031595942854;   // zeta(3) (Apery's constant)
        const int m = -s;                                      // s <= 0
        return (pow(2.0, m + 1) - 1.0) * bernoulli(m + 1) / (m + 1);
    };
    for (int si = 0; si < 2; ++si) {
        const int s = 2 + si;
        double fact = 1.0;
        for (int n = 0; n < kLiTerms; ++n) {
            if (n > 0) fact *= n;
            coef[si * kLiTerms + n] = -eta(s - n) / fact;
        }
    }
}

}  // namespace mala
