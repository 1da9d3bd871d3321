// Compile-time tables of the expansion coefficients u^J (Sec. 3.2.2, Eq.
// SNAPExpansion) in separated form.  With g = (a, b) the element (ma, mb) of
// U^J is, up to its normalisation, the coefficient of xi^mb eta^(J-mb) in
// (a xi - conj(b) eta)^ma (b xi + conj(a) eta)^(J-ma), and in every term of it
// the phases of a and b are the same:
//   U^J_{ma,mb} = a^k1 b^k2 P(t),  k1 = ma + mb - J,  k2 = mb - ma,  t = |a|^2,
// (a^-k meaning conj(a)^k), P a polynomial of degree n = (J - |k1| - |k2|) / 2.
// So u^J needs, per (k1, k2) of a half plane (the other half is conjugate), the
// neighbour sums of a^k1 b^k2 phi_n(t) for n = 0..(TJ - |k1| - |k2|) / 2 only:
// as many numbers as u has, each one multiply-add per neighbour, and every
// level's elements are fixed combinations of them, formed once per point.
//
// phi_n are Chebyshev polynomials of x(t) on the part of [0, 1] where the weight
// |a|^|k1| |b|^|k2| lies: with one interval for all (k1, k2) the combinations
// cancel up to 35-fold (FP32 error of u^10: 8.2e-7 against 5.9e-7 for a
// level-by-level recursion); with the interval chosen per (|k1|, |k2|)
// sum_n |c_n phi_n(t)| |a|^|k1| |b|^|k2| stays below 4.
#pragma once
#include "snap_core.h"

namespace mala {

constexpr int kUMaxN = kMaxTwojmax / 2;      // highest phi_n

// Intervals of t for the Chebyshev basis: [0,1], [0,3/4], [1/4,1], [0,1/2], [1/2,1].
constexpr int kUBases = 5;
__host__ __device__ constexpr double ub_half(int b) { return b == 0 ? 0.5 : b <= 2 ? 0.375 : 0.25; }
__host__ __device__ constexpr double ub_mid(int b) {
    return b == 0 ? 0.5 : b == 1 ? 0.375 : b == 2 ? 0.625 : b == 3 ? 0.25 : 0.75;
}
// The interval of (|k1|, |k2|): the better conditioned of the five.
__host__ __device__ constexpr int u_basis(int k1, int k2) {
    const int hi = k1 > k2 ? k1 : k2, lo = k1 > k2 ? k2 : k1;
    int narrow = 0;                          // 0: [0,1], 1: three quarters, 2: half
    if (lo == 0) narrow = hi == 0 ? 0 : hi <= 2 ? 1 : 2;
    else if (lo == 1) narrow = hi == 1 ? 0 : hi <= 3 ? 1 : 2;
    else if (lo == 2) narrow = hi == 2 ? 0 : hi <= 5 ? 1 : 2;
    else if (lo == 3) narrow = hi <= 4 ? 0 : 1;
    if (narrow == 0) return 0;
    const bool a_side = k1 > k2;             // weight towards t = 1
    return narrow == 1 ? (a_side ? 2 : 1) : (a_side ? 4 : 3);
}

struct UCoef {
    double c[kUMaxN + 1];
};

// Coefficients of phi_n in the normalised element (J, ma, mb).
__host__ __device__ constexpr UCoef u_coef(int J, int ma, int mb) {
    const int k1 = ma + mb - J, k2 = mb - ma;
    const int K1 = k1 < 0 ? -k1 : k1, K2 = k2 < 0 ? -k2 : k2, n = (J - K1 - K2) / 2;
    double p[kUMaxN + 1] = {};               // powers of t
    for (int s = 0; s <= ma; ++s) {
        if (mb - s < 0 || mb - s > J - ma) continue;
        const double c = ce_binom(ma, s) * ce_binom(J - ma, mb - s) * (((ma - s) & 1) ? -1.0 : 1.0);
        const int al = s < J - ma - mb + s ? s : J - ma - mb + s;        // |a|^2 to this power,
        for (int i = 0; i <= n - al; ++i)                                // |b|^2 = 1 - t to n - al
            p[al + i] += c * ce_binom(n - al, i) * ((i & 1) ? -1.0 : 1.0);
    }
    // t = mid + half x
    const double h = ub_half(u_basis(K1, K2)), m = ub_mid(u_basis(K1, K2));
    double q[kUMaxN + 1] = {};               // powers of x
    for (int i = n; i >= 0; --i) {           // Horner
        double r[kUMaxN + 1] = {};
        for (int k = 0; k <= kUMaxN; ++k) r[k] = m * q[k] + (k > 0 ? h * q[k - 1] : 0.0);
        for (int k = 0; k <= kUMaxN; ++k) q[k] = r[k];
        q[0] += p[i];
    }
    // x^k = 2^(1-k) sum_j binom(k, j) T_{k-2j} (half of it at T_0 for even k)
    const double nrm = ce_sqrt(ce_fact(mb) * ce_fact(J - mb) / (ce_fact(ma) * ce_fact(J - ma)));
    UCoef o{};
    for (int k = 0; k <= n; ++k) {
        double f = 2.0;
        for (int i = 0; i < k; ++i) f *= 0.5;
        for (int j = 0; 2 * j <= k; ++j)
            o.c[k - 2 * j] += nrm * q[k] * f * ce_binom(k, j) * (k == 2 * j ? 0.5 : 1.0);
    }
    return o;
}

// The sums are split over the block's four waves by |k1| (118, 120, 128 and 140
// sums at twojmax 10, 72, 68, 72 and 73 at 8).
constexpr int kUiWaves = 4;
__host__ __device__ constexpr int u_group_of(int /*tj*/, int k1) {
    return k1 == 1 || k1 >= 9 ? 0 : k1 == 2 || k1 == 6 ? 1 : k1 == 3 || k1 == 4 ? 2 : 3;
}
// Sums of (k1, k2 >= 0): products of the parts of a^k1 and b^k2, 4 in
// general (both signs of k2 from the same four), 2 on an axis, 1 at the origin.
__host__ __device__ constexpr int u_parts(int k1, int k2) { return (k1 > 0 ? 2 : 1) * (k2 > 0 ? 2 : 1); }
__host__ __device__ constexpr int u_ncount(int tj, int k1, int k2) { return (tj - k1 - k2) / 2 + 1; }
// First sum of (k1, k2) within the group of k1; (k1 = tj + 1) gives the group's size.
__host__ __device__ constexpr int u_slot(int tj, int g, int k1, int k2) {
    int s = 0;
    for (int i = 0; i <= tj; ++i) {
        if (u_group_of(tj, i) != g) continue;
        for (int k = 0; i + k <= tj; ++k) {
            if (i == k1 && k == k2) return s;
            s += u_parts(i, k) * u_ncount(tj, i, k);
        }
    }
    return s;
}
__host__ __device__ constexpr int u_group_size(int tj, int g) { return u_slot(tj, g, tj + 1, 0); }
// Largest k2, and highest phi_n of one basis, that a group needs.
__host__ __device__ constexpr int u_group_k2max(int tj, int g) {
    int m = 0;
    for (int i = 0; i <= tj; ++i)
        if (u_group_of(tj, i) == g && tj - i > m) m = tj - i;
    return m;
}
__host__ __device__ constexpr int u_basis_nmax(int tj, int g, int b) {
    int m = 0;
    for (int i = 0; i <= tj; ++i)
        for (int k = 0; u_group_of(tj, i) == g && i + k <= tj; ++k)
            if (u_basis(i, k) == b && u_ncount(tj, i, k) - 1 > m) m = u_ncount(tj, i, k) - 1;
    return m;
}
// Whether a group needs a^k: for its own k1, or on the way to one
// (a^k = a^(k - k/2) a^(k/2)).
__host__ __device__ constexpr bool u_power_needed(int tj, int g, int k) {
    bool need[2 * kMaxTwojmax + 2] = {};
    for (int i = 1; i <= tj; ++i)
        if (u_group_of(tj, i) == g) need[i] = true;
    for (int i = tj; i > 1; --i)
        if (need[i]) need[i / 2] = need[i - i / 2] = true;
    return need[k];
}

}  // namespace mala
