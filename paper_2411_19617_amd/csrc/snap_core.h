// Compile-time helpers of the bispectrum kernels (Sec. 3.2.2, Eq. SNAPExpansion,
// Eq. snap_dim) shared by the descriptor kernels and their adjoint: exact
// constants and the (row, row) pairs of the Z contraction.
#pragma once
#include "mala_internal.h"

namespace mala {

__host__ __device__ constexpr double ce_sqrt(double x) {
    if (x <= 0.0) return 0.0;
    double r = x > 1.0 ? x : 1.0;
    for (int i = 0; i < 64; ++i) r = 0.5 * (r + x / r);
    return r;
}

__host__ __device__ constexpr double ce_binom(int n, int k) {
    double r = 1.0;
    for (int i = 1; i <= k; ++i) r = r * (n - k + i) / i;
    return r;
}

__host__ __device__ constexpr double ce_fact(int n) {
    double f = 1.0;
    for (int i = 2; i <= n; ++i) f *= i;
    return f;
}

// Angle theta0 and cutoff phase of a neighbour at distance r, from their factors per
// unit distance, formed once (a quotient per neighbour is a full-precision division, a
// dozen instructions), each in two floats: the rounding of one would turn every
// neighbour the same way and add up where the others average out (descriptors
// 3.1e-7 -> 2.8e-7 against 64 bits).
struct PhaseFactors {
    float th, th_lo, cut, cut_lo;
    __device__ __forceinline__ explicit PhaseFactors(double rcut) {
        const double c = 3.14159265358979323846 / rcut, t = kRfac0 * c;
        th = (float)t;
        th_lo = (float)(t - th);
        cut = (float)c;
        cut_lo = (float)(c - cut);
    }
    __device__ __forceinline__ float angle(float r) const { return fmaf(th, r, th_lo * r); }
    __device__ __forceinline__ float cutoff(float r) const { return fmaf(cut, r, cut_lo * r); }
};

// x * (-1)^k for wave-uniform x and k, as a sign-bit flip on the scalar unit
__device__ __forceinline__ float flip_odd(float x, int k) {
    return __int_as_float(__float_as_int(x) ^ (int)((unsigned)(k & 1) << 31));
}

// Number of (ma, ma1) row pairs of a triple (rows ma <= J/2), their index,
// and which rows of u^{J1} and u^{J2} they use.
__host__ __device__ constexpr int zb_pairs(int J1, int J2, int J) {
    int n = 0;
    for (int ma = 0; ma <= J / 2; ++ma)
        for (int ma1 = 0; ma1 <= J1; ++ma1)
            if (zb_pair_ok(J1, J2, J, ma, ma1)) ++n;
    return n;
}
__host__ __device__ constexpr int zb_pair_index(int J1, int J2, int J, int ma, int ma1) {
    int n = 0;
    for (int a = 0; a <= J / 2; ++a)
        for (int a1 = 0; a1 <= J1; ++a1)
            if (zb_pair_ok(J1, J2, J, a, a1)) {
                if (a == ma && a1 == ma1) return n;
                ++n;
            }
    return -1;
}
// Scaling side of the dL/du column (the Z contraction of the adjoint).  It
// keeps the mirrored rows of the unscaled level unsigned: their sign
// (-1)^(row - column) alternates with the m1' column, so the pairs using them
// accumulate R <- P - R (a negated addend) and take the sign once, on the
// row CG factor in the fold.  The per-column scaling cost is then 2
// multiplies per used row of the scaled level, the smaller one scaled (ties
// as zb_scale2).
__host__ __device__ constexpr bool zy_scale2(int A, int B, int C) {
    const ZbRows r = zb_rows(A, B, C);
    return r.used2 < r.used1 || (r.used2 == r.used1 && zb_scale2(A, B, C));
}
__host__ __device__ constexpr int zy_scale_ops(int A, int B, int C) {
    const ZbRows r = zb_rows(A, B, C);
    return 2 * (zy_scale2(A, B, C) ? r.used2 : r.used1);
}
// Pair (ma, ma1) uses a mirrored row of the unscaled level, and which row.
__host__ __device__ constexpr bool zy_alt(int A, int B, int C, int ma, int ma1) {
    return zy_scale2(A, B, C) ? 2 * ma1 > A : 2 * (ma - ma1 + (A + B - C) / 2) > B;
}
__host__ __device__ constexpr int zy_alt_row(int A, int B, int C, int ma, int ma1) {
    return zy_scale2(A, B, C) ? ma1 : ma - ma1 + (A + B - C) / 2;
}
}  // namespace mala
