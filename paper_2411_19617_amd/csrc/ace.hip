// Grid-centred atomic cluster expansion descriptors (Sec. 3.2.3, Eqs.
// unweighted_ionicdensity, gridatom_basis, grid_base, product_grid_basis,
// ace_grid), one chemical element:
//   A_nlm = sum over atom images within rcut of R_n(r) Y_l^m(d/r), plus the
//   grid point's own delta on l = 0 (R_n(0) Y_0^0 = (-1)^n / sqrt(4 pi));
//   R_n(r) = T_n(2 r / rcut - 1) fc(r) (Chebyshev times the cosine cutoff);
//   rank 1: A_n00; rank 2: sum_m (-1)^m A_{n1 l m} A_{n2 l -m};
//   rank 3: sum (l1 l2 l3; m1 m2 m3) A A A over multisets of three (n, l);
//   rank 4: the generalized Clebsch-Gordan contraction with one intermediate
//   coupling L (k_ace4 below).
// Two kernels per chunk of points.  k_ace_proj: per 64-point tile (lane =
// point) the candidate atom images are gathered into LDS (shared with the
// other neighbour kernels), the waves build per-point neighbour lists and form
// A_{n l m} (m >= 0; A_{l,-m} = (-1)^m conj A_{l,m}) over a share of the lane's
// list each: T_n by the three-term recurrence, Y_l^m = N_lm Q_l^m(z/r)
// ((x + i y)/r)^m with Q_l^m = (-1)^m d^m P_l / dt^m by the associated
// Legendre recurrence in l; the tile's A goes to HBM (480 B per point,
// coalesced).  k_ace (ranks 1-3) and k_ace4 (rank 4) load a tile's A into
// LDS and contract it there.  Outputs are written point-major or
// descriptor-major (one plane per descriptor, coalesced stores).
#include <mutex>

#include "ace.h"
#include "tile_gather.h"

namespace mala {

constexpr int kAceN = kAceMaxN;          // radial functions held per point
constexpr int kAceL = kAceMaxL;          // largest l held
constexpr int kAceLm = 15;               // (l, m >= 0) entries per n: l(l+1)/2 + m
constexpr int kAceWaves = 4;            // projection: waves that share the neighbours

__host__ __device__ constexpr double ace_fact(int n) {
    double f = 1.0;
    for (int i = 2; i <= n; ++i) f *= i;
    return f;
}
__host__ __device__ constexpr double ace_sqrt(double x) {
    if (x <= 0.0) return 0.0;
    double r = x > 1.0 ? x : 1.0;
    for (int i = 0; i < 64; ++i) {
        const double next = 0.5 * (r + x / r);
        if (next == r) break;
        r = next;
    }
    return r;
}
// N_lm = sqrt((2l+1)/(4 pi) (l-m)!/(l+m)!)
__host__ __device__ constexpr double ace_norm_d(int l, int m) {
    return ace_sqrt((2 * l + 1) / (4.0 * 3.14159265358979323846) * ace_fact(l - m) / ace_fact(l + m));
}
__host__ __device__ constexpr float ace_norm(int l, int m) { return (float)ace_norm_d(l, m); }

// The tile's own point (lane = point) relative to the origins of its
// candidate atom images, gathered into cand (whole block).
struct AceTile {
    int64_t idx;      // point index within the launch range
    bool valid;
    PointFrame frame;
    int ncand;
};

__device__ __forceinline__ AceTile ace_tile(const BinState& bins, int Nx, int Ny, int Nz, double rcut, int64_t pt_begin,
                                            int64_t n_pts, float4* cand, int* scan_tmp, int* err) {
    const int lane = threadIdx.x & 63;
    const int64_t tile = blockIdx.x;
    AceTile t;
    t.idx = tile * kTile + lane;
    t.valid = t.idx < n_pts;
    const TilePoint pt = tile_point(bins, Nx, Ny, Nz, pt_begin + tile * kTile,
                                    (int)min((int64_t)kTile, n_pts - tile * kTile), lane);
    const TileBoxes& boxes = pt.boxes;
    int n0;
    const int base = gather_candidates(bins, boxes, rcut, cand, kMaxCand, scan_tmp, &n0);
    if (base > kMaxCand && threadIdx.x == 0) atomicOr(err, kErrCand);
    t.ncand = base < kMaxCand ? base : kMaxCand;
    t.frame = point_frame(boxes, n0, pt.x, pt.y, pt.z);
    return t;
}

// Real numbers of A_{n l m} for one n: Re of (l, m) at ace_re, Im (m > 0) behind it.
constexpr int kAceReals = (kAceL + 1) * (kAceL + 1);
__host__ __device__ constexpr int ace_re(int l, int m) { return l * l + (m ? 2 * m - 1 : 0); }

// One neighbour's R_n(r) Y_l^m for every n and (l, m), m >= 0, added to acc.
// Y_l^m = q_l^m(z/r) ((x + i y)/r)^m with q = N_lm Q_l^m by the recurrence in l
// (its factors and the norms are constants).
__device__ __forceinline__ void ace_add_neighbour(float dx, float dy, float dz, float k2, float kcut,
                                                  float (&acc)[kAceN][kAceReals]) {
    const float r2 = dx * dx + dy * dy + dz * dz;
    // 1/r and r from one hardware reciprocal square root (about 1 ulp)
    const bool at_point = !(r2 > kMinR2);
    const float inv = at_point ? 0.f : __builtin_amdgcn_rsqf(r2);
    const float r = r2 * inv;
    const float x = r * k2 - 1.f, fc = 0.5f * (cosf(kcut * r) + 1.f);
    float R[kAceN] = {fc, x * fc};
#pragma unroll
    for (int n = 2; n < kAceN; ++n) R[n] = fmaf(2.f * x, R[n - 1], -R[n - 2]);
    constexpr float y00 = ace_norm(0, 0);
#pragma unroll
    for (int n = 0; n < kAceN; ++n) {
        acc[n][0] = fmaf(R[n], y00, acc[n][0]);
        R[n] = at_point ? 0.f : R[n];                      // an atom on the point: l = 0 only
    }
    const float t = dz * inv, ur = dx * inv, ui = dy * inv;
    float er[kAceL + 1], ei[kAceL + 1];
    er[0] = 1.f;
    ei[0] = 0.f;
    er[1] = ur;
    ei[1] = ui;
#pragma unroll
    for (int m = 2; m <= kAceL; ++m) {
        er[m] = er[m - 1] * ur - ei[m - 1] * ui;
        ei[m] = er[m - 1] * ui + ei[m - 1] * ur;
    }
    static_for<0, kAceL + 1>([&](auto mc) {
        constexpr int m = decltype(mc)::value;
        // Q_m^m = (-1)^m (2m-1)!!
        constexpr double qmm = ((m & 1) ? -1.0 : 1.0) * (ace_fact(2 * m) / (ace_fact(m) * (double)(1 << m)));
        float q[kAceL + 1];
        static_for<(m ? m : 1), kAceL + 1>([&](auto lc) {
            constexpr int l = decltype(lc)::value;
            constexpr double nl = ace_norm_d(l, m);
            if constexpr (l == m) q[l] = (float)(nl * qmm);
            else if constexpr (l == m + 1) q[l] = (float)(nl * qmm * (2 * m + 1)) * t;
            else {
                constexpr float a = (float)(nl / ace_norm_d(l - 1, m) * (2 * l - 1) / (l - m));
                constexpr float b = (float)(nl / ace_norm_d(l - 2, m) * (l + m - 1) / (l - m));
                float q2;
                if constexpr (l == 2 && m == 0) q2 = y00;
                else q2 = q[l - 2];
                q[l] = fmaf(a * t, q[l - 1], -b * q2);
            }
            if constexpr (m == 0) {
#pragma unroll
                for (int n = 0; n < kAceN; ++n) acc[n][ace_re(l, 0)] = fmaf(R[n], q[l], acc[n][ace_re(l, 0)]);
            } else {
                const float yr = q[l] * er[m], yi = q[l] * ei[m];
#pragma unroll
                for (int n = 0; n < kAceN; ++n) {
                    acc[n][ace_re(l, m)] = fmaf(R[n], yr, acc[n][ace_re(l, m)]);
                    acc[n][ace_re(l, m) + 1] = fmaf(R[n], yi, acc[n][ace_re(l, m) + 1]);
                }
            }
        });
    });
}

// Bound by the VALU: about 200 instructions per neighbour and point, half of
// them the multiply-adds into A.  The waves share the neighbours (every wave all
// n and (l, m) of every fourth neighbour, so a neighbour's distance, cutoff and
// harmonics are formed once) and their sums meet in LDS at the end, wave n
// keeping radial index n.  Before, every wave formed them for its own n, behind
// a list that one wave built: 230 -> 142 us per 300,007 points of a solid.
__global__ __launch_bounds__(64 * kAceWaves, 3) void k_ace_proj(BinState bins, int Nx, int Ny, int Nz, double rcut,
                                                                int64_t pt_begin, int64_t n_pts,
                                                                float2* __restrict__ Ag, int* __restrict__ err) {
    static_assert(kAceWaves == 4 && kAceN == 4, "wave n keeps radial index n, in two phases of two");
    struct Lists {
        float4 cand[kMaxCand];
        unsigned short nbr[kMaxNbr][kTile];
        int nnbr[kAceWaves][kTile];
        int scan_tmp[16];
    };
    constexpr int kParts = 2 * (kAceWaves - 1);            // partial sums exchanged per phase
    __shared__ union {
        Lists l;
        float part[kParts][kAceReals][kTile];
    } sh;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const AceTile tl = ace_tile(bins, Nx, Ny, Nz, rcut, pt_begin, n_pts, sh.l.cand, sh.l.scan_tmp, err);
    __syncthreads();
    const float rcf = (float)rcut;
    const int my_n = build_neighbour_lists_block<kAceWaves>(sh.l.cand, tl.ncand, tl.frame, rcf, tl.valid, lane, wave,
                                                            sh.l.nbr, sh.l.nnbr, err);
    const int n_iter = wave_max_int(my_n);
    const float k2 = 2.f / rcf, kcut = 3.14159265358979323846f / rcf;      // per unit distance, formed once
    float acc[kAceN][kAceReals];
#pragma unroll
    for (int n = 0; n < kAceN; ++n)
#pragma unroll
        for (int e = 0; e < kAceReals; ++e) acc[n][e] = 0.f;
#pragma clang loop unroll(disable)
    for (int s = wave; s < n_iter; s += kAceWaves) {
        if (s >= my_n) continue;
        const int c = sh.l.nbr[s][lane];
        const float4 q = sh.l.cand[c];
        const float3 o = tl.frame.at(c);
        ace_add_neighbour(q.x - o.x, q.y - o.y, q.z - o.z, k2, kcut, acc);
    }
    float2* dst = Ag + ((int64_t)blockIdx.x * kAceN * kAceLm + wave * kAceLm) * kTile;
    static_for<0, kAceN / 2>([&](auto hc) {
        constexpr int h = decltype(hc)::value;
        __syncthreads();                                   // the lists, or the last phase's sums, are read
        static_for<2 * h, 2 * h + 2>([&](auto nc) {
            constexpr int n = decltype(nc)::value;
            if (wave == n) return;
            float (*to)[kTile] = sh.part[(n - 2 * h) * (kAceWaves - 1) + (wave < n ? wave : wave - 1)];
#pragma unroll
            for (int e = 0; e < kAceReals; ++e) to[e][lane] = acc[n][e];
        });
        __syncthreads();
        static_for<2 * h, 2 * h + 2>([&](auto nc) {
            constexpr int n = decltype(nc)::value;
            if (wave != n) return;
            float v[kAceReals];
#pragma unroll
            for (int e = 0; e < kAceReals; ++e) {
                v[e] = acc[n][e];
#pragma unroll
                for (int k = 0; k < kAceWaves - 1; ++k) v[e] += sh.part[(n - 2 * h) * (kAceWaves - 1) + k][e][lane];
            }
            constexpr float y00 = ace_norm(0, 0);
            v[0] += (n & 1) ? -y00 : y00;                  // the grid point's own delta: T_n(-1) Y_0^0
            static_for<0, kAceL + 1>([&](auto lc) {
                constexpr int l = decltype(lc)::value;
                static_for<0, l + 1>([&](auto mc) {
                    constexpr int m = decltype(mc)::value;
                    dst[(l * (l + 1) / 2 + m) * kTile + lane] =
                        make_float2(v[ace_re(l, m)], m ? v[ace_re(l, m) + 1] : 0.f);
                });
            });
        });
    });
}

// The tile's A from the projection kernel into LDS (whole block).
__device__ __forceinline__ void ace_load_tile(const float2* __restrict__ Ag, float2 (*sA)[kTile]) {
    const float2* src = Ag + (int64_t)blockIdx.x * kAceN * kAceLm * kTile;
    for (int e = threadIdx.x; e < kAceN * kAceLm * kTile; e += blockDim.x) sA[e / kTile][e % kTile] = src[e];
}

// 3j symbol (l1 l2 l3; m1 m2 m3) by Racah's sum, at compile time.
__host__ __device__ constexpr double ace_3j(int l1, int l2, int l3, int m1, int m2, int m3) {
    if (m1 + m2 + m3 != 0) return 0.0;
    double sum = 0.0;
    for (int k = 0; k <= l1 + l2 - l3; ++k) {
        const int a = l3 - l2 + k + m1, b = l3 - l1 + k - m2, c = l1 - k - m1, d = l2 - k + m2;
        if (a < 0 || b < 0 || c < 0 || d < 0) continue;
        sum += ((k & 1) ? -1.0 : 1.0) / (ace_fact(k) * ace_fact(l1 + l2 - l3 - k) * ace_fact(a) * ace_fact(b) *
                                         ace_fact(c) * ace_fact(d));
    }
    const double delta = ace_fact(l1 + l2 - l3) * ace_fact(l1 - l2 + l3) * ace_fact(l2 + l3 - l1) /
                         ace_fact(l1 + l2 + l3 + 1);
    const double root = ace_sqrt(delta * ace_fact(l1 + m1) * ace_fact(l1 - m1) * ace_fact(l2 + m2) *
                                 ace_fact(l2 - m2) * ace_fact(l3 + m3) * ace_fact(l3 - m3));
    return (((l1 - l2 - m3) & 1) ? -1.0 : 1.0) * root * sum;
}

// The l3 that couple with (l1, l2) at an even sum, up to lmax: l = |l1-l2| + 2 i.
struct AceL3 {
    int lo, n, reals;      // first l3, how many, real numbers of their A (2 l3 + 1 each)
};
__host__ __device__ constexpr AceL3 ace_l3(int l1, int l2, int lmax) {
    AceL3 r{l1 > l2 ? l1 - l2 : l2 - l1, 0, 0};
    for (int l = r.lo; l <= l1 + l2 && l <= lmax; l += 2) {
        ++r.n;
        r.reals += 2 * l + 1;
    }
    return r;
}
// Position of (l3, M >= 0)'s real part among them (the imaginary part of M > 0 behind it)
__host__ __device__ constexpr int ace_l3_re(int lo, int l3, int M) {
    int o = 0;
    for (int l = lo; l < l3; l += 2) o += 2 * l + 1;
    return o + (M ? 2 * M - 1 : 0);
}

// Where a lane's values of one tile go.  PT points per tile; the 64 / PT lane
// groups of a wave work on different pairs.  Point-major (PT = 16): whole rows in
// LDS, written at the end as one contiguous piece (segments of a row written when
// their pair was done left partial lines: 53 million write requests for 11
// million lines' worth at 300,007 points); a value that the lane's pair does not
// have goes to a spare word, which costs less than a branch around each.
// Descriptor-major (PT = 64): stored at once, one plane per column.
template <int PT>
struct AceOut {
    static constexpr bool kRows = PT < kTile;
    float* to;             // the lane's point: its row in LDS, or its element of plane 0
    float* spare;          // kAceMaxPairCols words per lane, a word apart between lanes (rows only)
    int64_t ds;            // plane stride
    bool valid;
    // value c of a pair whose own values begin at c = first, in column col0
    __device__ __forceinline__ void put(int col0, int c, int first, float v) const {
        if constexpr (kRows) (c >= first ? to + (col0 - first) : spare)[c] = v;
        else if (valid && c >= first) to[(col0 - first + c) * ds] = v;
    }
};

// A wave's place in its list of rounds: the kind of the round and the lane's pair.
template <int PT>
struct AceRounds {
    const int* r;          // this round (LDS)
    const int* end;
    int group;             // the lane's group
    int ints;              // of a round
    __device__ __forceinline__ bool more() const { return r < end; }
    __device__ __forceinline__ void next() { r += ints; }
    __device__ __forceinline__ int kind() const { return __builtin_amdgcn_readfirstlane(r[0]) & 255; }
    __device__ __forceinline__ int first_n3() const { return __builtin_amdgcn_readfirstlane(r[0]) >> 8; }
    __device__ __forceinline__ int pair() const {
        if constexpr (PT == kTile) return __builtin_amdgcn_readfirstlane(r[1]);
        else return r[1 + group];
    }
};

// Rank 3 of the pairs (n1 l1), (n2 l2), l1 <= l2, of the rounds of one kind, code
// specialised for (l1, l2).  For an even l-sum the terms of M and -M are conjugates, so
//   B = P(0) A_{l3,0} + sum_{M>=1} 2 (-1)^M Re[P(M) conj A_{l3,M}],
//   P(M) = sum_m1 (l1 l2 l3; m1, M - m1, -M) A1(m1) A2(M - m1);
// a product of the pair is formed once for every l3, A of the third factor stays
// in registers over the rounds, and every index, sign and 3j symbol is a constant.
template <int PT, int L1, int L2, int LMAX>
__device__ __forceinline__ void ace3_rounds(const float2* a, const AceOut<PT>& o, AceRounds<PT>& rounds, int nmax) {
    constexpr AceL3 S = ace_l3(L1, L2, LMAX);
    float a3[kAceN][S.reals];
    static_for<0, kAceN>([&](auto nc) {
        constexpr int n3 = decltype(nc)::value;
        static_for<0, S.n>([&](auto ic) {
            constexpr int l = S.lo + 2 * decltype(ic)::value;
            static_for<0, l + 1>([&](auto mc) {
                constexpr int M = decltype(mc)::value, e = ace_l3_re(S.lo, l, M);
                const float2 v = a[(n3 * kAceLm + l * (l + 1) / 2 + M) * PT];
                a3[n3][e] = v.x;
                if constexpr (M > 0) a3[n3][e + 1] = v.y;
            });
        });
    });
#pragma clang loop unroll(disable)
    do {
        const int pr = rounds.pair(), n3_lo = rounds.first_n3();
        const float2* s1 = a + (pr & 3) * (kAceLm * PT);
        const float2* s2 = a + ((pr >> 2) & 3) * (kAceLm * PT);
        float2 a1[L1 + 1], a2[L2 + 1];
        static_for<0, L1 + 1>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            a1[m] = s1[(L1 * (L1 + 1) / 2 + m) * PT];
        });
        static_for<0, L2 + 1>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            a2[m] = s2[(L2 * (L2 + 1) / 2 + m) * PT];
        });
        float p[S.reals];
        static_for<0, S.reals>([&](auto ec) { p[decltype(ec)::value] = 0.f; });
        static_for<0, (L1 < L2 ? L1 : L2) + 1>([&](auto mc) {             // M = 0: m1 = m, m2 = -m and their conjugates
            constexpr int m = decltype(mc)::value;
            const float x = m ? fmaf(a1[m].x, a2[m].x, a1[m].y * a2[m].y) : a1[0].x * a2[0].x;
            static_for<0, S.n>([&](auto ic) {
                constexpr int l = S.lo + 2 * decltype(ic)::value, e = ace_l3_re(S.lo, l, 0);
                constexpr float c = (float)(ace_3j(L1, L2, l, m, -m, 0) * (m == 0 ? 1.0 : (m & 1) ? -2.0 : 2.0));
                p[e] = fmaf(c, x, p[e]);
            });
        });
        static_for<1, S.lo + 2 * (S.n - 1) + 1>([&](auto Mc) {
            constexpr int M = decltype(Mc)::value;
            static_for<0, 2 * L1 + 1>([&](auto jc) {
                constexpr int m1 = decltype(jc)::value - L1, m2 = M - m1;
                if constexpr (m2 >= -L2 && m2 <= L2) {
                    constexpr int am1 = m1 < 0 ? -m1 : m1, am2 = m2 < 0 ? -m2 : m2;
                    // A_{l,-m} = (-1)^m conj A_{l,m}
                    constexpr bool neg = ((m1 < 0 && (am1 & 1)) != (m2 < 0 && (am2 & 1))) != ((M & 1) != 0);
                    const float ax = a1[am1].x, ay = m1 < 0 ? -a1[am1].y : a1[am1].y;
                    const float bx = a2[am2].x, by = m2 < 0 ? -a2[am2].y : a2[am2].y;
                    float xr, xi;
                    if constexpr (am1 == 0) { xr = ax * bx; xi = ax * by; }
                    else if constexpr (am2 == 0) { xr = ax * bx; xi = ay * bx; }
                    else { xr = fmaf(ax, bx, -ay * by); xi = fmaf(ax, by, ay * bx); }
                    static_for<0, S.n>([&](auto ic) {
                        constexpr int l = S.lo + 2 * decltype(ic)::value;
                        if constexpr (l >= M) {
                            constexpr int e = ace_l3_re(S.lo, l, M);
                            constexpr float c = (float)(ace_3j(L1, L2, l, m1, m2, -M) * (neg ? -2.0 : 2.0));
                            p[e] = fmaf(c, xr, p[e]);
                            p[e + 1] = fmaf(c, xi, p[e + 1]);
                        }
                    });
                }
            });
        });
        // the pair's columns are (n3, l3) in order, from its later key on
        const int first = (pr >> 4) & 15, col0 = pr >> 8;
        static_for<0, kAceN>([&](auto nc) {
            constexpr int n3 = decltype(nc)::value;
            if (n3 < n3_lo || n3 >= nmax) return;
            static_for<0, S.n>([&](auto ic) {
                constexpr int i = decltype(ic)::value, l = S.lo + 2 * i, e0 = ace_l3_re(S.lo, l, 0);
                float v = p[e0] * a3[n3][e0];
#pragma unroll
                for (int e = 1; e < 2 * l + 1; ++e) v = fmaf(p[e0 + e], a3[n3][e0 + e], v);
                o.put(col0, n3 * S.n + i, first, v);
            });
        });
        rounds.next();
    } while (rounds.more() && rounds.kind() == L1 * (kAceL + 1) + L2);
}

// Rank 2 of one l: sum_m (-1)^m A_{n1 l m} A_{n2 l -m}
//   = A_{n1 l 0} A_{n2 l 0} + 2 sum_{m>0} Re(A_{n1 l m} conj(A_{n2 l m})).
template <int PT, int L>
__device__ __forceinline__ void ace2_round(const float2* a, const AceOut<PT>& o, int pr) {
    const float2* s1 = a + ((pr & 3) * kAceLm + L * (L + 1) / 2) * PT;
    const float2* s2 = a + (((pr >> 2) & 3) * kAceLm + L * (L + 1) / 2) * PT;
    float s = 0.f;
    static_for<1, L + 1>([&](auto mc) {
        constexpr int m = decltype(mc)::value;
        const float2 x = s1[m * PT], y = s2[m * PT];
        s = fmaf(x.x, y.x, fmaf(x.y, y.y, s));
    });
    o.put(pr >> 8, 0, (pr >> 4) & 15, fmaf(2.f, s, s1[0].x * s2[0].x));
}

// A block's rows, n floats, from LDS (whole block).
__device__ __forceinline__ void ace_write_rows(const float* from, int n, float* __restrict__ to) {
    int done = 0;
    if ((reinterpret_cast<uintptr_t>(to) & 15) == 0) {
        done = n & ~3;
        for (int i = threadIdx.x; i < n / 4; i += blockDim.x)
            reinterpret_cast<float4*>(to)[i] = reinterpret_cast<const float4*>(from)[i];
    }
    for (int i = done + threadIdx.x; i < n; i += blockDim.x) to[i] = from[i];
}

// Ranks 1-3 of one tile from its projected A.  Bound by the VALU (17,000 of its
// instructions per 64 points in rank 3 at nmax = lmax = 4, if every lane group has
// a pair) beside the 2.4 KB of output per point.  Rounds of up to 64 / PT pairs of
// one (l1, l2) are dealt to the waves by their cost.  One product of a pair for
// all its l3, M >= 0 only, constant 3j symbols and whole rows written, where every
// (p1, p2, l3) formed its own products for every m3 from a table of symbols and
// wrote segments of rows: 745 -> 335 us per 300,007 points, point-major.
template <int PT, int LMAX>
__global__ __launch_bounds__(64 * kAce3Waves, 4) void k_ace(const float2* __restrict__ Ag, int nmax, int64_t n_pts,
                                                           const int* __restrict__ plan, int plan_ints, int n_desc,
                                                           float* __restrict__ out, int64_t ds) {
    extern __shared__ float4 ace_lds[];
    float2* sA = reinterpret_cast<float2*>(ace_lds);                       // [kAceAPerPoint][PT]
    int* sPlan = reinterpret_cast<int*>(sA + kAceAPerPoint * PT);
    // PT rows (point-major), as they lie in memory, and the spare words
    float* sO = reinterpret_cast<float*>(sPlan + (plan_ints + 3) / 4 * 4);
    const int lane = threadIdx.x & 63, pt = lane % PT;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t p0 = (int64_t)blockIdx.x * PT;
    {
        // the block's points of a 64-point tile of A
        const float2* src = Ag + p0 / kTile * (kAceAPerPoint * kTile) + p0 % kTile;
        for (int e = threadIdx.x; e < kAceAPerPoint * PT; e += blockDim.x) sA[e] = src[e / PT * kTile + e % PT];
        for (int e = threadIdx.x; e < plan_ints; e += blockDim.x) sPlan[e] = plan[e];
    }
    __syncthreads();
    AceOut<PT> o;
    o.ds = ds;
    o.valid = p0 + pt < n_pts;
    if constexpr (o.kRows) {
        o.to = sO + pt * n_desc;
        o.spare = sO + PT * n_desc + lane;
    } else {
        o.to = out + p0 + pt;
    }
    const float2* a = sA + pt;
    AceRounds<PT> rounds;
    rounds.group = lane / PT;
    rounds.ints = kTile / PT + 1;
    rounds.r = sPlan + __builtin_amdgcn_readfirstlane(sPlan[wave]);
    rounds.end = sPlan + __builtin_amdgcn_readfirstlane(sPlan[wave + 1]);
    while (rounds.more()) {
        const int kind = rounds.kind();
        if (kind >= kAceRank2) {
            const int pr = rounds.pair();
            static_for<0, LMAX + 1>([&](auto lc) {
                constexpr int L = decltype(lc)::value;
                if (kind == kAceRank2 + L) ace2_round<PT, L>(a, o, pr);
            });
            if (kind == kAceRank1) o.put(pr >> 8, 0, (pr >> 4) & 15, a[(pr & 3) * (kAceLm * PT)].x);
            rounds.next();
        } else {
            static_for<0, LMAX + 1>([&](auto c1) {
                static_for<decltype(c1)::value, LMAX + 1>([&](auto c2) {
                    constexpr int L1 = decltype(c1)::value, L2 = decltype(c2)::value;
                    if (kind == L1 * (kAceL + 1) + L2) ace3_rounds<PT, L1, L2, LMAX>(a, o, rounds, nmax);
                });
            });
        }
    }
    if constexpr (o.kRows) {
        __syncthreads();
        ace_write_rows(sO, (int)(n_pts - p0 < PT ? n_pts - p0 : PT) * n_desc, out + p0 * n_desc);
    }
}

// Position of the term (M, m1) in the Clebsch-Gordan block of a rank-4
// pair combination (l1, l2, L): M = 0..L, m1 = -l1..l1 with |M - m1| <= l2
// (the host builds the block in the same order).
__host__ __device__ constexpr int ace4_k(int L1, int L2, int M, int m1) {
    int k = 0;
    for (int a = 0; a <= M; ++a)
        for (int b = -L1; b <= L1; ++b) {
            if (a == M && b == m1) return k;
            if (a - b >= -L2 && a - b <= L2) ++k;
        }
    return k;
}

// P_a(M) = sum_m1 <l1 m1 l2 m2|L M> A1(m1) A2(m2), m2 = M - m1, for M = 0..L,
// code specialised for (L1, L2, LL): the pair's A values in registers,
// indices, conjugations and signs at compile time; written to dst[M][lane].
template <int L1, int L2, int LL>
__device__ __forceinline__ void ace4_pair(const float2 (*sA)[kTile], int b1, int b2, int lane,
                                          const float* __restrict__ cf, float2* __restrict__ dst) {
    float2 a1[L1 + 1], a2[L2 + 1];
    static_for<0, L1 + 1>([&](auto mc) { a1[decltype(mc)::value] = sA[b1 + decltype(mc)::value][lane]; });
    static_for<0, L2 + 1>([&](auto mc) { a2[decltype(mc)::value] = sA[b2 + decltype(mc)::value][lane]; });
    static_for<0, LL + 1>([&](auto ic) {
        constexpr int M = decltype(ic)::value;
        __builtin_amdgcn_sched_barrier(0);
        float xr = 0.f, xi = 0.f;
        static_for<0, 2 * L1 + 1>([&](auto jc) {
            constexpr int m1 = decltype(jc)::value - L1, m2 = M - m1;
            if constexpr (m2 >= -L2 && m2 <= L2) {
                constexpr int k = ace4_k(L1, L2, M, m1);
                constexpr int am1 = m1 < 0 ? -m1 : m1, am2 = m2 < 0 ? -m2 : m2;
                constexpr bool neg = ((m1 < 0 && (am1 & 1)) != (m2 < 0 && (am2 & 1)));
                const float c = neg ? -cf[k] : cf[k];
                const float ax = a1[am1].x, ay = m1 < 0 ? -a1[am1].y : a1[am1].y;
                const float bx = a2[am2].x, by = m2 < 0 ? -a2[am2].y : a2[am2].y;
                xr = fmaf(c, ax * bx - ay * by, xr);
                xi = fmaf(c, ax * by + ay * bx, xi);
            }
        });
        dst[M * kTile + lane] = make_float2(xr, xi);
    });
}

__host__ __device__ constexpr bool ace4_combo_valid(int c) {
    const int l1 = c / 28, l2 = (c / 7) % 4, L = c % 7;
    return L >= (l1 > l2 ? l1 - l2 : l2 - l1) && L <= l1 + l2;
}

// Rank 4 (one intermediate coupling L), descriptor-major.  Sixteen waves per 64-point tile
// (the projected A of the tile in LDS), in phases of one or more L: the
// coupled pairs P_a(M) = sum_m1 <l1 m1 l2 m2|L M> A_p1 A_p2 (M = 0..L) the
// descriptors of the phase need are formed into LDS (every wave takes every
// sixteenth pair, all its M by code specialised for (l1, l2, L)), then every
// wave evaluates a contiguous share of the phase's descriptors, B = f (Re P_a(0) conj P_b(0) + 2 sum_{M>0} Re P_a(M) conj P_b(M))
// (f = (-1)^(l3+l4) / sqrt(2L+1)), keeping P_a in registers while consecutive
// descriptors share it.  Terms and descriptors come from wave-uniform loads.
constexpr int kAce4Waves = 16;

__global__ __launch_bounds__(64 * kAce4Waves) void k_ace4(const float2* __restrict__ Ag, int n_phases, int64_t n_pts,
                                                          const int* __restrict__ l_units,
                                                          const int4* __restrict__ units,
                                                          const float* __restrict__ coef,
                                                          const int* __restrict__ l_descs,
                                                          const int4* __restrict__ descs, int n4,
                                                          float* __restrict__ out, int64_t ds) {
    __shared__ float2 sA[kAceN * kAceLm][kTile];
    __shared__ int4 sD[kAce4MaxDescsL];     // this phase's descriptor entries
    extern __shared__ float2 sP[];          // [slots][kTile]

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    AceTile tl;
    tl.idx = (int64_t)blockIdx.x * kTile + lane;
    tl.valid = tl.idx < n_pts;
    ace_load_tile(Ag, sA);
    __syncthreads();

    float* o = out + (tl.valid ? tl.idx : 0);         // descriptor k at o[k * ds]
    for (int ph = 0; ph < n_phases; ++ph) {
        // this phase's descriptor entries into LDS, read back as broadcasts:
        // a scalar load per descriptor would hold every LDS wait of the loop
        // below until the scalar cache answered
        const int d0 = l_descs[ph], nd = l_descs[ph + 1] - d0;
        for (int i = threadIdx.x; i < nd; i += blockDim.x) sD[i] = descs[d0 + i];
        // coupled pairs of this phase's couplings L into sP
        const int u0 = l_units[ph], u1 = l_units[ph + 1];
        for (int u = u0 + wave; u < u1; u += kAce4Waves) {
            const int4 h = units[u];
            const float* cf = coef + __builtin_amdgcn_readfirstlane(h.x);
            const int combo = __builtin_amdgcn_readfirstlane(h.y), slot = __builtin_amdgcn_readfirstlane(h.z);
            const int bb = __builtin_amdgcn_readfirstlane(h.w);
            const int b1 = bb & 255, b2 = bb >> 8;
            static_for<0, 4 * 4 * 7>([&](auto cc) {
                constexpr int C = decltype(cc)::value;
                if constexpr (ace4_combo_valid(C)) {
                    if (combo == C) ace4_pair<C / 28, (C / 7) % 4, C % 7>(sA, b1, b2, lane, cf, sP + slot * kTile);
                }
            });
        }
        __syncthreads();
        // this phase's descriptors, a contiguous share per wave
        const int db = nd * wave / kAce4Waves, de = nd * (wave + 1) / kAce4Waves;
        int cached = -1;
        float2 pa[2 * kAce4MaxL + 1];
        for (int d = db; d < de; ++d) {
            const int4 q = sD[d];
            const int sx = __builtin_amdgcn_readfirstlane(q.x), sb = __builtin_amdgcn_readfirstlane(q.y);
            const int sa = sx & 0xffff, L = sx >> 16;             // a slot identifies its L too
            const int ok = __builtin_amdgcn_readfirstlane(q.z);
            const float f = __int_as_float(__builtin_amdgcn_readfirstlane(q.w));
            // code per L: a descriptor's LDS reads issue together, with no
            // branch per M between them
            float v = 0.f;
            static_for<0, 2 * kAce4MaxL + 1>([&](auto lc) {
                constexpr int LL = decltype(lc)::value;
                if (L != LL) return;
                if (sa != cached) {
#pragma unroll
                    for (int M = 0; M <= LL; ++M) pa[M] = sP[(sa + M) * kTile + lane];
                    cached = sa;
                }
                float2 b[LL + 1];
#pragma unroll
                for (int M = 0; M <= LL; ++M) b[M] = sP[(sb + M) * kTile + lane];
                float acc = 0.f;
#pragma unroll
                for (int M = 1; M <= LL; ++M) acc = fmaf(pa[M].x, b[M].x, fmaf(pa[M].y, b[M].y, acc));
                v = f * fmaf(2.f, acc, pa[0].x * b[0].x + pa[0].y * b[0].y);
            });
            if (tl.valid) o[ok * ds] = v;
        }
        __syncthreads();
    }
}

// Clebsch-Gordan coefficient <l1 m1 l2 m2 | L M> at compile time.
__host__ __device__ constexpr double ace_cg(int l1, int m1, int l2, int m2, int L, int M) {
    return (((l1 - l2 + M) & 1) ? -1.0 : 1.0) * ace_sqrt(2 * L + 1) * ace_3j(l1, l2, L, m1, m2, -M);
}

// P_a(M) of the pairs (n1 l1), (n2 l2), l1 <= l2, of the rounds of one kind, for
// every L their descriptors need (the others go to spare slots): a product of the
// pair is formed once for all L.  a, pairs: the lane's point.
template <int L1, int L2>
__device__ __forceinline__ void ace4_pair_rounds(const float2* a, float2* pairs, AceRounds<kAce4RowPoints>& rounds) {
    constexpr int PT = kAce4RowPoints, LO = L2 - L1, HI = L1 + L2;
#pragma clang loop unroll(disable)
    do {
        const int* e = rounds.r + 1 + rounds.group * kAce4PairInts;
        const int pr = e[0];
        float2 a1[L1 + 1], a2[L2 + 1];
        static_for<0, L1 + 1>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            a1[m] = a[((pr & 3) * kAceLm + L1 * (L1 + 1) / 2 + m) * PT];
        });
        static_for<0, L2 + 1>([&](auto mc) {
            constexpr int m = decltype(mc)::value;
            a2[m] = a[((pr >> 2) * kAceLm + L2 * (L2 + 1) / 2 + m) * PT];
        });
        float2* to[HI - LO + 1];
        static_for<0, HI - LO + 1>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            to[i] = pairs + ((e[1 + i / 3] >> (10 * (i % 3))) & 1023) * PT;
        });
        static_for<0, HI + 1>([&](auto Mc) {
            constexpr int M = decltype(Mc)::value, L0 = M > LO ? M : LO;
            float xr[HI + 1], xi[HI + 1];
            static_for<L0, HI + 1>([&](auto Lc) { xr[decltype(Lc)::value] = xi[decltype(Lc)::value] = 0.f; });
            static_for<0, 2 * L1 + 1>([&](auto jc) {
                constexpr int m1 = decltype(jc)::value - L1, m2 = M - m1;
                if constexpr (m2 >= -L2 && m2 <= L2) {
                    constexpr int am1 = m1 < 0 ? -m1 : m1, am2 = m2 < 0 ? -m2 : m2;
                    constexpr bool neg = (m1 < 0 && (am1 & 1)) != (m2 < 0 && (am2 & 1));
                    const float ax = a1[am1].x, ay = m1 < 0 ? -a1[am1].y : a1[am1].y;
                    const float bx = a2[am2].x, by = m2 < 0 ? -a2[am2].y : a2[am2].y;
                    float pr_, pi_;
                    if constexpr (am1 == 0) { pr_ = ax * bx; pi_ = ax * by; }
                    else if constexpr (am2 == 0) { pr_ = ax * bx; pi_ = ay * bx; }
                    else { pr_ = fmaf(ax, bx, -ay * by); pi_ = fmaf(ax, by, ay * bx); }
                    static_for<L0, HI + 1>([&](auto Lc) {
                        constexpr int L = decltype(Lc)::value;
                        constexpr double cg = ace_cg(L1, m1, L2, m2, L, M);
                        if constexpr (cg > 1e-12 || cg < -1e-12) {
                            constexpr float c = (float)(neg ? -cg : cg);
                            xr[L] = fmaf(c, pr_, xr[L]);
                            xi[L] = fmaf(c, pi_, xi[L]);
                        }
                    });
                }
            });
            static_for<L0, HI + 1>([&](auto Lc) {
                constexpr int L = decltype(Lc)::value;
                to[L - LO][M * PT] = make_float2(xr[L], xi[L]);
            });
        });
        rounds.next();
    } while (rounds.more() && rounds.kind() == L1 * (kAce4MaxL + 1) + L2);
}

// Rank 4, point-major: blocks of kAce4RowPoints points with every coupled pair and
// the whole rows in LDS, so that the pairs are formed and the descriptors
// evaluated in one pass each and the rows leave as one contiguous piece.  The
// lane groups of the waves take contiguous shares of the descriptors of one L
// (sorted by their first pair, whose P_a stays in registers).  Bound by the VALU
// and the LDS reads of P_b beside 4 n4 bytes of output per point.  Writing planes
// (in phases of the L that fit) and transposing them moved every value three
// times: 660 -> 345 us per 150,001 points at nmax4 = lmax4 = 3.  Blocks of 8
// points leave room for two on a CU (79 KB each).
__global__ __launch_bounds__(64 * kAce4RowWaves) void k_ace4_rows(const float2* __restrict__ Ag, int64_t n_pts,
                                                                  const int* __restrict__ plan, int plan_ints,
                                                                  int n_slots, int n4, float* __restrict__ out) {
    constexpr int PT = kAce4RowPoints, G = kTile / PT;
    extern __shared__ float4 ace_lds[];
    float2* sA = reinterpret_cast<float2*>(ace_lds);                       // [kAce4ARows][PT]
    float2* sP = sA + kAce4ARows * PT;                                     // [n_slots][PT]
    float* sO = reinterpret_cast<float*>(sP + n_slots * PT);               // [PT][n4], spare words
    int* sPlan = reinterpret_cast<int*>(sO + PT * n4 + 64);
    const int lane = threadIdx.x & 63, pt = lane % PT, group = lane / PT;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t p0 = (int64_t)blockIdx.x * PT;
    {
        const float2* src = Ag + p0 / kTile * (kAceAPerPoint * kTile) + p0 % kTile;
        for (int e = threadIdx.x; e < kAce4ARows * PT; e += blockDim.x) sA[e] = src[e / PT * kTile + e % PT];
        for (int e = threadIdx.x; e < plan_ints; e += blockDim.x) sPlan[e] = plan[e];
    }
    __syncthreads();
    AceRounds<PT> rounds;
    rounds.group = group;
    rounds.ints = 1 + G * kAce4PairInts;
    rounds.r = sPlan + __builtin_amdgcn_readfirstlane(sPlan[wave]);
    rounds.end = sPlan + __builtin_amdgcn_readfirstlane(sPlan[wave + 1]);
    while (rounds.more()) {
        const int kind = rounds.kind();
        static_for<0, kAce4MaxL + 1>([&](auto c1) {
            static_for<decltype(c1)::value, kAce4MaxL + 1>([&](auto c2) {
                constexpr int L1 = decltype(c1)::value, L2 = decltype(c2)::value;
                if (kind == L1 * (kAce4MaxL + 1) + L2) ace4_pair_rounds<L1, L2>(sA + pt, sP + pt, rounds);
            });
        });
    }
    __syncthreads();
    float* row = sO + pt * n4;
    float* spare = sO + PT * n4 + lane;
    const float2* pairs = sP + pt;
    static_for<0, 2 * kAce4MaxL + 1>([&](auto lc) {
        constexpr int L = decltype(lc)::value;
        const int d0 = __builtin_amdgcn_readfirstlane(sPlan[kAce4RowWaves + 1 + L]);
        const int d1 = __builtin_amdgcn_readfirstlane(sPlan[kAce4RowWaves + 2 + L]);
        const int share = (d1 - d0 + kAce4RowWaves * G - 1) / (kAce4RowWaves * G);
        const int first = d0 + (wave * G + group) * share;
        constexpr float f = (float)(1.0 / ace_sqrt(2 * L + 1));
        int cached = -1;
        float2 pa[L + 1];
#pragma clang loop unroll(disable)
        for (int k = 0; k < share; ++k) {
            const int d = first + k, q = sPlan[d < d1 ? d : d1 - 1];
            const int sa = q & 1023, sb = (q >> 10) & 1023;
            if (sa != cached) {
                static_for<0, L + 1>([&](auto mc) { pa[decltype(mc)::value] = pairs[(sa + decltype(mc)::value) * PT]; });
                cached = sa;
            }
            float2 b[L + 1];
            static_for<0, L + 1>([&](auto mc) { b[decltype(mc)::value] = pairs[(sb + decltype(mc)::value) * PT]; });
            float acc = 0.f;
#pragma unroll
            for (int M = 1; M <= L; ++M) acc = fmaf(pa[M].x, b[M].x, fmaf(pa[M].y, b[M].y, acc));
            const float v = fmaf(2.f, acc, pa[0].x * b[0].x + pa[0].y * b[0].y) * (q < 0 ? -f : f);
            *(d < d1 ? row + ((q >> 20) & 1023) : spare) = v;
        }
    });
    __syncthreads();
    ace_write_rows(sO, (int)(n_pts - p0 < PT ? n_pts - p0 : PT) * n4, out + p0 * n4);
}

hipError_t launch_ace_proj(hipStream_t s, const BinState& bins, const int N[3], double rcut, int64_t pt_begin,
                           int64_t n_pts, float2* Ag, int* err) {
    if (n_pts <= 0) return hipSuccess;
    const int64_t n_tiles = (n_pts + kTile - 1) / kTile;
    hipLaunchKernelGGL(k_ace_proj, dim3((unsigned)n_tiles), dim3(64 * kAceWaves), 0, s, bins, N[0], N[1], N[2], rcut,
                       pt_begin, n_pts, Ag, err);
    return hipGetLastError();
}

hipError_t launch_ace4(hipStream_t s, const float2* Ag, int lmax4, int n_phases, int64_t n_pts, const int* l_units,
                       const int4* units, const float* coef, const int* l_descs, const int4* descs, int max_slots,
                       int n4, float* out, int64_t ds) {
    if (n_pts <= 0 || n4 <= 0) return hipSuccess;
    if (lmax4 < 0 || lmax4 > kAce4MaxL) return hipErrorInvalidValue;
    const size_t lds = sizeof(float2) * (size_t)max_slots * kTile;
    static std::once_flag attr_once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(attr_once, [] {
        attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_ace4),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kAce4LdsBudget);
    });
    if (attr_err != hipSuccess) return attr_err;
    if (lds > kAce4LdsBudget) return hipErrorInvalidValue;
    const int64_t n_tiles = (n_pts + kTile - 1) / kTile;
    hipLaunchKernelGGL(k_ace4, dim3((unsigned)n_tiles), dim3(64 * kAce4Waves), lds, s, Ag, n_phases, n_pts, l_units,
                       units, coef, l_descs, descs, n4, out, ds);
    return hipGetLastError();
}

hipError_t launch_ace4_rows(hipStream_t s, const float2* Ag, int64_t n_pts, const int* plan, int plan_ints, int n_slots,
                            int n4, float* out) {
    if (n_pts <= 0 || n4 <= 0) return hipSuccess;
    constexpr int PT = kAce4RowPoints;
    const size_t lds = ace4_rows_lds(plan_ints, n_slots, n4);
    if (lds > kAce4RowsLds) return hipErrorInvalidValue;
    static std::once_flag attr_once;
    static hipError_t attr_err = hipSuccess;
    std::call_once(attr_once, [] {
        attr_err = hipFuncSetAttribute(reinterpret_cast<const void*>(&k_ace4_rows),
                                       hipFuncAttributeMaxDynamicSharedMemorySize, (int)kAce4RowsLds);
    });
    if (attr_err != hipSuccess) return attr_err;
    hipLaunchKernelGGL(k_ace4_rows, dim3((unsigned)((n_pts + PT - 1) / PT)), dim3(64 * kAce4RowWaves), lds, s, Ag, n_pts,
                       plan, plan_ints, n_slots, n4, out);
    return hipGetLastError();
}

template <int PT, int LMAX>
static hipError_t ace_run(hipStream_t s, const float2* Ag, int nmax, int64_t n_pts, const int* plan, int plan_ints,
                          int n_desc, float* out, int64_t ds) {
    const size_t lds = sizeof(float2) * kAceAPerPoint * PT + sizeof(int) * ((plan_ints + 3) / 4 * 4) +
                       (PT < kTile ? sizeof(float) * (PT * n_desc + 64 + kAceMaxPairCols) : 0);
    hipLaunchKernelGGL((k_ace<PT, LMAX>), dim3((unsigned)((n_pts + PT - 1) / PT)), dim3(64 * kAce3Waves), lds, s, Ag,
                       nmax, n_pts, plan, plan_ints, n_desc, out, ds);
    return hipGetLastError();
}

template <int PT>
static hipError_t ace_lmax(hipStream_t s, const float2* Ag, int nmax, int lmax, int64_t n_pts, const int* plan,
                           int plan_ints, int n_desc, float* out, int64_t ds) {
    switch (lmax) {
    case 0: return ace_run<PT, 0>(s, Ag, nmax, n_pts, plan, plan_ints, n_desc, out, ds);
    case 1: return ace_run<PT, 1>(s, Ag, nmax, n_pts, plan, plan_ints, n_desc, out, ds);
    case 2: return ace_run<PT, 2>(s, Ag, nmax, n_pts, plan, plan_ints, n_desc, out, ds);
    case 3: return ace_run<PT, 3>(s, Ag, nmax, n_pts, plan, plan_ints, n_desc, out, ds);
    case 4: return ace_run<PT, 4>(s, Ag, nmax, n_pts, plan, plan_ints, n_desc, out, ds);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_ace(hipStream_t s, const float2* Ag, int nmax, int lmax, int64_t n_pts, const int* plan,
                      int plan_ints, bool rows, int n_desc, float* out, int64_t ds) {
    if (n_pts <= 0) return hipSuccess;
    if (nmax < 1 || nmax > kAceN) return hipErrorInvalidValue;
    return rows ? ace_lmax<kAceRowPoints>(s, Ag, nmax, lmax, n_pts, plan, plan_ints, n_desc, out, ds)
                : ace_lmax<kTile>(s, Ag, nmax, lmax, n_pts, plan, plan_ints, n_desc, out, ds);
}

}  // namespace mala
