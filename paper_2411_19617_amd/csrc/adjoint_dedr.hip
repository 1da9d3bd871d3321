// Adjoint of the bispectrum descriptors, second step: dL/dR from Y = dL/du
// (the descriptor factor of the force expression, Eq. forcesmala).  With
// u^J = I + sum_k fc(r_k) U^J(Delta_k) (Eq. SNAPExpansion), per grid point
// and neighbour image k,
//   dL/dDelta_k = fc sum Re(conj(Y) dU/dDelta) + fc' n_k sum Re(conj(Y) U)
// (rows below the middle of a level twice, by the shared conjugate symmetry).
// In the separated form of u_basis.h sum Re(conj(Y) U) is, per point, a fixed
//   g(a, b) = sum over (k1, k2, n) of W phi_n(|a|^2) . parts of a^k1 b^k2
// whose W are combinations of Y, formed once per point and kept in registers
// (split over the waves by k1); a neighbour needs g and its four derivatives.
// Per candidate image the lanes' terms are summed in LDS, then added to its
// atom's gradient with one FP64 atomic per component (the order of those
// additions is not fixed).  An atom sitting exactly on a grid point is left out
// of that point's gradient: the map from the displacement to U has no derivative
// at r = 0.
#include "snap_core.h"
#include "tile_gather.h"
#include "u_basis.h"

namespace mala {
// ------------------------------------------------------------------ dL/dDelta
// The group's W from the point's Y (the transpose of the combinations that form
// u from its sums).
template <int TJ, int G, int NACC>
__device__ __forceinline__ void dedr_weights(const float2* __restrict__ yt, float (&W)[NACC]) {
    static_for<0, NACC>([&](auto ec) { W[decltype(ec)::value] = 0.f; });
    static_for<0, TJ + 1>([&](auto Jc) {
        constexpr int J = decltype(Jc)::value;
        static_for<0, J / 2 + 1>([&](auto mac) {
            constexpr int ma = decltype(mac)::value;
            static_for<0, J + 1>([&](auto mbc) {
                constexpr int mb = decltype(mbc)::value, k1 = ma + mb - J, k2 = mb - ma;
                constexpr int K1 = k1 < 0 ? -k1 : k1, K2 = k2 < 0 ? -k2 : k2;
                if constexpr (u_group_of(TJ, K1) == G) {
                    constexpr UCoef cf = u_coef(J, ma, mb);
                    constexpr int NP = u_parts(K1, K2), S = u_slot(TJ, G, K1, K2);
                    constexpr bool cj = k1 < 0 || (k1 == 0 && k2 < 0);       // conjugate of (-k1, -k2)
                    constexpr bool bneg = cj ? -k2 < 0 : k2 < 0;             // conj(b)^K2 beside a^K1
                    constexpr float w = 2 * ma == J ? 1.f : 2.f;
                    const float2 y = yt[(half_off(J) + ma * (J + 1) + mb) * kTile];
                    const float yr = w * y.x, yi = cj ? -w * y.y : w * y.y;
                    static_for<0, (J - K1 - K2) / 2 + 1>([&](auto nc) {
                        constexpr int n = decltype(nc)::value;
                        constexpr float c = (float)cf.c[n];
                        constexpr int o = S + NP * n;
                        W[o] = fmaf(c, yr, W[o]);
                        if constexpr (NP == 4) {          // rr, ii, ri, ir
                            W[o + 1] = fmaf(bneg ? c : -c, yr, W[o + 1]);
                            W[o + 2] = fmaf(bneg ? -c : c, yi, W[o + 2]);
                            W[o + 3] = fmaf(c, yi, W[o + 3]);
                        } else if constexpr (NP == 2) {
                            W[o + 1] = fmaf(c, yi, W[o + 1]);
                        }
                    });
                }
            });
        });
    });
}

// The group's part of g and of its derivatives: out = g, d/d(a_r, a_i, b_r, b_i).
template <int TJ, int G, int NACC>
__device__ __forceinline__ void dedr_neighbour(float ar, float ai, float br, float bi, const float (&W)[NACC],
                                               float (&out)[5]) {
    // phi_n = T_n(x) of the bases the group uses, and d phi_n / dx
    const float x0 = fmaf(ai, ai, fmaf(ar, ar, -fmaf(br, br, bi * bi)));
    float phi[kUBases][kUMaxN + 1], dphi[kUBases][kUMaxN + 1];
    static_for<0, kUBases>([&](auto bc) {
        constexpr int B = decltype(bc)::value, NM = u_basis_nmax(TJ, G, B);
        if constexpr (NM >= 1) {
            if constexpr (B == 0) phi[B][1] = x0;
            else phi[B][1] = fmaf(x0, (float)(0.5 / ub_half(B)), (float)((0.5 - ub_mid(B)) / ub_half(B)));
            const float x2 = 2.f * phi[B][1];
            dphi[B][1] = 1.f;
            static_for<2, NM + 1>([&](auto nc) {
                constexpr int n = decltype(nc)::value;
                if constexpr (n == 2) {
                    phi[B][2] = fmaf(x2, phi[B][1], -1.f);
                    dphi[B][2] = 2.f * x2;
                } else {
                    phi[B][n] = fmaf(x2, phi[B][n - 1], -phi[B][n - 2]);
                    dphi[B][n] = fmaf(x2, dphi[B][n - 1], fmaf(2.f, phi[B][n - 1], -dphi[B][n - 2]));
                }
            });
        }
    });
    constexpr int K1M = [] { int m = 0; for (int i = 0; i <= TJ; ++i) if (u_group_of(TJ, i) == G) m = i; return m; }();
    float pr[K1M + 1], pi[K1M + 1];           // a^k1
    pr[0] = 1.f;
    pi[0] = 0.f;
    static_for<1, K1M + 1>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        if constexpr (k == 1) {
            pr[1] = ar;
            pi[1] = ai;
        } else {
            pr[k] = fmaf(pr[k - 1], ar, -pi[k - 1] * ai);
            pi[k] = fmaf(pr[k - 1], ai, pi[k - 1] * ar);
        }
    });
    float car[K1M + 1], cai[K1M + 1];         // coefficients of Re, Im a^k1, summed over k2
    static_for<0, K1M + 1>([&](auto kc) { car[decltype(kc)::value] = cai[decltype(kc)::value] = 0.f; });
    float g = 0.f, gbr = 0.f, gbi = 0.f, dx = 0.f;
    float qr = 1.f, qi = 0.f;                 // b^k2
    static_for<0, u_group_k2max(TJ, G) + 1>([&](auto k2c) {
        constexpr int k2 = decltype(k2c)::value;
        const float lr = qr, li = qi;         // b^(k2 - 1)
        if constexpr (k2 == 1) {
            qr = br;
            qi = bi;
        } else if constexpr (k2 > 1) {
            qr = fmaf(lr, br, -li * bi);
            qi = fmaf(lr, bi, li * br);
        }
        float cbr = 0.f, cbi = 0.f;           // coefficients of Re, Im b^k2, summed over k1
        static_for<0, TJ + 1 - k2>([&](auto k1c) {
            constexpr int k1 = decltype(k1c)::value;
            if constexpr (u_group_of(TJ, k1) == G) {
                constexpr int NP = u_parts(k1, k2), NN = u_ncount(TJ, k1, k2), S = u_slot(TJ, G, k1, k2), B = u_basis(k1, k2);
                constexpr float scale = (float)(0.5 / ub_half(B));        // dx_B / dx0
                float h[NP], d[NP];
                static_for<0, NP>([&](auto pc) {
                    constexpr int p = decltype(pc)::value;
                    h[p] = W[S + p];
                    d[p] = 0.f;
                    static_for<1, NN>([&](auto nc) {
                        constexpr int n = decltype(nc)::value;
                        h[p] = fmaf(W[S + NP * n + p], phi[B][n], h[p]);
                        if constexpr (n == 1) d[p] = W[S + NP + p];
                        else d[p] = fmaf(W[S + NP * n + p], dphi[B][n], d[p]);
                    });
                });
                if constexpr (NP == 4) {      // rr, ii, ri, ir
                    car[k1] = fmaf(h[0], qr, fmaf(h[2], qi, car[k1]));
                    cai[k1] = fmaf(h[1], qi, fmaf(h[3], qr, cai[k1]));
                    cbr = fmaf(h[0], pr[k1], fmaf(h[3], pi[k1], cbr));
                    cbi = fmaf(h[1], pi[k1], fmaf(h[2], pr[k1], cbi));
                    if constexpr (NN > 1) {
                        const float er = fmaf(d[0], pr[k1], d[3] * pi[k1]), ei = fmaf(d[1], pi[k1], d[2] * pr[k1]);
                        dx = fmaf(scale, fmaf(er, qr, ei * qi), dx);
                    }
                } else if constexpr (k2 == 0 && k1 > 0) {
                    car[k1] += h[0];
                    cai[k1] += h[1];
                    if constexpr (NN > 1) dx = fmaf(scale, fmaf(d[0], pr[k1], d[1] * pi[k1]), dx);
                } else if constexpr (k2 > 0) {
                    cbr += h[0];
                    cbi += h[1];
                    g = fmaf(h[0], qr, fmaf(h[1], qi, g));
                    if constexpr (NN > 1) dx = fmaf(scale, fmaf(d[0], qr, d[1] * qi), dx);
                } else {
                    g += h[0];
                    if constexpr (NN > 1) dx = fmaf(scale, d[0], dx);
                }
            }
        });
        if constexpr (k2 > 0) {               // d b^k2 = k2 b^(k2-1) db
            gbr = fmaf((float)k2, fmaf(cbr, lr, cbi * li), gbr);
            gbi = fmaf((float)k2, fmaf(cbi, lr, -cbr * li), gbi);
        }
    });
    float gar = 0.f, gai = 0.f;
    static_for<1, K1M + 1>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        if constexpr (u_group_of(TJ, k) == G) {
            g = fmaf(car[k], pr[k], fmaf(cai[k], pi[k], g));
            gar = fmaf((float)k, fmaf(car[k], pr[k - 1], cai[k] * pi[k - 1]), gar);
            gai = fmaf((float)k, fmaf(cai[k], pr[k - 1], -car[k] * pi[k - 1]), gai);
        }
    });
    dx *= 2.f;                                // x0 = |a|^2 - |b|^2
    out[0] = g;
    out[1] = fmaf(dx, ar, gar);
    out[2] = fmaf(dx, ai, gai);
    out[3] = fmaf(-dx, br, gbr);
    out[4] = fmaf(-dx, bi, gbi);
}

// Neighbours are taken four at a time: wave w forms the w-th one's (a, b), every
// wave adds its group's part of g and the derivatives, and wave w turns their sum
// into the gradient.  Bound by the VALU: about 2,300 instructions per neighbour
// and point at twojmax 10, where the rows of every level and their derivatives
// took 9,700 and each wave its own geometry: 991 -> 219 us per 65,537 points.
template <int TJ>
__global__ __launch_bounds__(64 * kUiWaves, 2) void k_dedr(BinState bins, int Nx, int Ny, int Nz,
                                                           double rcut, int64_t pt_begin, int64_t n_pts,
                                                           const float2* __restrict__ y_in,
                                                           double* __restrict__ dLdR, int* __restrict__ err) {
    constexpr int NH = n_half(TJ);
    constexpr int NG = kUiWaves;
    __shared__ float4 cand[kMaxCand];
    __shared__ unsigned short nbr[kMaxNbr][kTile];
    __shared__ int nnbr[NG][kTile];
    __shared__ int scan_tmp[16];
    __shared__ float cgrad[kMaxCand][3];
    __shared__ float4 geo[NG][kTile];                 // a, b of the four neighbours
    __shared__ float part[NG][NG][5][kTile];          // [neighbour][wave]

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t tile = blockIdx.x;
    const int64_t idx = tile * kTile + lane;
    const bool valid = idx < n_pts;
    const TilePoint pt = tile_point(bins, Nx, Ny, Nz, pt_begin + tile * kTile,
                                    (int)min((int64_t)kTile, n_pts - tile * kTile), lane);
    const TileBoxes& boxes = pt.boxes;

    int n0;
    const int base = gather_candidates(bins, boxes, rcut, cand, kMaxCand, scan_tmp, &n0);
    if (base > kMaxCand && threadIdx.x == 0) atomicOr(err, kErrCand);
    const int ncand = base < kMaxCand ? base : kMaxCand;
    for (int c = threadIdx.x; c < ncand; c += blockDim.x) cgrad[c][0] = cgrad[c][1] = cgrad[c][2] = 0.f;
    __syncthreads();

    const PointFrame frame = point_frame(boxes, n0, pt.x, pt.y, pt.z);
    const float rcf = (float)rcut;
    const int nn = build_neighbour_lists_block<NG>(cand, ncand, frame, rcf, valid, lane, wave, nbr, nnbr, err);
    const int nmax = wave_max_int(nn);                // the same in every wave

    const float2* yt = y_in + tile * NH * kTile + lane;
    const PhaseFactors phase(rcut);
    // a loop per wave with the same count of barriers in each (nmax is the same in every
    // wave; the hardware counts the waves that have reached one, wherever in the code)
    static_for<0, NG>([&](auto gc) {
        constexpr int G = decltype(gc)::value;
        if (wave != G) return;
        constexpr int NACC = u_group_size(TJ, G) > 0 ? u_group_size(TJ, G) : 1;
        float W[NACC];
        dedr_weights<TJ, G, NACC>(yt, W);
        for (int s0 = 0; s0 < nmax; s0 += NG) {
            const int s = s0 + G;                     // the neighbour this wave forms and finishes
            const bool act = s < nn;
            const int c = act ? nbr[s][lane] : 0;
            const float4 q = cand[c];
            const float3 o = frame.at(c);
            const float dx = q.x - o.x, dy = q.y - o.y, dz = q.z - o.z;
            const float r2 = dx * dx + dy * dy + dz * dz;
            const bool on = act && r2 > kMinR2;       // an atom on the point has no derivative: left out
            const float inv = on ? inverse_distance(r2) : 1.f;
            const float r = on ? r2 * inv : 1.f;
            const float n[3] = {dx * inv, dy * inv, dz * inv};
            float sn, cs;
            sincosf(phase.angle(r), &sn, &cs);
            geo[G][lane] = on ? make_float4(cs, -n[2] * sn, -n[1] * sn, -n[0] * sn) : make_float4(1.f, 0.f, 0.f, 0.f);
            __syncthreads();
            const int cnt = min(NG, nmax - s0);
#pragma clang loop unroll(disable)
            for (int i = 0; i < cnt; ++i) {
                const float4 ab = geo[i][lane];
                float v[5];
                dedr_neighbour<TJ, G, NACC>(ab.x, ab.y, ab.z, ab.w, W, v);
#pragma unroll
                for (int k = 0; k < 5; ++k) part[i][G][k][lane] = v[k];
            }
            __syncthreads();                          // the parts are whole, geo no longer read
            if (on) {
                float v[5];
#pragma unroll
                for (int k = 0; k < 5; ++k) {
                    v[k] = part[G][0][k][lane];
#pragma unroll
                    for (int w = 1; w < NG; ++w) v[k] += part[G][w][k][lane];
                }
                const float x = phase.cutoff(r);
                const float fc = 0.5f * (cosf(x) + 1.f), dfc = -0.5f * phase.cutoff(sinf(x));
#pragma unroll
                for (int d = 0; d < 3; ++d) {
                    // theta' = n_d theta0 / r, n_i' = (delta_id - n_i n_d) / r
                    const float dth = phase.angle(n[d]);
                    const float dnx = ((d == 0 ? 1.f : 0.f) - n[0] * n[d]) * inv;
                    const float dny = ((d == 1 ? 1.f : 0.f) - n[1] * n[d]) * inv;
                    const float dnz = ((d == 2 ? 1.f : 0.f) - n[2] * n[d]) * inv;
                    const float dar = -sn * dth;
                    const float dai = -(dnz * sn + n[2] * cs * dth);
                    const float dbr = -(cs * dth * n[1] + sn * dny);
                    const float dbi = -(cs * dth * n[0] + sn * dnx);
                    const float gd = dar * v[1] + dai * v[2] + dbr * v[3] + dbi * v[4];
                    atomicAdd(&cgrad[c][d], fc * gd + dfc * n[d] * v[0]);
                }
            }
        }
    });
    __syncthreads();
    for (int c = threadIdx.x; c < ncand; c += blockDim.x) {
        const int atom = __float_as_int(cand[c].w);
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            const float v = cgrad[c][d];
            if (v != 0.f) atomicAdd(&dLdR[3 * atom + d], (double)v);
        }
    }
}

// ------------------------------------------------------------------ launch
__global__ void k_zero_f64(double* __restrict__ p, int64_t n) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0;
}

hipError_t launch_zero_f64(hipStream_t s, double* p, int64_t n) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_zero_f64, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

template <int TJ>
static hipError_t dedr_tj(hipStream_t s, const BinState& bins, const int N[3], double rcut, int64_t pt_begin,
                          int64_t n_pts, const float2* y, double* dLdR, int* err) {
    const int64_t n_tiles = (n_pts + kTile - 1) / kTile;
    if (n_tiles == 0) return hipSuccess;
    hipLaunchKernelGGL(k_dedr<TJ>, dim3((unsigned)n_tiles), dim3(64 * kUiWaves), 0, s, bins, N[0], N[1], N[2],
                       rcut, pt_begin, n_pts, y, dLdR, err);
    return hipGetLastError();
}

hipError_t launch_dedr(hipStream_t s, int twojmax, const BinState& bins, const int N[3], double rcut,
                       int64_t pt_begin, int64_t n_pts, const float2* y, double* dLdR, int* err) {
    switch (twojmax) {
    case 2: return dedr_tj<2>(s, bins, N, rcut, pt_begin, n_pts, y, dLdR, err);
    case 4: return dedr_tj<4>(s, bins, N, rcut, pt_begin, n_pts, y, dLdR, err);
    case 6: return dedr_tj<6>(s, bins, N, rcut, pt_begin, n_pts, y, dLdR, err);
    case 8: return dedr_tj<8>(s, bins, N, rcut, pt_begin, n_pts, y, dLdR, err);
    case 10: return dedr_tj<10>(s, bins, N, rcut, pt_begin, n_pts, y, dLdR, err);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace mala
