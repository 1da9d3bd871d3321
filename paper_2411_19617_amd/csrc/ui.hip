// Expansion coefficients of the grid bispectrum descriptors on gfx950 (Sec.
// 3.2.2: Eqs. ionicdensity, SNAPExpansion), per tile of 64 consecutive grid
// points (one point per lane): neighbour gather and u^J = I + sum_k f_c(r_k)
// U^J(g_k) in the separated form of u_basis.h: a neighbour adds
// a^k1 b^k2 phi_n(|a|^2) to one sum per (k1, k2, n), a multiply-add each, and
// the levels' elements are combined from the sums once per point.  The sums
// are split over the waves of the block by k1, so that each wave keeps its
// share in registers over the whole neighbour loop; the neighbours' (a, b, f_c)
// are formed once, by the waves in turn, and passed through LDS.  Only rows
// ma <= J/2 are written; the rest follow from
// u_{J-ma,J-mb} = (-1)^(ma-mb) conj(u_{ma,mb}).
//
// Bound by the VALU: about 1,000 instructions per neighbour and point at
// twojmax 10 where a recursion over the levels takes 2,600.  Against the
// recursion with wave 0 listing the neighbours: twojmax 10, 200,003 points of a
// liquid, 445 -> 240 us; twojmax 8, 8,000 points of a 32-atom cell (125 blocks,
// where the list's serial chain counts), 59 -> 32 us.
#include "snap_core.h"
#include "tile_gather.h"
#include "u_basis.h"

namespace mala {

// Add one neighbour to the group's sums.
template <int TJ, int G, int NACC>
__device__ __forceinline__ void ui_neighbour(float ar, float ai, float br, float bi, float fc, float (&acc)[NACC]) {
    // phi_n of the bases the group uses: phi_0 = 1, phi_n = 2 x phi_{n-1} - phi_{n-2}
    // (from 2 t - 1 as |a|^2 - |b|^2, whose rounding does not favour one end of
    // [0, 1]: with t = |a|^2 the sums were 8% further from 64 bits)
    const float x0 = fmaf(ai, ai, fmaf(ar, ar, -fmaf(br, br, bi * bi)));
    float phi[kUBases][kUMaxN + 1];
    static_for<0, kUBases>([&](auto bc) {
        constexpr int B = decltype(bc)::value, NM = u_basis_nmax(TJ, G, B);
        if constexpr (NM >= 1) {
            if constexpr (B == 0) phi[B][1] = x0;
            else phi[B][1] = fmaf(x0, (float)(0.5 / ub_half(B)), (float)((0.5 - ub_mid(B)) / ub_half(B)));
            const float x2 = 2.f * phi[B][1];
            static_for<2, NM + 1>([&](auto nc) {
                constexpr int n = decltype(nc)::value;
                if constexpr (n == 2) phi[B][2] = fmaf(x2, phi[B][1], -1.f);
                else phi[B][n] = fmaf(x2, phi[B][n - 1], -phi[B][n - 2]);
            });
        }
    });
    // f_c a^k1 of the group's k1
    float pr[TJ + 1], pi[TJ + 1];
    pr[1] = ar;
    pi[1] = ai;
    static_for<2, TJ + 1>([&](auto kc) {
        constexpr int k = decltype(kc)::value, h = k / 2;
        if constexpr (u_power_needed(TJ, G, k)) {
            if constexpr (2 * h == k) {
                pr[k] = fmaf(pr[h], pr[h], -pi[h] * pi[h]);
                pi[k] = 2.f * pr[h] * pi[h];
            } else {
                pr[k] = fmaf(pr[h], pr[h + 1], -pi[h] * pi[h + 1]);
                pi[k] = fmaf(pr[h], pi[h + 1], pi[h] * pr[h + 1]);
            }
        }
    });
    static_for<1, TJ + 1>([&](auto kc) {
        constexpr int k = decltype(kc)::value;
        if constexpr (u_group_of(TJ, k) == G) {
            pr[k] *= fc;
            pi[k] *= fc;
        }
    });
    pr[0] = fc;
    float qr = 1.f, qi = 0.f;                 // b^k2
    static_for<0, u_group_k2max(TJ, G) + 1>([&](auto k2c) {
        constexpr int k2 = decltype(k2c)::value;
        if constexpr (k2 == 1) {
            qr = br;
            qi = bi;
        } else if constexpr (k2 > 1) {
            const float r = fmaf(qr, br, -qi * bi);
            qi = fmaf(qr, bi, qi * br);
            qr = r;
        }
        static_for<0, TJ + 1 - k2>([&](auto k1c) {
            constexpr int k1 = decltype(k1c)::value;
            if constexpr (u_group_of(TJ, k1) == G) {
                constexpr int NP = u_parts(k1, k2), NN = u_ncount(TJ, k1, k2), S = u_slot(TJ, G, k1, k2), B = u_basis(k1, k2);
                if constexpr (NP == 4) {      // rr, ii, ri, ir
                    const float x[4] = {pr[k1], pi[k1], pr[k1], pi[k1]}, y[4] = {qr, qi, qi, qr};
                    static_for<0, 4>([&](auto pc) {
                        constexpr int p = decltype(pc)::value;
                        if constexpr (NN == 1) {
                            acc[S + p] = fmaf(x[p], y[p], acc[S + p]);
                        } else {
                            const float v = x[p] * y[p];
                            acc[S + p] += v;
                            static_for<1, NN>([&](auto nc) {
                                constexpr int n = decltype(nc)::value;
                                acc[S + 4 * n + p] = fmaf(v, phi[B][n], acc[S + 4 * n + p]);
                            });
                        }
                    });
                } else {                      // an axis: f_c a^k1, or f_c b^k2
                    float v[NP];
                    if constexpr (k2 == 0) {
                        v[0] = pr[k1];
                        if constexpr (NP == 2) v[1] = pi[k1];
                    } else {
                        v[0] = pr[0] * qr;
                        v[1] = pr[0] * qi;
                    }
                    static_for<0, NP>([&](auto pc) {
                        constexpr int p = decltype(pc)::value;
                        acc[S + p] += v[p];
                        static_for<1, NN>([&](auto nc) {
                            constexpr int n = decltype(nc)::value;
                            acc[S + NP * n + p] = fmaf(v[p], phi[B][n], acc[S + NP * n + p]);
                        });
                    });
                }
            }
        });
    });
}

// Neighbours whose (a, b, f_c) are in LDS at once (two sets: one is formed
// while the other is summed).
constexpr int kUiChunk = 8;

// Bound: FP32 VALU.  Per neighbour about 1,000 instructions over the four waves
// at twojmax 10 (506 of them the multiply-adds into the sums) against 2,600
// for the recursion over the rows of each level that this replaces.
template <int TJ>
__global__ __launch_bounds__(64 * kUiWaves, 2) void k_ui(BinState bins, int Nx, int Ny, int Nz,
                                                          double rcut, int64_t pt_begin, int64_t n_pts,
                                                          float2* __restrict__ u_out,
                                                          int* __restrict__ err) {
    constexpr int NG = kUiWaves;
    constexpr int NH = n_half(TJ);
    __shared__ float4 cand[kMaxCand];
    __shared__ unsigned short nbr[kMaxNbr][kTile];
    __shared__ int nnbr[NG][kTile];
    __shared__ int scan_tmp[16];
    __shared__ float4 geo_ab[2][kUiChunk][kTile];
    __shared__ float geo_fc[2][kUiChunk][kTile];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t tile = blockIdx.x;
    const int64_t idx = tile * kTile + lane;
    const bool valid = idx < n_pts;
    const TilePoint pt = tile_point(bins, Nx, Ny, Nz, pt_begin + tile * kTile,
                                    (int)min((int64_t)kTile, n_pts - tile * kTile), lane);
    const TileBoxes& boxes = pt.boxes;

    // ---- candidate atom images within rcut of the boxes, in a fixed order
    int n0;
    const int base = gather_candidates(bins, boxes, rcut, cand, kMaxCand, scan_tmp, &n0);
    if (base > kMaxCand && threadIdx.x == 0) atomicOr(err, kErrCand);
    const int ncand = base < kMaxCand ? base : kMaxCand;
    __syncthreads();

    // ---- per-point neighbour lists, in candidate order, by all waves
    const PointFrame frame = point_frame(boxes, n0, pt.x, pt.y, pt.z);
    const float rcf = (float)rcut;
    const int my_n = build_neighbour_lists_block<NG>(cand, ncand, frame, rcf, valid, lane, wave, nbr, nnbr, err);
    const int n_iter = wave_max_int(my_n);            // the same in every wave

    // ---- expansion coefficients, this wave's group of sums
    const PhaseFactors phase(rcut);
    auto form = [&](int s0) {                         // this wave's share of the chunk from s0
#pragma unroll
        for (int q = 0; q < kUiChunk / NG; ++q) {
            const int i = wave * (kUiChunk / NG) + q, s = s0 + i;
            if (s >= n_iter) continue;
            float ar = 1.f, ai = 0.f, br = 0.f, bi = 0.f, fc = 0.f;
            if (s < my_n) {
                const int c = nbr[s][lane];
                const float4 v = cand[c];
                const float3 o = frame.at(c);
                const float dx = v.x - o.x, dy = v.y - o.y, dz = v.z - o.z;
                const float r2 = dx * dx + dy * dy + dz * dz;
                const float inv = r2 > kMinR2 ? inverse_distance(r2) : 0.f;      // an atom on the point: r = 0
                const float r = r2 * inv;
                float sn, cs;
                sincosf(phase.angle(r), &sn, &cs);
                ar = cs;
                ai = -dz * inv * sn;
                br = -dy * inv * sn;
                bi = -dx * inv * sn;
                fc = 0.5f * (cosf(phase.cutoff(r)) + 1.f);
            }
            geo_ab[(s0 / kUiChunk) & 1][i][lane] = make_float4(ar, ai, br, bi);
            geo_fc[(s0 / kUiChunk) & 1][i][lane] = fc;
        }
    };
    if (n_iter > 0) form(0);
    // a loop per wave, each with code of its own: its barriers are met by every wave
    // because n_iter is the same in all of them (the hardware counts the waves that
    // have reached a barrier, wherever in the code)
    static_for<0, NG>([&](auto gc) {
        constexpr int G = decltype(gc)::value;
        if (wave != G) return;
        constexpr int NACC = u_group_size(TJ, G) > 0 ? u_group_size(TJ, G) : 1;
        float acc[NACC];
        static_for<0, NACC>([&](auto ec) { acc[decltype(ec)::value] = 0.f; });
        for (int s0 = 0; s0 < n_iter; s0 += kUiChunk) {
            __syncthreads();                          // the chunk is whole, the other set no longer read
            if (s0 + kUiChunk < n_iter) form(s0 + kUiChunk);
            const int cnt = min(kUiChunk, n_iter - s0), set = (s0 / kUiChunk) & 1;
#pragma clang loop unroll(disable)
            for (int i = 0; i < cnt; ++i) {
                const float4 ab = geo_ab[set][i][lane];
                ui_neighbour<TJ, G, NACC>(ab.x, ab.y, ab.z, ab.w, geo_fc[set][i][lane], acc);
            }
        }
        // elements of the group's |k1|: the combination of their sums, the self
        // term (the identity), write-out
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
                        float re = ma == mb ? 1.f : 0.f, im = 0.f;
                        static_for<0, (J - K1 - K2) / 2 + 1>([&](auto nc) {
                            constexpr int n = decltype(nc)::value;
                            constexpr float c = (float)cf.c[n];
                            constexpr int o = S + NP * n;
                            if constexpr (NP == 4) {      // rr, ii, ri, ir
                                re = fmaf(c, bneg ? acc[o] + acc[o + 1] : acc[o] - acc[o + 1], re);
                                im = fmaf(c, bneg ? acc[o + 3] - acc[o + 2] : acc[o + 2] + acc[o + 3], im);
                            } else {
                                re = fmaf(c, acc[o], re);
                                if constexpr (NP == 2) im = fmaf(c, acc[o + 1], im);
                            }
                        });
                        constexpr int e = half_off(J) + ma * (J + 1) + mb;
                        u_out[(tile * NH + e) * kTile + lane] = make_float2(re, cj ? -im : im);
                    }
                });
            });
        });
    });
}

template <int TJ>
static hipError_t ui_tj(hipStream_t s, const BinState& bins, const int N[3], double rcut, int64_t pt_begin,
                        int64_t n_pts, float2* u_scratch, int* err_flag) {
    const int64_t n_tiles = (n_pts + kTile - 1) / kTile;
    if (n_tiles == 0) return hipSuccess;
    hipLaunchKernelGGL(k_ui<TJ>, dim3((unsigned)n_tiles), dim3(64 * kUiWaves), 0, s, bins, N[0], N[1],
                       N[2], rcut, pt_begin, n_pts, u_scratch, err_flag);
    return hipGetLastError();
}

hipError_t launch_ui(hipStream_t s, int twojmax, const BinState& bins, const int N[3], double rcut,
                     int64_t pt_begin, int64_t n_pts, float2* u_scratch, int* err_flag) {
    switch (twojmax) {
    case 2: return ui_tj<2>(s, bins, N, rcut, pt_begin, n_pts, u_scratch, err_flag);
    case 4: return ui_tj<4>(s, bins, N, rcut, pt_begin, n_pts, u_scratch, err_flag);
    case 6: return ui_tj<6>(s, bins, N, rcut, pt_begin, n_pts, u_scratch, err_flag);
    case 8: return ui_tj<8>(s, bins, N, rcut, pt_begin, n_pts, u_scratch, err_flag);
    case 10: return ui_tj<10>(s, bins, N, rcut, pt_begin, n_pts, u_scratch, err_flag);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace mala
