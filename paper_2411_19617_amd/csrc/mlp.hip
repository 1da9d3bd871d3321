// Per-point feed-forward network (Sec. 2.4, Eq. ffnn) on MFMA, with the LDOS
// reductions of Sec. 2.3 / 3.4 fused into the output epilogue.
//
// A block takes NP = 16*NT grid points at a time from its fixed, contiguous
// range (one block of 8 waves per CU).  One activation tile in LDS serves every layer: a wave keeps its
// share of a layer's output (unit tiles w, w + 8, ... against all point tiles,
// so every weight operand fetched from L2 feeds NT products) in registers, and
// after the barrier that ends the reading of the input the output is written
// over it.
//
// Epilogues:
//   LDOS       d = out_scale*y + out_shift stored as float32 [n][n_e]
//   DOS        d summed over points in FP64 into a per-block FP64 row
//              (fixed assignment: deterministic); optional row stride to run
//              on a strided subsample of the points
//   DOS_WINDOW DOS as above, plus per point the FP64 prefix sum of the fully
//              occupied part sum_{e<lo} tw_e d_e and the float32 LDOS values
//              of the energy window [lo, hi] around the estimated E_F
//   DENSITY    n(p) = sum_e w_e d_e(p) (FP64) with the solved Fermi weights;
//              runs only when the stored window did not cover E_F.
#include "mlp_core.h"

namespace mala {

template <int P, int MODE, int NT, int MT, int RS>
__global__ __launch_bounds__(kWaves * 64, waves_per_simd(MT)) void k_mlp(MlpArgs a, const float* __restrict__ B, int64_t n_pts,
                                                        int row_stride, MlpOut o) {
    constexpr int NP = 16 * NT, OT = out_unit_tiles(MT);      // output tiles of a wave, at most
    constexpr bool WINDOW = MODE == kModeDosWindow, DENSITY = MODE == kModeDensity;
    constexpr bool DOS = MODE == kModeDos || WINDOW;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ double s_w[WINDOW || DENSITY ? kMlpMaxOut : 1];
    __shared__ unsigned s_max[3][NP];          // largest input of each layer per point (FP32 weights)

    const int lane0 = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int lo = 0, W = 0;
    if constexpr (DENSITY) {
        if (o.res->status != 0 || o.win->covered) return;      // nothing to recompute
    }
    if constexpr (WINDOW) {
        lo = o.win->lo;
        W = o.win->valid ? o.win->hi - o.win->lo + 1 : 0;
    }
    const int in_tiles = a.in_pad / 16;
    const ActTile<P, NT, RS> act{reinterpret_cast<unsigned short*>(smem)};

    if constexpr (WINDOW || DENSITY) {
        // weights of the per-point energy sum: density -> Fermi weights w_e,
        // window prefix -> trapezoid weight de (de/2 at e = 0) below lo
        for (int e = threadIdx.x; e < kMlpMaxOut; e += blockDim.x) {
            double we = 0.0;
            if (DENSITY) we = e < a.n_out ? o.fermi_w[e] : 0.0;
            else we = (e < lo) ? (e == 0 ? 0.5 * o.de : o.de) : 0.0;
            s_w[e] = we;
        }
    }

    const int64_t n_it = (n_pts + NP - 1) / NP;
    const int nb = gridDim.x;
    const int64_t it_begin = n_it * blockIdx.x / nb, it_end = n_it * (blockIdx.x + 1) / nb;
    const int n_in = a.n_in;
    auto rows_of = [&](int64_t it) {
        const int64_t left = n_pts - it * NP;
        return (int)(left < NP ? left : NP);
    };

    // DOS column sums: every lane keeps the FP64 sums of its 4 OT energies over
    // all of its points and iterations; the 16 point lanes are combined once
    // at the end (fixed order)
    double dacc[OT][4] = {};
    const float mu[2] = {lane0 < n_in ? a.in_mean[lane0] : 0.f, lane0 + 64 < n_in ? a.in_mean[lane0 + 64] : 0.f};
    const float rstd[2] = {lane0 < n_in ? a.in_rstd[lane0] : 0.f, lane0 + 64 < n_in ? a.in_rstd[lane0 + 64] : 0.f};
    const bool fast_act = a.slope > 0.f && a.slope <= 1.f;
    // the stored LDOS goes out through the activation tile, SP points at a time
    constexpr int SP = ActTile<P, NT, RS>::kBytes / (sizeof(float) * 16 * kWaves * OT) >= NP ? NP : 16;
    const bool wide = (reinterpret_cast<uintptr_t>(o.ldos) & 15) == 0;      // a tile's rows start on 16 bytes then

    for (int64_t it = it_begin; it < it_end; ++it) {
        const int64_t p0 = it * NP;
        const int rows = rows_of(it);
        // the empty asm makes the lane loop-variant: biases, first weights and
        // addresses are formed where they are used and not held across the loop
        int lane = lane0;
        asm volatile("" : "+v"(lane));
        const int j = lane & 15, g = lane >> 4;
        stage_rows(B, p0, rows, row_stride, n_in, a.in_pad, mu, rstd, act, s_max[0], wave, lane);
        if constexpr (P == 2)
            for (int i = threadIdx.x; i < NP; i += blockDim.x) s_max[1][i] = s_max[2][i] = 0;
        __syncthreads();
        Acc<NT, MT> acc;
#pragma clang loop unroll(disable)
        for (int l = 0; l < 2; ++l) {
            const float* bias = l == 0 ? a.b1 : a.b2;
            const Share<NT> sh(l == 0 ? a.h1_tiles : a.h2_tiles, wave, MT > 1);
            f4 b0{};                                 // one unit tile per wave: its bias comes during the products
            if (MT == 1 && sh.cnt > 0) b0 = bias4(bias, 16 * wave + 4 * g);
            layer_mm<P, NT, MT, RS, (MT > 1)>(l == 0 ? a.W1 : a.W2, l == 0 ? in_tiles : a.h1_tiles, sh, act, wave, lane, acc);
            float c[NT];
#pragma unroll
            for (int n = 0; n < NT; ++n) c[n] = unscale<P>(s_max[l], 16 * n + j, a.wexp[l]);
            auto out = [&](auto fast) {
                layer_out<P, NT, MT, RS>(acc, sh, act, s_max[l + 1], wave, lane, [&](auto slot, int mt, int n, f4& v) {
                    const f4 b = MT == 1 ? b0 : bias4(bias, 16 * mt + 4 * g);
                    float cn;
                    if constexpr (decltype(slot)::value < MT) cn = c[n];
                    else cn = unscale<P>(s_max[l], 16 * n + j, a.wexp[l]);
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        v[r] = leaky<decltype(fast)::value>(P == 2 ? fmaf(v[r], cn, b[r]) : v[r] + b[r], a.slope);
                });
            };
            if (fast_act) out(std::true_type{});
            else out(std::false_type{});
        }
        Acc<NT, OT> acc3;
        f4 out0[3] = {};
        {
            const Share<NT> sh(a.out_tiles, wave, false);
            if (MT == 1 && sh.cnt > 0) {
                const int e0 = 16 * wave + 4 * g;
                out0[0] = bias4(a.b3, e0);
                out0[1] = bias4(a.out_scale, e0);
                out0[2] = bias4(a.out_shift, e0);
            }
            layer_mm<P, NT, OT, RS, false>(a.W3, a.h2_tiles, sh, act, wave, lane, acc3);
        }

        // ---- epilogue
        float c3[NT];
#pragma unroll
        for (int n = 0; n < NT; ++n) c3[n] = unscale<P>(s_max[2], 16 * n + j, a.wexp[2]);
        double part[NT];
#pragma unroll
        for (int n = 0; n < NT; ++n) part[n] = 0.0;
        static_for<0, OT>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            const int ot = wave + kWaves * i, e0 = 16 * ot + 4 * g;
            if (ot >= a.out_tiles) return;
            // every mode forms the same float LDOS value d = s y + c (affine map
            // in FP64, rounded once), so that the stored LDOS, the DOS, the
            // window, its prefix and a recomputed density all use identical numbers
            // (bias and scaler rows are zero-padded: energies past n_out give zero)
            const f4 b = MT == 1 ? out0[0] : bias4(a.b3, e0), scf = MT == 1 ? out0[1] : bias4(a.out_scale, e0),
                     shf = MT == 1 ? out0[2] : bias4(a.out_shift, e0);
            float df[4][NT];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double sc = (double)scf[r], sh = (double)shf[r];
#pragma unroll
                for (int n = 0; n < NT; ++n) {
                    float yv = P == 2 ? fmaf(acc3.t[i][n][r], c3[n], b[r]) : acc3.t[i][n][r] + b[r];
                    if (a.out_act) yv = leaky<false>(yv, a.slope);
                    df[r][n] = (float)(sc * (double)yv + sh);
                }
            }
            if constexpr (MODE == kModeLdos) {
                static_for<0, NT>([&](auto nc) {
                    constexpr int n = decltype(nc)::value;
                    acc3.t[i][n] = f4{df[0][n], df[1][n], df[2][n], df[3][n]};
                });
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int e = e0 + r;
                    double dsum = 0.0;
#pragma unroll
                    for (int n = 0; n < NT; ++n) {
                        const bool pv = 16 * n + j < rows;
                        const double d = (double)df[r][n];
                        if constexpr (WINDOW || DENSITY) part[n] += s_w[e] * d;
                        if constexpr (DOS) dsum += pv ? d : 0.0;
                        if constexpr (WINDOW)
                            if (pv && e >= lo && e < lo + W) o.window[(p0 + 16 * n + j) * W + (e - lo)] = df[r][n];
                    }
                    if constexpr (DOS) dacc[i][r] += dsum;
                }
            }
            __builtin_amdgcn_sched_barrier(0);       // one output tile at a time: fewer values live
        });
        if constexpr (MODE == kModeLdos) {
            // [point][energy] rows in LDS, then one contiguous run of memory: a lane's
            // own values are 16 bytes of a row, each of a wave's 16 points in another
            // row; stored from there they took 80 of the BF16 kernel's 380 us per
            // 262,147 points, this way 16
            float* out = reinterpret_cast<float*>(smem);
            static_for<0, NP / SP>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                __syncthreads();
                static_for<0, OT>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    const int e0 = 16 * (wave + kWaves * i) + 4 * g;
                    static_for<k * SP / 16, (k + 1) * SP / 16>([&](auto nc) {
                        constexpr int n = decltype(nc)::value;
                        float* d = out + (16 * n - k * SP + j) * a.n_out + e0;
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (e0 + r < a.n_out) d[r] = acc3.t[i][n][r];
                    });
                });
                __syncthreads();
                const int nf = max(0, min(SP, rows - k * SP)) * a.n_out, n4 = wide ? nf >> 2 : 0;
                float* g_out = o.ldos + (p0 + k * SP) * a.n_out;
                for (int q = threadIdx.x; q < n4; q += kWaves * 64)
                    reinterpret_cast<float4*>(g_out)[q] = reinterpret_cast<const float4*>(out)[q];
                for (int q = 4 * n4 + threadIdx.x; q < nf; q += kWaves * 64) g_out[q] = out[q];
            });
        }
        if constexpr (MODE == kModeLdos && P == 2) {
            // (the reductions work on descriptors of the library's own, which are finite)
            unsigned long long again = infinite_points(s_max, 3, rows, lane);
            if (again) {
                PlainPoint& q = *reinterpret_cast<PlainPoint*>(smem);
                __syncthreads();                     // the rows in LDS are out
                for (; again; again &= again - 1) {
                    const int64_t p = p0 + __ffsll(again) - 1;
                    const int t = plain_thread();
                    const MlpPlain& w = *a.plain;
                    plain_hidden(w, B + p * row_stride * w.n[0], q, t);
                    plain_layer(w, 2, q.z2, t, [&](int e, float y) {
                        if (w.out_act) y = leaky<false>(y, w.slope);
                        o.ldos[p * w.n[3] + e] = (float)((double)w.out_scale[e] * (double)y + (double)w.out_shift[e]);
                    });
                    __syncthreads();
                }
            }
        }
        if constexpr (WINDOW || DENSITY) {
            double* s_part = reinterpret_cast<double*>(smem);      // [wave][point], over the activation tile
            __syncthreads();
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                double v = part[n];
                v += __shfl_xor(v, 16, 64);
                v += __shfl_xor(v, 32, 64);
                if (g == 0) s_part[wave * NP + 16 * n + j] = v;
            }
            __syncthreads();
            if ((int)threadIdx.x < NP && (int)threadIdx.x < rows) {
                double v = 0.0;
                for (int w = 0; w < kWaves; ++w) v += s_part[w * NP + threadIdx.x];
                const int64_t q = p0 + threadIdx.x;
                if constexpr (DENSITY) o.density[q] = v;
                else o.prefix[q] = v;
            }
        }
        // every wave has read the activation tile (and the point sums, which the
        // next tile's waves write four barriers later)
        __syncthreads();
    }
    if constexpr (DOS) {
        __syncthreads();
        const int j = lane0 & 15, g = lane0 >> 4;
        double* s_dos = reinterpret_cast<double*>(smem);       // the activation tile is free
        for (int e = threadIdx.x; e < kMlpMaxOut; e += blockDim.x) s_dos[e] = 0.0;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < OT; ++i) {
            const int ot = wave + kWaves * i;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                double v = dacc[i][r];
                v += __shfl_xor(v, 1, 16);
                v += __shfl_xor(v, 2, 16);
                v += __shfl_xor(v, 4, 16);
                v += __shfl_xor(v, 8, 16);
                const int e = 16 * ot + 4 * g + r;
                if (j == 0 && ot < a.out_tiles && e < a.n_out) s_dos[e] = v;
            }
        }
        __syncthreads();
        for (int e = threadIdx.x; e < kMlpMaxOut; e += blockDim.x)
            o.partials[(size_t)blockIdx.x * kMlpMaxOut + e] = s_dos[e];
    }
}

template <int P, int MODE, int NT, int MT, int RS>
static hipError_t launch_pmn(hipStream_t s, const MlpArgs& a, const float* B, int64_t n_pts, int row_stride,
                             int n_blocks, const MlpOut& o) {
    constexpr size_t lds = ActTile<P, NT, RS>::kBytes;
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_mlp<P, MODE, NT, MT, RS>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL((k_mlp<P, MODE, NT, MT, RS>), dim3(n_blocks), dim3(kWaves * 64), lds, s, a, B, n_pts, row_stride, o);
    return hipGetLastError();
}

// Point tiles per block: 64 points, or 96 for BF16 (one plane of activations)
// where no layer has more than 400 units; larger tiles read fewer weights per
// point but hold so many accumulators that the epilogues spill (96 points of FP32
// weights: the same 1.4 ms per 729,000 points, 2% more with the DOS epilogue;
// 128 of BF16: 0.38 ms per 262,147 points against 0.28).  32 points where that
// shortens the busiest block, counted as tiles times (point tiles + 1.5): a
// tile's fixed part (staging, barriers, weight latency) costs about as much as
// 1.5 point tiles, so few points are spread over more blocks.
int mlp_point_tiles(const MlpArgs& a, int64_t n_pts, int n_blocks) {
    auto cost = [&](int NT) {
        const int64_t tiles = (n_pts + 16 * NT - 1) / (16 * NT);
        return (double)((tiles + n_blocks - 1) / n_blocks) * (NT + 1.5);
    };
    int best = cost(4) <= cost(2) ? 4 : 2;
    if (a.precision == 1 && !mlp_rows_small(a) && mlp_rows_wide(a) && cost(6) <= cost(best)) best = 6;
    return best;
}

template <int P, int MODE>
static hipError_t launch_pm(hipStream_t s, const MlpArgs& a, const float* B, int64_t n_pts, int row_stride,
                            int n_blocks, const MlpOut& o) {
    const int nt = mlp_point_tiles(a, n_pts, n_blocks);
    if (mlp_rows_small(a)) {
        if (nt == 4) return launch_pmn<P, MODE, 4, 1, kRowSmall>(s, a, B, n_pts, row_stride, n_blocks, o);
        return launch_pmn<P, MODE, 2, 1, kRowSmall>(s, a, B, n_pts, row_stride, n_blocks, o);
    }
    if (mlp_rows_wide(a)) {
        if constexpr (P == 1)
            if (nt == 6) return launch_pmn<P, MODE, 6, 3, kRowWide>(s, a, B, n_pts, row_stride, n_blocks, o);
        if (nt == 4) return launch_pmn<P, MODE, 4, 3, kRowWide>(s, a, B, n_pts, row_stride, n_blocks, o);
        return launch_pmn<P, MODE, 2, 3, kRowWide>(s, a, B, n_pts, row_stride, n_blocks, o);
    }
    if (nt == 4) return launch_pmn<P, MODE, 4, 4, kRowMax>(s, a, B, n_pts, row_stride, n_blocks, o);
    return launch_pmn<P, MODE, 2, 4, kRowMax>(s, a, B, n_pts, row_stride, n_blocks, o);
}

// One block per CU, or per_cu, fewer when there are not that many 32-point tiles.
int mlp_blocks(int64_t n_pts, int per_cu) {
    const int64_t it = (n_pts + 31) / 32, most = (int64_t)kMlpBlocks * per_cu;
    return (int)(it < most ? (it > 0 ? it : 1) : most);
}

// Weights W [fout][fin] (or, transposed, the layer with the widths swapped) as A
// operands in lane order, [unit tile][step][plane][lane][8]: lane l holds row
// 16 mt + l % 16 and, in step s, units 32 s + 8 (l / 16) + 0..7 (in the last step
// of an odd tile count 16 (kt - 1) + 4 (l / 16) + 0..3 and four zeros).  One thread
// per element.
__global__ __launch_bounds__(256) void k_pack_weights(const float* __restrict__ W, int fout, int fin, int transposed,
                                                      int mtiles, int kt, int planes, float scale,
                                                      unsigned short* __restrict__ out) {
    const int steps = w_steps(kt);
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)mtiles * steps * planes * 512) return;
    const int q = (int)(i & 7), lane = (int)(i >> 3) & 63, pl = (int)((i >> 9) % planes);
    const int st = (int)((i >> 9) / planes % steps), mt = (int)((i >> 9) / planes / steps);
    const int per = 32 * st + 32 <= 16 * kt ? 8 : 4;
    const int row = 16 * mt + (lane & 15), k = 32 * st + per * (lane >> 4) + q;
    const int rows = transposed ? fin : fout, cols = transposed ? fout : fin;
    float v = 0.f;
    if (q < per && row < rows && k < cols) v = transposed ? W[(size_t)k * fin + row] : W[(size_t)row * fin + k];
    unsigned short h;
    if (planes == 1) {                                  // BF16, round to nearest even
        const unsigned x = (unsigned)__float_as_int(v);
        h = (unsigned short)((x + 0x7FFFu + ((x >> 16) & 1u)) >> 16);
    } else {                                            // v scale = hi + lo / 2^kLoBits
        const float x = v * scale;
        const _Float16 hi = (_Float16)x;
        h = bits_as<unsigned short>(pl == 0 ? hi : (_Float16)((x - (float)hi) * (float)(1 << kLoBits)));
    }
    out[i] = h;
}

size_t packed_weight_elems(int mtiles, int kt, int planes) { return (size_t)mtiles * w_steps(kt) * planes * 512; }

hipError_t launch_pack_weights(hipStream_t s, const float* W, int fout, int fin, bool transposed, int mtiles, int kt,
                               int planes, int wexp, void* out) {
    const size_t n = packed_weight_elems(mtiles, kt, planes);
    hipLaunchKernelGGL(k_pack_weights, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, W, fout, fin,
                       transposed ? 1 : 0, mtiles, kt, planes, ldexpf(1.f, wexp), static_cast<unsigned short*>(out));
    return hipGetLastError();
}

hipError_t launch_mlp(hipStream_t s, const MlpArgs& a, int mode, const float* B, int64_t n_pts, int row_stride,
                      int n_blocks, const MlpOut& o) {
    if (n_pts <= 0 || n_blocks <= 0) return hipSuccess;
#define MALA_MLP_CASE(P, M) return launch_pm<P, M>(s, a, B, n_pts, row_stride, n_blocks, o)
    if (a.precision == 0) {
        if (mode == kModeLdos) MALA_MLP_CASE(2, kModeLdos);
        if (mode == kModeDos) MALA_MLP_CASE(2, kModeDos);
        if (mode == kModeDosWindow) MALA_MLP_CASE(2, kModeDosWindow);
        if (mode == kModeDensity) MALA_MLP_CASE(2, kModeDensity);
    } else {
        if (mode == kModeLdos) MALA_MLP_CASE(1, kModeLdos);
        if (mode == kModeDos) MALA_MLP_CASE(1, kModeDos);
        if (mode == kModeDosWindow) MALA_MLP_CASE(1, kModeDosWindow);
        if (mode == kModeDensity) MALA_MLP_CASE(1, kModeDensity);
    }
#undef MALA_MLP_CASE
    return hipErrorInvalidValue;
}

}  // namespace mala
