// Vector-Jacobian product of the per-point network: the network factor of
// the force expression (Eq. forcesmala).  For every grid point p and a given
// vector v(p) over the energies, g(p) = (dd(p)/dB(p))^T v(p), where
// d = s .* sigma(W3 sigma(W2 sigma(W1 x + b1) + b2) + b3) + c and
// x = (B - mean) / std (sigma on the output layer only with output
// activation).  Backpropagation, with sigma'(z) = 1 for z > 0 and slope
// otherwise:
//   delta3 = s .* v .* sigma'(z3),  delta2 = (W3^T delta3) .* sigma'(z2),
//   delta1 = (W2^T delta2) .* sigma'(z1),  g = (W1^T delta1) ./ std.
//
// Six MFMA layers over one activation tile in LDS, as in the network kernel:
// the forward layers, then the same over the transposed weights.  No
// activation is kept for the way back: only the signs of the two hidden layers
// matter there, and a backward layer's output units belong to the same lane as
// the forward layer's, so each lane keeps them as bits in registers.  FP32
// weights only (two FP16 planes).
#include "mlp_core.h"

namespace mala {

template <int NT, int MT, int RS>
__global__ __launch_bounds__(kWaves * 64, waves_per_simd(MT)) void k_mlp_vjp(MlpArgs a, const float* __restrict__ B,
                                                            const float* __restrict__ v, int64_t n_pts,
                                                            float* __restrict__ g_out) {
    constexpr int NP = 16 * NT;
    static_assert(NT * 4 <= 32, "one mask word per unit tile");
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ unsigned s_max[6][NP];        // largest input of each layer per point
    const int lane0 = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n_in = a.n_in, n_out = a.n_out, in_tiles = a.in_pad / 16;
    const float slope = a.slope;
    const ActTile<2, NT, RS> act{reinterpret_cast<unsigned short*>(smem)};

    const int64_t n_it = (n_pts + NP - 1) / NP;
    const int nb = gridDim.x;
    const int64_t it_begin = n_it * blockIdx.x / nb, it_end = n_it * (blockIdx.x + 1) / nb;
    auto rows_of = [&](int64_t it) {
        const int64_t left = n_pts - it * NP;
        return (int)(left < NP ? left : NP);
    };
    const float mu[2] = {lane0 < n_in ? a.in_mean[lane0] : 0.f, lane0 + 64 < n_in ? a.in_mean[lane0 + 64] : 0.f};
    const float rstd[2] = {lane0 < n_in ? a.in_rstd[lane0] : 0.f, lane0 + 64 < n_in ? a.in_rstd[lane0 + 64] : 0.f};

    for (int64_t it = it_begin; it < it_end; ++it) {
        const int64_t p0 = it * NP;
        const int rows = rows_of(it);
        int lane = lane0;                      // loop-variant, as in the network kernel
        asm volatile("" : "+v"(lane));
        const int j = lane & 15, g = lane >> 4;
        stage_rows(B, p0, rows, 1, n_in, a.in_pad, mu, rstd, act, s_max[0], wave, lane);
        for (int i = threadIdx.x; i < 5 * NP; i += blockDim.x) s_max[1][i] = 0;
        __syncthreads();
        Acc<NT, MT> acc;
        unsigned mask[2][MT + 1];              // sigma' of the two hidden layers: bit 4 n + r of word m; the item's in the last
        // forward: the hidden layers, their signs kept
        static_for<0, 2>([&](auto lc) {
            constexpr int l = decltype(lc)::value;
            const float* bias = l == 0 ? a.b1 : a.b2;
            const Share<NT> sh(l == 0 ? a.h1_tiles : a.h2_tiles, wave, MT > 1);
            f4 b0{};                           // one unit tile per wave: its bias comes during the products
            if (MT == 1 && sh.cnt > 0) b0 = bias4(bias, 16 * wave + 4 * g);
            layer_mm<2, NT, MT, RS, (MT > 1)>(l == 0 ? a.W1 : a.W2, l == 0 ? in_tiles : a.h1_tiles, sh, act, wave, lane, acc);
            float c[NT];
#pragma unroll
            for (int n = 0; n < NT; ++n) c[n] = unscale<2>(s_max[l], 16 * n + j, a.wexp[l]);
#pragma unroll
            for (int m = 0; m <= MT; ++m) mask[l][m] = 0;
            layer_out<2, NT, MT, RS>(acc, sh, act, s_max[l + 1], wave, lane, [&](auto slotc, int mt, int n, f4& z) {
                constexpr int slot = decltype(slotc)::value;
                const f4 b = MT == 1 ? b0 : bias4(bias, 16 * mt + 4 * g);
                float cn;
                if constexpr (slot < MT) cn = c[n];
                else cn = unscale<2>(s_max[l], 16 * n + j, a.wexp[l]);
                unsigned bits = 0;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const float x = fmaf(z[r], cn, b[r]);
                    bits |= x > 0.f ? 1u << r : 0u;
                    z[r] = leaky<false>(x, slope);
                }
                mask[l][slot] |= bits << (slot < MT ? 4 * n : 0);
            });
        });
        // output layer and delta3 = s .* v .* sigma'(z3)
        {
            const Share<NT> sh(a.out_tiles, wave, false);
            auto vector = [&](int n, int e) {
                return v[(p0 + min(16 * n + j, rows - 1)) * n_out + min(e, n_out - 1)];
            };
            f4 b0{}, s0{}, v0[MT == 1 ? NT : 1] = {};      // as the hidden layers' bias
            if constexpr (MT == 1)
                if (sh.cnt > 0) {
                    const int e0 = 16 * wave + 4 * g;
                    b0 = bias4(a.b3, e0);
                    s0 = bias4(a.out_scale, e0);
#pragma unroll
                    for (int n = 0; n < NT; ++n)
#pragma unroll
                        for (int r = 0; r < 4; ++r) v0[n][r] = vector(n, e0 + r);
                }
            layer_mm<2, NT, MT, RS, false>(a.W3, a.h2_tiles, sh, act, wave, lane, acc);
            float c[NT];
#pragma unroll
            for (int n = 0; n < NT; ++n) c[n] = unscale<2>(s_max[2], 16 * n + j, a.wexp[2]);
            layer_out<2, NT, MT, RS>(acc, sh, act, s_max[3], wave, lane, [&](auto, int mt, int n, f4& z) {
                const f4 b = MT == 1 ? b0 : bias4(a.b3, 16 * mt + 4 * g);
                const int pj = 16 * n + j;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int e = 16 * mt + 4 * g + r;
                    float x;
                    if constexpr (MT == 1) x = v0[n][r] * s0[r];
                    else x = vector(n, e) * a.out_scale[e];
                    if (a.out_act && !(fmaf(z[r], c[n], b[r]) > 0.f)) x *= slope;
                    z[r] = (pj < rows && e < n_out) ? x : 0.f;
                }
            });
        }
        // delta2 = (W3^T delta3) .* sigma'(z2), delta1 = (W2^T delta2) .* sigma'(z1)
        static_for<0, 2>([&](auto lc) {
            constexpr int l = decltype(lc)::value;
            const Share<NT> sh(l == 0 ? a.h2_tiles : a.h1_tiles, wave, MT > 1);
            const int we = a.wexp[l == 0 ? 2 : 1];
            layer_mm<2, NT, MT, RS, (MT > 1)>(l == 0 ? a.W3T : a.W2T, l == 0 ? a.out_tiles : a.h2_tiles, sh, act, wave, lane, acc);
            float c[NT];
#pragma unroll
            for (int n = 0; n < NT; ++n) c[n] = unscale<2>(s_max[3 + l], 16 * n + j, we);
            layer_out<2, NT, MT, RS>(acc, sh, act, s_max[4 + l], wave, lane, [&](auto slotc, int, int n, f4& z) {
                constexpr int slot = decltype(slotc)::value;
                float cn;
                if constexpr (slot < MT) cn = c[n];
                else cn = unscale<2>(s_max[3 + l], 16 * n + j, we);
                const unsigned bits = mask[1 - l][slot] >> (slot < MT ? 4 * n : 0);
#pragma unroll
                for (int r = 0; r < 4; ++r) z[r] = z[r] * cn * ((bits >> r) & 1u ? 1.f : slope);
            });
        });
        // g = (W1^T delta1) ./ std
        const Share<NT> sh(in_tiles, wave, false);
        layer_mm<2, NT, MT, RS, false>(a.W1T, a.h1_tiles, sh, act, wave, lane, acc);
        if (sh.cnt > 0) {                      // at most eight input tiles: one per wave
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                const int pj = 16 * n + j;
                const float c = unscale<2>(s_max[5], pj, a.wexp[0]);
                if (pj >= rows) continue;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int k = 16 * wave + 4 * g + r;
                    if (k < n_in) g_out[(p0 + pj) * n_in + k] = acc.t[0][n][r] * c * a.in_rstd[k];
                }
            }
        }
        unsigned long long again = infinite_points(s_max, 6, rows, lane);
        __syncthreads();                       // every wave has read the activation tile
        for (; again; again &= again - 1) {
            PlainPoint& q = *reinterpret_cast<PlainPoint*>(smem);
            const int64_t p = p0 + __ffsll(again) - 1;
            const int t = plain_thread();
            const MlpPlain& w = *a.plain;
            plain_hidden(w, B + p * w.n[0], q, t);
            plain_layer(w, 2, q.z2, t, [&](int e, float y) {
                q.d[e] = v[p * w.n[3] + e] * w.out_scale[e] * (w.out_act && !(y > 0.f) ? w.slope : 1.f);
            });
            // delta over the units of `z` in place, from the delta of the layer W leads to
            auto back = [&](const float* W, int fout, const float* delta, int n, auto&& f) {
                __syncthreads();
                for (int u = t; u < n; u += kWaves * 64) {
                    float z = 0.f;
#pragma clang loop unroll(disable)
                    for (int i = 0; i < fout; ++i) z = fmaf(W[(unsigned)(i * n + u)], delta[i], z);
                    f(u, z);
                }
            };
            auto through = [&](float* z) { return [z, slope = w.slope](int u, float d) { z[u] = d * (z[u] > 0.f ? 1.f : slope); }; };
            back(w.W[2], w.n[3], q.d, w.n[2], through(q.z2));
            back(w.W[1], w.n[2], q.z2, w.n[1], through(q.z1));
            back(w.W[0], w.n[1], q.z1, w.n[0], [&](int k, float z) { g_out[p * w.n[0] + k] = z * w.in_rstd[k]; });
            __syncthreads();
        }
    }
}

// The widths the call accepts, part of its interface: both hidden layers and the
// wider of input and output, each rounded up to 64 units, of at most 1152 together.
// It is no limit of this kernel, whose one tile holds any layer: a form that kept
// the activations of all three in LDS had it, and callers choose their path by it.
bool mlp_vjp_supported(const MlpArgs& a) {
    auto padded = [](int w) { return (w + 63) / 64 * 64; };
    return padded(a.h1_tiles * 16) + padded(a.h2_tiles * 16) + padded(std::max(a.in_pad, a.out_tiles * 16)) <= 1152;
}

template <int NT, int MT, int RS>
static hipError_t launch_vjp_n(hipStream_t s, const MlpArgs& a, const float* B, const float* v, int64_t n_pts,
                               float* g_out, int n_blocks) {
    constexpr size_t lds = ActTile<2, NT, RS>::kBytes;
    (void)hipFuncSetAttribute(reinterpret_cast<const void*>(&k_mlp_vjp<NT, MT, RS>),
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL((k_mlp_vjp<NT, MT, RS>), dim3(n_blocks), dim3(kWaves * 64), lds, s, a, B, v, n_pts, g_out);
    return hipGetLastError();
}

// Point tiles per block by the rule of the network kernel.
hipError_t launch_mlp_vjp(hipStream_t s, const MlpArgs& a, const float* B, const float* v, int64_t n_pts,
                          float* g_out) {
    if (n_pts <= 0) return hipSuccess;
    if (a.precision != 0 || !a.W1T || !a.W2T || !a.W3T || !mlp_vjp_supported(a)) return hipErrorInvalidValue;
    const int nb = mlp_blocks(n_pts, mlp_rows_small(a) ? 2 : 1), nt = mlp_point_tiles(a, n_pts, nb);
    if (mlp_rows_small(a)) {
        if (nt == 4) return launch_vjp_n<4, 1, kRowSmall>(s, a, B, v, n_pts, g_out, nb);
        return launch_vjp_n<2, 1, kRowSmall>(s, a, B, v, n_pts, g_out, nb);
    }
    if (mlp_rows_wide(a)) {
        if (nt == 4) return launch_vjp_n<4, 3, kRowWide>(s, a, B, v, n_pts, g_out, nb);
        return launch_vjp_n<2, 3, kRowWide>(s, a, B, v, n_pts, g_out, nb);
    }
    if (nt == 4) return launch_vjp_n<4, 4, kRowMax>(s, a, B, v, n_pts, g_out, nb);
    return launch_vjp_n<2, 4, kRowMax>(s, a, B, v, n_pts, g_out, nb);
}

}  // namespace mala
