// MFMA building blocks of the per-point network (Sec. 2.4, Eq. ffnn): the
// number formats, the matrix product of one layer and the activation tile in
// LDS.  Shared by the forward kernel and its vector-Jacobian product.
//
// Layers are computed transposed, out^T = W in^T: output units are the MFMA
// M dimension, the points of the block's tile the N dimension.
//
// FP32 weights run as two FP16 planes per operand on the 16-bit matrix unit:
// x = hi + lo / 2^11 with hi = fp16(x), lo = fp16(2^11 (x - hi)), after a
// power-of-two scale that puts the largest value near 2^14 (per layer for the
// weights, per point for the activations, taken from the values themselves, so
// nothing overflows).  hi + lo / 2^11 keeps x to at most one unit of the last FP32
// place (exactly for three values in four) from the largest value down to 2^-27 of
// it; below that a bit is lost per binade (as lo = fp16(x - hi) it was from 2^-16 on).
// FP32 has its precision at any size, so the loader first evens out the network's
// inputs, units and outputs (even_out in api.cpp): what is left below 2^-27 of
// the largest then counts only beside values that no unit adds to it.  The products
// hi hi and hi lo + lo hi are accumulated in FP32, in a sum each, and lo lo (2^-24
// of the product) is dropped.  Against the 16x16x4 FP32 instruction that is
// three 16x16x32 instructions of 16 cycles per 32 units instead of eight of
// 32, and fewer FP32 roundings of the running sum (one per 32 units).  Error
// against 64 bits of the plain network output (2-norm, x ~ N(0, 1)): 2.6e-7
// with that instruction and 1.9e-7 here at 55-64-64-250, 5.5e-7 and 2.5e-7 at
// 91-400-400-250, 6.1e-7 and 2.6e-7 at 128-512-512-256; the same with units
// spread over 14 decades, and 3.8e-7 and 2.6e-7 with two halves of a network 1e8
// apart.  The sum of its own for the small products costs 1 to 2%.
// Time at 91-400-400-250: 4.12 -> 1.46 ms per 729,000 points with the LDOS stored,
// 14.6 -> 5.0 to 5.3 us per 1,000 points for the vector-Jacobian product.  What bounds it
// now: the products are 0.65 ms of the 1.46 at the 1.9 GHz the card holds under
// them, the epilogues (activation, scales, LDS writes) as much, and the weights
// from L2 most of the rest.
// BF16 weights use one plane, rounded once, without scales.
#pragma once
#include "mala_internal.h"

namespace mala {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf4 __attribute__((ext_vector_type(4)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef short s4 __attribute__((ext_vector_type(4)));

constexpr int kLoBits = 11;        // binary places by which the second plane is raised (FP32 weights)
constexpr int kWaves = 8;          // waves of a network block (two per SIMD, one block per CU)

// sigma(x) = slope x for x < 0, else x.  For 0 < slope <= 1 that is the larger of
// the two, for every x (infinities and NaN included): one instruction less.
template <bool FAST>
__device__ __forceinline__ float leaky(float x, float s) {
    if constexpr (FAST) return fmaxf(x, s * x);
    else return x < 0.f ? s * x : x;
}
__device__ __forceinline__ f4 bias4(const float* b, int off) {
    const float4 v = *reinterpret_cast<const float4*>(b + off);
    return f4{v.x, v.y, v.z, v.w};
}

template <typename To, typename From>
__device__ __forceinline__ To bits_as(const From& v) {
    static_assert(sizeof(To) == sizeof(From), "size");
    To t;
    __builtin_memcpy(&t, &v, sizeof(t));
    return t;
}

// acc += A B over 32 (mfma32) or 16 (mfma16) units: lane l of A holds row
// l % 16 and units 8 (l / 16) + 0..7 (4 (l / 16) + 0..3), of B the same for its point.
template <int P>
__device__ __forceinline__ f4 mfma32(uint4 a, uint4 b, f4 c) {
    if constexpr (P == 2) return __builtin_amdgcn_mfma_f32_16x16x32_f16(bits_as<h8>(a), bits_as<h8>(b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x32_bf16(bits_as<bf8>(a), bits_as<bf8>(b), c, 0, 0, 0);
}
template <int P>
__device__ __forceinline__ f4 mfma16(uint2 a, uint2 b, f4 c) {
    if constexpr (P == 2) return __builtin_amdgcn_mfma_f32_16x16x16f16(bits_as<h4>(a), bits_as<h4>(b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(bits_as<s4>(a), bits_as<s4>(b), c, 0, 0, 0);
}

// Unit tiles of the output layer a wave holds, and waves per SIMD, of a kernel whose waves
// hold MT of a hidden layer.
__host__ __device__ constexpr int out_unit_tiles(int MT) { return MT == 1 ? 1 : kMlpMaxOut / 16 / kWaves; }
constexpr int waves_per_simd(int MT) { return MT == 1 ? 4 : 2; }

// The activation tile of a block, [plane][point][unit], for NT point tiles and
// layers of at most RS units.  The row stride RS (16-bit elements) is an odd
// multiple of 8 dwords, chosen for the 128-bit operand reads (16 points x 4
// groups of 8 units), which then spread over all banks, and a constant, so that
// every operand and output address is one register plus an immediate.  The 8-byte
// writes of a layer's output pay for it (points j and j + 8 share banks): 0.70 of
// the conflicts that the counters show for FP32 weights (0.35 of the LDS cycles,
// LDOS stored), the rows of the stored LDOS another 0.08.
template <int P, int NT, int RS>
struct ActTile {
    static constexpr int kPlane = 16 * NT * RS;
    static constexpr size_t kBytes = (size_t)P * kPlane * 2;
    unsigned short* p;
};

// What one wave computes of a layer of TO unit tiles: tiles wave, wave + 8, ...
// (`cnt` of them) against every point tile, and, where TO leaves so few tiles
// over after the full rounds that their (unit tile, point tile) products give
// each wave at most one, such an item, so that no wave runs a whole extra tile.
template <int NT>
struct Share {
    int cnt;
    int it_mt, it_n;       // it_mt < 0: none
    __device__ __forceinline__ Share(int TO, int wave, bool items) {
        const int full = TO / kWaves, r = TO % kWaves;
        const bool split = items && full > 0 && r * NT <= kWaves;
        cnt = full + (!split && wave < r ? 1 : 0);
        const bool on = split && wave < r * NT;
        it_mt = on ? kWaves * full + wave / NT : -1;
        it_n = on ? wave % NT : 0;
    }
};

// Weights are packed in lane order, [unit tile][step][plane][lane][16 bytes]:
// (T + 1) / 2 steps of 32 units for T unit tiles of input; in the last step of
// an odd T a lane's first 8 bytes hold its 4 of the 16 units.
__host__ __device__ __forceinline__ int w_steps(int T) { return (T + 1) / 2; }

template <int P>
__device__ __forceinline__ void fetch_tile(const void* W, int mt, int T, int s, int lane, uint4 (&d)[P]) {
    // uniform base plus a 32-bit lane offset: no per-lane 64-bit address arithmetic
    const char* base = static_cast<const char*>(W) + ((size_t)mt * w_steps(T) + s) * (P * 1024);
#pragma unroll
    for (int p = 0; p < P; ++p) d[p] = *reinterpret_cast<const uint4*>(base + p * 1024 + (unsigned)lane * 16u);
}

// The accumulators of one wave: MT unit tiles x NT point tiles, and the item.
template <int NT, int MT>
struct Acc {
    f4 t[MT][NT];
    f4 it;
};

// Half a step: the first 8 bytes of the weight operand, 16 units.
template <int P>
__device__ __forceinline__ void half_products(const uint4 (&w)[P], const uint2 (&b)[P], f4& c, f4& cl) {
    auto lo = [](const uint4& v) { return make_uint2(v.x, v.y); };
    c = mfma16<P>(lo(w[0]), b[0], c);
    if constexpr (P == 2) {
        cl = mfma16<P>(lo(w[0]), b[P - 1], cl);
        cl = mfma16<P>(lo(w[P - 1]), b[0], cl);
    }
}

// The sum of hi hi and that of the two cross products, 2^kLoBits larger.
__device__ __forceinline__ f4 join_planes(f4 c, f4 cl) {
    constexpr float f = 1.f / (float)(1 << kLoBits);
    return f4{fmaf(cl[0], f, c[0]), fmaf(cl[1], f, c[1]), fmaf(cl[2], f, c[2]), fmaf(cl[3], f, c[3])};
}

// t[m][n] = the wave's unit tile m times point tile n over T unit tiles of
// input: T / 2 steps of 32 units and, for odd T, one of 16.  A step takes the
// unit tiles at once, or in two halves where two sets of them would not fit
// the registers; the weights of the next step (half) come from L2 while this
// one's products run, the LDS operand of the next point tile while this one's
// do.  The scheduling barriers keep the compiler from reading all operands
// first, which spills.
template <int P, int NT, int MT, int RS, int M>
__device__ __forceinline__ void mm(const void* W, int T, const ActTile<P, NT, RS>& in, int wave, int lane,
                                   f4 (&t)[MT][NT]) {
    constexpr int NC = M * P > 6 ? 2 : 1, H0 = (M + NC - 1) / NC;      // chunks per step, tiles of the first
    constexpr int PS = ActTile<P, NT, RS>::kPlane;
    const int KS = T >> 1, KL = w_steps(T) - 1, g = lane >> 4;
    const unsigned short* row = in.p + (lane & 15) * RS;
    uint4 a[2][H0][P], b[2][P];
    f4 tl[P == 2 ? M : 1][NT];            // the cross products of the planes
    auto fetch = [&](int s, auto hc, uint4 (&d)[H0][P]) {
        constexpr int h = decltype(hc)::value;
#pragma unroll
        for (int m = 0; m < H0; ++m)
            if (h * H0 + m < M) fetch_tile<P>(W, wave + kWaves * (h * H0 + m), T, s < KL ? s : KL, lane, d[m]);
    };
    auto fetch_b = [&](int n, int s, uint4 (&d)[P]) {
#pragma unroll
        for (int p = 0; p < P; ++p)
            d[p] = *reinterpret_cast<const uint4*>(row + n * 16 * RS + p * PS + 32 * s + 8 * g);
    };
    constexpr std::integral_constant<int, 0> c0{};
    constexpr std::integral_constant<int, 1> c1{};
    constexpr std::integral_constant<int, NC - 1> clast{};
    fetch(0, c0, a[0]);
    static_for<0, M>([&](auto mc) {
        static_for<0, NT>([&](auto nc) {
            if constexpr (P == 2) tl[decltype(mc)::value][decltype(nc)::value] = f4{0.f, 0.f, 0.f, 0.f};
        });
    });
    if (KS > 0) fetch_b(0, 0, b[0]);
    // step s, the I-th of the loop body: its first chunk lies in a[I * NC % 2],
    // its first LDS operand in b[I * NC * NT % 2]
    auto step = [&](int s, auto ic) {
        constexpr int Q = decltype(ic)::value * NC % 2, G0 = decltype(ic)::value * NC * NT % 2;
        static_for<0, NC>([&](auto hc) {
            constexpr int h = decltype(hc)::value, MH = M - h * H0 < H0 ? M - h * H0 : H0;
            const uint4 (&ac)[H0][P] = a[(Q + h) % 2];
            if constexpr (h + 1 < NC) fetch(s, clast, a[(Q + h + 1) % 2]);
            else fetch(s + 1, c0, a[(Q + h + 1) % 2]);
            static_for<0, NT>([&](auto nc) {
                constexpr int n = decltype(nc)::value, G = G0 + h * NT + n;
                const uint4 (&bc)[P] = b[G % 2];
                if constexpr (n + 1 < NT) fetch_b(n + 1, s, b[(G + 1) % 2]);
                else fetch_b(0, h + 1 < NC ? s : min(s + 1, KS - 1), b[(G + 1) % 2]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int m = 0; m < MH; ++m) t[h * H0 + m][n] = mfma32<P>(ac[m][0], bc[0], t[h * H0 + m][n]);
                if constexpr (P == 2) {
#pragma unroll
                    for (int m = 0; m < MH; ++m) tl[h * H0 + m][n] = mfma32<P>(ac[m][0], bc[P - 1], tl[h * H0 + m][n]);
#pragma unroll
                    for (int m = 0; m < MH; ++m) tl[h * H0 + m][n] = mfma32<P>(ac[m][P - 1], bc[0], tl[h * H0 + m][n]);
                }
                __builtin_amdgcn_sched_barrier(0);
            });
        });
    };
    // the half step of an odd T; its first chunk lies in a[0]
    auto tail = [&]() {
        if constexpr (NC == 2) fetch(KL, clast, a[1]);
        static_for<0, NT>([&](auto nc) {
            constexpr int n = decltype(nc)::value;
            uint2 bt[P];
#pragma unroll
            for (int p = 0; p < P; ++p) bt[p] = *reinterpret_cast<const uint2*>(row + n * 16 * RS + p * PS + 32 * KS + 4 * g);
            static_for<0, M>([&](auto mc) {
                constexpr int m = decltype(mc)::value;
                half_products<P>(a[m / H0][m % H0], bt, t[m][n], tl[P == 2 ? m : 0][n]);
            });
        });
    };
    int s = 0;
    if constexpr (NC == 2) {
#pragma clang loop unroll(disable)
        for (; s < KS; ++s) step(s, c0);
    } else {
#pragma clang loop unroll(disable)
        for (; s + 2 <= KS; s += 2) {
            step(s, c0);
            step(s + 1, c1);
        }
        if (s < KS) {
            step(s, c0);
            static_for<0, H0>([&](auto mc) {
                static_for<0, P>([&](auto pc) { a[0][decltype(mc)::value][decltype(pc)::value] = a[1][decltype(mc)::value][decltype(pc)::value]; });
            });
        }
    }
    if (T & 1) tail();
    if constexpr (P == 2)
        static_for<0, M>([&](auto mc) {
            static_for<0, NT>([&](auto nc) {
                constexpr int m = decltype(mc)::value, n = decltype(nc)::value;
                t[m][n] = join_planes(t[m][n], tl[m][n]);
            });
        });
}

// The wave's item: one unit tile times one point tile.  Three products per
// step cover little of a weight read, so six steps of weights are in flight.
// The sum runs in the order of mm: whether a unit tile is an item depends on the
// point tiles of a block and with them on the number of points of the call, and
// a point's values must not.
template <int P, int NT, int RS>
__device__ __forceinline__ f4 mm_item(const void* W, int T, const Share<NT>& sh, const ActTile<P, NT, RS>& in, int lane) {
    constexpr int D = 6, PS = ActTile<P, NT, RS>::kPlane;
    const int KS = T >> 1, KL = w_steps(T) - 1, g = lane >> 4;
    const unsigned short* row = in.p + (16 * sh.it_n + (lane & 15)) * RS;
    uint4 a[D][P];
    static_for<0, D>([&](auto dc) { fetch_tile<P>(W, sh.it_mt, T, min((int)decltype(dc)::value, KL), lane, a[decltype(dc)::value]); });
    f4 t = {}, tl = {};
    auto step = [&](int s, uint4 (&w)[P]) {
        uint4 b[P];
#pragma unroll
        for (int p = 0; p < P; ++p) b[p] = *reinterpret_cast<const uint4*>(row + p * PS + 32 * s + 8 * g);
        t = mfma32<P>(w[0], b[0], t);
        if constexpr (P == 2) {
            tl = mfma32<P>(w[0], b[P - 1], tl);
            tl = mfma32<P>(w[P - 1], b[0], tl);
        }
        fetch_tile<P>(W, sh.it_mt, T, min(s + D, KL), lane, w);
    };
    int s = 0;
#pragma clang loop unroll(disable)
    for (; s + D <= KS; s += D) static_for<0, D>([&](auto dc) { step(s + decltype(dc)::value, a[decltype(dc)::value]); });
    // the last KS % D steps, then the half step: a[i] holds step s + i
    static_for<0, D>([&](auto dc) {
        constexpr int i = decltype(dc)::value;
        if (s + i < KS) step(s + i, a[i]);
        else if (s + i == KS && (T & 1)) {
            uint2 bt[P];
#pragma unroll
            for (int p = 0; p < P; ++p) bt[p] = *reinterpret_cast<const uint2*>(row + p * PS + 32 * KS + 4 * g);
            half_products<P>(a[i], bt, t, tl);
        }
    });
    if constexpr (P == 2) return join_planes(t, tl);
    else return t;
}

// acc = W in for the wave's share of a layer.
template <int P, int NT, int MT, int RS, bool ITEMS>
__device__ __forceinline__ void layer_mm(const void* W, int T, const Share<NT>& sh, const ActTile<P, NT, RS>& in,
                                         int wave, int lane, Acc<NT, MT>& acc) {
    // every tile, also those this wave has none of: what they held before would
    // stay live beside the products
    static_for<0, MT>([&](auto mc) {
        static_for<0, NT>([&](auto nc) { acc.t[decltype(mc)::value][decltype(nc)::value] = f4{0.f, 0.f, 0.f, 0.f}; });
    });
    if constexpr (ITEMS) acc.it = f4{0.f, 0.f, 0.f, 0.f};
    static_for<1, MT + 1>([&](auto mc) {
        if (sh.cnt == decltype(mc)::value) mm<P, NT, MT, RS, decltype(mc)::value>(W, T, in, wave, lane, acc.t);
    });
    if constexpr (ITEMS)
        if (sh.it_mt >= 0) acc.it = mm_item<P, NT, RS>(W, T, sh, in, lane);
}

// Power-of-two exponent that brings a value of largest magnitude `bits` (FP32
// bit pattern, sign cleared) to [2^14, 2^15); 0 for infinities and NaN, at
// most 100 so that its inverse and products with weight scales stay normal.
__device__ __forceinline__ int act_exponent(unsigned bits) {
    const int e = (int)(bits >> 23);
    if (e == 255) return 0;
    return min(14 - (e - 127), 100);
}
__device__ __forceinline__ float pow2f(int k) { return __int_as_float((127 + k) << 23); }      // |k| <= 126

// Largest magnitude of mx and four values (NaN passes by: it stays NaN under any scale).
__device__ __forceinline__ float max_abs4(float mx, f4 v) {
    mx = fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), mx);
    return fmaxf(fmaxf(fabsf(v[2]), fabsf(v[3])), mx);
}

// hi = fp16(v scale), lo = fp16(2^kLoBits (v scale - hi)) of two values, each
// half one mixed-precision FMA that rounds once (v scale is exact: a power of two).
__device__ __forceinline__ void split2(float v0, float v1, float scale, unsigned& hi, unsigned& lo) {
    constexpr float f = (float)(1 << kLoBits);
    const float s0 = v0 * (scale * f), s1 = v1 * (scale * f);
    asm("v_fma_mixlo_f16 %0, %1, %2, 0" : "=v"(hi) : "v"(v0), "v"(scale));
    asm("v_fma_mixhi_f16 %0, %1, %2, 0" : "+v"(hi) : "v"(v1), "v"(scale));
    asm("v_fma_mixlo_f16 %0, %1, %2, %3 op_sel_hi:[1,0,0]" : "=v"(lo) : "v"(hi), "s"(-f), "v"(s0));
    asm("v_fma_mixhi_f16 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "+v"(lo) : "v"(hi), "s"(-f), "v"(s1));
}

// Four consecutive units of one point into the tile (scale: FP32 weights only).
template <int P, int NT, int RS>
__device__ __forceinline__ void put4(const ActTile<P, NT, RS>& t, int point, int unit, f4 v, float scale) {
    unsigned short* d = t.p + point * RS + unit;
    if constexpr (P == 1) {
        const bf4 h = {(__bf16)v[0], (__bf16)v[1], (__bf16)v[2], (__bf16)v[3]};
        *reinterpret_cast<bf4*>(d) = h;
    } else {
        uint2 hi, lo;
        split2(v[0], v[1], scale, hi.x, lo.x);
        split2(v[2], v[3], scale, hi.y, lo.y);
        *reinterpret_cast<uint2*>(d) = hi;
        *reinterpret_cast<uint2*>(d + ActTile<P, NT, RS>::kPlane) = lo;
    }
}

// Largest magnitude per point of a layer's output over the block: `m` is the
// lane's own maximum for point 16 n + j; out must start at zero.
__device__ __forceinline__ void point_max(unsigned* out, int n, int lane, float m) {
    m = fmaxf(m, __shfl_xor(m, 16, 64));
    m = fmaxf(m, __shfl_xor(m, 32, 64));
    if ((lane >> 4) == (n & 3)) atomicMax(out + 16 * n + (lane & 15), (unsigned)__float_as_int(m));
}

// Largest unsigned value over the wave, in a scalar register: shifts inside
// each row of 16 lanes, then the row results broadcast upwards (lane 63 ends
// with all of them).
__device__ __forceinline__ unsigned wave_max_u32(unsigned v) {
#define MALA_DPP_MAX(ctrl) v = max(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, 0xf, 0xf, false))
    MALA_DPP_MAX(0x111);      // row_shr 1, 2, 4, 8
    MALA_DPP_MAX(0x112);
    MALA_DPP_MAX(0x114);
    MALA_DPP_MAX(0x118);
    MALA_DPP_MAX(0x142);      // row_bcast 15, 31
    MALA_DPP_MAX(0x143);
#undef MALA_DPP_MAX
    return (unsigned)__builtin_amdgcn_readlane((int)v, 63);
}

// One layer's output into the tile that also held its input, as the next
// layer's input: ep(slot, mt, n, acc) forms the four values of the lane's units
// of (unit tile mt, point tile n) in place (slot: the wave's tile, MT the
// item); then, once every wave has read the input, the values are written with
// the point's scale.
template <int P, int NT, int MT, int RS, typename Ep>
__device__ __forceinline__ void layer_out(Acc<NT, MT>& acc, const Share<NT>& sh, const ActTile<P, NT, RS>& t,
                                          unsigned* s_max, int wave, int lane, Ep&& ep) {
    const int j = lane & 15, g = lane >> 4;
    float mx[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) mx[n] = 0.f;
    static_for<0, MT>([&](auto mc) {
        constexpr int m = decltype(mc)::value;
        if (m < sh.cnt) {
            static_for<0, NT>([&](auto nc) {
                constexpr int n = decltype(nc)::value;
                ep(mc, wave + kWaves * m, n, acc.t[m][n]);
                if constexpr (P == 2) mx[n] = max_abs4(mx[n], acc.t[m][n]);
            });
        }
    });
    if (sh.it_mt >= 0) {
        ep(std::integral_constant<int, MT>{}, sh.it_mt, sh.it_n, acc.it);
        if constexpr (P == 2) point_max(s_max, sh.it_n, lane, max_abs4(0.f, acc.it));
    }
    if constexpr (P == 2)
        if (sh.cnt > 0) {
#pragma unroll
            for (int n = 0; n < NT; ++n) point_max(s_max, n, lane, mx[n]);
        }
    __syncthreads();
    float sc[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) sc[n] = P == 2 ? pow2f(act_exponent(s_max[16 * n + j])) : 1.f;
#pragma unroll
    for (int m = 0; m < MT; ++m)
        if (m < sh.cnt) {
#pragma unroll
            for (int n = 0; n < NT; ++n)
                put4(t, 16 * n + j, 16 * (wave + kWaves * m) + 4 * g, acc.t[m][n], sc[n]);
        }
    if (sh.it_mt >= 0) {
        const int p = 16 * sh.it_n + j;
        put4(t, p, 16 * sh.it_mt + 4 * g, acc.it, P == 2 ? pow2f(act_exponent(s_max[p])) : 1.f);
    }
    __syncthreads();
}

// Factor that takes an accumulated product back to its true scale: the inverse
// of the point's activation scale (its largest magnitude in s_max) and of the
// layer's weight scale 2^wexp.
template <int P>
__device__ __forceinline__ float unscale(const unsigned* s_max, int point, int wexp) {
    if constexpr (P == 1) return 1.f;
    else return pow2f(-act_exponent(s_max[point])) * pow2f(-wexp);
}

// Standardised descriptor rows of a tile into LDS: wave w takes rows w R ..
// w R + R - 1, lane = columns lane and lane + 64, at most twelve rows'
// reads in flight.  A row past the last valid point repeats that point (its
// results are not used), a pad column the last one.
template <int P, int NT, int RS>
__device__ __forceinline__ void stage_rows(const float* __restrict__ B, int64_t p0, int rows, int row_stride, int n_in,
                                           int in_pad, const float (&mu)[2], const float (&rstd)[2],
                                           const ActTile<P, NT, RS>& t, unsigned* s_max, int wave, int lane) {
    constexpr int R = 16 * NT / kWaves, C = R % 12 == 0 ? 12 : R % 8 == 0 ? 8 : 4, PS = ActTile<P, NT, RS>::kPlane;
    const int c0 = min(lane, n_in - 1), c1 = min(lane + 64, n_in - 1);
#pragma clang loop unroll(disable)
    for (int q0 = 0; q0 < R; q0 += C) {
        float v[C][2];
#pragma unroll
        for (int q = 0; q < C; ++q) {
            const float* r = B + (p0 + min(wave * R + q0 + q, rows - 1)) * row_stride * n_in;
            v[q][0] = r[c0];
            v[q][1] = n_in > 64 ? r[c1] : 0.f;
        }
#pragma unroll
        for (int q = 0; q < C; ++q) {
            const int p = wave * R + q0 + q;
            // a pad column is zero also where the last one is infinite
            const float x0 = lane < n_in ? (v[q][0] - mu[0]) * rstd[0] : 0.f;
            const float x1 = lane + 64 < n_in ? (v[q][1] - mu[1]) * rstd[1] : 0.f;
            unsigned short* d = t.p + p * RS + lane;
            if constexpr (P == 2) {
                const unsigned mx = wave_max_u32(max((unsigned)__float_as_int(x0) & 0x7fffffffu, (unsigned)__float_as_int(x1) & 0x7fffffffu));
                s_max[p] = mx;                                   // every lane the same value
                unsigned hi, lo;
                split2(x0, x1, pow2f(act_exponent(mx)), hi, lo);
                if (lane < in_pad) {
                    d[0] = (unsigned short)hi;
                    d[PS] = (unsigned short)lo;
                }
                if (lane + 64 < in_pad) {
                    d[64] = (unsigned short)(hi >> 16);
                    d[PS + 64] = (unsigned short)(lo >> 16);
                }
            } else {
                if (lane < in_pad) *reinterpret_cast<__bf16*>(d) = (__bf16)x0;
                if (lane + 64 < in_pad) *reinterpret_cast<__bf16*>(d + 64) = (__bf16)x1;
            }
        }
    }
}

// The FP16 planes of an infinity are infinity and NaN, and its product with the second
// plane of a weight has any sign, so a point with an infinite input or activation
// comes out of the matrix unit as NaN where FP32 has an infinity: its units' signs,
// and with them the gradient, would be lost.  Such points are done again, one at a
// time by the whole block, in plain FP32.  The tile's points that need it (NaN
// without an infinity does not): s_max holds the largest magnitude of each of the
// layers' inputs.
template <int NP>
__device__ __forceinline__ unsigned long long infinite_points(const unsigned (*s_max)[NP], int layers, int rows, int lane) {
    static_assert(NP <= 64, "one lane per point");
    bool inf = false;
    for (int l = 0; l < layers; ++l) inf = inf || s_max[l][lane % NP] == 0x7f800000u;
    return __ballot(inf && lane < rows);
}

// Units of layer l of one point: f(unit, W sigma(in) + b), in: the layer before in LDS
// (z, or x for l = 0).  t: the thread, in a register of its own, or the addresses
// formed from it stay in registers all along.
template <typename F>
__device__ __forceinline__ void plain_layer(const MlpPlain& w, int l, const float* in, int t, F&& f) {
    const int n_in = w.n[l], n_out = w.n[l + 1];
    const float* W = w.W[l];
    for (int u = t; u < n_out; u += kWaves * 64) {
        float z = w.b[l][u];
#pragma clang loop unroll(disable)
        for (int k = 0; k < n_in; ++k) z = fmaf(W[(unsigned)(u * n_in + k)], l ? leaky<false>(in[k], w.slope) : in[k], z);
        f(u, z);
    }
}
__device__ __forceinline__ int plain_thread() {
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// Inputs and hidden z of one point in plain FP32 (LDS of PlainPoint; a barrier has
// passed since the last write).
struct PlainPoint {
    float x[kMlpMaxIn], z1[kMlpMaxHidden], z2[kMlpMaxHidden], d[kMlpMaxOut];
};
__device__ __forceinline__ void plain_hidden(const MlpPlain& w, const float* __restrict__ row, PlainPoint& q, int t) {
    for (int k = t; k < w.n[0]; k += kWaves * 64) q.x[k] = (row[k] - w.in_mean[k]) * w.in_rstd[k];
    __syncthreads();
    plain_layer(w, 0, q.x, t, [&](int u, float z) { q.z1[u] = z; });
    __syncthreads();
    plain_layer(w, 1, q.z1, t, [&](int u, float z) { q.z2[u] = z; });
    __syncthreads();
}

}  // namespace mala
