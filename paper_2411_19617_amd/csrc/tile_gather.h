// Device helpers shared by the kernels that visit, for a tile of grid
// points, every atom image within a cutoff (the neighbour sums of
// Eq. ionicdensity and the Gaussian descriptors): wave reductions, a block
// scan, and the candidate gather over the cell list.
#pragma once

#include "mala_internal.h"

namespace mala {

__device__ __forceinline__ int wave_max_int(int v) {
    for (int off = 32; off > 0; off >>= 1) v = max(v, __shfl_xor(v, off, 64));
    return v;
}

// Block-wide exclusive scan of one int per thread (blockDim <= 1024).
__device__ __forceinline__ int block_exclusive_scan(int v, int* tmp, int* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    int x = v;
    for (int off = 1; off < 64; off <<= 1) {
        int y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    if (lane == 63) tmp[wave] = x;
    __syncthreads();
    int wbase = 0, tot = 0;
    for (int w = 0; w < nw; ++w) {
        if (w < wave) wbase += tmp[w];
        tot += tmp[w];
    }
    __syncthreads();
    *total = tot;
    return wbase + x - v;
}

// Bounding boxes of a tile of consecutive flat grid indices: box 0 holds the
// points in the first one's run (its z-row when a row has at least 64 points, else
// its x-plane), box 1 the others.
// A tile that crosses a row or a plane would otherwise get one box spanning
// the cell's whole cross-section, and with it far more candidate images.
struct TileBoxes {
    double lo[2][3], hi[2][3];
    int n;            // 1, or 2 when the tile crosses a run boundary
    // The origin of a box's candidates and points: its middle, which keeps their FP32
    // coordinates half as large as its lower corner would and so their rounding, the
    // largest part of the kernels' error against 64 bits (descriptors 3.1e-7 ->
    // 2.9e-7, their gradient 9.6e-7 -> 8.5e-7, grid ACE 2.5e-7 -> 2.2e-7).  The middle
    // for a whole tile of 64 points, also where the range ends before: a point's
    // values must not depend on that.
    double mid[2][3];
};

// The lane's point of the tile of `count` points (1..64) that starts at flat
// index p0 (lanes past the last point take the first), and the tile's boxes.
// One division of p0 by the grid's row and plane, in 32 bits where it fits, and
// the rest from the offset in the tile: 64-bit divisions per lane and reductions of
// the coordinates over the wave cost 1.3 us of a 64 us call for 8,000 points.
struct TilePoint {
    double x, y, z;
    TileBoxes boxes;
};
__device__ __forceinline__ TilePoint tile_point(const BinState& bins, int Nx, int Ny, int Nz, int64_t p0, int count,
                                                int lane) {
    const int64_t plane = (int64_t)Ny * Nz;
    int i0, j0, k0;
    if (((p0 | plane) >> 32) == 0) {
        const unsigned q = (unsigned)p0, pl = (unsigned)plane, i = q / pl, rem = q - i * pl, j = rem / (unsigned)Nz;
        i0 = (int)i;
        j0 = (int)j;
        k0 = (int)(rem - j * (unsigned)Nz);
    } else {
        i0 = (int)(p0 / plane);
        const int64_t rem = p0 - i0 * plane;
        j0 = (int)(rem / Nz);
        k0 = (int)(rem - (int64_t)j0 * Nz);
    }
    auto index = [&](int d, int (&c)[3]) {            // of point p0 + d, d < 64
        const unsigned t = (unsigned)k0 + d, q = t / (unsigned)Nz, u = (unsigned)j0 + q, q2 = u / (unsigned)Ny;
        c[2] = (int)(t - q * (unsigned)Nz);
        c[1] = (int)(u - q2 * (unsigned)Ny);
        c[0] = i0 + (int)q2;
    };
    const int N[3] = {Nx, Ny, Nz};
    auto coord = [&](int d, int c) { return (double)c * bins.L[d] / N[d]; };
    TilePoint t;
    int c[3];
    index(lane < count ? lane : 0, c);
    t.x = coord(0, c[0]);
    t.y = coord(1, c[1]);
    t.z = coord(2, c[2]);
    // points p0 + d0 .. p0 + d1: a range that leaves its row covers whole rows' z, one
    // that leaves its plane whole planes
    auto box = [&](int d0, int d1, double (&from)[3], double (&to)[3]) {
        int a[3], b[3];
        index(d0, a);
        index(d1, b);
        const bool planes = a[0] != b[0], rows = planes || a[1] != b[1];
        const int lo[3] = {a[0], planes ? 0 : a[1], rows ? 0 : a[2]};
        const int hi[3] = {b[0], planes ? Ny - 1 : b[1], rows ? Nz - 1 : b[2]};
        for (int d = 0; d < 3; ++d) {
            from[d] = coord(d, lo[d]);
            to[d] = coord(d, hi[d]);
        }
    };
    const int64_t left = Nz >= 64 ? Nz - k0 : plane - ((int64_t)j0 * Nz + k0);      // points left in the run
    const int n0 = left < count ? (int)left : count;
    t.boxes.n = n0 < count ? 2 : 1;
    box(0, n0 - 1, t.boxes.lo[0], t.boxes.hi[0]);
    box(n0 < count ? n0 : 0, count - 1, t.boxes.lo[1], t.boxes.hi[1]);
    auto middle = [&](int k, const double (&from)[3], const double (&to)[3]) {
        for (int d = 0; d < 3; ++d) t.boxes.mid[k][d] = 0.5 * (from[d] + to[d]);
    };
    if (count == kTile) {
        for (int k = 0; k < 2; ++k) middle(k, t.boxes.lo[k], t.boxes.hi[k]);
    } else {
        const int whole = left < kTile ? (int)left : kTile;
        double from[3], to[3];
        box(0, whole - 1, from, to);
        middle(0, from, to);
        box(whole < kTile ? whole : 0, kTile - 1, from, to);
        middle(1, from, to);
    }
    return t;
}

__device__ __forceinline__ bool near_box(const double lo[3], const double hi[3], double X, double Y, double Z,
                                         double rc2) {
    const double dx = fmax(0.0, fmax(lo[0] - X, X - hi[0]));
    const double dy = fmax(0.0, fmax(lo[1] - Y, Y - hi[1]));
    const double dz = fmax(0.0, fmax(lo[2] - Z, Z - hi[2]));
    return dx * dx + dy * dy + dz * dz < rc2;
}

// One pass of the candidate gather: every image in the cells overlapping box
// `k` grown by rcut that lies within rcut of that box (and, for k = 1, not
// within rcut of box 0, whose pass took it already), appended after `base`
// in a fixed order (cells in index order, atoms in cell order), relative to
// the box's middle.
__device__ __forceinline__ int gather_pass(const BinState& bins, const TileBoxes& tb, int k, double rcut,
                                           float4* cand, int cap, int* scan_tmp, int base) {
    const double rc2 = rcut * rcut;
    const double* lo = tb.lo[k];
    const double* hi = tb.hi[k];
    const double* mid = tb.mid[k];
    int c_lo[3], c_n[3];
    for (int d = 0; d < 3; ++d) {
        c_lo[d] = (int)floor((lo[d] - rcut) / bins.cs[d]);
        c_n[d] = (int)floor((hi[d] + rcut) / bins.cs[d]) - c_lo[d] + 1;
    }
    const int ncells = c_n[0] * c_n[1] * c_n[2];
    for (int c0 = 0; c0 < ncells; c0 += blockDim.x) {
        const int c = c0 + threadIdx.x;
        int cnt = 0, b = 0, e = 0;
        double sx = 0, sy = 0, sz = 0;
        if (c < ncells) {
            const int cz = c % c_n[2], cy = (c / c_n[2]) % c_n[1], cx = c / (c_n[2] * c_n[1]);
            const int gx = c_lo[0] + cx, gy = c_lo[1] + cy, gz = c_lo[2] + cz;
            const int wx = ((gx % bins.nc[0]) + bins.nc[0]) % bins.nc[0];
            const int wy = ((gy % bins.nc[1]) + bins.nc[1]) % bins.nc[1];
            const int wz = ((gz % bins.nc[2]) + bins.nc[2]) % bins.nc[2];
            sx = (double)((gx - wx) / bins.nc[0]) * bins.L[0];
            sy = (double)((gy - wy) / bins.nc[1]) * bins.L[1];
            sz = (double)((gz - wz) / bins.nc[2]) * bins.L[2];
            const int cell = (wx * bins.nc[1] + wy) * bins.nc[2] + wz;
            b = bins.cell_start[cell];
            e = bins.cell_start[cell + 1];
            for (int a = b; a < e; ++a) {
                const double4 at = bins.atoms[a];
                const double X = at.x + sx, Y = at.y + sy, Z = at.z + sz;
                cnt += near_box(lo, hi, X, Y, Z, rc2) && !(k == 1 && near_box(tb.lo[0], tb.hi[0], X, Y, Z, rc2));
            }
        }
        int total;
        int off = base + block_exclusive_scan(cnt, scan_tmp, &total);
        for (int a = b; a < e; ++a) {
            const double4 at = bins.atoms[a];
            const double X = at.x + sx, Y = at.y + sy, Z = at.z + sz;
            if (near_box(lo, hi, X, Y, Z, rc2) && !(k == 1 && near_box(tb.lo[0], tb.hi[0], X, Y, Z, rc2))) {
                if (off < cap)
                    cand[off] = make_float4((float)(X - mid[0]), (float)(Y - mid[1]), (float)(Z - mid[2]),
                                            __int_as_float((int)at.w));
                ++off;
            }
        }
        base += total;
    }
    return base;
}

// Candidate atom images of a tile with boxes `tb`: every image within rcut
// of one of its boxes, each once, as float4 in cand[0 .. cap) (w holds the
// bits of the atom's index).  Box 0's pass comes first and is stored
// relative to box 0's middle; box 1's pass, from index *n0 on, relative
// to box 1's, so that offsets stay as small as the boxes (a tile crossing a
// row spans the cell).  Called by the whole block; returns the total count,
// which exceeds cap when the list overflowed (only the first cap are
// stored).  scan_tmp holds blockDim/64 ints.
__device__ __forceinline__ int gather_candidates(const BinState& bins, const TileBoxes& tb, double rcut,
                                                 float4* cand, int cap, int* scan_tmp, int* n0) {
    int base = gather_pass(bins, tb, 0, rcut, cand, cap, scan_tmp, 0);
    *n0 = base;
    if (tb.n == 2) base = gather_pass(bins, tb, 1, rcut, cand, cap, scan_tmp, base);
    return base;
}

// Squared displacements below this (r < 1e-15 A) count as an atom on the
// point (r = 0): it keeps the hardware reciprocal square root away from
// denormal inputs, and the terms left out are below FP32 resolution.
constexpr float kMinR2 = 1e-30f;

// 1/r from r^2 > kMinR2: the hardware's reciprocal square root (about 1 ulp, off to one
// side on the whole, which neighbours share) and a Newton step.
__device__ __forceinline__ float inverse_distance(float r2) {
    const float y = __builtin_amdgcn_rsqf(r2), h = r2 * y;
    return fmaf(fmaf(-h, y, 1.f), 0.5f * y, y);
}

// A lane's point relative to the two origins its candidates are stored
// against: candidate c is compared with at(c).
struct PointFrame {
    float3 p0, p1;
    int n0;
    __device__ __forceinline__ float3 at(int c) const { return c < n0 ? p0 : p1; }
};

__device__ __forceinline__ PointFrame point_frame(const TileBoxes& tb, int n0, double rx, double ry, double rz) {
    PointFrame f;
    f.p0 = make_float3((float)(rx - tb.mid[0][0]), (float)(ry - tb.mid[0][1]), (float)(rz - tb.mid[0][2]));
    f.p1 = tb.n == 2 ? make_float3((float)(rx - tb.mid[1][0]), (float)(ry - tb.mid[1][1]), (float)(rz - tb.mid[1][2]))
                     : f.p0;
    f.n0 = n0;
    return f;
}

// Per-point neighbour lists by all NW waves of the block (called by all of them):
// the indices of the candidates within rc of the lane's point, in candidate order,
// at most kMaxNbr (more sets kErrNbr in *err); invalid lanes get empty lists.  Wave w
// takes the w-th part of the candidates, marks each point's hits in bit masks,
// and writes the marked indices behind those of the waves before it.  Most candidates miss (about 300 for 50 neighbours on a row
// of 64 points): a marked candidate costs one pass over the few bits set, where
// a second scan for the writes cost as much as the first (k_ace_proj 160 ->
// 142 us per 300,007 points).
// Returns the lane's list length; a barrier has passed since the last write.
template <int NW>
__device__ __forceinline__ int build_neighbour_lists_block(const float4* cand, int ncand, const PointFrame& f, float rc,
                                                           bool valid, int lane, int wave,
                                                           unsigned short (*nbr)[kTile], int (*nnbr)[kTile], int* err) {
    constexpr int kWords = (kMaxCand + 32 * NW - 1) / (32 * NW);
    const int begin = ncand * wave / NW, end = ncand * (wave + 1) / NW;
    const float rc2 = rc * rc;
    unsigned mask[kWords];
    int cnt = 0;
#pragma unroll
    for (int w = 0; w < kWords; ++w) {
        mask[w] = 0u;
        const int lo = begin + 32 * w, hi = min(lo + 32, end);
        auto part = [&](int c0, int c1, float3 p) {
#pragma unroll 4
            for (int c = c0; c < c1; ++c) {
                const float4 q = cand[c];
                const float dx = q.x - p.x, dy = q.y - p.y, dz = q.z - p.z;
                mask[w] |= dx * dx + dy * dy + dz * dz < rc2 ? 1u << (c - lo) : 0u;
            }
        };
        const int split = min(max(f.n0, lo), hi);
        part(lo, split, f.p0);
        part(split, hi, f.p1);
        cnt += __popc(mask[w]);
    }
    nnbr[wave][lane] = cnt;
    __syncthreads();
    int at = 0, total = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const int c = nnbr[w][lane];
        if (w < wave) at += c;
        total += c;
    }
#pragma unroll
    for (int w = 0; w < kWords; ++w)
        for (unsigned m = mask[w]; m; m &= m - 1) {
            if (at < kMaxNbr) nbr[at][lane] = (unsigned short)(begin + 32 * w + __ffs(m) - 1);
            ++at;
        }
    if (total > kMaxNbr && wave == 0) atomicOr(err, kErrNbr);
    __syncthreads();
    return valid ? min(total, kMaxNbr) : 0;
}

}  // namespace mala
