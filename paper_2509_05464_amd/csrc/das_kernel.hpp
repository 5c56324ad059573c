// Delay-and-sum kernel of das_beamform (gfx950), shared by the files that instantiate it
// for the block lengths FB = 1 .. 8 (das_fb*.hip).
//
// One workgroup of 256 threads sums one tile of 512 voxels (two consecutive z per thread)
// for FB frames over all elements and the AT transmits of a pass.  For every (transmit,
// element) the delay rows that the tile touches (FB complex samples each) are staged in
// LDS and every thread takes its taps from there.
//
// Calls too small to fill the chip that way split the elements: a workgroup of 1024 threads
// works as G = 4 or 16 groups on one tile of 256 or 64 voxels, group g sums the elements
// g, g + G, ..., and the groups' sums are added in LDS in a fixed order at the end (16
// wavefronts a workgroup in place of 4, on smaller tiles; no memory and no atomics).
//
//  * Staging is asynchronous: the rows go from the baseband straight to LDS
//    (buffer_load ... lds, no registers), one half of an element's transmits ahead of the
//    half being summed, into two LDS arrays that take turns: one barrier per half.  Rows
//    outside the record read as zero through the buffer descriptor's bounds.  Only the
//    rows between the tile's nearest and farthest delay are fetched.
//  * Delays are 32-bit fixed point with 24 fraction bits: a transmit part per (voxel,
//    transmit) and a receive part per (voxel, element), both relative to integer row
//    bases of the tile and rounded once from FP64.  One integer add gives row and
//    fraction (the fraction, below 2^24, converts to FP32 exactly; its scale 2^-24 is
//    folded into the phase factor).  Windows beyond 248 rows keep whole rows beside it.
//  * The phase exp(i 2 pi fc tau) is a per-(voxel, transmit) factor times a
//    per-(voxel, element) factor, each from an FP64 cycle count.  With few frames
//    (AT * FB <= 16) every transmit keeps its own sums and its factor is applied once at
//    the end instead of once per element.
//
// What bounds it: a unit (voxel, element, transmit, frame) reads 16 bytes from LDS and
// costs 8 FMAs, plus per (voxel, element, transmit) about 12 instructions shared by the FB
// frames; 24 frames of 128^3 voxels x 1024 elements x 9 transmits read 7.4 TB from LDS.
#pragma once

#include <type_traits>

#include "fq_common.hpp"

namespace fq {

constexpr int DAS_MAX_FB = 8;         // frames per block, at most
constexpr int DAS_THREADS = 256;      // one group
constexpr int DAS_SPLIT_THREADS = 1024;
constexpr int DAS_MAX_AT = 9;         // transmits per pass
constexpr int DAS_ROWS = 320;         // rows of one LDS array (half the transmits of a pass)
constexpr int DAS_ROWS_WIDE = 832;    // the same at most, for windows beyond 248 rows (AT <= 2: one window an array)
__host__ __device__ constexpr int das_group_threads(int G) { return G == 1 ? DAS_THREADS : DAS_SPLIT_THREADS / G; }
__host__ __device__ constexpr int das_vz(int G) { return G == 1 ? 2 : 1; }   // voxels per thread, consecutive in z
constexpr int DAS_W_NARROW = 248;     // fixed point with 24 fraction bits holds 256 rows
constexpr int DAS_SLACK = 16;         // bytes after a window (odd row sizes are copied in 16-byte pieces)

// LDS bytes of a row: the 16-byte reads of 16 consecutive rows fall in distinct banks for
// every FB but 4 and 8, whose rows get one 16-byte pad
__host__ __device__ constexpr int das_row_lds(int fb) { return fb == 8 ? 80 : fb == 4 ? 48 : 8 * fb; }

// rows of one LDS array of a group
__host__ __device__ constexpr int das_rows(int G, bool wide, int fb) {
    return wide ? DAS_ROWS_WIDE : G == 1 ? DAS_ROWS : (fb == 8 ? 960 : 1280) / G;
}

struct DasArgs {
    const char* bb;        // baseband [block][A][E][TR][FB] complex64
    float2* iq;            // [F][Nv]
    int nx, ny, nz;
    int sx, sy, sz;        // log2 of the tile's threads along x, y, z (sum 8)
    int ntx, nty;          // tiles along x, y
    int ntiles;            // tiles of the grid
    int64_t nwork;         // (tile, frame block) pairs of this launch
    double x0, y0, z0, dx, dy, dz;
    int nx_el;
    double pitch_x, pitch_y;
    double fs_c, fc_fs;    // fs/c, fc/fs
    int A, E, TR, F;       // TR: rows of a trace (T, or T + 1 where a row of zeros is added)
    int a0;                // first transmit of this pass
    int fb0;               // first global frame block of this launch
    int W;                 // window rows, at most
    int WB;                // bytes between the windows of two transmits
    int accumulate;
    float inv_A;
    double ux[DAS_MAX_AT], uy[DAS_MAX_AT], uz[DAS_MAX_AT], t0s[DAS_MAX_AT];   // t0s = t0 * fs
    uint32_t dzs[DAS_MAX_AT];                                // transmit delay of one z step, fixed point
    int dzr[DAS_MAX_AT];                                     // its whole rows (wide windows)
    float2 zeta[DAS_MAX_AT];                                 // exp(i 2 pi fc uz dz / c)
};

using DasFn = void (*)(const DasArgs);

__device__ __forceinline__ double das_lane(double x, int l) {
    const long long u = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readlane((int)u, l), hi = __builtin_amdgcn_readlane((int)(u >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

template <int AT, int INTERP, int FB, bool WIDE, int G>
__global__ void __launch_bounds__(G == 1 ? DAS_THREADS : DAS_SPLIT_THREADS, G > 1 ? 1 : 3) das_kernel(const DasArgs a) {
    constexpr int VZ = das_vz(G);
    constexpr int TPG = das_group_threads(G), WPG = TPG / 64;   // threads and wavefronts of a group
    constexpr int NT = INTERP ? 4 : 2;         // taps per delay
    constexpr int J0 = INTERP ? -1 : 0;        // first tap offset
    constexpr int SH = 24;                     // fraction bits of a delay
    constexpr uint32_t MASK = (1u << SH) - 1u;
    constexpr int ROWG = 8 * FB;               // row bytes in the baseband
    constexpr int ROWL = das_row_lds(FB);      // row bytes in LDS
    constexpr bool PADDED = ROWL != ROWG;
    constexpr int LPR = ROWL / 16;             // padded: lanes per row, the last one idle
    constexpr int RPI = PADDED ? 64 / LPR : 1; // padded: rows per wavefront-wide copy
    constexpr int H1 = (AT + 1) / 2;           // transmits of the first half
    constexpr bool OWN = AT * FB <= 16;        // every transmit keeps its own sums
    constexpr int NS = OWN ? AT : 1;
    constexpr int LDS_BYTES = WIDE ? 16 : das_rows(G, WIDE, FB) * ROWL;   // of a group
    __shared__ __attribute__((aligned(16))) char ldsA[G * LDS_BYTES];
    __shared__ __attribute__((aligned(16))) char ldsB[G * LDS_BYTES];
    extern __shared__ __attribute__((aligned(16))) char wide_lds[];   // wide: two windows
    const int grp = G == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / TPG);
    char* const winA = WIDE ? wide_lds : ldsA + grp * LDS_BYTES;
    char* const winB = WIDE ? wide_lds + a.WB : ldsB + grp * LDS_BYTES;

    // Workgroup id -> (tile, frame block), tiles fastest.  (Handing each XCD a contiguous
    // run of tiles cut the HBM traffic ~3x but ran 5.6% slower: the neighbouring tiles of one
    // XCD request the same delay rows at the same time.)
    const int64_t g = blockIdx.x;
    const int tile = (int)(g % a.ntiles), fbl = (int)(g / a.ntiles);
    const int fb = a.fb0 + fbl;
    const int txi = tile % a.ntx, tyi = (tile / a.ntx) % a.nty, tzi = tile / (a.ntx * a.nty);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((threadIdx.x % TPG) >> 6);
    // thread -> voxel column: up to 8 x 8 columns per wavefront (neighbouring delays)
    int t = threadIdx.x % TPG;
    const int bx = min(a.sx, 3), by = min(a.sy, 3);
    int lx = t & ((1 << bx) - 1);
    t >>= bx;
    int ly = t & ((1 << by) - 1);
    t >>= by;
    lx |= (t & ((1 << (a.sx - bx)) - 1)) << bx;
    t >>= a.sx - bx;
    ly |= (t & ((1 << (a.sy - by)) - 1)) << by;
    t >>= a.sy - by;
    const int ix = (txi << a.sx) + lx, iy = (tyi << a.sy) + ly, iz0 = ((tzi << a.sz) + t) * VZ;

    // voxels past the grid's edge repeat the last one (their sums are not stored)
    const int ixl = txi << a.sx, iyl = tyi << a.sy, izl = (tzi << a.sz) * VZ;
    const double bx0 = a.x0 + ixl * a.dx, bx1 = a.x0 + min(ixl + (1 << a.sx) - 1, a.nx - 1) * a.dx;
    const double by0 = a.y0 + iyl * a.dy, by1 = a.y0 + min(iyl + (1 << a.sy) - 1, a.ny - 1) * a.dy;
    const double bz0 = a.z0 + izl * a.dz, bz1 = a.z0 + min(izl + (VZ << a.sz) - 1, a.nz - 1) * a.dz;
    const double xv = a.x0 + min(ix, a.nx - 1) * a.dx, yv = a.y0 + min(iy, a.ny - 1) * a.dy;
    double zv[VZ];
#pragma unroll
    for (int k = 0; k < VZ; ++k) zv[k] = a.z0 + min(iz0 + k, a.nz - 1) * a.dz;

    // Transmit delays: tile bounds (uniform) and this thread's voxels.  Lane j of l_tlo
    // holds transmit j's row base, an integer at least one row below its lowest delay, and
    // l_dtx the spread above it in 1/16 rows.
    int l_tlo = 0, l_dtx = 0;
    uint32_t ftx[AT];
    int itx[AT];                               // wide windows: whole rows, ftx the fraction
    float2 ptx[AT];
    const uint32_t smax = ((uint32_t)(a.W - NT) << SH) | MASK;
    constexpr double ONE = (double)(1u << SH);
    double tlo = 1e300;
#pragma unroll
    for (int j = 0; j < AT; ++j) {
        const double lo = (a.ux[j] * (a.ux[j] > 0 ? bx0 : bx1) + a.uy[j] * (a.uy[j] > 0 ? by0 : by1) + a.uz[j] * bz0) *
                              a.fs_c - a.t0s[j];
        const double hi = (a.ux[j] * (a.ux[j] > 0 ? bx1 : bx0) + a.uy[j] * (a.uy[j] > 0 ? by1 : by0) + a.uz[j] * bz1) *
                              a.fs_c - a.t0s[j];
        const double fl = floor(lo) - 1.0;
        tlo = fmin(tlo, fl);
        if (lane == j) {
            l_tlo = (int)fl;
            l_dtx = (int)ceil((hi - fl) * 16.0);
        }
        const double x = (a.ux[j] * xv + a.uy[j] * yv + a.uz[j] * zv[0]) * a.fs_c - a.t0s[j];
        const double xf = WIDE ? floor(x) : fl;
        itx[j] = WIDE ? (int)(xf - fl) : 0;
        ftx[j] = (uint32_t)fma(x - xf, ONE, 0.5);
        float2 p = cis_cycles(x * a.fc_fs);
        if (!INTERP) p = make_float2(p.x * (1.0f / ONE), p.y * (1.0f / ONE));   // the weights' scale
        ptx[j] = p;
    }

    float2 acc[NS][VZ][FB];
#pragma unroll
    for (int j = 0; j < NS; ++j)
#pragma unroll
        for (int k = 0; k < VZ; ++k)
#pragma unroll
            for (int q = 0; q < FB; ++q) acc[j][k][q] = make_float2(0.0f, 0.0f);

    const int ny_el = a.E / a.nx_el;
    // A tile whose nearest delay lies past the record sums nothing.  (Its rows' byte offsets could
    // also wrap at 2^32; a tile that reaches back into the record is too near for that.)
    const double hx = fabs(0.5 * (a.nx_el - 1) * a.pitch_x), hy = fabs(0.5 * (ny_el - 1) * a.pitch_y);
    const double nx = fmax(fmax(bx0 - hx, -hx - bx1), 0.0), ny = fmax(fmax(by0 - hy, -hy - by1), 0.0);
    const bool past = __builtin_amdgcn_readfirstlane(
        tlo + floor(sqrt(nx * nx + ny * ny + bz0 * bz0) * a.fs_c) - 2.0 > (double)a.TR);
    const int64_t trace_bytes = (int64_t)a.TR * ROWG;
    const char* bb = a.bb + ((int64_t)fbl * a.A + a.a0) * a.E * trace_bytes;

    // Element geometry, 64 elements at a time (one per lane): position, the integer row
    // below the tile's nearest receive delay and the spread above it in 1/16 rows.
    double l_px = 0.0, l_py = 0.0;
    int l_lo = 0, l_dr = 0;
    double pex_n = 0.0, pey_n = 0.0;   // of the element whose rows are requested next
    int rlo_n = 0, drx_n = 0;
    // n counts the elements of this group
    const int n_el = past ? 0 : G == 1 ? a.E : (a.E - grp + G - 1) / G;
    auto element = [&](int n) {
        if ((n & 63) == 0) {
            const int el = min((n + lane) * G + grp, a.E - 1);
            l_px = ((el % a.nx_el) - 0.5 * (a.nx_el - 1)) * a.pitch_x;
            l_py = ((el / a.nx_el) - 0.5 * (ny_el - 1)) * a.pitch_y;
            const double cx = fmin(fmax(l_px, bx0), bx1) - l_px, cy = fmin(fmax(l_py, by0), by1) - l_py;
            const double fx = fmax(fabs(bx0 - l_px), fabs(bx1 - l_px)), fy = fmax(fabs(by0 - l_py), fabs(by1 - l_py));
            const double rlo = floor(sqrt(cx * cx + cy * cy + bz0 * bz0) * a.fs_c) - 1.0;
            l_lo = (int)rlo;
            l_dr = (int)ceil((sqrt(fx * fx + fy * fy + bz1 * bz1) * a.fs_c - rlo) * 16.0);
        }
        const int l = n & 63;
        pex_n = das_lane(l_px, l);
        pey_n = das_lane(l_py, l);
        rlo_n = __builtin_amdgcn_readlane(l_lo, l);
        drx_n = __builtin_amdgcn_readlane(l_dr, l);
    };

    // Request the rows of transmits [j0, j1) of an element into one of the LDS arrays.
    typedef __attribute__((address_space(3))) void lds_void;
    const int lrow = lane / LPR, lcol = lane % LPR;   // padded copies
    auto request = [&](char* win, auto J0C, auto J1C, int n, int rlo, int drx) {
        const int e = G == 1 ? n : n * G + grp;
        constexpr int ja = decltype(J0C)::value, jb = decltype(J1C)::value;
#pragma unroll
        for (int j = ja; j < jb; ++j) {
            const int first = __builtin_amdgcn_readlane(l_tlo, j) + rlo + J0;
            const int rows = min(a.W, ((__builtin_amdgcn_readlane(l_dtx, j) + drx) >> 4) + NT + 1);
            const char* src = bb + ((int64_t)j * a.E + e) * trace_bytes;
            auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(src), 0, (int)trace_bytes, 0x00020000);
            char* dst = win + (j - ja) * a.WB;
            if (PADDED) {
                for (int r0 = wave * RPI; r0 < rows; r0 += WPG * RPI) {
                    if (lcol < LPR - 1 && lrow < RPI && r0 + lrow < rows)
                        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void*)(dst + r0 * ROWL), 16,
                                                                 (first + r0 + lrow) * ROWG + lcol * 16, 0, 0, 0);
                }
            } else {
                const int begin = (first * ROWG) & ~15;   // odd row sizes start up to 8 bytes early
                const int pieces = ((first + rows) * ROWG - begin + 15) >> 4;
                for (int p0 = wave * 64; p0 < pieces; p0 += TPG) {
                    if (p0 + lane < pieces)
                        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void*)(dst + p0 * 16), 16,
                                                                 begin + (p0 + lane) * 16, 0, 0, 0);
                }
            }
        }
    };

    uint32_t frx[VZ];
    int irx[VZ];
    float2 prx[VZ];
    // receive geometry of the thread's voxels (FP64 distance, shared by all transmits)
    auto receive = [&](double pex, double pey, int rlo) {
        const double ddx = xv - pex, ddy = yv - pey;
        const double dxy2 = ddx * ddx + ddy * ddy;
        const double off = 0.5 - (double)rlo * ONE;
#pragma unroll
        for (int k = 0; k < VZ; ++k) {
            const double xr = sqrt_nr(fma(zv[k], zv[k], dxy2)) * a.fs_c;
            if (WIDE) {
                const double xf = floor(xr);
                irx[k] = (int)xf - rlo;
                frx[k] = (uint32_t)fma(xr - xf, ONE, 0.5);
            } else {
                frx[k] = (uint32_t)fma(xr, ONE, off);
            }
            prx[k] = cis_cycles(xr * a.fc_fs);
        }
    };

    // Sum transmits [j0, j1) of an element from one of the LDS arrays.
    auto sum = [&](const char* win, auto J0C, auto J1C, int rlo) {
        constexpr int ja = decltype(J0C)::value, jb = decltype(J1C)::value;
#pragma unroll
        for (int j = ja; j < jb; ++j) {
            const char* wj = win + (j - ja) * a.WB;
            if (ROWG % 16) wj += ((__builtin_amdgcn_readlane(l_tlo, j) + rlo + J0) * ROWG) & 15;
#pragma unroll
            for (int k = 0; k < VZ; ++k) {
                // The window holds every tap of the tile; the bound keeps the LDS reads in it
                // whatever the input.
                uint32_t x = ftx[j] + frx[k] + (k ? a.dzs[j] : 0u);
                if (!WIDE) x = min(x, smax);
                uint32_t row = x >> SH;
                if (WIDE) row = (uint32_t)min(max(itx[j] + irx[k] + (int)row + (k ? a.dzr[j] : 0), 0), a.W - NT);
                const char* rp = wj + row * (uint32_t)ROWL;
                const float fr = (float)(x & MASK);
                float w[NT];
                if (INTERP == 0) {
                    w[0] = (float)ONE - fr;   // exact
                    w[1] = fr;
                } else {
                    const float al = fr * (1.0f / ONE);
                    const float a2 = al * al, a3 = a2 * al;
                    w[0] = 0.5f * (-a3 + 2.0f * a2 - al);
                    w[1] = 0.5f * (3.0f * a3 - 5.0f * a2 + 2.0f);
                    w[2] = 0.5f * (-3.0f * a3 + 4.0f * a2 + al);
                    w[3] = 0.5f * (a3 - a2);
                }
                float2 P = prx[k];
                if (!OWN) {
                    P = cmul(ptx[j], P);
                    if (k > 0) P = cmul(P, a.zeta[j]);
                }
                // taps combined with the real weights, then rotated: acc += P * sum_t w_t b_t
                auto add = [&](float2& c, float bx_, float by_) {
                    c.x = fmaf(P.x, bx_, c.x);
                    c.x = fmaf(-P.y, by_, c.x);
                    c.y = fmaf(P.x, by_, c.y);
                    c.y = fmaf(P.y, bx_, c.y);
                };
                if (FB % 2 == 0) {
#pragma unroll
                    for (int q = 0; q < FB; q += 2) {
                        const float4 b0 = *reinterpret_cast<const float4*>(rp + 8 * q);
                        float4 B = make_float4(w[0] * b0.x, w[0] * b0.y, w[0] * b0.z, w[0] * b0.w);
#pragma unroll
                        for (int s = 1; s < NT; ++s) {
                            const float4 b = *reinterpret_cast<const float4*>(rp + s * ROWL + 8 * q);
                            B.x = fmaf(w[s], b.x, B.x);
                            B.y = fmaf(w[s], b.y, B.y);
                            B.z = fmaf(w[s], b.z, B.z);
                            B.w = fmaf(w[s], b.w, B.w);
                        }
                        add(acc[OWN ? j : 0][k][q], B.x, B.y);
                        add(acc[OWN ? j : 0][k][q + 1 < FB ? q + 1 : q], B.z, B.w);
                    }
                } else {
#pragma unroll
                    for (int q = 0; q < FB; ++q) {
                        const float2 b0 = *reinterpret_cast<const float2*>(rp + 8 * q);
                        float2 B = make_float2(w[0] * b0.x, w[0] * b0.y);
#pragma unroll
                        for (int s = 1; s < NT; ++s) {
                            const float2 b = *reinterpret_cast<const float2*>(rp + s * ROWL + 8 * q);
                            B.x = fmaf(w[s], b.x, B.x);
                            B.y = fmaf(w[s], b.y, B.y);
                        }
                        add(acc[OWN ? j : 0][k][q], B.x, B.y);
                    }
                }
                // the sums end here: deferred past the next barrier, the taps would pile up in registers
#pragma unroll
                for (int q = 0; q < FB; ++q) asm volatile("" : "+v"(acc[OWN ? j : 0][k][q].x), "+v"(acc[OWN ? j : 0][k][q].y));
            }
        }
    };
    // this wavefront's requests have landed and every wavefront is done with the other array
    auto arrive = [] {
        __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
        __syncthreads();
    };

    using I0 = std::integral_constant<int, 0>;
    using IH = std::integral_constant<int, H1>;
    using IA = std::integral_constant<int, AT>;
    // (a group that is out of elements keeps the barriers of the others)
    const int n_max = past ? 0 : G == 1 ? a.E : (a.E + G - 1) / G;
    element(0);
    if (n_el > 0) request(winA, I0{}, IH{}, 0, rlo_n, drx_n);
    if (AT > 1) {
        for (int n = 0; n < n_max; ++n) {
            const bool live = G == 1 || n < n_el;
            const double pex = pex_n, pey = pey_n;
            const int rlo = rlo_n, drx = drx_n;
            arrive();
            if (live) {
                request(winB, IH{}, IA{}, n, rlo, drx);
                receive(pex, pey, rlo);
                sum(winA, I0{}, IH{}, rlo);
            }
            arrive();
            if (n + 1 < n_el) {
                element(n + 1);
                request(winA, I0{}, IH{}, n + 1, rlo_n, drx_n);
            }
            if (live) sum(winB, IH{}, IA{}, rlo);
        }
    } else {
        for (int n = 0; n < n_max; n += 2) {   // one transmit: the arrays take turns by element
            double pex = pex_n, pey = pey_n;
            int rlo = rlo_n;
            arrive();
            if (n + 1 < n_el) {
                element(n + 1);
                request(winB, I0{}, IH{}, n + 1, rlo_n, drx_n);
            }
            if (G == 1 || n < n_el) {
                receive(pex, pey, rlo);
                sum(winA, I0{}, IH{}, rlo);
            }
            if (n + 1 >= n_max) break;
            pex = pex_n;
            pey = pey_n;
            rlo = rlo_n;
            arrive();
            if (n + 2 < n_el) {
                element(n + 2);
                request(winA, I0{}, IH{}, n + 2, rlo_n, drx_n);
            }
            if (G == 1 || n + 1 < n_el) {
                receive(pex, pey, rlo);
                sum(winB, I0{}, IH{}, rlo);
            }
        }
    }

    // every transmit's own sums, rotated
    float2 tot[VZ][FB];
#pragma unroll
    for (int k = 0; k < VZ; ++k)
#pragma unroll
        for (int q = 0; q < FB; ++q) {
            float2 s = acc[0][k][q];
            if (OWN) {
                s = make_float2(0.0f, 0.0f);
#pragma unroll
                for (int j = 0; j < AT; ++j) {
                    const float2 P = k ? cmul(ptx[j], a.zeta[j]) : ptx[j];
                    const float2 p = cmul(P, acc[OWN ? j : 0][k][q]);
                    s.x += p.x;
                    s.y += p.y;
                }
            }
            tot[k][q] = s;
        }
    if (G > 1) {   // the groups' sums: group 0 adds the others' in order
        static_assert(G == 1 || (size_t)(G - 1) * TPG * FB * VZ * 8 <= 2 * (size_t)G * LDS_BYTES, "sums fit the windows");
        constexpr int PER = G * LDS_BYTES / (TPG * 8);   // values (of a thread) that one array holds
        float2* sA = reinterpret_cast<float2*>(ldsA);
        float2* sB = reinterpret_cast<float2*>(ldsB);
        auto place = [&](int i) -> float2& { return i < PER ? sA[i * TPG + (threadIdx.x % TPG)] : sB[(i - PER) * TPG + (threadIdx.x % TPG)]; };
        __syncthreads();
        if (grp > 0) {
#pragma unroll
            for (int q = 0; q < FB; ++q) place((grp - 1) * FB + q) = tot[0][q];
        }
        __syncthreads();
        if (grp > 0) return;
#pragma unroll 1
        for (int g = 1; g < G; ++g)
#pragma unroll
            for (int q = 0; q < FB; ++q) {
                const float2 x = place((g - 1) * FB + q);
                tot[0][q].x += x.x;
                tot[0][q].y += x.y;
            }
    }

    if (ix >= a.nx || iy >= a.ny) return;
    const int64_t nv = (int64_t)a.nx * a.ny * a.nz;
#pragma unroll
    for (int k = 0; k < VZ; ++k) {
        const int iz = iz0 + k;
        if (iz >= a.nz) break;
        const int64_t v = ix + (int64_t)a.nx * (iy + (int64_t)a.ny * iz);
#pragma unroll
        for (int q = 0; q < FB; ++q) {
            const int f = fb * FB + q;
            if (f >= a.F) break;
            const float2 s = tot[k][q];
            float2* o = a.iq + (int64_t)f * nv + v;
            float2 r = make_float2(s.x * a.inv_A, s.y * a.inv_A);
            if (a.accumulate) {
                const float2 old = *o;
                r.x += old.x;
                r.y += old.y;
            }
            *o = r;
        }
    }
}

// Kernel of a pass of `at` transmits and blocks of FB frames.
template <int FB, bool WIDE, int G>
DasFn das_pick_at(int at, int interp) {
    switch (at) {
        case 1: return interp ? das_kernel<1, 1, FB, WIDE, G> : das_kernel<1, 0, FB, WIDE, G>;
        case 2: return interp ? das_kernel<2, 1, FB, WIDE, G> : das_kernel<2, 0, FB, WIDE, G>;
        default: break;
    }
    if constexpr (!WIDE) {
        switch (at) {
            case 3: return interp ? das_kernel<3, 1, FB, WIDE, G> : das_kernel<3, 0, FB, WIDE, G>;
            case 4: return interp ? das_kernel<4, 1, FB, WIDE, G> : das_kernel<4, 0, FB, WIDE, G>;
            case 5: return interp ? das_kernel<5, 1, FB, WIDE, G> : das_kernel<5, 0, FB, WIDE, G>;
            case 6: return interp ? das_kernel<6, 1, FB, WIDE, G> : das_kernel<6, 0, FB, WIDE, G>;
            case 7: return interp ? das_kernel<7, 1, FB, WIDE, G> : das_kernel<7, 0, FB, WIDE, G>;
            case 8: return interp ? das_kernel<8, 1, FB, WIDE, G> : das_kernel<8, 0, FB, WIDE, G>;
            default: return interp ? das_kernel<9, 1, FB, WIDE, G> : das_kernel<9, 0, FB, WIDE, G>;
        }
    }
    return nullptr;
}
template <int FB>
DasFn das_pick(int at, int interp, bool wide, int groups) {
    if (wide) return das_pick_at<FB, true, 1>(at, interp);
    if (groups == 1) return das_pick_at<FB, false, 1>(at, interp);
    return groups == 4 ? das_pick_at<FB, false, 4>(at, interp) : das_pick_at<FB, false, 16>(at, interp);
}

// one per das_fb*.hip
DasFn das_fn1(int at, int interp, bool wide, int groups);
DasFn das_fn2(int at, int interp, bool wide, int groups);
DasFn das_fn3(int at, int interp, bool wide, int groups);
DasFn das_fn4(int at, int interp, bool wide, int groups);
DasFn das_fn5(int at, int interp, bool wide, int groups);
DasFn das_fn6(int at, int interp, bool wide, int groups);
DasFn das_fn7(int at, int interp, bool wide, int groups);
DasFn das_fn8(int at, int interp, bool wide, int groups);

}  // namespace fq
