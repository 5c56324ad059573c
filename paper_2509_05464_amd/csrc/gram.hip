// casorati_gram: G = S^H S of the Casorati matrix on the gfx950 matrix cores.
//
// With S = A + iB (voxels x frames), Re G = A^T A + B^T B and Im G = A^T B - B^T A.
// G is Hermitian, so only the 32x32 frame tiles (I, J) with I <= J are formed.  A
// workgroup owns a group of four tiles on at most four frame blocks and one voxel range
// (split over the contraction dimension): each stage of the 128 frames is staged in LDS once,
// and each of the four waves forms the four real products Re.Re, Im.Im, Re.Im and Im.Re of
// its own tile with MFMA, so every staged value feeds two tiles' products.  Up to 32 frames
// there is one tile: the four waves then take four quarters of the voxels.
//   FP32 mode       : v_mfma_f32_32x32x2_f32.  A lane's operands of four products are one
//                     16-byte read: a stage keeps the even voxels of each eight ahead of the odd.
//   split-BF16 mode : x = hi + lo with hi = bf16(x), lo = bf16(x - hi) (round to nearest
//                     even), split once when the stage is written to LDS; three
//                     v_mfma_f32_32x32x16_bf16 products hi.hi + hi.lo + lo.hi.
//   split-BF16 x4   : hi.hi + hi.lo + lo.hi + lo.lo.  The three-product form drops
//                     sum_v lo lo^H, a positive semi-definite term of about 2^-18 of the
//                     Gram's trace that biases every eigenvalue below that level; the
//                     fourth product removes it.
//   BF16 mode       : hi.hi only (negative control).
// What bounds it: FP32, the matrix cores (6.6M voxels x 400 frames: 42.4 ms, MFMA busy 0.77; 51.4 ms
// while every load was waited for in a branch of its own); the split modes, LDS traffic beside
// the products (2.1M x 200, four products: 1.9 ms, busy 0.50; 2.76 before).  20 frames x 65536
// voxels: 11 us on 256 workgroups of four busy wavefronts, 192 us on 32 with one.
// Accumulation is FP32 inside each 64-voxel stage and FP64 across stages (a long FP32
// running sum of same-sign terms grows its rounding error with the sum; short blocks
// keep the Gram exact to ~1e-8 of lambda_1, which the clutter subspace near the cutoff
// needs); the partial tiles of all voxel ranges are then summed in FP64 in a fixed
// order (deterministic).
// Workgroups that share a voxel range are placed on the same XCD so the range is read
// from HBM once and served to the other groups from that XCD's L2.
#include <algorithm>
#include <cstring>
#include <mutex>
#include <vector>

#include "fq_common.hpp"

namespace fq {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int GT = 32;            // tile edge, frames
constexpr int GR = 2 * GT;        // LDS stage: 4 frame blocks (2 GR rows)
constexpr int GMAX = 34;          // tile groups at n_t = 512 (136 tiles, 4 per group)
constexpr int KC = 64;            // voxels per LDS stage
constexpr int GRAM_THREADS = 256;
constexpr int NXCD = 8;

// A workgroup's four tiles (one per wavefront; 255 = none) and the at most four frame
// blocks they read (255 = none): the blocks fill the LDS stage's four 32-row slots.
struct GroupTab {
    unsigned char ij[GMAX][4][2];
    unsigned char blk[GMAX][4];
};

struct GramArgs {
    const float2* iq;     // [nt][nv]
    double* part;         // [nsplit][ntiles][2][GT*GT]: Re G, Im G partial tiles
    int64_t nv;
    int64_t chunk;        // voxels per split
    int nt, nb, ntiles, nsplit;
    int ngroups;          // tile groups
    GroupTab tab;
};

// two BF16 terms of two values, packed, with the hardware pair conversion (round to nearest
// even): hi = bf16(x), lo = bf16(x - hi)
__device__ __forceinline__ void split2(float x, float y, unsigned int& hi, unsigned int& lo) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 v = {(__bf16)x, (__bf16)y};
    hi = __builtin_bit_cast(unsigned int, v);
    const bf16x2 r = {(__bf16)(x - __uint_as_float(hi << 16)), (__bf16)(y - __uint_as_float(hi & 0xffff0000u))};
    lo = __builtin_bit_cast(unsigned int, r);
}

// flip the sign bits of 8 packed bf16 values
__device__ __forceinline__ uint4 neg8(uint4 x) {
    return make_uint4(x.x ^ 0x80008000u, x.y ^ 0x80008000u, x.z ^ 0x80008000u, x.w ^ 0x80008000u);
}

template <int MODE>
struct GramShape {
    static constexpr bool SPLIT = MODE != FQ_GRAM_FP32;
    static constexpr int NP = SPLIT ? 2 : 1;                     // terms of a value
    static constexpr int LD = SPLIT ? (KC + 8) * 2 : (KC + 4) * 4;   // LDS row, bytes: 16-byte reads of 8 rows on distinct banks
    static constexpr int PLANE = 2 * GR * LD;                    // bytes: one term of Re or Im of the 128 rows
    static constexpr int LDS = 2 * NP * PLANE;
    // a lane loads 8 consecutive voxels of a frame: one or two 16-byte LDS writes per plane, and
    // the loads of a wavefront stay within 8 rows at a time
    static constexpr int VPT = 8;
    static constexpr int LPR = KC / VPT;                         // lanes per row
    static constexpr int RPP = 64 / LPR;                         // rows per pass
    static constexpr int NPASS = GT / RPP;
};

template <int MODE, bool ONE, bool EVEN>
__global__ void __launch_bounds__(GRAM_THREADS, 2) gram_kernel(const GramArgs a) {
    using S = GramShape<MODE>;
    constexpr int NP = S::NP, PLANE = S::PLANE, VPT = S::VPT;
    __shared__ __align__(16) unsigned char lds[S::LDS];   // planes [Re, Im][term][128 rows][LD]

    // XCD-aware decode: workgroups id, id+8, ... run on one XCD; give them one voxel range.
    const int id = blockIdx.x;
    const int xcd = id % NXCD, loc = id / NXCD;
    const int grp = ONE ? 0 : loc % a.ngroups;
    const int split = (ONE ? loc : loc / a.ngroups) * NXCD + xcd;
    if (split >= a.nsplit) return;
    const int64_t v_begin = (int64_t)split * a.chunk;
    const int64_t v_end = min(a.nv, v_begin + a.chunk);

    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / 64), l = threadIdx.x % 64;
    const int I = ONE ? 0 : a.tab.ij[grp][w][0], J = ONE ? 0 : a.tab.ij[grp][w][1];
    const bool active = I != 255;
    int xrow = w * GT, yrow = w * GT;   // stage rows of blocks I and J
    if (!ONE) {
        xrow = yrow = 0;
#pragma unroll
        for (int sl = 0; sl < 4; ++sl) {
            if (a.tab.blk[grp][sl] == I) xrow = sl * GT;
            if (a.tab.blk[grp][sl] == J) yrow = sl * GT;
        }
    }

    // Re G = Re.Re + Im.Im and Im G = Re.Im - Im.Re accumulate directly (the second term of
    // Im G through a negated operand): FP32 within a stage, FP64 across stages
    floatx16 acc_re, acc_im;
    double sum_re[16], sum_im[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        acc_re[r] = acc_im[r] = 0.0f;
        sum_re[r] = sum_im[r] = 0.0;
    }

    // Wavefront w loads block slot w (one tile: the w-th quarter of the stage's voxels); the
    // next stage is in flight to registers while the current one is multiplied.  The loads of
    // a full stage have no condition on them (frames past the end read the last one: their
    // tile elements are not stored): where lanes or rows were tested, every load sat in a
    // branch of its own that waited for it, and nothing was in flight during the products.
    const int lr = l / S::LPR, lv = (l % S::LPR) * VPT;
    const int lblk = ONE ? 0 : a.tab.blk[grp][w];
    const bool lact = lblk != 255;
    const float2* src[S::NPASS];
#pragma unroll
    for (int p = 0; p < S::NPASS; ++p)
        src[p] = a.iq + (int64_t)min((lact ? lblk : 0) * GT + p * S::RPP + lr, a.nt - 1) * a.nv + v_begin +
                 (ONE ? w * KC : 0) + lv;
    float4 in[S::NPASS][VPT / 2];
    auto load = [&] {
#pragma unroll
        for (int p = 0; p < S::NPASS; ++p) {
#pragma unroll
            for (int q = 0; q < VPT / 2; ++q) {
                if (EVEN) {
                    in[p][q] = reinterpret_cast<const float4*>(src[p])[q];
                } else {   // rows start on 8-byte boundaries
                    const float2 x = src[p][2 * q], y = src[p][2 * q + 1];
                    in[p][q] = make_float4(x.x, x.y, y.x, y.y);
                }
            }
            src[p] += ONE ? 4 * KC : KC;
        }
    };
    // the last, partial stage, of `left` voxels
    auto load_tail = [&](int left) {
        left -= (ONE ? w * KC : 0) + lv;
#pragma unroll
        for (int p = 0; p < S::NPASS; ++p)
#pragma unroll
            for (int q = 0; q < VPT / 2; ++q) {
                float2 x = make_float2(0.f, 0.f), y = x;
                if (2 * q < left) x = src[p][2 * q];
                if (2 * q + 1 < left) y = src[p][2 * q + 1];
                in[p][q] = make_float4(x.x, x.y, y.x, y.y);
            }
    };

    const int i = l % 32, h = l / 32;
    constexpr int STEP = ONE ? 4 * KC : KC;
    const int len = (int)max((int64_t)0, v_end - v_begin), nfull = len / STEP, left = len % STEP;
    if (lact && nfull) load();
    for (int stage = 0; stage < nfull + (left ? 1 : 0); ++stage) {
        __syncthreads();
        if (lact) {
            if (stage == nfull) load_tail(left);
#pragma unroll
            for (int p = 0; p < S::NPASS; ++p) {
                unsigned char* d = lds + (w * GT + p * S::RPP + lr) * S::LD + lv * (S::SPLIT ? 2 : 4);
                if constexpr (!S::SPLIT) {
                    const float4* x = in[p];
                    *reinterpret_cast<float4*>(d) = make_float4(x[0].x, x[1].x, x[2].x, x[3].x);
                    *reinterpret_cast<float4*>(d + 16) = make_float4(x[0].z, x[1].z, x[2].z, x[3].z);
                    *reinterpret_cast<float4*>(d + PLANE) = make_float4(x[0].y, x[1].y, x[2].y, x[3].y);
                    *reinterpret_cast<float4*>(d + PLANE + 16) = make_float4(x[0].w, x[1].w, x[2].w, x[3].w);
                } else {
                    unsigned int re[2][4], im[2][4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        split2(in[p][q].x, in[p][q].z, re[0][q], re[1][q]);
                        split2(in[p][q].y, in[p][q].w, im[0][q], im[1][q]);
                    }
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        *reinterpret_cast<uint4*>(d + t * PLANE) = make_uint4(re[t][0], re[t][1], re[t][2], re[t][3]);
                        *reinterpret_cast<uint4*>(d + (2 + t) * PLANE) = make_uint4(im[t][0], im[t][1], im[t][2], im[t][3]);
                    }
                }
            }
        }
        __syncthreads();
        if (lact && stage + 1 < nfull) load();
        if (!active) continue;
        const unsigned char* X = lds + (xrow + i) * S::LD + h * 16;
        const unsigned char* Y = lds + (yrow + i) * S::LD + h * 16;
        if constexpr (!S::SPLIT) {
#pragma unroll
            for (int kk = 0; kk < KC; kk += 8) {
                const float4 xr = *reinterpret_cast<const float4*>(X + kk * 4);
                const float4 xi = *reinterpret_cast<const float4*>(X + PLANE + kk * 4);
                const float4 yr = *reinterpret_cast<const float4*>(Y + kk * 4);
                const float4 yi = *reinterpret_cast<const float4*>(Y + PLANE + kk * 4);
                auto step = [&](float ar, float ai, float br, float bi) {   // the accumulators take turns
                    acc_re = __builtin_amdgcn_mfma_f32_32x32x2f32(ar, br, acc_re, 0, 0, 0);
                    acc_im = __builtin_amdgcn_mfma_f32_32x32x2f32(ar, bi, acc_im, 0, 0, 0);
                    acc_re = __builtin_amdgcn_mfma_f32_32x32x2f32(ai, bi, acc_re, 0, 0, 0);
                    acc_im = __builtin_amdgcn_mfma_f32_32x32x2f32(-ai, br, acc_im, 0, 0, 0);
                };
                step(xr.x, xi.x, yr.x, yi.x);
                step(xr.y, xi.y, yr.y, yi.y);
                step(xr.z, xi.z, yr.z, yi.z);
                step(xr.w, xi.w, yr.w, yi.w);
            }
        } else {
#pragma unroll
            for (int kk = 0; kk < KC; kk += 16) {
                uint4 xr[2], xi[2], xn[2], yr[2], yi[2];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    xr[t] = *reinterpret_cast<const uint4*>(X + t * PLANE + kk * 2);
                    xi[t] = *reinterpret_cast<const uint4*>(X + (2 + t) * PLANE + kk * 2);
                    yr[t] = *reinterpret_cast<const uint4*>(Y + t * PLANE + kk * 2);
                    yi[t] = *reinterpret_cast<const uint4*>(Y + (2 + t) * PLANE + kk * 2);
                    xn[t] = neg8(xi[t]);
                }
                auto mul = [](const uint4& x, const uint4& y, floatx16& acc) {
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, x),
                                                                  __builtin_bit_cast(bf16x8, y), acc, 0, 0, 0);
                };
                // Re.Re and Re.Im, then Im.Im and -Im.Re; the two accumulators take turns
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const uint4* xa = c ? xi : xr;
                    const uint4* xb = c ? xn : xr;
                    const uint4* ya = c ? yi : yr;
                    const uint4* yb = c ? yr : yi;
                    auto product = [&](int p, int q) {
                        mul(xa[p], ya[q], acc_re);
                        mul(xb[p], yb[q], acc_im);
                    };
                    product(0, 0);
                    if constexpr (MODE != FQ_GRAM_BF16) {
                        product(0, 1);
                        product(1, 0);
                    }
                    if constexpr (MODE == FQ_GRAM_SPLIT4_BF16) product(1, 1);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            sum_re[r] += (double)acc_re[r];
            sum_im[r] += (double)acc_im[r];
            acc_re[r] = acc_im[r] = 0.0f;
        }
    }
    if (ONE) {   // the four waves' sums, in a fixed order
        double* part = reinterpret_cast<double*>(lds);   // [3][16][64], Re then Im
        static_assert(3 * 16 * 64 * sizeof(double) <= S::LDS, "partial sums fit the stage");
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            double* sum = c ? sum_im : sum_re;
            __syncthreads();
            if (w > 0) {
#pragma unroll
                for (int r = 0; r < 16; ++r) part[((w - 1) * 16 + r) * 64 + l] = sum[r];
            }
            __syncthreads();
            if (w == 0) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    sum[r] = (sum[r] + part[r * 64 + l]) + (part[(16 + r) * 64 + l] + part[(32 + r) * 64 + l]);
            }
        }
        if (w > 0) return;
    }
    if (!active) return;

    // 32x32 accumulator layout: lane l holds column l%32, rows 8*(r/4) + 4*(l/32) + r%4
    const int t = I * a.nb - I * (I - 1) / 2 + (J - I);
    const int col = l % 32;
    double* out = a.part + ((int64_t)split * a.ntiles + t) * 2 * (GT * GT);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int row = 8 * (r / 4) + 4 * (l / 32) + (r % 4);
        out[row * GT + col] = sum_re[r];
        out[GT * GT + row * GT + col] = sum_im[r];
    }
}

struct ReduceArgs {
    const double* part;
    double2* gram;        // [nt][nt]
    int nt, nb, ntiles, nsplit;
};

// One thread per element of the partial tiles and per eighth of the voxel ranges (consecutive
// threads read consecutive words of each range's tiles); the eight part sums are added in a
// fixed order (deterministic).  Tile element (i, j) of tile (I, J) is G[f][g], f = 32 I + i,
// g = 32 J + j; elements with f < g are written with their mirror conj(G[f][g]) at G[g][f], the
// diagonal with a zero imaginary part, and the lower half of the diagonal tiles is not read.
constexpr int RED_GROUPS = 8;
__global__ void __launch_bounds__(256) gram_reduce_kernel(const ReduceArgs a) {
    __shared__ double sums[RED_GROUPS][32];
    const int le = threadIdx.x % 32, rg = threadIdx.x / 32;
    const int64_t per_split = (int64_t)a.ntiles * 2 * GT * GT;
    const int64_t e = (int64_t)blockIdx.x * 32 + le;
    double acc = 0.0;
    if (e < per_split)
        for (int sp = rg; sp < a.nsplit; sp += RED_GROUPS) acc += a.part[(int64_t)sp * per_split + e];
    sums[rg][le] = acc;
    __syncthreads();
    if (rg != 0 || e >= per_split) return;
    double tot = sums[0][le];
#pragma unroll
    for (int q = 1; q < RED_GROUPS; ++q) tot += sums[q][le];
    int t = (int)(e / (2 * GT * GT));
    const int rem = (int)(e % (2 * GT * GT));
    const int c = rem / (GT * GT), i = (rem % (GT * GT)) / GT, j = rem % GT;
    int I = 0;
    while (t >= a.nb - I) {   // tile t of the row-major upper triangle -> (I, J)
        t -= a.nb - I;
        ++I;
    }
    const int J = I + t;
    const int f = I * GT + i, g = J * GT + j;
    if (f >= a.nt || g >= a.nt || f > g) return;
    double* G = reinterpret_cast<double*>(a.gram);   // [nt][nt] x (Re, Im)
    if (f == g) {
        G[((int64_t)f * a.nt + g) * 2 + c] = c ? 0.0 : tot;
        return;
    }
    G[((int64_t)f * a.nt + g) * 2 + c] = tot;
    G[((int64_t)g * a.nt + f) * 2 + c] = c ? -tot : tot;
}

struct Plan {
    int nb, ntiles, ngroups, nsplit;
    int64_t chunk;
    size_t bytes;
    GroupTab tab;
};

// Tiles (I <= J) into groups of four that read at most four frame blocks: first every full
// 2x2 block of tiles off the diagonal between the block pairs (2a, 2a+1) and (2b, 2b+1), then
// the remaining tiles in row-major order, each group seeded with the first left and grown by
// the tile that adds the fewest new blocks.  This reaches ceil(ntiles / 4) groups for every
// nb <= 16 (a 2x2 tiling of the triangle needs up to 36% more, its diagonal and edge groups
// being partly empty).
void group_tiles(int nb, Plan& p) {
    std::memset(&p.tab, 255, sizeof(p.tab));
    std::vector<std::pair<int, int>> rest;
    std::vector<char> used(nb * nb, 0);
    int g = 0;
    auto put = [&](int gi, const std::vector<std::pair<int, int>>& ts) {
        int nbk = 0;
        for (size_t w = 0; w < ts.size(); ++w) {
            p.tab.ij[gi][w][0] = (unsigned char)ts[w].first;
            p.tab.ij[gi][w][1] = (unsigned char)ts[w].second;
            for (int x : {ts[w].first, ts[w].second}) {
                bool have = false;
                for (int k = 0; k < nbk; ++k) have |= p.tab.blk[gi][k] == x;
                if (!have) p.tab.blk[gi][nbk++] = (unsigned char)x;
            }
        }
    };
    for (int a2 = 0; a2 + 1 < nb; a2 += 2)
        for (int b2 = a2 + 2; b2 + 1 < nb; b2 += 2) {
            const std::vector<std::pair<int, int>> ts = {{a2, b2}, {a2, b2 + 1}, {a2 + 1, b2}, {a2 + 1, b2 + 1}};
            for (auto& t : ts) used[t.first * nb + t.second] = 1;
            put(g++, ts);
        }
    for (int I = 0; I < nb; ++I)
        for (int J = I; J < nb; ++J)
            if (!used[I * nb + J]) rest.push_back({I, J});
    while (!rest.empty()) {
        std::vector<std::pair<int, int>> ts = {rest.front()};
        rest.erase(rest.begin());
        std::vector<int> blocks = {ts[0].first};
        if (ts[0].second != ts[0].first) blocks.push_back(ts[0].second);
        while (ts.size() < 4) {
            int best = -1, best_add = 3;
            for (size_t c = 0; c < rest.size(); ++c) {
                int add = 0;
                for (int x : {rest[c].first, rest[c].second}) {
                    if (std::find(blocks.begin(), blocks.end(), x) == blocks.end()) ++add;
                }
                if (rest[c].first == rest[c].second && add == 2) add = 1;
                if ((int)blocks.size() + add <= 4 && add < best_add) {
                    best = (int)c;
                    best_add = add;
                }
            }
            if (best < 0) break;
            for (int x : {rest[best].first, rest[best].second})
                if (std::find(blocks.begin(), blocks.end(), x) == blocks.end()) blocks.push_back(x);
            ts.push_back(rest[best]);
            rest.erase(rest.begin() + best);
        }
        put(g++, ts);
    }
    p.ngroups = g;
}

Plan plan(int64_t nv, int nt, size_t max_bytes = 0) {
    Plan p{};
    p.nb = (nt + GT - 1) / GT;
    p.ntiles = p.nb * (p.nb + 1) / 2;
    group_tiles(p.nb, p);
    // about 16384 workgroups (short voxel ranges: the groups of one range stay close enough
    // in step to share its stages through the L2); ranges are whole multiples of 2048 voxels
    int64_t want = std::max<int64_t>(1, 16384 / p.ngroups);
    if (max_bytes) {
        // at most max_bytes of partial tiles: whole multiples of NXCD voxel ranges
        const size_t per_split = (size_t)p.ntiles * 2 * GT * GT * sizeof(double);
        const int64_t cap = (int64_t)(max_bytes / per_split) / NXCD * NXCD;
        want = std::max<int64_t>(1, std::min<int64_t>(want, cap));
    }
    // Few workgroups: as many ranges as fill the 512 places on the chip (two workgroups a
    // compute unit) a whole number of times, down to 256 voxels each.  262144 voxels x 200 frames
    // are 73 ranges x 7 groups, one round, where 2048-voxel ranges made 1.75.
    int64_t rounds = (nv * p.ngroups + 512 * 2048 - 1) / (512 * 2048);
    if (rounds <= 4) {
        const int64_t ranges = std::max<int64_t>(NXCD, 512 * rounds / p.ngroups / NXCD * NXCD);
        want = std::min(ranges, max_bytes ? want : ranges);
        p.chunk = std::max<int64_t>(256, round_up((size_t)((nv + want - 1) / want), 64));
    } else {
        p.chunk = std::max<int64_t>(2048, round_up((size_t)((nv + want - 1) / want), 2048));
    }
    const int64_t ns = (nv + p.chunk - 1) / p.chunk;
    p.nsplit = (int)round_up((size_t)ns, NXCD);
    p.bytes = (size_t)p.nsplit * p.ntiles * 2 * GT * GT * sizeof(double);
    return p;
}

// The least workspace that casorati_gram takes: ranges of whole multiples of 2048 voxels.  It
// grows with n_vox up to 16384 workgroups and drops where the multiple rises beyond (n_t = 512:
// 1020 MiB at 980000 voxels, 527 at 1000000): a workspace for several sizes takes the largest of
// their queries.  With less than plan() asks for, the call runs on as many ranges as fit.
size_t least_bytes(int64_t nv, const Plan& p) {
    const int64_t want = std::max<int64_t>(1, 16384 / p.ngroups);
    const int64_t chunk = round_up((size_t)((nv + want - 1) / want), 2048);
    return round_up((size_t)((nv + chunk - 1) / chunk), NXCD) * p.ntiles * 2 * GT * GT * sizeof(double);
}

}  // namespace
}  // namespace fq

// Partial tiles of casorati_gram_noalloc: a static device array (each GPU the library runs
// on holds its own copy until the process ends).  Host code never passes the symbol
// itself to a kernel: its device address is looked up once per device.
static __device__ __align__(256) unsigned char scratch[FQ_GRAM_SCRATCH_BYTES];

namespace fq {
namespace {
constexpr int MAX_DEVICES = 64;
void* g_scratch_ptr[MAX_DEVICES];
std::mutex g_scratch_mu;

int scratch_for_current_device(void** out) {
    int dev = -1;
    FQ_HIP(hipGetDevice(&dev));
    FQ_REQUIRE(dev >= 0 && dev < MAX_DEVICES, "device ordinal %d out of range", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        FQ_HIP(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        FQ_REQUIRE(ptr != nullptr, "no device address for the Gram scratch array");
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return FQ_OK;
}

using GramFn = void (*)(const GramArgs);
template <int MODE>
GramFn gram_mode_fn(bool one, bool even) {
    if (one) return even ? gram_kernel<MODE, true, true> : gram_kernel<MODE, true, false>;
    return even ? gram_kernel<MODE, false, true> : gram_kernel<MODE, false, false>;
}
GramFn gram_fn(int mode, bool one, bool even) {
    switch (mode) {
        case FQ_GRAM_FP32: return gram_mode_fn<FQ_GRAM_FP32>(one, even);
        case FQ_GRAM_SPLIT_BF16: return gram_mode_fn<FQ_GRAM_SPLIT_BF16>(one, even);
        case FQ_GRAM_SPLIT4_BF16: return gram_mode_fn<FQ_GRAM_SPLIT4_BF16>(one, even);
        default: return gram_mode_fn<FQ_GRAM_BF16>(one, even);
    }
}

int launch_gram(const float* iq, int64_t n_vox, int32_t n_t, int32_t gram_mode, const Plan& p, void* ws,
                double* gram, hipStream_t s) {
    GramArgs ga{};
    ga.iq = reinterpret_cast<const float2*>(iq);
    ga.part = reinterpret_cast<double*>(ws);
    ga.nv = n_vox;
    ga.chunk = p.chunk;
    ga.nt = n_t;
    ga.nb = p.nb;
    ga.ntiles = p.ntiles;
    ga.nsplit = p.nsplit;
    ga.ngroups = p.ngroups;
    ga.tab = p.tab;
    const unsigned nwg = (unsigned)(p.ngroups * p.nsplit);
    const GramFn fn = gram_fn(gram_mode, p.ntiles == 1, n_vox % 2 == 0);
    hipLaunchKernelGGL(fn, dim3(nwg), dim3(GRAM_THREADS), 0, s, ga);
    FQ_LAUNCH_CHECK();
    ReduceArgs ra{reinterpret_cast<const double*>(ws), reinterpret_cast<double2*>(gram), n_t, p.nb, p.ntiles,
                  p.nsplit};
    const int64_t per_split = (int64_t)p.ntiles * 2 * GT * GT;
    hipLaunchKernelGGL(gram_reduce_kernel, dim3((unsigned)((per_split + 31) / 32)), dim3(256), 0, s, ra);
    FQ_LAUNCH_CHECK();
    return FQ_OK;
}

int check_gram_args(const float* iq, int64_t n_vox, int32_t n_t, int32_t gram_mode, double* gram) {
    FQ_REQUIRE(n_t >= 1 && n_t <= FQ_MAX_NT, "n_t must be 1..%d", FQ_MAX_NT);
    FQ_REQUIRE(n_vox >= 1, "n_vox must be >= 1");
    FQ_REQUIRE(gram_mode == FQ_GRAM_FP32 || gram_mode == FQ_GRAM_SPLIT_BF16 || gram_mode == FQ_GRAM_BF16 ||
                   gram_mode == FQ_GRAM_SPLIT4_BF16,
               "bad gram_mode");
    FQ_REQUIRE(iq && gram && aligned16(iq) && aligned16(gram), "null or misaligned pointer");
    return FQ_OK;
}
}  // namespace
}  // namespace fq

using namespace fq;

extern "C" int casorati_gram_noalloc(const float* iq, int64_t n_vox, int32_t n_t, int32_t gram_mode, double* gram,
                                     void* stream) {
    int st = check_gram_args(iq, n_vox, n_t, gram_mode, gram);
    if (st != FQ_OK) return st;
    const Plan p = plan(n_vox, n_t, FQ_GRAM_SCRATCH_BYTES);
    if (p.bytes > FQ_GRAM_SCRATCH_BYTES) {
        set_error("n_t = %d needs %zu bytes of partial tiles, above the %zu-byte static scratch", n_t, p.bytes,
                  (size_t)FQ_GRAM_SCRATCH_BYTES);
        return FQ_E_INVALID;
    }
    void* ws = nullptr;
    if ((st = scratch_for_current_device(&ws)) != FQ_OK) return st;
    return launch_gram(iq, n_vox, n_t, gram_mode, p, ws, gram, as_stream(stream));
}

extern "C" size_t gram_workspace_size(int64_t n_vox, int32_t n_t, int32_t gram_mode) {
    (void)gram_mode;
    if (n_vox < 1 || n_t < 1) return 0;
    const Plan p = plan(n_vox, n_t);
    return std::max(p.bytes, least_bytes(n_vox, p));
}

extern "C" int casorati_gram(const float* iq, int64_t n_vox, int32_t n_t, int32_t gram_mode, void* ws, size_t ws_bytes,
                             double* gram, void* stream) {
    int st = check_gram_args(iq, n_vox, n_t, gram_mode, gram);
    if (st != FQ_OK) return st;
    FQ_REQUIRE(ws && aligned16(ws), "null or misaligned workspace");
    Plan p = plan(n_vox, n_t);
    const size_t least = least_bytes(n_vox, p);
    if (ws_bytes < least) {
        set_error("workspace too small: %zu < %zu bytes", ws_bytes, least);
        return FQ_E_WORKSPACE;
    }
    if (ws_bytes < p.bytes) p = plan(n_vox, n_t, ws_bytes);
    return launch_gram(iq, n_vox, n_t, gram_mode, p, ws, gram, as_stream(stream));
}
