// Learned slow-time clutter filter on gfx950: BF16 matrix-core training and inference.
//
// Network (per voxel series, T frames): x = [Re, Im](s)/r, r = sqrt(mean |s|^2 + eps),
//   h1 = GELU(conv9(x; W1[32][2][9]) + b1), h2 = GELU(conv9(h1; W2) + b2),
//   h3 = GELU(conv9(h2; W3) + b3),          y  = W4[2][32] h3 + b4,
// blood estimate r (y0 + i y1).  conv9 has "same" zero padding (taps t-4..t+4).
//
// Each 32->32 conv is an implicit GEMM on v_mfma_f32_32x32x16_bf16:
//   C[o][t] = sum_kk A[o][kk] B[kk][t],  kk = k*32 + i (tap-major),
//   A = weights (held in registers as MFMA fragments for the whole kernel),
//   B[kk][t] = h[t + k - 4][i] read from a time-major LDS image h[row][32 channels]
//   (row = t + 4): the 8 consecutive kk a lane supplies are 8 consecutive channels of
//   one row, one 16-byte LDS read.  The 2-channel input layer uses an 8-channel image
//   (kk = k*8 + i, channels 2..7 zero).  Output C tiles are 32 channels x 32 frames.
// Backward: dgrad is the same conv on dz with the transposed, time-flipped kernel
// (A[i][k'*32+o] = W[o][i][8-k']); wgrad reduces over time,
//   dW[o][i][k] = sum_t dz[t][o] h[t+k-4][i],
// with K = time: its operands come from the time-major images by transposing LDS reads.
// Rounding points (round to nearest even): weights (BF16 copy kept by Adam), the
// network input, every stored activation (z and h of layers 1-3) and every dz; all
// accumulation, biases, GELU and the output layer are FP32.
#include "fq_common.hpp"

namespace fq {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));
typedef unsigned short u16x4 __attribute__((ext_vector_type(4)));

constexpr int CH = 32, KW = 9, PADT = 4;
constexpr int OFF_W1 = 0, OFF_B1 = 576, OFF_W2 = 608, OFF_B2 = 9824, OFF_W3 = 9856, OFF_B3 = 19072,
              OFF_W4 = 19104, OFF_B4 = 19168, NPAR = 19170;
constexpr int K1C = 2;    // layer-1 K chunks: 9 taps x 2 channels = 18 -> 32
constexpr int K2C = 18;   // 32->32 K chunks: 9 taps x 32 channels = 288
constexpr int NWB = 256;          // workgroups of the backward pass, at most
constexpr int PART = NPAR + 1;    // partial gradient of a workgroup, then its loss sum

__device__ __forceinline__ unsigned short f2bf(float x) {
    unsigned int u = __float_as_uint(x);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}
__device__ __forceinline__ float bf2f(unsigned short b) { return __uint_as_float((unsigned int)b << 16); }
// GELU in its tanh form (Hendrycks & Gimpel): GELU(z) = z (1 + tanh u)/2, u = C (z + A z^3),
// C = sqrt(2/pi), A = 0.044715.  With (1 + tanh u)/2 = 1/(1 + exp(-2u)) and exp(-2u) =
// 2^(z (K1 + K3 z^2)), K1 = -2 C log2 e, K3 = -2 C A log2 e: three multiply/FMAs, one
// exponential, one add, one reciprocal and a product (z -> -inf: 2^y overflows, the
// reciprocal gives 0 and GELU -0; z -> +inf: GELU = z).
constexpr float GELU_K1 = -2.3022081982f, GELU_K3 = -0.10294324f;
__device__ __forceinline__ float gelu_fwd(float z) {
    const float y = z * fmaf(GELU_K3, z * z, GELU_K1);
    return z * __builtin_amdgcn_rcpf(__builtin_amdgcn_exp2f(y) + 1.0f);
}
// two floats to BF16 (round to nearest even) with the hardware pair conversion
__device__ __forceinline__ unsigned int f2bf2(float lo, float hi) {
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 v = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(unsigned int, v);
}
// d GELU / dz = s + 2 C z s (1 - s) (1 + 3 A z^2), s = (1 + tanh u)/2; the hardware
// exponential and reciprocal (1 ulp each) are far below the BF16 rounding of the product
__device__ __forceinline__ float gelu_grad(float z) {
    const float z2 = z * z;
    const float s = __builtin_amdgcn_rcpf(__builtin_amdgcn_exp2f(z * fmaf(GELU_K3, z2, GELU_K1)) + 1.0f);
    return fmaf(1.5957691216f * z * s * (1.0f - s), fmaf(0.134145f, z2, 1.0f), s);
}
__device__ __forceinline__ float wave_sum(float v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}
__device__ __forceinline__ floatx16 mfma(const u16x8& a, const u16x8& b, const floatx16& c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c,
                                                   0, 0, 0);
}

struct Geo {
    int T, TT, TP;   // frames, 32-frame tiles, image rows (32*TT + 8)
    __device__ Geo(int t) : T(t), TT((t + 31) / 32), TP(32 * ((t + 31) / 32) + 8) {}
};

// per-series activation record (u16): h0 [T][2] hi terms, [T][2] lo terms (padded to 8) |
// z1 h1 z2 h2 z3 h3, T*32 each; every slot starts on a 16-byte boundary.  A slot holds its
// 32-frame tiles in the order the accumulators hold them, so that one 16-byte store or load
// per lane and half tile moves contiguous memory: piece g of lane (frame j, half h) has
// channels 8 (2g + e/4) + 4h + e%4, e = 0..7, at ((g nf + j) 2 + h) 8 of the tile, nf the
// frames of the tile.
__host__ __device__ inline int64_t h0_len(int T) { return ((int64_t)4 * T + 7) / 8 * 8; }
__host__ __device__ inline int64_t act_stride(int T) { return h0_len(T) + (int64_t)6 * T * CH; }
__host__ __device__ inline int64_t act_off(int which, int T) {   // 0:h0 1:z1 2:h1 3:z2 4:h2 5:z3 6:h3
    return which == 0 ? 0 : h0_len(T) + (int64_t)(which - 1) * T * CH;
}

__device__ __forceinline__ int64_t act_piece(int which, int T, int u, int g, int j, int h) {
    return act_off(which, T) + u * 1024 + ((g * min(32, T - 32 * u) + j) * 2 + h) * 8;
}

// ---------------------------------------------------------------- fragment loads
// A lane's 8 channels x 9 taps of a chunk pair are 72 consecutive weights (nine 16-byte
// loads; OFF_W2, OFF_W3 and the row length are multiples of 8).
__device__ void frag_fwd32(const uint16_t* wb, int base, int l, u16x8* fr) {
    const int o = l % 32, h = l / 32;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const u16x8* src = reinterpret_cast<const u16x8*>(wb + base + o * 288 + (16 * b + 8 * h) * 9);
        u16x8 row[KW];
#pragma unroll
        for (int m = 0; m < KW; ++m) row[m] = src[m];
#pragma unroll
        for (int k = 0; k < KW; ++k)
#pragma unroll
            for (int q = 0; q < 8; ++q) fr[2 * k + b][q] = row[(q * 9 + k) / 8][(q * 9 + k) % 8];
    }
}
// 32x32 accumulator layout: lane l holds frame column l%32 and channel rows
// 8*(r/4) + 4*(l/32) + r%4, r = 0..15 (four groups of four consecutive channels).
__device__ __forceinline__ int acc_row(int r, int l) { return 8 * (r / 4) + 4 * (l / 32) + (r % 4); }

// ---------------------------------------------------------------- forward
struct FwdArgs {
    const float* w;
    const uint16_t* wb;
    const float2* x;      // [T][N]
    uint16_t* act;        // or null
    float2* y;            // [T][N] or null
    float* pd;            // [N] or null
    int64_t N;
    int T;
    float eps;
};

// An FP32 bias enters the products exactly as three BF16 terms (hi + mid + lo = b: each
// split leaves a remainder with 8 fewer significant bits), each times a B entry of 1.
__device__ __forceinline__ void split3(float b, unsigned short* o) {
    o[0] = f2bf(b);
    const float r1 = b - bf2f(o[0]);
    o[1] = f2bf(r1);
    o[2] = f2bf(r1 - bf2f(o[1]));
}
constexpr unsigned int BF_ONE2 = 0x3F803F80u;   // two BF16 ones
// Row stride (elements) of the forward pass's 32-channel image: 80 bytes, so the 16-byte
// reads of consecutive rows by consecutive lanes fall in distinct banks (a 64-byte stride
// puts every other row, or every fourth, on the same banks).
constexpr int RS = 40;

// input layer: kk = 2k + i (tap-major over the 2 input channels), 18 used of 32; the bias
// terms sit at kk = 18, 19, 20 (chunk 1, lanes h = 0, elements 2..4)
__device__ void frag_fwd1(const uint16_t* wb, const float* w, int l, u16x8* fr) {
    const int o = l % 32, h = l / 32;
#pragma unroll
    for (int c = 0; c < K1C; ++c) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int kk = 16 * c + 8 * h + q, k = kk / 2, i = kk % 2;
            fr[c][q] = k < KW ? wb[OFF_W1 + o * 18 + i * 9 + k] : (unsigned short)0;
        }
    }
    unsigned short bs[3];
    split3(w[OFF_B1 + o], bs);
    if (h == 0) {
        fr[1][2] = bs[0];
        fr[1][3] = bs[1];
        fr[1][4] = bs[2];
    }
}
// bias chunk of a 32->32 layer (kk = 288..290, lanes h = 0)
__device__ u16x8 frag_bias(const float* w, int off, int l) {
    u16x8 fr;
#pragma unroll
    for (int q = 0; q < 8; ++q) fr[q] = 0;
    unsigned short bs[3];
    split3(w[off + l % 32], bs);
    if (l < 32) {
        fr[0] = bs[0];
        fr[1] = bs[1];
        fr[2] = bs[2];
    }
    return fr;
}
// output layer as a 32-row product (rows 0, 1 used) over the 32 channels of h3 in the
// order the layer-3 accumulator holds them: chunk c, element e is channel
// 8 (2c + e/4) + 4h + e%4
__device__ void frag_out(const uint16_t* wb, int l, u16x8* fr) {
    const int o = l % 32, h = l / 32;
#pragma unroll
    for (int c = 0; c < 2; ++c) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int ch = 8 * (2 * c + e / 4) + 4 * h + e % 4;
            fr[c][e] = o < 2 ? wb[OFF_W4 + o * CH + ch] : (unsigned short)0;
        }
    }
}

// the input layer's conv: 2-channel image, 4 bytes per row; a lane's 8 consecutive kk are
// taps 8c + 4h .. 8c + 4h + 3 of both channels, 16 contiguous bytes (4-byte aligned)
// The input is two BF16 terms per value (hi = bf16(x), lo = bf16(x - hi)): the same
// weights multiply the hi image and the lo image.
__device__ __forceinline__ floatx16 conv2(const unsigned short* img, const unsigned short* img_lo, int t0,
                                         const u16x8* fr, int l) {
    const int j = l % 32, h = l / 32;
    const unsigned int* im = reinterpret_cast<const unsigned int*>(img);
    const unsigned int* il = reinterpret_cast<const unsigned int*>(img_lo);
    floatx16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
    for (int c = 0; c < K1C; ++c) {
        const int row = t0 + j + 8 * c + 4 * h;
        uint4 w = make_uint4(im[row], im[row + 1], im[row + 2], im[row + 3]);
        uint4 wl = make_uint4(il[row], il[row + 1], il[row + 2], il[row + 3]);
        if (c == 1 && h == 0) {   // B = 1 against the bias terms, once
            w.y = w.z = BF_ONE2;
            wl.y = wl.z = 0u;
        }
        acc = mfma(fr[c], __builtin_bit_cast(u16x8, w), acc);
        acc = mfma(fr[c], __builtin_bit_cast(u16x8, wl), acc);
    }
    return acc;
}
// a 32->32 conv tile with its bias chunk
__device__ __forceinline__ floatx16 conv32b(const unsigned short* img, int t0, const u16x8* fr, const u16x8& fb,
                                           int l) {
    const int j = l % 32, h = l / 32;
    u16x8 one;
#pragma unroll
    for (int q = 0; q < 8; ++q) one[q] = q < 3 ? (unsigned short)0x3F80 : (unsigned short)0;
    floatx16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
    __builtin_amdgcn_s_setprio(1);
    acc = mfma(fb, one, acc);
#pragma unroll
    for (int c = 0; c < K2C; ++c) {
        const int k = c / 2, ch0 = (c % 2) * 16 + 8 * h;
        const u16x8 b = *reinterpret_cast<const u16x8*>(img + (t0 + j + k) * RS + ch0);
        acc = mfma(fr[c], b, acc);
    }
    __builtin_amdgcn_s_setprio(0);
    return acc;
}

// GELU of one 32x32 output tile u (this lane: frame 32 u + j, channels 8q + 4h + p),
// rounded to BF16 (zero for frames past the end: they are the next layer's padding).  With
// an activation record, z and h of the layer are stored too.
template <bool ACT>
__device__ __forceinline__ void gelu_tile(const floatx16& acc, uint16_t* actv, int layer, int u, int T, int j, int h,
                                          uint2* hv) {
    const bool live = 32 * u + j < T;
    uint2 zv[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float z[4] = {acc[4 * q], acc[4 * q + 1], acc[4 * q + 2], acc[4 * q + 3]};
        hv[q] = live ? make_uint2(f2bf2(gelu_fwd(z[0]), gelu_fwd(z[1])), f2bf2(gelu_fwd(z[2]), gelu_fwd(z[3])))
                     : make_uint2(0u, 0u);
        if (ACT) zv[q] = make_uint2(f2bf2(z[0], z[1]), f2bf2(z[2], z[3]));
    }
    if (ACT && live) {
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            *reinterpret_cast<uint4*>(actv + act_piece(2 * layer - 1, T, u, g, j, h)) =
                make_uint4(zv[2 * g].x, zv[2 * g].y, zv[2 * g + 1].x, zv[2 * g + 1].y);
            *reinterpret_cast<uint4*>(actv + act_piece(2 * layer, T, u, g, j, h)) =
                make_uint4(hv[2 * g].x, hv[2 * g].y, hv[2 * g + 1].x, hv[2 * g + 1].y);
        }
    }
}

// Layers 1-3 are streamed over 32-frame tiles: step s computes layer 1 on tile s, layer 2
// on tile s-1 and layer 3 on tile s-2, so each layer's output only needs a ring of three
// tile slots.  A slot holds its tile's 32 rows between 4 halo rows on each side (the taps
// reach 4 frames into the neighbouring tiles): a tile's first 4 rows are also written into
// the after-halo of the previous tile's slot and its last 4 into the before-halo of the
// next one, so a tile's products read one contiguous 40-row window.  The halos outside the
// series (before tile 0, after the last tile) are cleared.
constexpr int SLOT = 40;   // rows per ring slot
constexpr int RING_ELEMS = 3 * SLOT * RS;

__device__ __forceinline__ void ring_store(unsigned short* ring, int s, int j, int h, const uint2* hv) {
    const int cur = s % 3, prev = (s + 2) % 3, next = (s + 1) % 3;
    unsigned short* body = ring + (cur * SLOT + 4 + j) * RS + 4 * h;
#pragma unroll
    for (int q = 0; q < 4; ++q) *reinterpret_cast<uint2*>(body + 8 * q) = hv[q];
    if (j < 4) {
        unsigned short* p = ring + (prev * SLOT + 36 + j) * RS + 4 * h;
#pragma unroll
        for (int q = 0; q < 4; ++q) *reinterpret_cast<uint2*>(p + 8 * q) = hv[q];
    } else if (j >= 28) {
        unsigned short* p = ring + (next * SLOT + j - 28) * RS + 4 * h;
#pragma unroll
        for (int q = 0; q < 4; ++q) *reinterpret_cast<uint2*>(p + 8 * q) = hv[q];
    }
}
__device__ __forceinline__ void ring_clear(unsigned short* ring, int first_row, int l) {
    for (int i = l; i < 4 * RS / 4; i += 64) reinterpret_cast<uint2*>(ring + first_row * RS)[i] = make_uint2(0u, 0u);
}

// One wave per series at a time (grid-stride), two waves per SIMD: one wave's GELU
// epilogue overlaps the other's matrix products.  Every layer, biases and the output
// layer included, runs on the matrix cores; the weights stay in registers as MFMA
// fragments.  The next series' samples are fetched into registers (XR per lane, frames
// l, l+64, ...) while the current one is processed.
// Up to 256 frames (XR = 4) one image of the whole series serves layers 1 and 2 (about
// 20 KB, eight workgroups per CU); longer series stream the layers over tile rings, whose
// size does not grow with the series.
template <int XR, bool ACT>
__global__ void __launch_bounds__(64, 2) lcf_fwd_kernel(const FwdArgs a) {
    constexpr bool STREAM = XR > 4;
    extern __shared__ float4 smem4[];
    const Geo g(a.T);
    const int l = threadIdx.x;
    // streamed: ring of layer-1 tiles, ring of layer-2 tiles, input images (hi, lo) [TP+8][2]
    // whole:    input images (hi, lo) [TP+8][2], image [TP][RS] of layer 1, then layer 2 in place
    unsigned short* ra = reinterpret_cast<unsigned short*>(smem4);
    unsigned short* rb = ra + RING_ELEMS;
    unsigned short* h0 = STREAM ? rb + RING_ELEMS : ra;
    unsigned short* hl = h0 + (g.TP + 8) * 2;   // lo terms of the input, [TP+8][2]
    unsigned short* hb = hl + (g.TP + 8) * 2;

    u16x8 f1[K1C], f2[K2C], f3[K2C], f4[2];
    frag_fwd1(a.wb, a.w, l, f1);
    frag_fwd32(a.wb, OFF_W2, l, f2);
    frag_fwd32(a.wb, OFF_W3, l, f3);
    frag_out(a.wb, l, f4);
    const u16x8 fb2 = frag_bias(a.w, OFF_B2, l), fb3 = frag_bias(a.w, OFF_B3, l);
    const float b40 = a.w[OFF_B4], b41 = a.w[OFF_B4 + 1];
    for (int i = l; i < (g.TP + 8) * 4 + (STREAM ? 0 : g.TP * RS); i += 64) h0[i] = 0;   // padding rows stay zero
    __builtin_amdgcn_wave_barrier();

    const int h = l / 32, j = l % 32;
    const int last = (g.TT - 1) % 3;   // slot of the last tile
    float2 xn[XR];
    auto fetch = [&](int64_t v) {
#pragma unroll
        for (int q = 0; q < XR; ++q) {
            const int t = l + 64 * q;
            xn[q] = (v < a.N && t < g.T) ? a.x[(int64_t)t * a.N + v] : make_float2(0.f, 0.f);
        }
    };
    fetch(blockIdx.x);
    for (int64_t v = blockIdx.x; v < a.N; v += gridDim.x) {
        float2 xc[XR];
#pragma unroll
        for (int q = 0; q < XR; ++q) xc[q] = xn[q];
        fetch(v + gridDim.x);
        float ss = 0.0f;
#pragma unroll
        for (int q = 0; q < XR; ++q) ss += xc[q].x * xc[q].x + xc[q].y * xc[q].y;
        const float r = sqrtf(wave_sum(ss) / (float)g.T + a.eps);
        const float ir = 1.0f / r;
        uint16_t* actv = ACT ? a.act + v * act_stride(g.T) : nullptr;
#pragma unroll
        for (int q = 0; q < XR; ++q) {
            const int t = l + 64 * q;
            if (t < g.T) {
                const float xr = xc[q].x * ir, xi = xc[q].y * ir;
                const unsigned int p = f2bf2(xr, xi);
                const unsigned int pl = f2bf2(xr - __uint_as_float(p << 16), xi - __uint_as_float(p & 0xffff0000u));
                *reinterpret_cast<unsigned int*>(h0 + (t + PADT) * 2) = p;
                *reinterpret_cast<unsigned int*>(hl + (t + PADT) * 2) = pl;
                if (ACT) {
                    *reinterpret_cast<unsigned int*>(actv + act_off(0, g.T) + 2 * t) = p;
                    *reinterpret_cast<unsigned int*>(actv + act_off(0, g.T) + 2 * g.T + 2 * t) = pl;
                }
            }
        }
        float pdacc = 0.0f;
        // layer 3 and the output layer on tile u of the image img (rows of tile u start at
        // row 0): y = W4 h3 (rows 0 and 1 of a 32-row product whose B operand is h3 as this
        // lane holds it) + b4
        auto layer3 = [&](const unsigned short* img, int u) {
            const floatx16 acc = conv32b(img, 0, f3, fb3, l);
            const int t = 32 * u + j;
            uint2 hv[4];
            gelu_tile<ACT>(acc, actv, 3, u, g.T, j, h, hv);
            floatx16 yo;
#pragma unroll
            for (int i = 0; i < 16; ++i) yo[i] = 0.0f;
            yo = mfma(f4[0], __builtin_bit_cast(u16x8, make_uint4(hv[0].x, hv[0].y, hv[1].x, hv[1].y)), yo);
            yo = mfma(f4[1], __builtin_bit_cast(u16x8, make_uint4(hv[2].x, hv[2].y, hv[3].x, hv[3].y)), yo);
            if (h == 0 && t < g.T) {   // rows 0 and 1 of column j
                const float y0 = yo[0] + b40, y1 = yo[1] + b41;
                pdacc += y0 * y0 + y1 * y1;
                if (a.y) a.y[(int64_t)t * a.N + v] = make_float2(r * y0, r * y1);
            }
        };
        if (STREAM) {
            ring_clear(ra, 0, l);   // before tile 0
            ring_clear(rb, 0, l);
            __builtin_amdgcn_wave_barrier();
            for (int s = 0; s < g.TT + 2; ++s) {
                if (s < g.TT) {   // layer 1, tile s
                    const floatx16 acc = conv2(h0, hl, 32 * s, f1, l);
                    uint2 hv[4];
                    gelu_tile<ACT>(acc, actv, 1, s, g.T, j, h, hv);
                    ring_store(ra, s, j, h, hv);
                } else if (s == g.TT) {
                    ring_clear(ra, last * SLOT + 36, l);   // after the last tile
                }
                if (s >= 1 && s <= g.TT) {   // layer 2, tile s - 1
                    const int u = s - 1;
                    const floatx16 acc = conv32b(ra + (u % 3) * SLOT * RS, 0, f2, fb2, l);
                    uint2 hv[4];
                    gelu_tile<ACT>(acc, actv, 2, u, g.T, j, h, hv);
                    ring_store(rb, u, j, h, hv);
                } else if (s == g.TT + 1) {
                    ring_clear(rb, last * SLOT + 36, l);
                }
                if (s >= 2) layer3(rb + ((s - 2) % 3) * SLOT * RS, s - 2);
            }
        } else {
            __builtin_amdgcn_wave_barrier();
            // layer 1 -> hb; layer 2 -> hb in place: the output of a 32-frame tile is
            // stored only after the next tile's products have read their inputs (the taps
            // reach 4 frames into the neighbouring tiles)
            for (int tt = 0; tt < g.TT; ++tt) {
                const floatx16 acc = conv2(h0, hl, 32 * tt, f1, l);
                const int t = 32 * tt + j;
                uint2 hv[4];
                gelu_tile<ACT>(acc, actv, 1, tt, g.T, j, h, hv);
#pragma unroll
                for (int q = 0; q < 4; ++q) *reinterpret_cast<uint2*>(hb + (t + PADT) * RS + 8 * q + 4 * h) = hv[q];
            }
            __builtin_amdgcn_wave_barrier();
            uint2 pend[4];
            for (int tt = 0; tt < g.TT; ++tt) {
                const floatx16 acc = conv32b(hb, 32 * tt, f2, fb2, l);
                if (tt > 0) {
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        *reinterpret_cast<uint2*>(hb + (32 * tt - 32 + j + PADT) * RS + 8 * q + 4 * h) = pend[q];
                }
                gelu_tile<ACT>(acc, actv, 2, tt, g.T, j, h, pend);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<uint2*>(hb + (32 * g.TT - 32 + j + PADT) * RS + 8 * q + 4 * h) = pend[q];
            __builtin_amdgcn_wave_barrier();
            for (int tt = 0; tt < g.TT; ++tt) layer3(hb + 32 * tt * RS, tt);
        }
        pdacc = wave_sum(pdacc);
        if (a.pd && l == 0) a.pd[v] = r * r * pdacc / (float)g.T;
        __builtin_amdgcn_wave_barrier();
    }
}

// ---------------------------------------------------------------- backward
struct BwdArgs {
    const float* w;
    const uint16_t* wb;
    const float2* x;      // [T][N]
    const float2* tgt;    // [T][N]
    uint16_t* act;
    float* part;          // [workgroups][PART]: gradient in parameter order, loss sum
    int64_t N;
    int T;
    float eps;
    float inv_count;      // 1 / (N * 2 * T)
};

// Two kernels, one per 32->32 layer L: dz_L comes in, dW_L and the dz of the layer below go
// out.  L = 3 forms dz3 from the output layer and the target, adds dW4 and stores dz2 over z2;
// L = 2 reads it back and adds dW1.  One wavefront takes a series through a kernel, streaming
// 32-frame tiles: step s puts tile s of dz_L into a ring of three slots (as the forward pass
// streams its layers) and works on tile s-1, whose neighbours are then there.
//
//  * The gradient of layer L takes 9 taps x 16 registers and stays in registers for all the
//    series of a wavefront (one wavefront per SIMD; both layers at once would need more
//    accumulators than the 256 there are); the dgrad weight fragments, the same for all
//    four wavefronts, are read from LDS.
//  * wgrad's K dimension is time.  dz is read from its time-major slot by transposing LDS
//    reads, 16 frames per lane once; the 9 taps are 9 shifts of them in registers.
//  * One more accumulator tile collects what is left, by column: 0..17 dW1 (tap 2k + i; the
//    input rows overlap, so the read needs no copy per tap), 18..20 db1..db3 (ones), 21..26
//    dW4 (rows = channels; dL/dy as three BF16 terms per output).
//  * dL/dy enters the products exactly (three BF16 terms), like the biases of the forward pass.
//  * The accumulators truncate; over 1024 wavefronts the sums still lose no more than FP32 FMAs in
//    256 did.  Gradient of 64 series repeated to 4096, against the 64 themselves (200 frames,
//    relative L2, FMAs / here): db1 2.9e-7 / 7.6e-8, db2 2.2e-7 / 8.2e-8, db3 3.8e-7 / 6.9e-8, dW4
//    2.8e-7 / 8.2e-8; the whole gradient against 64 bits with the same BF16 roundings, 8 sizes:
//    5.15e-6 / 5.14e-6 (the quotient of GELU' by IEEE division / by the hardware reciprocal).
//
// Bound by the VALU (GELU' of 96 values a frame) and the matrix products, with one wavefront
// per SIMD to issue both.  4096 series x 200 frames: 242 us for the two kernels, where one
// for the dz (256 wavefronts, weights in registers) and three for the weight gradients took
// 1262 us.
constexpr int BWD_WAVES = 4;
constexpr int BSLOT = 48;                  // ring slot rows (40 used; 48 keeps the chunk rotation in phase)
constexpr int BRING = 3 * BSLOT * 64;      // bytes
constexpr int BTILE = 32 * 64;
constexpr int BG = 6 * 64;                 // dL/dy terms [6][32]
constexpr int BH0 = 192;                   // one copy of an input window (48 rows)
constexpr int BWD_WAVE = BRING + 2 * BTILE + 4 * BH0;   // the terms of dL/dy share the second tile
constexpr int BWD_FRAG = K2C * 64 * 16 + 2 * CH * 4;   // dgrad fragments, W4 in FP32
constexpr int BWD_PART = OFF_W3;           // parameters of a kernel, at most
constexpr size_t BWD_LDS = std::max<size_t>(BWD_FRAG + BWD_WAVES * BWD_WAVE, 2 * BWD_PART * sizeof(float));
static_assert(BWD_LDS <= 160 * 1024 && PART - OFF_W3 <= BWD_PART && BG <= BTILE, "LDS of a compute unit");

// byte of 16-byte chunk c (8 channels) of a row of 32 channels: chunks are rotated by the
// row group so that 16 consecutive rows' chunks fall in distinct banks
__device__ __forceinline__ int chunk_at(int row, int c) { return row * 64 + ((c ^ ((row >> 2) & 3)) << 4); }

// Transposing read: lane i of each 16 lanes supplies 4 columns of row i / 4 and receives the
// 4 rows of column i.
__device__ __forceinline__ uint2 tr_read(const char* p) {
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)p));
}
__device__ __forceinline__ u16x8 frag4(unsigned int a, unsigned int b, unsigned int c, unsigned int d) {
    return __builtin_bit_cast(u16x8, make_uint4(a, b, c, d));
}

template <int LAYER, int XR>
__global__ void __launch_bounds__(64 * BWD_WAVES, 1) lcf_bwd_kernel(const BwdArgs a) {
    extern __shared__ float4 smem4[];
    char* sm = reinterpret_cast<char*>(smem4);
    const int T = a.T, TT = (T + 31) / 32;
    const int l = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = l / 32, j = l % 32;

    // dgrad fragments: A[i][k'*32 + o] = W[o][i][8 - k']
    constexpr int OFF_W = LAYER == 3 ? OFF_W3 : OFF_W2;
    u16x8* frag = reinterpret_cast<u16x8*>(sm);
    for (int it = threadIdx.x; it < K2C * 64; it += 64 * BWD_WAVES) {
        const int c = it / 64, i = it % 32, o0 = (c % 2) * 16 + 8 * ((it / 32) % 2);
        u16x8 f;
#pragma unroll
        for (int q = 0; q < 8; ++q) f[q] = a.wb[OFF_W + (o0 + q) * 288 + i * 9 + (8 - c / 2)];
        frag[it] = f;
    }
    float* w4 = reinterpret_cast<float*>(sm + K2C * 64 * 16);   // [2][32]
    if (threadIdx.x < 2 * CH) w4[threadIdx.x] = bf2f(a.wb[OFF_W4 + threadIdx.x]);
    __syncthreads();
    const u16x8* fr = frag + l;
    char* ring = sm + BWD_FRAG + wv * BWD_WAVE;   // dz of this layer
    char* ht = ring + BRING;                      // h tile
    char* d1 = ht + BTILE;                        // L = 2: dz1 tile
    char* gst = d1;                               // L = 3: dL/dy terms
    char* h0 = d1 + BTILE;                        // input window: hi, hi one row on, lo, lo one row on

    // output layer: W4^T against the terms of dL/dy
    u16x8 f4t;
#pragma unroll
    for (int e = 0; e < 8; ++e) f4t[e] = h == 0 && e < 6 ? a.wb[OFF_W4 + (e % 2) * CH + j] : (unsigned short)0;
    const float b40 = a.w[OFF_B4], b41 = a.w[OFF_B4 + 1];

    // lane offsets: conv rows j + k (chunk h; chunk 2 + h is 32 bytes off by xor), transposing
    // reads of rows 8h + 4m + 0..3, the same of the input window
    int co[KW], tro[4], tr0[2];
#pragma unroll
    for (int k = 0; k < KW; ++k) co[k] = chunk_at(j + k, h);
    const int i16 = l % 16, g2 = (l / 16) % 2;
#pragma unroll
    for (int m = 0; m < 4; ++m) tro[m] = chunk_at(8 * h + 4 * m + i16 / 4, 2 * g2 + (i16 % 4) / 2) + 8 * (i16 % 2);
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const int t = 8 * h + 4 * m + i16 / 4;
        tr0[m] = (t & 1) * BH0 + 4 * (t & ~1) + 8 * (i16 % 4 + 4 * g2);
    }

    floatx16 accw[KW], accm;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        accm[r] = 0.0f;
#pragma unroll
        for (int k = 0; k < KW; ++k) accw[k][r] = 0.0f;
    }
    float db40 = 0.0f, db41 = 0.0f, lossacc = 0.0f;

    auto conv = [&](const char* slot) {
        floatx16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
        for (int c = 0; c < K2C; ++c)
            acc = mfma(fr[c * 64], *reinterpret_cast<const u16x8*>(slot + (co[c / 2] ^ (32 * (c % 2)))), acc);
        return acc;
    };
    // gradient of the 9 taps from a dz slot (rows 32u-4 .. 32u+35) and the h tile in ht; db in
    // column `col` of accm
    auto wgrad = [&](const char* slot, int col) {
        const unsigned int one = j == col ? BF_ONE2 : 0u;
#pragma unroll
        for (int t0 = 0; t0 < 32; t0 += 16) {
            unsigned int e[8], o[7];   // frames 2d, 2d + 1 and 2d + 1, 2d + 2 of this lane's 16
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const uint2 v = tr_read(slot + t0 * 64 + tro[m]);
                e[2 * m] = v.x;
                e[2 * m + 1] = v.y;
            }
            const uint2 b0 = tr_read(ht + t0 * 64 + tro[0]), b1 = tr_read(ht + t0 * 64 + tro[1]);
            const u16x8 B = frag4(b0.x, b0.y, b1.x, b1.y);
#pragma unroll
            for (int d = 0; d < 7; ++d) o[d] = __builtin_amdgcn_alignbit(e[d + 1], e[d], 16);
#pragma unroll
            for (int k = 0; k < KW; ++k) {   // dz[t' + 4 - k]: 8 - k frames into the window
                const int m = (8 - k) / 2;
                const u16x8 A = k % 2 ? frag4(o[m], o[m + 1], o[m + 2], o[m + 3]) : frag4(e[m], e[m + 1], e[m + 2], e[m + 3]);
                accw[k] = mfma(A, B, accw[k]);
            }
            accm = mfma(frag4(e[2], e[3], e[4], e[5]), frag4(one, one, one, one), accm);
        }
    };
    // dz = dh GELU'(z) of tile u, BF16, zero past the end
    auto dz_tile = [&](const floatx16& dh, const uint4& za, const uint4& zb, bool live, uint2* out) {
        const unsigned int z[8] = {za.x, za.y, za.z, za.w, zb.x, zb.y, zb.z, zb.w};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            unsigned int v[2];
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                const unsigned int zz = z[2 * q + p];
                v[p] = f2bf2(dh[4 * q + 2 * p] * gelu_grad(__uint_as_float(zz << 16)),
                             dh[4 * q + 2 * p + 1] * gelu_grad(__uint_as_float(zz & 0xffff0000u)));
            }
            out[q] = live ? make_uint2(v[0], v[1]) : make_uint2(0u, 0u);
        }
    };
    auto row_store = [&](char* base, int row, const uint2* v) {
#pragma unroll
        for (int q = 0; q < 4; ++q) *reinterpret_cast<uint2*>(base + chunk_at(row, q) + 8 * h) = v[q];
    };
    auto dz_store = [&](int s, const uint2* v) {
        row_store(ring + (s % 3) * BSLOT * 64, 4 + j, v);
        if (j < 4) row_store(ring + ((s + 2) % 3) * BSLOT * 64, 36 + j, v);
        else if (j >= 28) row_store(ring + ((s + 1) % 3) * BSLOT * 64, j - 28, v);
    };
    auto halo_clear = [&](char* rows) {   // 4 rows
        *reinterpret_cast<unsigned int*>(rows + 4 * l) = 0u;
    };
    auto h_store = [&](const uint4& pa, const uint4& pb) {
        const uint2 v[4] = {make_uint2(pa.x, pa.y), make_uint2(pa.z, pa.w), make_uint2(pb.x, pb.y), make_uint2(pb.z, pb.w)};
        row_store(ht, j, v);
    };

    const int64_t stride = (int64_t)gridDim.x * BWD_WAVES;
    for (int64_t v = (int64_t)blockIdx.x * BWD_WAVES + wv; v < a.N; v += stride) {
        uint16_t* av = a.act + v * act_stride(T);
        // record pieces, loaded one step before they are used
        auto load = [&](int which, int u, uint4& pa, uint4& pb) {
            pa = pb = make_uint4(0u, 0u, 0u, 0u);
            if (u < TT && 32 * u + j < T) {
                pa = *reinterpret_cast<const uint4*>(av + act_piece(which, T, u, 0, j, h));
                pb = *reinterpret_cast<const uint4*>(av + act_piece(which, T, u, 1, j, h));
            }
        };
        auto load_tgt = [&](int u) {
            const int t = 32 * u + j;
            return h == 0 && u < TT && t < T ? a.tgt[(int64_t)t * a.N + v] : make_float2(0.0f, 0.0f);
        };
        auto load_in = [&](int u, unsigned int& hi, unsigned int& lo) {
            const int t = 32 * u - PADT + l;
            hi = lo = 0u;
            if (l < 40 && u < TT && t >= 0 && t < T) {
                hi = *reinterpret_cast<const unsigned int*>(av + 2 * t);
                lo = *reinterpret_cast<const unsigned int*>(av + 2 * T + 2 * t);
            }
        };
        uint4 za, zb, ha, hb;        // z and h of the layer below
        uint4 za3, zb3, ha3, hb3;    // L = 3: z3 and h3
        uint4 da, db;                // L = 2: dz2
        unsigned int xhi = 0u, xlo = 0u;
        float2 tg = make_float2(0.0f, 0.0f);
        float ir = 0.0f;
        load(LAYER == 3 ? 3 : 1, 0, za, zb);
        load(LAYER == 3 ? 4 : 2, 0, ha, hb);
        if (LAYER == 3) {
            tg = load_tgt(0);
            load(5, 0, za3, zb3);
            load(6, 0, ha3, hb3);
            float ss = 0.0f;
#pragma unroll
            for (int q = 0; q < XR; ++q) {
                const int t = l + 64 * q;
                const float2 xv = t < T ? a.x[(int64_t)t * a.N + v] : make_float2(0.0f, 0.0f);
                ss += xv.x * xv.x + xv.y * xv.y;
            }
            ir = 1.0f / sqrtf(wave_sum(ss) / (float)T + a.eps);
        } else {
            load(3, 0, da, db);
            load_in(0, xhi, xlo);
        }
        halo_clear(ring);   // before tile 0
        __builtin_amdgcn_wave_barrier();

        for (int s = 0; s <= TT; ++s) {
            if (s == TT) {
                halo_clear(ring + ((TT - 1) % 3) * BSLOT * 64 + 36 * 64);   // after the last tile
                __builtin_amdgcn_wave_barrier();
            } else if (LAYER == 2) {   // dz2, tile s
                const uint2 dz[4] = {make_uint2(da.x, da.y), make_uint2(da.z, da.w), make_uint2(db.x, db.y),
                                     make_uint2(db.z, db.w)};
                dz_store(s, dz);
                load(3, s + 1, da, db);
                __builtin_amdgcn_wave_barrier();
            } else {   // output layer and dz3, tile s
                const bool live = 32 * s + j < T;
                floatx16 zero;
#pragma unroll
                for (int r = 0; r < 16; ++r) zero[r] = 0.0f;
                // y = W4 h3 + b4 by FMAs: its terms cancel to a hundredth of their size, and the
                // matrix cores' truncated sums put a bias of 1e-6 on the loss
                float y0 = 0.0f, y1 = 0.0f;
                {
                    const unsigned int hw[8] = {ha3.x, ha3.y, ha3.z, ha3.w, hb3.x, hb3.y, hb3.z, hb3.w};
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float4 wa = *reinterpret_cast<const float4*>(w4 + 8 * q + 4 * h);
                        const float4 wc = *reinterpret_cast<const float4*>(w4 + CH + 8 * q + 4 * h);
                        const float v0 = __uint_as_float(hw[2 * q] << 16), v1 = __uint_as_float(hw[2 * q] & 0xffff0000u);
                        const float v2 = __uint_as_float(hw[2 * q + 1] << 16), v3 = __uint_as_float(hw[2 * q + 1] & 0xffff0000u);
                        y0 = fmaf(wa.w, v3, fmaf(wa.z, v2, fmaf(wa.y, v1, fmaf(wa.x, v0, y0))));
                        y1 = fmaf(wc.w, v3, fmaf(wc.z, v2, fmaf(wc.y, v1, fmaf(wc.x, v0, y1))));
                    }
                    y0 += __shfl_xor(y0, 32);
                    y1 += __shfl_xor(y1, 32);
                }
                h_store(ha3, hb3);
                float g0 = 0.0f, g1 = 0.0f;
                if (h == 0 && live) {
                    const float e0 = y0 + b40 - tg.x * ir, e1 = y1 + b41 - tg.y * ir;
                    lossacc += e0 * e0 + e1 * e1;
                    g0 = 2.0f * e0 * a.inv_count;
                    g1 = 2.0f * e1 * a.inv_count;
                    db40 += g0;
                    db41 += g1;
                }
                unsigned short t0[3], t1[3];
                split3(g0, t0);
                split3(g1, t1);
                unsigned int gp[3];
#pragma unroll
                for (int m = 0; m < 3; ++m) {
                    gp[m] = t0[m] | ((unsigned int)t1[m] << 16);
                    if (h == 0) {
                        reinterpret_cast<unsigned short*>(gst)[(2 * m) * 32 + j] = t0[m];
                        reinterpret_cast<unsigned short*>(gst)[(2 * m + 1) * 32 + j] = t1[m];
                    }
                }
                const floatx16 dh = mfma(f4t, frag4(gp[0], gp[1], gp[2], 0u), zero);
                uint2 dz[4];
                dz_tile(dh, za3, zb3, live, dz);
                tg = load_tgt(s + 1);
                load(5, s + 1, za3, zb3);
                load(6, s + 1, ha3, hb3);
                dz_store(s, dz);
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int k0 = 0; k0 < 32; k0 += 16) {   // dW4
                    const uint2 a0 = tr_read(ht + k0 * 64 + tro[0]), a1 = tr_read(ht + k0 * 64 + tro[1]);
                    const bool in = j >= 21 && j < 27;
                    const uint4 b = *reinterpret_cast<const uint4*>(gst + (in ? (j - 21) * 64 : 0) + (k0 + 8 * h) * 2);
                    accm = mfma(frag4(a0.x, a0.y, a1.x, a1.y),
                                frag4(in ? b.x : 0u, in ? b.y : 0u, in ? b.z : 0u, in ? b.w : 0u), accm);
                }
                __builtin_amdgcn_wave_barrier();
            }
            if (s == 0) continue;
            // dW of this layer and dz of the one below, tile u
            const int u = s - 1;
            const char* slot = ring + (u % 3) * BSLOT * 64;
            h_store(ha, hb);
            if (LAYER == 2 && l < 48) {
                unsigned int* hw = reinterpret_cast<unsigned int*>(h0);
                hw[l] = xhi;
                hw[2 * BH0 / 4 + l] = xlo;
                if (l > 0) {
                    hw[BH0 / 4 + l - 1] = xhi;
                    hw[3 * BH0 / 4 + l - 1] = xlo;
                }
            }
            __builtin_amdgcn_wave_barrier();
            const floatx16 dh = conv(slot);
            wgrad(slot, LAYER == 3 ? 20 : 19);
            uint2 dz[4];
            const bool live = 32 * u + j < T;
            dz_tile(dh, za, zb, live, dz);
            load(LAYER == 3 ? 3 : 1, s, za, zb);
            load(LAYER == 3 ? 4 : 2, s, ha, hb);
            if (LAYER == 3) {   // dz2 replaces z2
                if (live) {
#pragma unroll
                    for (int g = 0; g < 2; ++g)
                        *reinterpret_cast<uint4*>(av + act_piece(3, T, u, g, j, h)) =
                            make_uint4(dz[2 * g].x, dz[2 * g].y, dz[2 * g + 1].x, dz[2 * g + 1].y);
                }
                __builtin_amdgcn_wave_barrier();
                continue;
            }
            load_in(s, xhi, xlo);
            row_store(d1, j, dz);
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int k0 = 0; k0 < 32; k0 += 16) {
                const uint2 a0 = tr_read(d1 + k0 * 64 + tro[0]), a1 = tr_read(d1 + k0 * 64 + tro[1]);
                const u16x8 A = frag4(a0.x, a0.y, a1.x, a1.y);
#pragma unroll
                for (int p = 0; p < 2; ++p) {   // hi terms, with the ones of db1; lo terms
                    const uint2 b0 = tr_read(h0 + 2 * p * BH0 + k0 * 4 + tr0[0]);
                    const uint2 b1 = tr_read(h0 + 2 * p * BH0 + k0 * 4 + tr0[1]);
                    const unsigned int one = p == 0 && j == 18 ? BF_ONE2 : 0u;
                    const bool in = j < 18;
                    accm = mfma(A, frag4(in ? b0.x : one, in ? b0.y : one, in ? b1.x : one, in ? b1.y : one), accm);
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
    }

    // sum over the wavefronts in LDS, in a fixed order: waves 0, 1 store, 2, 3 add
    constexpr int FIRST = LAYER == 3 ? OFF_W3 : 0, LAST = LAYER == 3 ? PART : OFF_W3;
    __syncthreads();
    float* reg = reinterpret_cast<float*>(smem4) + (wv & 1) * BWD_PART - FIRST;
    if (LAYER == 3) {
        db40 = wave_sum(db40);
        db41 = wave_sum(db41);
        lossacc = wave_sum(lossacc);
    }
    auto put = [&](bool add) {
        auto one = [&](int idx, float x) { reg[idx] = add ? reg[idx] + x : x; };
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int o = acc_row(r, l);
#pragma unroll
            for (int k = 0; k < KW; ++k) one(OFF_W + o * 288 + j * 9 + k, accw[k][r]);
            const float x = accm[r];
            if (LAYER == 3) {
                const float x3 = x + __shfl_down(x, 2) + __shfl_down(x, 4);   // the three terms of dW4
                if (j == 20) one(OFF_B3 + o, x);
                else if (j == 21 || j == 22) one(OFF_W4 + (j - 21) * CH + o, x3);
            } else {
                if (j < 18) one(OFF_W1 + o * 18 + (j % 2) * 9 + j / 2, x);
                else if (j == 18) one(OFF_B1 + o, x);
                else if (j == 19) one(OFF_B2 + o, x);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (LAYER == 3 && l == 0) {
            one(OFF_B4, db40);
            one(OFF_B4 + 1, db41);
            one(NPAR, lossacc);
        }
    };
    for (int turn = 0; turn < 2; ++turn) {
        if (wv / 2 == turn) put(turn == 1);
        __syncthreads();
    }
    const float* sum = reinterpret_cast<const float*>(smem4);
    for (int p = threadIdx.x; p < LAST - FIRST; p += 64 * BWD_WAVES)
        a.part[(int64_t)blockIdx.x * PART + FIRST + p] = sum[p] + sum[BWD_PART + p];
}

// deterministic sum of the workgroups' partials: 16 waves share the partials of 64 parameters
constexpr int RED_GROUPS = 16;
__global__ void __launch_bounds__(64 * RED_GROUPS) lcf_reduce_kernel(const float* part, int nwg, float* grad, float* loss,
                                                                    float inv_count) {
    __shared__ float s[RED_GROUPS][64];
    const int l = threadIdx.x & 63, g = threadIdx.x >> 6;
    const int p = blockIdx.x * 64 + l;
    float x = 0.0f;
    if (p < PART) {
#pragma unroll 8
        for (int w = g; w < nwg; w += RED_GROUPS) x += part[(int64_t)w * PART + p];
    }
    s[g][l] = x;
    __syncthreads();
    if (g > 0 || p >= PART) return;
#pragma unroll
    for (int k = 1; k < RED_GROUPS; ++k) x += s[k][l];
    if (p < NPAR) grad[p] = x;
    else *loss = x * inv_count;
}

// ---------------------------------------------------------------- optimiser, batches, fallback
__global__ void adam_kernel(float* w, uint16_t* wb, float* m, float* v, const float* g, int n, float lr, float b1,
                            float b2, float eps, float c1, float c2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float wi = w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    w[i] = wi;
    wb[i] = f2bf(wi);
}

// One thread an element, series fastest: neighbouring workgroups read one frame at a time, which
// stays in the L2s.  (Eight frames a thread: 65536 of 262144 series x 200 frames 183 -> 208 us,
// and no faster for 4096.)
__global__ void gather_kernel(const float2* src, int64_t nv, int T, const int64_t* idx, int64_t B, float2* dst) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (int64_t)T * B) return;
    const int t = (int)(i / B);
    const int64_t b = i - (int64_t)t * B;
    const int64_t gi = idx[b];
    const int64_t vol = gi / nv, vv = gi - vol * nv;
    dst[i] = src[(vol * T + t) * nv + vv];
}

__global__ void fb_partial_kernel(const float* pl, const float* ps, int64_t n, double* part) {
    __shared__ double s0[256], s1[256], s2[256];
    double a0 = 0.0, a1 = 0.0, a2 = 0.0;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
        const float x = pl[i], y = ps[i];
        if (!isfinite(x)) a2 += 1.0;
        else {
            const double d = (double)x - (double)y;
            a0 += d * d;
        }
        a1 += (double)y * (double)y;
    }
    s0[threadIdx.x] = a0;
    s1[threadIdx.x] = a1;
    s2[threadIdx.x] = a2;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) {
            s0[threadIdx.x] += s0[threadIdx.x + o];
            s1[threadIdx.x] += s1[threadIdx.x + o];
            s2[threadIdx.x] += s2[threadIdx.x + o];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[3 * blockIdx.x] = s0[0];
        part[3 * blockIdx.x + 1] = s1[0];
        part[3 * blockIdx.x + 2] = s2[0];
    }
}

// Every block reduces the partials itself, in the same order (12 KB out of L2), and block
// 0 stores the judgement: one thread adding them alone took 60 us.  Eight blocks a compute unit at
// most share the values: a block for every 256 of 20 million took 214 us, mostly reductions, as
// against 148 before the partials were reduced here.
__global__ void __launch_bounds__(256) fb_select_kernel(const float* pl, const float* ps, int64_t n, const double* part,
                                                        int nblk, float tau_db, int* flag, float* d_db, float* out) {
    __shared__ double s[3][4];
    double v[3] = {0.0, 0.0, 0.0};
    for (int b = threadIdx.x; b < nblk; b += 256)
#pragma unroll
        for (int q = 0; q < 3; ++q) v[q] += part[3 * b + q];
#pragma unroll
    for (int q = 0; q < 3; ++q) {
        for (int o = 32; o > 0; o >>= 1) v[q] += __shfl_xor(v[q], o);
        if ((threadIdx.x & 63) == 0) s[q][threadIdx.x >> 6] = v[q];
    }
    __syncthreads();
    double a[3];
#pragma unroll
    for (int q = 0; q < 3; ++q) a[q] = (s[q][0] + s[q][1]) + (s[q][2] + s[q][3]);
    const double d = a[1] > 0.0 ? 10.0 * log10(fmax(a[0], 1e-300) / a[1]) : 0.0;
    const int f = (a[2] > 0.0) || !(a[1] > 0.0) || !(d <= (double)tau_db);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *flag = f;
        *d_db = a[2] > 0.0 ? __builtin_nanf("") : (float)d;
    }
    const float* src = f ? ps : pl;
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) out[i] = src[i];
}

constexpr int FB_BLOCKS = 512;
constexpr int64_t FB_SELECT_BLOCKS = 2048;

size_t fwd_lds(int T) {   // the launch below takes the streamed kernel above 256 frames
    const int TP = 32 * ((T + 31) / 32) + 8;
    return (T > 256 ? 2 * (size_t)RING_ELEMS * 2 : (size_t)TP * RS * 2) + (size_t)(TP + 8) * 4 * 2;
}
size_t act_bytes(int64_t n, int T) { return round_up((size_t)n * act_stride(T) * 2, 256); }
size_t part_bytes() { return (size_t)NWB * PART * 4; }

}  // namespace
}  // namespace fq

using namespace fq;

extern "C" size_t lcf_act_size(int64_t n_series, int32_t n_t) {
    if (n_series < 1 || n_t < 1) return 0;
    return act_bytes(n_series, n_t) + part_bytes();
}

extern "C" int lcf_forward(const float* w, const uint16_t* w_bf16, const float* x, int64_t n_series, int32_t n_t,
                           float eps, uint16_t* act, float* y, float* pd, void* stream) {
    FQ_REQUIRE(w && w_bf16 && x && aligned16(w_bf16) && aligned16(x), "null or misaligned pointer");
    FQ_REQUIRE(n_series >= 1 && n_t >= 1 && n_t <= FQ_MAX_NT, "bad sizes");
    FQ_REQUIRE(!act || aligned16(act), "misaligned act");
    FQ_REQUIRE(eps >= 0.0f, "eps must be >= 0");
    const size_t lds = fwd_lds(n_t);
    FQ_REQUIRE(lds <= 160 * 1024, "n_t too large");
    FwdArgs fa{w, w_bf16, reinterpret_cast<const float2*>(x), act, reinterpret_cast<float2*>(y), pd, n_series, n_t, eps};
    const unsigned grid = (unsigned)std::min<int64_t>(n_series, 8192);
    auto kern = n_t <= 256 ? (act ? lcf_fwd_kernel<4, true> : lcf_fwd_kernel<4, false>)
                           : (act ? lcf_fwd_kernel<8, true> : lcf_fwd_kernel<8, false>);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64), lds, as_stream(stream), fa);
    FQ_LAUNCH_CHECK();
    return FQ_OK;
}

extern "C" int lcf_backward(const float* w, const uint16_t* w_bf16, const float* x, const float* target,
                            int64_t n_series, int32_t n_t, float eps, uint16_t* act, float* grad, float* loss,
                            void* stream) {
    FQ_REQUIRE(w && w_bf16 && x && target && act && grad && loss, "null pointer");
    FQ_REQUIRE(aligned16(w_bf16) && aligned16(x) && aligned16(target) && aligned16(act), "misaligned pointer");
    FQ_REQUIRE(n_series >= 1 && n_t >= 1 && n_t <= FQ_MAX_NT, "bad sizes");
    hipStream_t s = as_stream(stream);
    float* part = reinterpret_cast<float*>(reinterpret_cast<char*>(act) + act_bytes(n_series, n_t));
    const float inv_count = (float)(1.0 / ((double)n_series * 2.0 * n_t));
    const int nwg = (int)std::min<int64_t>(NWB, (n_series + BWD_WAVES - 1) / BWD_WAVES);
    BwdArgs ba{w, w_bf16, reinterpret_cast<const float2*>(x), reinterpret_cast<const float2*>(target), act, part,
               n_series, n_t, eps, inv_count};
    hipLaunchKernelGGL((n_t <= 256 ? lcf_bwd_kernel<3, 4> : lcf_bwd_kernel<3, 8>), dim3(nwg), dim3(64 * BWD_WAVES),
                       BWD_LDS, s, ba);
    FQ_LAUNCH_CHECK();
    hipLaunchKernelGGL((lcf_bwd_kernel<2, 1>), dim3(nwg), dim3(64 * BWD_WAVES), BWD_LDS, s, ba);
    FQ_LAUNCH_CHECK();
    hipLaunchKernelGGL(lcf_reduce_kernel, dim3((PART + 63) / 64), dim3(64 * RED_GROUPS), 0, s, part, nwg, grad, loss,
                       inv_count);
    FQ_LAUNCH_CHECK();
    return FQ_OK;
}

extern "C" int lcf_adam_step(float* w, uint16_t* w_bf16, float* m, float* v, const float* grad, int32_t n_param,
                             float lr, float beta1, float beta2, float eps, int32_t step, void* stream) {
    FQ_REQUIRE(w && w_bf16 && m && v && grad, "null pointer");
    FQ_REQUIRE(n_param >= 1 && step >= 1, "bad n_param / step");
    FQ_REQUIRE(beta1 >= 0 && beta1 < 1 && beta2 >= 0 && beta2 < 1 && eps > 0 && lr >= 0, "bad Adam hyper-parameters");
    const float c1 = (float)(1.0 - std::pow((double)beta1, step));
    const float c2 = (float)(1.0 - std::pow((double)beta2, step));
    hipLaunchKernelGGL(adam_kernel, dim3((n_param + 255) / 256), dim3(256), 0, as_stream(stream), w, w_bf16, m, v,
                       grad, n_param, lr, beta1, beta2, eps, c1, c2);
    FQ_LAUNCH_CHECK();
    return FQ_OK;
}

extern "C" int lcf_gather(const float* src, int64_t n_vox, int32_t n_t, int64_t n_vol, const int64_t* idx,
                          int64_t batch, float* dst, void* stream) {
    FQ_REQUIRE(src && idx && dst && aligned16(src) && aligned16(dst), "null or misaligned pointer");
    FQ_REQUIRE(n_vox >= 1 && n_t >= 1 && n_vol >= 1 && batch >= 1, "bad sizes");
    const int64_t total = (int64_t)n_t * batch;
    hipLaunchKernelGGL(gather_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, as_stream(stream),
                       reinterpret_cast<const float2*>(src), n_vox, n_t, idx, batch, reinterpret_cast<float2*>(dst));
    FQ_LAUNCH_CHECK();
    return FQ_OK;
}

extern "C" size_t fallback_workspace_size(int64_t n) {
    (void)n;
    return (size_t)FB_BLOCKS * 3 * sizeof(double);
}

extern "C" int lcf_fallback(const float* pd_l, const float* pd_s, int64_t n, float tau_db, void* ws, size_t ws_bytes,
                            float* out, int32_t* flag, float* d_db, void* stream) {
    FQ_REQUIRE(pd_l && pd_s && out && flag && d_db && ws, "null pointer");
    FQ_REQUIRE(n >= 1, "n must be >= 1");
    if (ws_bytes < fallback_workspace_size(n)) {
        set_error("workspace too small");
        return FQ_E_WORKSPACE;
    }
    hipStream_t s = as_stream(stream);
    double* part = reinterpret_cast<double*>(ws);
    hipLaunchKernelGGL(fb_partial_kernel, dim3(FB_BLOCKS), dim3(256), 0, s, pd_l, pd_s, n, part);
    FQ_LAUNCH_CHECK();
    hipLaunchKernelGGL(fb_select_kernel, dim3((unsigned)std::min<int64_t>((n + 255) / 256, FB_SELECT_BLOCKS)), dim3(256), 0, s, pd_l, pd_s, n, part,
                       FB_BLOCKS, tau_db, flag, d_db, out);
    FQ_LAUNCH_CHECK();
    return FQ_OK;
}
