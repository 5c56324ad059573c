// display_db and mip: log-compressed display of B-mode and power-Doppler volumes over a
// dynamic range, and their maximum-intensity projections (Section 2.4.2; the results
// show B-mode over 75 dB, power Doppler over 60 dB, and MIPs onto the x-y, x-z and y-z
// planes).  All passes are HBM-bound streams.
//
//   displayed power p = PD (power) or |IQ|^2 (complex IQ; 20 log10 |IQ| = 10 log10 |IQ|^2)
//   out = max(-dr, 10 log10(p / max p));  max p == 0 shows everything at -dr;
//   or, as grey levels, 1 + out / dr in [0, 1].
// The reference max p comes from block maxima that every block of the second pass reduces
// again; a maximum does not depend on the order of its operands, so the result is exact
// and deterministic.  The logarithms use the hardware log2 (error far below 1e-4 dB).
#include "fq_common.hpp"

namespace fq {
namespace {

constexpr int DISP_THREADS = 256;
constexpr int DISP_MAX_BLOCKS = 1024;
constexpr float TEN_LOG10_2 = 3.0102999566398120f;   // 10 log10(2)

__device__ __forceinline__ float wave_max(float m) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) m = fmaxf(m, __shfl_xor(m, o));
    return m;
}

// max over the block of 256 threads (4 waves); valid in thread 0
__device__ __forceinline__ float block_max(float m, float* s) {
    m = wave_max(m);
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = m;
    __syncthreads();
    return fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3]));
}

// displayed power of value i, and of the values of one 16-byte load (four powers, or two
// IQ samples)
template <bool IQ>
__device__ __forceinline__ float power_at(const float* in, int64_t i) {
    if (IQ) {
        const float2 z = reinterpret_cast<const float2*>(in)[i];
        return z.x * z.x + z.y * z.y;
    }
    return in[i];
}

template <bool IQ>
struct Quad {
    static constexpr int N = IQ ? 2 : 4;
    float p[N];
    __device__ __forceinline__ Quad(const float* in, int64_t q) {
        const float4 v = reinterpret_cast<const float4*>(in)[q];
        if constexpr (IQ) {
            p[0] = v.x * v.x + v.y * v.y;
            p[1] = v.z * v.z + v.w * v.w;
        } else {
            p[0] = v.x;
            p[1] = v.y;
            p[2] = v.z;
            p[3] = v.w;
        }
    }
};

template <bool IQ>
__global__ void __launch_bounds__(DISP_THREADS) peak_partial_kernel(const float* in, int64_t n, float* part) {
    constexpr int N = Quad<IQ>::N;
    __shared__ float s[4];
    float m = 0.0f;
    const int64_t i0 = (int64_t)blockIdx.x * DISP_THREADS + threadIdx.x, step = (int64_t)gridDim.x * DISP_THREADS;
    for (int64_t q = i0; q < n / N; q += step) {
        const Quad<IQ> v(in, q);
#pragma unroll
        for (int k = 0; k < N; ++k) m = fmaxf(m, v.p[k]);
    }
    if (i0 < n % N) m = fmaxf(m, power_at<IQ>(in, n - 1 - i0));
    m = block_max(m, s);
    if (threadIdx.x == 0) part[blockIdx.x] = m;
}

// Every block reduces the block maxima itself (at most DISP_MAX_BLOCKS words out of L2):
// a launch of one block between the two passes cost 3 us and its gap.
template <bool IQ>
__global__ void __launch_bounds__(DISP_THREADS) db_kernel(const float* in, int64_t n, const float* part, int nb,
                                                          float* peak, float neg_dr, int unit, float* out) {
    constexpr int N = Quad<IQ>::N;
    __shared__ float s[4];
    float pk = 0.0f;
    for (int i = threadIdx.x; i < nb; i += DISP_THREADS) pk = fmaxf(pk, part[i]);
    pk = block_max(pk, s);
    if (peak && blockIdx.x == 0 && threadIdx.x == 0) *peak = pk;
    const float lpk = __builtin_amdgcn_logf(pk);   // log2
    auto level = [&](float p) {
        float d = neg_dr;
        if (pk > 0.0f && p > 0.0f) d = fmaxf(neg_dr, TEN_LOG10_2 * (__builtin_amdgcn_logf(p) - lpk));
        // grey level (d + dr) / dr: exactly 0 at the floor and 1 at the peak
        return unit ? (d - neg_dr) / -neg_dr : d;
    };
    const int64_t i0 = (int64_t)blockIdx.x * DISP_THREADS + threadIdx.x, step = (int64_t)gridDim.x * DISP_THREADS;
    for (int64_t q = i0; q < n / N; q += step) {
        const Quad<IQ> v(in, q);
        if constexpr (IQ)
            reinterpret_cast<float2*>(out)[q] = make_float2(level(v.p[0]), level(v.p[1]));
        else
            reinterpret_cast<float4*>(out)[q] = make_float4(level(v.p[0]), level(v.p[1]), level(v.p[2]), level(v.p[3]));
    }
    if (i0 < n % N) {
        const int64_t i = n - 1 - i0;
        out[i] = level(power_at<IQ>(in, i));
    }
}

// MIP onto x-y (max over z) or x-z (max over y): SEG wavefronts share the planes (or rows) of 64
// consecutive output pixels (mip_segments).
constexpr int64_t MIP_MAX_BLOCKS = 1 << 20;   // (a launch holds 2^32 threads) larger planes loop
template <int SEG>
__global__ void __launch_bounds__(SEG > 4 ? 64 * SEG : 256) mip_strided_kernel(const float* vol, int nx, int ny, int nz,
                                                                              int over_z, float* out) {
    constexpr int PIX = SEG >= 4 ? 64 : 256 / SEG;   // pixels of a workgroup
    __shared__ float s[SEG > 1 ? SEG : 1][SEG > 1 ? PIX : 1];
    const int l = threadIdx.x % PIX, seg = threadIdx.x / PIX;
    const int64_t n_out = over_z ? (int64_t)nx * ny : (int64_t)nx * nz;
    for (int64_t i0 = (int64_t)blockIdx.x * PIX; i0 < n_out; i0 += (int64_t)gridDim.x * PIX) {
        const int64_t idx = i0 + l;
        float m = -INFINITY;
        if (idx < n_out) {
            // over z: pixel (ix, iy) is voxel idx of every plane; over y: pixel (ix, iz) starts at row iz * ny
            const int64_t o = idx / nx, plane = (int64_t)nx * ny;
            const float* src = vol + (over_z ? idx : idx + o * (plane - nx));
            const int64_t stride = over_z ? plane : nx;
            const int len = over_z ? nz : ny;
#pragma unroll 4
            for (int k = seg; k < len; k += SEG) m = fmaxf(m, src[k * stride]);
        }
        if (SEG == 1) {
            if (idx < n_out) out[idx] = m;
            continue;
        }
        s[seg][l] = m;
        __syncthreads();
        if (seg == 0 && idx < n_out) {
#pragma unroll
            for (int k = 1; k < SEG; ++k) m = fmaxf(m, s[k][l]);
            out[idx] = m;
        }
        __syncthreads();
    }
}

// MIP onto y-z (max over x): one wave per row of x.
__global__ void __launch_bounds__(DISP_THREADS) mip_rows_kernel(const float* vol, int nx, int64_t n_rows, float* out) {
    const int64_t row = (int64_t)blockIdx.x * (DISP_THREADS / 64) + (threadIdx.x >> 6);
    if (row >= n_rows) return;
    const int l = threadIdx.x & 63;
    const float* r = vol + row * nx;
    float m = -INFINITY;
    for (int ix = l; ix < nx; ix += 64) m = fmaxf(m, r[ix]);
    m = wave_max(m);
    if (l == 0) out[row] = m;
}

// blocks of the two display passes: one 16-byte load per thread and pass until the block
// maxima fill their workspace
int blocks_for(int64_t n, int per_thread) {
    const int64_t per = (int64_t)DISP_THREADS * per_thread;
    return (int)std::max<int64_t>(1, std::min<int64_t>(DISP_MAX_BLOCKS, (n + per - 1) / per));
}

// Wavefronts that share 64 pixels' reduction: few pixels leave the chip idle in chains of dependent
// reads, many are a stream of their own and only pay for the exchange.  1, 4 and 16 wavefronts:
// 128 x 128 pixels of 1024 planes 68, 20, 11 us; 256 x 256 of 256 planes 20, 11, 11; 1024 x 1024 of 8
// planes 10, 10, 28 and of 64 planes 42, 39, 47; 4096 x 4096 of 4 planes 62, 135, 503.
int mip_segments(int64_t pixels) { return pixels <= 32768 ? 16 : pixels <= 524288 ? 4 : 1; }

template <bool IQ>
int launch_display(const float* in, int64_t n, float* part, float* peak, float neg_dr, int unit, float* out,
                   hipStream_t s) {
    const int nb = blocks_for(n, Quad<IQ>::N);
    hipLaunchKernelGGL(peak_partial_kernel<IQ>, dim3(nb), dim3(DISP_THREADS), 0, s, in, n, part);
    FQ_LAUNCH_CHECK();
    hipLaunchKernelGGL(db_kernel<IQ>, dim3(nb), dim3(DISP_THREADS), 0, s, in, n, part, nb, peak, neg_dr, unit, out);
    FQ_LAUNCH_CHECK();
    return FQ_OK;
}

}  // namespace
}  // namespace fq

using namespace fq;

extern "C" size_t display_workspace_size(int64_t n) {
    (void)n;
    return sizeof(float) * (DISP_MAX_BLOCKS + 64);
}

extern "C" int display_db(const float* in, int64_t n, int32_t kind, float dr_db, void* ws, size_t ws_bytes, float* out,
                          float* peak, void* stream) {
    FQ_REQUIRE(n >= 1, "n must be >= 1");
    const bool unit = (kind & FQ_DISP_UNIT) != 0;
    kind &= ~FQ_DISP_UNIT;
    FQ_REQUIRE(kind == FQ_DISP_POWER || kind == FQ_DISP_IQ, "kind must be FQ_DISP_POWER or FQ_DISP_IQ (| FQ_DISP_UNIT)");
    FQ_REQUIRE(dr_db > 0.0f && dr_db < 1000.0f, "dr_db must be in (0, 1000)");
    FQ_REQUIRE(in && out && ws && aligned16(in) && aligned16(out) && aligned16(ws), "null or misaligned pointer");
    if (ws_bytes < display_workspace_size(n)) {
        set_error("workspace too small: %zu < %zu bytes", ws_bytes, display_workspace_size(n));
        return FQ_E_WORKSPACE;
    }
    hipStream_t s = as_stream(stream);
    float* part = reinterpret_cast<float*>(ws);
    return kind == FQ_DISP_IQ ? launch_display<true>(in, n, part, peak, -dr_db, unit ? 1 : 0, out, s)
                              : launch_display<false>(in, n, part, peak, -dr_db, unit ? 1 : 0, out, s);
}

extern "C" int mip(const float* vol, int32_t nx, int32_t ny, int32_t nz, int32_t plane, float* out, void* stream) {
    FQ_REQUIRE(nx >= 1 && ny >= 1 && nz >= 1, "bad volume size");
    FQ_REQUIRE(plane == FQ_MIP_XY || plane == FQ_MIP_XZ || plane == FQ_MIP_YZ, "bad plane");
    FQ_REQUIRE(vol && out && aligned16(vol) && aligned16(out), "null or misaligned pointer");
    hipStream_t s = as_stream(stream);
    if (plane == FQ_MIP_YZ) {
        const int64_t rows = (int64_t)ny * nz;
        const unsigned nb = (unsigned)((rows + DISP_THREADS / 64 - 1) / (DISP_THREADS / 64));
        hipLaunchKernelGGL(mip_rows_kernel, dim3(nb), dim3(DISP_THREADS), 0, s, vol, nx, rows, out);
    } else {
        const int over_z = plane == FQ_MIP_XY ? 1 : 0;
        const int64_t n_out = over_z ? (int64_t)nx * ny : (int64_t)nx * nz;
        const int seg = mip_segments(n_out);
        const int pix = seg >= 4 ? 64 : 256 / seg;
        const unsigned nb = (unsigned)std::min<int64_t>((n_out + pix - 1) / pix, MIP_MAX_BLOCKS);
        auto kern = seg == 16 ? mip_strided_kernel<16> : seg == 4 ? mip_strided_kernel<4> : mip_strided_kernel<1>;
        hipLaunchKernelGGL(kern, dim3(nb), dim3(seg * pix), 0, s, vol, nx, ny, nz, over_z, out);
    }
    FQ_LAUNCH_CHECK();
    return FQ_OK;
}
