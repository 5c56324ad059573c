// image_quality: MSE, PSNR and SSIM of an image against its ground truth (Section 2.4.3;
// the paper applies them to maximum-intensity projections).  SSIM after Wang, Bovik,
// Sheikh and Simoncelli (IEEE TIP 2004): 11 x 11 Gaussian window (sigma 1.5, weights
// summing to 1), K1 = 0.01, K2 = 0.03, window-weighted moments, averaged over the
// positions where the window lies inside the image.  The images are small (projections)
// and the call has no workspace, so one workgroup computes everything in FP64 and reduces
// in a fixed order (deterministic).
//
// The window is separable: a tile of up to 60 x 54 positions first forms the five moment
// sums along x of every row (four neighbouring positions per thread share their pixels)
// in LDS, then sums them along y (up to three positions per thread).  110 FP64
// multiply-adds a position and moment set instead of 605 and their products: 33.5 us -> 13.6 us
// for a 64 x 64 image, launch included, on the one compute unit.
#include "fq_common.hpp"

namespace fq {
namespace {

constexpr int IQM_THREADS = 1024;
constexpr int IQM_WIN = 11;

struct IqmArgs {
    const float* a;
    const float* b;
    double* out;      // [3]: MSE, PSNR, SSIM
    int nx, ny;
    int bx, by;       // positions of a tile; bx = 0: every position by itself
    double c1, c2, range2;
    double w[IQM_WIN];
};

constexpr int IQM_TX = 60, IQM_TY = 54;            // positions of a tile
constexpr int IQM_PLANE = (IQM_TY + IQM_WIN - 1) * IQM_TX;   // sums along x of its image rows
constexpr int IQM_QX = 4, IQM_QY = 3;              // positions of a thread in the two passes
constexpr size_t IQM_LDS = sizeof(double) * 5 * IQM_PLANE;

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

__global__ void __launch_bounds__(IQM_THREADS) image_quality_kernel(const IqmArgs p) {
    extern __shared__ double hs[];   // [5][IQM_PLANE]: [row][bx] sums along x
    __shared__ double red[2][IQM_THREADS / 64];
    constexpr int PLANE = IQM_PLANE;
    const int tid = threadIdx.x;
    const int n = p.nx * p.ny;
    double m = 0.0;
    auto similarity = [&](const double (&v)[5]) {   // from the window's moments
        const double ma = v[0], mb = v[1];
        const double sa = v[2] - ma * ma, sb = v[3] - mb * mb, sab = v[4] - ma * mb;
        return ((2.0 * ma * mb + p.c1) * (2.0 * sab + p.c2)) / ((ma * ma + mb * mb + p.c1) * (sa + sb + p.c2));
    };
    const int ox = p.nx - IQM_WIN + 1, oy = p.ny - IQM_WIN + 1;
    const int bx = p.bx, by = p.by;
    double ss = 0.0;
    if (bx == 0) {
        for (int i = tid; i < n; i += IQM_THREADS) {
            const double d = (double)p.a[i] - (double)p.b[i];
            m = fma(d, d, m);
        }
        for (int q = tid; q < ox * oy; q += IQM_THREADS) {
            const int y = q / ox, x = q - y * ox;
            double v[5] = {};
            for (int dy = 0; dy < IQM_WIN; ++dy) {
                const float* ra = p.a + (int64_t)(y + dy) * p.nx + x;
                const float* rb = p.b + (int64_t)(y + dy) * p.nx + x;
#pragma unroll
                for (int dx = 0; dx < IQM_WIN; ++dx) {
                    const double w = p.w[dy] * p.w[dx], va = ra[dx], vb = rb[dx];
                    v[0] = fma(w, va, v[0]);
                    v[1] = fma(w, vb, v[1]);
                    v[2] = fma(w * va, va, v[2]);
                    v[3] = fma(w * vb, vb, v[3]);
                    v[4] = fma(w * va, vb, v[4]);
                }
            }
            ss += similarity(v);
        }
    }
    for (int y0 = 0; bx > 0 && y0 < oy; y0 += by)
        for (int x0 = 0; x0 < ox; x0 += bx) {
            const int w = min(bx, ox - x0), h = min(by, oy - y0);
            const int rows = h + IQM_WIN - 1, quads = (w + IQM_QX - 1) / IQM_QX;
            for (int i = tid; i < rows * quads; i += IQM_THREADS) {
                const int r = i / quads, c0 = (i - r * quads) * IQM_QX;
                const int64_t at = (int64_t)(y0 + r) * p.nx;
                double acc[5][IQM_QX] = {};
                // each pixel's squared error is counted once: in its own tile and group of
                // four, the image's last rows and columns in the last ones
                const bool own_row = r < h || y0 + h == oy, own_tail = x0 + w == ox && c0 + IQM_QX >= w;
#pragma unroll
                for (int k = 0; k < IQM_WIN + IQM_QX - 1; ++k) {
                    const int x = min(x0 + c0 + k, p.nx - 1);   // past the tile: not stored
                    const double va = p.a[at + x], vb = p.b[at + x];
                    const double v[5] = {va, vb, va * va, vb * vb, va * vb};
                    const bool own = own_row && x0 + c0 + k < p.nx && (own_tail || (k < IQM_QX && c0 + k < w));
                    const double d = own ? va - vb : 0.0;
                    m = fma(d, d, m);
#pragma unroll
                    for (int j = 0; j < IQM_QX; ++j) {
                        if (k - j < 0 || k - j >= IQM_WIN) continue;
#pragma unroll
                        for (int q = 0; q < 5; ++q) acc[q][j] = fma(p.w[k - j], v[q], acc[q][j]);
                    }
                }
#pragma unroll
                for (int j = 0; j < IQM_QX; ++j)
                    if (c0 + j < w) {
#pragma unroll
                        for (int q = 0; q < 5; ++q) hs[q * PLANE + r * bx + c0 + j] = acc[q][j];
                    }
            }
            __syncthreads();
            const int runs = (h + IQM_QY - 1) / IQM_QY;
            for (int i = tid; i < runs * w; i += IQM_THREADS) {
                const int g = i / w, x = i - g * w, r0 = g * IQM_QY;
                double acc[5][IQM_QY] = {};
#pragma unroll
                for (int k = 0; k < IQM_WIN + IQM_QY - 1; ++k) {
                    const int r = min(r0 + k, rows - 1);   // past the tile: not counted
#pragma unroll
                    for (int q = 0; q < 5; ++q) {
                        const double v = hs[q * PLANE + r * bx + x];
#pragma unroll
                        for (int j = 0; j < IQM_QY; ++j)
                            if (k - j >= 0 && k - j < IQM_WIN) acc[q][j] = fma(p.w[k - j], v, acc[q][j]);
                    }
                }
#pragma unroll
                for (int j = 0; j < IQM_QY; ++j) {
                    const double v[5] = {acc[0][j], acc[1][j], acc[2][j], acc[3][j], acc[4][j]};
                    const double sim = similarity(v);
                    if (r0 + j < h) ss += sim;
                }
            }
            __syncthreads();
        }
    m = wave_sum(m);
    ss = wave_sum(ss);
    if ((tid & 63) == 0) {
        red[0][tid >> 6] = m;
        red[1][tid >> 6] = ss;
    }
    __syncthreads();
    if (tid == 0) {
        for (int k = 1; k < IQM_THREADS / 64; ++k) {
            m += red[0][k];
            ss += red[1][k];
        }
        const double mse = m / (double)n;
        p.out[0] = mse;
        p.out[1] = mse > 0.0 ? 10.0 * log10(p.range2 / mse) : __builtin_inf();
        p.out[2] = ss / ((double)ox * (double)oy);
    }
}

// Positions of a tile: 60 x 54, or in an image narrower than that in one direction as many in the
// other as the sums leave room for (400 x 16 pixels: 18.8 us, 38.7 with at most 54 rows).  Every
// position by itself where that takes fewer rounds of the workgroup than there are tiles: a tile
// and a round take about 8 us each, and the windows of one to three rows of positions share
// little (1000 x 11 pixels, x fastest: 15 us, 32 in tiles; x 14: 45 and 42).
void choose_tiles(int ox, int oy, int& bx, int& by) {
    bx = std::min(ox, IQM_TX);
    by = std::min(oy, IQM_TY);
    if (ox < IQM_TX) by = std::min(oy, IQM_PLANE / bx - (IQM_WIN - 1));
    else if (oy < IQM_TY) bx = std::min(ox, IQM_PLANE / (by + IQM_WIN - 1));
    const int tx = (ox + bx - 1) / bx, ty = (oy + by - 1) / by;
    bx = (ox + tx - 1) / tx;
    by = (oy + ty - 1) / ty;
    if ((ox * oy + IQM_THREADS - 1) / IQM_THREADS < tx * ty) bx = 0;
}

}  // namespace
}  // namespace fq

using namespace fq;

extern "C" int image_quality(const float* img, const float* ref, int32_t nx, int32_t ny, double data_range,
                             double* out, void* stream) {
    FQ_REQUIRE(nx >= IQM_WIN && ny >= IQM_WIN, "images must be at least %d x %d (SSIM window)", IQM_WIN, IQM_WIN);
    FQ_REQUIRE((int64_t)nx * ny <= ((int64_t)1 << 24), "image larger than 2^24 pixels");
    FQ_REQUIRE(data_range > 0.0, "data_range must be > 0");
    FQ_REQUIRE(img && ref && out, "null pointer");
    IqmArgs p{};
    p.a = img;
    p.b = ref;
    p.out = out;
    p.nx = nx;
    p.ny = ny;
    p.c1 = (0.01 * data_range) * (0.01 * data_range);
    p.c2 = (0.03 * data_range) * (0.03 * data_range);
    p.range2 = data_range * data_range;
    choose_tiles(nx - IQM_WIN + 1, ny - IQM_WIN + 1, p.bx, p.by);
    double sum = 0.0;
    for (int i = 0; i < IQM_WIN; ++i) {
        const double t = i - 0.5 * (IQM_WIN - 1);
        p.w[i] = std::exp(-t * t / (2.0 * 1.5 * 1.5));
        sum += p.w[i];
    }
    for (int i = 0; i < IQM_WIN; ++i) p.w[i] /= sum;
    hipLaunchKernelGGL(image_quality_kernel, dim3(1), dim3(IQM_THREADS), IQM_LDS, as_stream(stream), p);
    FQ_LAUNCH_CHECK();
    return FQ_OK;
}
