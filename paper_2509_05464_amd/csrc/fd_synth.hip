// fd_synth: frequency-domain RF synthesis of point scatterers (Appendix D, Eq. 1 and
// Eq. 2; the scatterer-block partition and frequency stepping of Algorithm 2).
//
// Per frequency sample f_j = j df (k_j = 2 pi f_j / c), with the element response
//   H_e(s, f) = sum over the v sub-elements mu of element e (the coherent sub-element
//               sum of Eq. 2; Eq. 1 sums every transmitting sub-element) of
//               (r_ref / r) e^{(i k - alpha) r} sinc(k b_x u_x) sinc(k b_y u_y),
// the field of transmit a at scatterer s and the echo at receive element m are
//   T_a(s, f) = sum_e W_e e^{i 2 pi f dtau_ae} H_e(s, f),
//   P_a(m, f) = sum_s H_m(s, f) R_s T_a(s, f),
// and the RF is  rf_a(m, t) = 2 Re sum_j w_j P_a(m, f_j) e^{-i 2 pi j t / N},
// w_j = q_j S(f_j) df with S the Fourier transform of the Gaussian pulse (q = 1/2 at
// j = 0 and j = N/2).  Three kernels per scatterer block and batch of frames (the first two in
// one, fd_both_kernel, for few transmits and elements):
//   fd_tx_kernel   lane = scatterer: T for a chunk of KC consecutive frequencies and the
//                  transmits of a group; the four wavefronts of a workgroup take every fourth
//                  block of elements, whose W_e e^{i 2 pi f dtau_ae} they hold in LDS, and add up
//                  their sums at the end;
//   fd_rx_kernel   lane = receive element: P for the chunk, scatterers staged in LDS
//                  blocks with R_s T_a(s, f); scatterer ranges split for occupancy, partial
//                  sums kept apart and added in a fixed order;
//   fd_idft_kernel workgroup = (elements, transmit): the weighted inverse transform of the
//                  band, the complex exponential stepped in frequency, shared by the
//                  elements and re-anchored from an exact integer phase every 64 samples.
// Frames go through the kernels in batches as large as the workspace holds: one frame of a
// small scene (500 scatterers, 405 frequencies) fills a quarter of the chip for 0.6 ms.
//
// Element response: within a chunk e^{i k r} is stepped from frequency to frequency by one
// complex multiplication (the frequency-stepping propagation update of Algorithm 2),
// outwards from the chunk's middle, whose phase is taken in FP64 (cycles = j df r / c), so the
// error does not grow with j and is at most KC/2 steps.  The directivity sines (a few cycles
// at most) come straight from the hardware sine.  The
// kernels are bound by the VALU work of this response (FP64 path and reduction to a turn,
// 16 transcendentals, ~110 FP32 multiply-adds per sub-element and chunk); the products with
// the NA transmits add 4 NA KC.  Chunks of 8 cost 0.55 of chunks of 4 with a sine per
// frequency and axis; kernels compiled for the group's number of transmits do not compute
// 9 for 3.  (16 x 16 elements of 2 x 2, 3 transmits, 2000 static + 20 x 500 scatterers:
// 9.8 ms against 23.6.)
// Scatterer blocks bound the transmit-field buffer by the workspace (the memory partition
// of Algorithm 2); their echoes add up in P.
#include "fq_common.hpp"

namespace fq {
namespace {

constexpr int FD_THREADS = 256;
constexpr int KC = 8;         // frequencies per chunk
constexpr int AG = 9;         // transmits per launch group, at most
constexpr int EB = 16;        // elements per LDS block (transmit field) and wavefront
constexpr int SB = 32;        // scatterers per LDS block (echo)
constexpr int FD_MAX_K = 4096;
constexpr int FD_MIN_BLOCK = 256;
constexpr int MC = 8;         // elements of an inverse-transform workgroup, at most
constexpr int MC_MAX_K = 1024;   // band that MC elements' spectra fit in LDS for; two beyond
constexpr int64_t IDFT_WG = 1024;   // inverse-transform workgroups that fill the chip
constexpr double TWO_PI = 6.283185307179586;

struct FdArgs {
    const float* pos;       // [S][3] of the batch's first frame
    const float* amp;       // [S]
    const float* apod;      // [E] or null
    float2* T;              // [frame][chunk][nsb][nq][NA], nq = frequencies of the chunk
    float2* P;              // [frame][split][chunk][E][nq][NA]
    const float* w;         // [K] 2 w_j
    float* rf;              // output of the inverse transform
    int64_t s0, ns, nsb;    // scatterer block [s0, s0 + ns), T row stride nsb
    int64_t pos_stride;     // floats between frames of pos
    int n_elem, nx_el, K, j_lo, N, chunks;
    int vx, vy;
    int na;                 // transmits in this group (<= AG)
    int nsplit, p_acc;      // echo splits; P accumulates over scatterer blocks
    int rx_groups;          // wavefront groups of an echo workgroup that share its scatterers
    int dir;                // elements have a size
    double pitch_x, pitch_y, hx, hy;   // element pitch; (n-1)/2 pitch offsets
    double wx, wy;          // element size
    double df_c;            // df / c: cycles per metre per frequency step
    double alpha2_df;       // attenuation, powers of two per metre per frequency step
    double bx_df_c, by_df_c;   // directivity cycles per step per unit direction cosine (b df / c)
    double df;
    float r_ref;
    double ux[AG], uy[AG], t0[AG];   // transmit directions and first-firing offsets (s)
    double inv_c;
    // inverse transform
    int T_len, n_frames_out, frame0, n_angles_total, a0, accumulate;
};

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
    return make_float2(fmaf(a.x, b.x, -a.y * b.y), fmaf(a.x, b.y, a.y * b.x));
}

__device__ __forceinline__ void elem_xy(const FdArgs& a, int e, double& ex, double& ey) {
    ex = (e % a.nx_el) * a.pitch_x - a.hx;
    ey = (e / a.nx_el) * a.pitch_y - a.hy;
}

// h[q] = sum_mu (r_ref/r) e^{(i k - alpha) r} D for f = (j0 + q) df, q < KC, of an element whose
// centre is (dxc, dyc) off the scatterer; D = sinc sinc of the sub-element's direction.
__device__ __forceinline__ void elem_resp(const FdArgs& a, double dxc, double dyc, double sz2, int j0,
                                          const float* invj2, float2* h) {
    constexpr int M = KC / 2;
#pragma unroll
    for (int q = 0; q < KC; ++q) h[q] = make_float2(0.f, 0.f);
    float h0 = 0.0f;   // the response at f = 0
    const float tmin = 1e-12f * __builtin_amdgcn_rcpf((float)(j0 + KC));
    for (int mx = 0; mx < a.vx; ++mx) {
        const double dx = dxc - ((mx + 0.5) / a.vx - 0.5) * a.wx;
        const double dx2 = fma(dx, dx, sz2);
        for (int my = 0; my < a.vy; ++my) {
            const double dy = dyc - ((my + 0.5) / a.vy - 0.5) * a.wy;
            // r and 1/r (to about 1e-14, rounded to FP32 once) from one estimate
            const double d2 = fma(dy, dy, dx2), y = __builtin_amdgcn_rsq(d2), r0 = d2 * y;
            const double r = fma(fma(-r0, r0, d2), 0.5 * y, r0);
            const float rinv = (float)fma(fma(-r, y, 1.0), y, y);
            const double cyc = a.df_c * r;                        // phase cycles per frequency step
            const float2 zm = cis_cycles((double)(j0 + M) * cyc);
            const float2 st = cis_cycles(cyc);
            const float ar = (float)(a.alpha2_df * r);
            // Amplitudes of the lower half, from j0 up, and of the middle: a scatterer whose
            // attenuation over a step passes FP32's range decays to zero (steps down from the middle
            // would grow past it, from nothing).
            const float at = __builtin_amdgcn_exp2f(-ar);
            float am[M + 1];
            am[0] = __builtin_amdgcn_exp2f(-ar * (float)j0);
#pragma unroll
            for (int q = 0; q < M; ++q) am[q + 1] = am[q] * at;
            const float2 up = make_float2(st.x * at, st.y * at), dn = make_float2(st.x, -st.y);
            float g = a.r_ref * rinv;
            h0 += g;
            if (!a.dir) {
                const float2 z0 = make_float2(zm.x * g, zm.y * g);
                float2 z = make_float2(z0.x * am[M], z0.y * am[M]);
#pragma unroll
                for (int q = M; q < KC; ++q) {
                    h[q].x += z.x;
                    h[q].y += z.y;
                    z = cmul(z, up);
                }
                z = z0;
#pragma unroll
                for (int q = M - 1; q >= 0; --q) {
                    z = cmul(z, dn);
                    h[q].x = fmaf(z.x, am[q], h[q].x);
                    h[q].y = fmaf(z.y, am[q], h[q].y);
                }
                continue;
            }
            // sinc(2 pi j t) = sin(2 pi j t) / (2 pi j t), t = b df u / c turns per frequency step, the
            // sine straight from the hardware (argument reduced to a turn); 1 / j^2 of both axes
            // comes last.  Where |j t| stays below 1e-12 (an offset of about 1e-14 m: the rounding
            // error of an element's position, seen from a scatterer on its axis) j stands for the
            // sine: the product of two such t, in the one reciprocal of both axes, is below FP32's
            // range and its reciprocal infinite.  (The fraction c - floor(c) of a small negative c keeps
            // FP32's grid just below 1: the sinc is off by up to 3e-8 / |c|, and lost below 3e-8 turns.)
            const float tx = (float)(a.bx_df_c * dx) * rinv, ty = (float)(a.by_df_c * dy) * rinv;
            const bool axis_x = fabsf(tx) < tmin, axis_y = fabsf(ty) < tmin;
            float d[KC];
            {
                float s[KC];
#pragma unroll
                for (int q = 0; q < KC; ++q) {
                    const float c = tx * (float)(j0 + q);
                    d[q] = __builtin_amdgcn_sinf(c - floorf(c));
                }
#pragma unroll
                for (int q = 0; q < KC; ++q) {
                    const float c = ty * (float)(j0 + q);
                    s[q] = __builtin_amdgcn_sinf(c - floorf(c));
                }
                if (axis_x) {
#pragma unroll
                    for (int q = 0; q < KC; ++q) d[q] = (float)(j0 + q);
                }
                if (axis_y) {
#pragma unroll
                    for (int q = 0; q < KC; ++q) s[q] = (float)(j0 + q);
                }
#pragma unroll
                for (int q = 0; q < KC; ++q) d[q] *= s[q];
            }
            g *= __builtin_amdgcn_rcpf((axis_x ? 1.0f : (float)TWO_PI * tx) * (axis_y ? 1.0f : (float)TWO_PI * ty));
            const float2 z0 = make_float2(zm.x * g, zm.y * g);
            float2 z = make_float2(z0.x * am[M], z0.y * am[M]);
#pragma unroll
            for (int q = M; q < KC; ++q) {
                h[q].x = fmaf(z.x, d[q], h[q].x);
                h[q].y = fmaf(z.y, d[q], h[q].y);
                z = cmul(z, up);
            }
            z = z0;
#pragma unroll
            for (int q = M - 1; q >= 0; --q) {
                z = cmul(z, dn);
                d[q] *= am[q];
                h[q].x = fmaf(z.x, d[q], h[q].x);
                h[q].y = fmaf(z.y, d[q], h[q].y);
            }
        }
    }
    if (a.dir) {
#pragma unroll
        for (int q = 0; q < KC; ++q) {
            h[q].x *= invj2[q];
            h[q].y *= invj2[q];
        }
    }
    if (j0 == 0) h[0] = make_float2(h0, 0.0f);
}

__device__ __forceinline__ void chunk_invj2(int j0, float* invj2) {
#pragma unroll
    for (int q = 0; q < KC; ++q) invj2[q] = 1.0f / ((float)max(1, j0 + q) * (float)max(1, j0 + q));
}

// Transmit field T_a(s, f) of one chunk of frequencies; lane = scatterer.
template <int NA>
__global__ void __launch_bounds__(FD_THREADS) fd_tx_kernel(const FdArgs a) {
    constexpr int W = FD_THREADS / 64;
    constexpr int TAB = EB * KC * NA, SUM = 64 * KC * NA;   // float2
    __shared__ float2 lds[W * TAB > SUM ? W * TAB : SUM];
    const int chunk = blockIdx.y, fr = blockIdx.z;
    const int j0 = a.j_lo + chunk * KC;
    const int l = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t sl = (int64_t)blockIdx.x * 64 + l;
    const bool valid = sl < a.ns;
    double sx = 0.0, sy = 0.0, sz = 1.0;
    if (valid) {
        const float* p = a.pos + fr * a.pos_stride + 3 * (a.s0 + sl);
        sx = p[0];
        sy = p[1];
        sz = p[2];
    }
    const bool live = valid && sz > 0.0;
    if (!live) sz = 1.0;
    const double sz2 = sz * sz;
    float invj2[KC];
    chunk_invj2(j0, invj2);
    float2 acc[KC][NA];
#pragma unroll
    for (int q = 0; q < KC; ++q)
#pragma unroll
        for (int g = 0; g < NA; ++g) acc[q][g] = make_float2(0.f, 0.f);

    float2* tab = lds + w * TAB;   // [EB][KC][NA] of this wavefront
    const int eb = min(EB, (a.n_elem + W - 1) / W);   // (up to 64 elements: shared evenly)
    for (int e0 = w * eb; e0 < a.n_elem; e0 += W * eb) {
        __builtin_amdgcn_wave_barrier();
        for (int i = l; i < TAB; i += 64) {
            const int el = i / (KC * NA), q = (i / NA) % KC, g = i % NA;
            const int e = e0 + el;
            float2 v = make_float2(0.f, 0.f);
            if (e < a.n_elem) {
                double ex, ey;
                elem_xy(a, e, ex, ey);
                const double dtau = (a.ux[g] * ex + a.uy[g] * ey) * a.inv_c - a.t0[g];
                v = cis_cycles((double)(j0 + q) * a.df * dtau);
                const float wgt = a.apod ? a.apod[e] : 1.0f;
                v.x *= wgt;
                v.y *= wgt;
            }
            tab[i] = v;
        }
        __builtin_amdgcn_wave_barrier();
        const int ne = min(eb, a.n_elem - e0);
        for (int el = 0; el < ne; ++el) {
            double ex, ey;
            elem_xy(a, e0 + el, ex, ey);
            float2 h[KC];
            elem_resp(a, sx - ex, sy - ey, sz2, j0, invj2, h);
#pragma unroll
            for (int q = 0; q < KC; ++q)
#pragma unroll
                for (int g = 0; g < NA; ++g) {
                    const float2 E = tab[(el * KC + q) * NA + g];
                    acc[q][g].x = fmaf(h[q].x, E.x, fmaf(-h[q].y, E.y, acc[q][g].x));
                    acc[q][g].y = fmaf(h[q].x, E.y, fmaf(h[q].y, E.x, acc[q][g].y));
                }
        }
    }
    // the wavefronts' sums, in order; lane-minor, so that a wavefront's accesses are contiguous
    for (int turn = 0; turn < W; ++turn) {
        __syncthreads();
        if (w == turn) {
#pragma unroll
            for (int q = 0; q < KC; ++q)
#pragma unroll
                for (int g = 0; g < NA; ++g) {
                    float2& s = lds[(q * NA + g) * 64 + l];
                    s = turn ? make_float2(s.x + acc[q][g].x, s.y + acc[q][g].y) : acc[q][g];
                }
        }
    }
    __syncthreads();
    const int row = min(KC, a.K - chunk * KC) * NA;
    float2* dst = a.T + ((int64_t)fr * a.K + chunk * KC) * a.nsb * NA + (int64_t)blockIdx.x * 64 * row;
    const int n = (int)min((int64_t)64, a.ns - (int64_t)blockIdx.x * 64);
    // (dead scatterers' fields are not used: their echo is skipped)
    for (int i = threadIdx.x; i < n * row; i += FD_THREADS) dst[i] = lds[(i % row) * 64 + i / row];
}

// Echo P_a(m, f) of one chunk of frequencies and one scatterer split; lane = element.  Up to 64
// (128) elements the workgroup's wavefronts form 4 (2) groups that share the scatterers, and
// the groups' sums are added in order at the end: one wavefront a workgroup left the chip half
// empty (8 x 8 elements, 9 transmits, 6837 scatterers, splits bound by the
// workspace: 4.1 ms a call, 1.9 so).
template <int NA>
__global__ void __launch_bounds__(FD_THREADS) fd_rx_kernel(const FdArgs a) {
    __shared__ float4 spos[SB];
    __shared__ float2 xs[SB * KC * NA];
    const int chunk = blockIdx.y, fr = blockIdx.z / a.nsplit, split = blockIdx.z % a.nsplit;
    const int j0 = a.j_lo + chunk * KC;
    const int lanes = blockDim.x / a.rx_groups;   // elements of the workgroup, a multiple of 64
    const int grp = __builtin_amdgcn_readfirstlane(threadIdx.x / lanes), le = threadIdx.x - grp * lanes;
    const int m = blockIdx.x * lanes + le;
    const int64_t per = (a.ns + a.nsplit - 1) / a.nsplit;
    const int64_t sb0 = split * per;
    const int64_t sb1 = a.ns < sb0 + per ? a.ns : sb0 + per;
    const float* pos = a.pos + fr * a.pos_stride + 3 * a.s0;
    const float* amp = a.amp + a.s0;
    const int row = min(KC, a.K - chunk * KC) * NA;
    const float2* T = a.T + ((int64_t)fr * a.K + chunk * KC) * a.nsb * NA;
    double ex = 0.0, ey = 0.0;
    if (m < a.n_elem) elem_xy(a, m, ex, ey);
    float invj2[KC];
    chunk_invj2(j0, invj2);
    float2 acc[KC][NA];
#pragma unroll
    for (int q = 0; q < KC; ++q)
#pragma unroll
        for (int g = 0; g < NA; ++g) acc[q][g] = make_float2(0.f, 0.f);

    for (int64_t b = sb0; b < sb1; b += SB) {
        const int nb = sb1 - b < SB ? (int)(sb1 - b) : SB;
        __syncthreads();
        for (int i = threadIdx.x; i < nb; i += blockDim.x) {
            const float* p = pos + 3 * (b + i);
            spos[i] = make_float4(p[0], p[1], p[2], 0.f);
        }
        for (int i = threadIdx.x; i < nb * row; i += blockDim.x) {
            const float2 v = T[b * row + i];
            const float r = amp[b + i / row];
            xs[i] = make_float2(v.x * r, v.y * r);
        }
        __syncthreads();
        if (m < a.n_elem) {
            for (int sl = grp; sl < nb; sl += a.rx_groups) {
                const float4 p = spos[sl];
                if (!(p.z > 0.0f)) continue;
                const double sz = p.z;
                float2 h[KC];
                elem_resp(a, (double)p.x - ex, (double)p.y - ey, sz * sz, j0, invj2, h);
#pragma unroll
                for (int q = 0; q < KC; ++q)
#pragma unroll
                    for (int g = 0; g < NA; ++g) {
                        const float2 X = xs[sl * row + q * NA + g];   // (past the chunk: not stored)
                        acc[q][g].x = fmaf(h[q].x, X.x, fmaf(-h[q].y, X.y, acc[q][g].x));
                        acc[q][g].y = fmaf(h[q].x, X.y, fmaf(h[q].y, X.x, acc[q][g].y));
                    }
            }
        }
    }
    if (a.rx_groups > 1) {   // the others' sums to group 0, one frequency at a time
        static_assert(3 * 64 <= SB * KC && 128 <= SB * KC, "the groups' sums of a frequency fit the scatterers' block");
#pragma unroll
        for (int q = 0; q < KC; ++q) {
            __syncthreads();
            if (grp > 0) {
#pragma unroll
                for (int g = 0; g < NA; ++g) xs[((grp - 1) * NA + g) * lanes + le] = acc[q][g];
            }
            __syncthreads();
            if (grp == 0)
                for (int k = 1; k < a.rx_groups; ++k)
#pragma unroll
                    for (int g = 0; g < NA; ++g) {
                        const float2 v = xs[((k - 1) * NA + g) * lanes + le];
                        acc[q][g].x += v.x;
                        acc[q][g].y += v.y;
                    }
        }
    }
    if (m >= a.n_elem || grp > 0) return;
    float2* dst = a.P + (((int64_t)fr * a.nsplit + split) * a.K + chunk * KC) * a.n_elem * NA + (int64_t)m * row;
#pragma unroll
    for (int q = 0; q < KC; ++q)
#pragma unroll
        for (int g = 0; g < NA; ++g) {
            if (q * NA >= row) break;
            float2 v = acc[q][g];
            if (a.p_acc) {
                v.x += dst[q * NA + g].x;
                v.y += dst[q * NA + g].y;
            }
            dst[q * NA + g] = v;
        }
}

// Both legs of one chunk of frequencies in one workgroup, thread = element: the response of a
// scatterer is formed once, summed over the workgroup into its transmit field (a halving
// exchange over the wavefront, the wavefronts' sums through LDS) and multiplied into the echo.
// Taken where the registers hold it, for up to BOTH_NA transmits and BOTH_MAX_E elements: the
// response is most of the work of either leg (16 x 16 elements, 3 transmits, 2000 static and 20 x
// 500 scatterers: 6.8 ms, 9.8 with the legs apart).
constexpr int BOTH_NA = 3, BOTH_MAX_E = 512;
constexpr int SF = 4;          // scatterers between barriers

template <int CTRL>
__device__ __forceinline__ float dpp_add(float x) {
    return x + __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}

// Sums of the NV values of v over the wavefront: row r of 16 lanes ends with values
// r NV/4 .. (r + 1) NV/4 - 1 in v[0 .. NV/4 - 1], the same in its 16 lanes.
template <int NV>
__device__ __forceinline__ void wave_sums(float (&v)[NV]) {
#pragma unroll
    for (int i = 0; i < NV / 2; ++i) {
        const auto p = __builtin_amdgcn_permlane32_swap(__float_as_int(v[i]), __float_as_int(v[i + NV / 2]), false, false);
        v[i] = __int_as_float(p[0]) + __int_as_float(p[1]);
    }
#pragma unroll
    for (int i = 0; i < NV / 4; ++i) {
        const auto p = __builtin_amdgcn_permlane16_swap(__float_as_int(v[i]), __float_as_int(v[i + NV / 4]), false, false);
        v[i] = __int_as_float(p[0]) + __int_as_float(p[1]);
        v[i] = dpp_add<0x128>(v[i]);   // row rotations by 8, 4, 2, 1
        v[i] = dpp_add<0x124>(v[i]);
        v[i] = dpp_add<0x122>(v[i]);
        v[i] = dpp_add<0x121>(v[i]);
    }
}

template <int NA>
size_t both_lds(int threads) {
    return sizeof(float) * ((size_t)2 * KC * NA * threads + (size_t)(threads / 64 + 1) * SF * 2 * KC * NA);
}

template <int NA>
__global__ void __launch_bounds__(BOTH_MAX_E) fd_both_kernel(const FdArgs a) {
    constexpr int NV = 2 * KC * NA;   // a transmit field: [q][g][re, im]
    extern __shared__ float4 lds4[];
    __shared__ float4 spos[SF];
    const int nthr = blockDim.x, nw = nthr / 64;
    float2* tab = reinterpret_cast<float2*>(lds4);                    // [KC NA][threads] W e^{i 2 pi f dtau}
    float* part = reinterpret_cast<float*>(tab + KC * NA * nthr);     // [wavefront][SF][NV]
    float* xs = part + nw * SF * NV;                                  // [SF][NV] R T
    const int chunk = blockIdx.x, fr = blockIdx.z, split = blockIdx.y;
    const int j0 = a.j_lo + chunk * KC;
    const int m = threadIdx.x, l = m & 63, w = __builtin_amdgcn_readfirstlane(m >> 6);
    const int64_t per = (a.ns + a.nsplit - 1) / a.nsplit;
    const int64_t sb0 = split * per;
    const int64_t sb1 = a.ns < sb0 + per ? a.ns : sb0 + per;
    const float* pos = a.pos + fr * a.pos_stride + 3 * a.s0;
    const float* amp = a.amp + a.s0;
    double ex, ey;
    elem_xy(a, m, ex, ey);
    const float wgt = m >= a.n_elem ? 0.0f : a.apod ? a.apod[m] : 1.0f;
#pragma unroll
    for (int g = 0; g < NA; ++g) {
        const double dtau = (a.ux[g] * ex + a.uy[g] * ey) * a.inv_c - a.t0[g];
#pragma unroll
        for (int q = 0; q < KC; ++q) {
            const float2 v = cis_cycles((double)(j0 + q) * a.df * dtau);
            tab[(q * NA + g) * nthr + m] = make_float2(v.x * wgt, v.y * wgt);
        }
    }
    float invj2[KC];
    chunk_invj2(j0, invj2);
    float2 acc[KC][NA];
#pragma unroll
    for (int q = 0; q < KC; ++q)
#pragma unroll
        for (int g = 0; g < NA; ++g) acc[q][g] = make_float2(0.f, 0.f);

    for (int64_t b = sb0; b < sb1; b += SF) {
        const int nb = sb1 - b < SF ? (int)(sb1 - b) : SF;
        __syncthreads();
        if (m < SF) {
            float4 v = make_float4(0.f, 0.f, -1.f, 0.f);
            if (m < nb) v = make_float4(pos[3 * (b + m)], pos[3 * (b + m) + 1], pos[3 * (b + m) + 2], amp[b + m]);
            if (!(v.z > 0.0f)) v.w = 0.0f;   // behind the array: not in either leg
            spos[m] = v;
        }
        __syncthreads();
        float2 h[SF][KC];
#pragma unroll
        for (int i = 0; i < SF; ++i) {
            const float4 p = spos[i];
            if (p.z > 0.0f) {
                const double sz = p.z;
                elem_resp(a, (double)p.x - ex, (double)p.y - ey, sz * sz, j0, invj2, h[i]);
            } else {
#pragma unroll
                for (int q = 0; q < KC; ++q) h[i][q] = make_float2(0.f, 0.f);
            }
            float v[NV];
#pragma unroll
            for (int q = 0; q < KC; ++q)
#pragma unroll
                for (int g = 0; g < NA; ++g) {
                    const float2 E = tab[(q * NA + g) * nthr + m];
                    v[2 * (q * NA + g)] = fmaf(h[i][q].x, E.x, -h[i][q].y * E.y);
                    v[2 * (q * NA + g) + 1] = fmaf(h[i][q].x, E.y, h[i][q].y * E.x);
                }
            wave_sums<NV>(v);
            if ((l & 15) == 0) {
                float4* dst = reinterpret_cast<float4*>(part + (w * SF + i) * NV + (l >> 4) * (NV / 4));
#pragma unroll
                for (int c = 0; c < NV / 16; ++c) dst[c] = make_float4(v[4 * c], v[4 * c + 1], v[4 * c + 2], v[4 * c + 3]);
            }
        }
        __syncthreads();
        for (int i = m; i < SF * NV; i += nthr) {
            float t = part[i];
            for (int k = 1; k < nw; ++k) t += part[k * SF * NV + i];
            xs[i] = t * spos[i / NV].w;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < SF; ++i)
#pragma unroll
            for (int q = 0; q < KC; ++q)
#pragma unroll
                for (int g = 0; g < NA; ++g) {
                    const float2 X = *reinterpret_cast<const float2*>(xs + i * NV + 2 * (q * NA + g));
                    acc[q][g].x = fmaf(h[i][q].x, X.x, fmaf(-h[i][q].y, X.y, acc[q][g].x));
                    acc[q][g].y = fmaf(h[i][q].x, X.y, fmaf(h[i][q].y, X.x, acc[q][g].y));
                }
    }
    if (m >= a.n_elem) return;
    const int row = min(KC, a.K - chunk * KC) * NA;
    float2* dst = a.P + (((int64_t)fr * a.nsplit + split) * a.K + chunk * KC) * a.n_elem * NA + (int64_t)m * row;
#pragma unroll
    for (int q = 0; q < KC; ++q)
#pragma unroll
        for (int g = 0; g < NA; ++g) {
            if (q * NA >= row) break;
            dst[q * NA + g] = acc[q][g];
        }
}

// Inverse transform of NM elements of one transmit: rf(t) = sum_j Re(Q_j e^{-i 2 pi j t / N}),
// Q_j = 2 w_j sum_split P; written to n_frames_out consecutive frames from frame0.
template <int NM>
__global__ void __launch_bounds__(FD_THREADS) fd_idft_kernel(const FdArgs a) {
    extern __shared__ float2 Q[];   // [K][NM]
    const int m0 = blockIdx.x * NM, g = blockIdx.y, fr = blockIdx.z;
    for (int i = threadIdx.x; i < a.K * NM; i += FD_THREADS) {
        const int kk = i / NM, m = min(m0 + i % NM, a.n_elem - 1);
        const int c0 = kk / KC * KC, row = min(KC, a.K - c0) * a.na;
        float2 s = make_float2(0.f, 0.f);
        for (int sp = 0; sp < a.nsplit; ++sp) {
            const float2 v = a.P[(((int64_t)fr * a.nsplit + sp) * a.K + c0) * a.n_elem * a.na + (int64_t)m * row +
                                 (kk - c0) * a.na + g];
            s.x += v.x;
            s.y += v.y;
        }
        const float wk = a.w[kk];
        Q[i] = make_float2(s.x * wk, s.y * wk);
    }
    __syncthreads();
    const int an = a.a0 + g, nm = min(NM, a.n_elem - m0);
    for (int t = threadIdx.x; t < a.T_len; t += FD_THREADS) {
        // e^{-i 2 pi j t / N}, stepped in j; exact integer phase every 64 samples
        const float2 st = cis_cycles(-(double)t / a.N);
        float acc[NM];
#pragma unroll
        for (int c = 0; c < NM; ++c) acc[c] = 0.0f;
        for (int k0 = 0; k0 < a.K; k0 += 64) {
            const int64_t ph = ((int64_t)(a.j_lo + k0) * t) % a.N;
            float2 z = cis_cycles(-(double)ph / a.N);
            const int k1 = min(a.K, k0 + 64);
#pragma unroll 4
            for (int kk = k0; kk < k1; ++kk) {
#pragma unroll
                for (int c = 0; c < NM; ++c) {
                    const float2 q = Q[kk * NM + c];
                    acc[c] = fmaf(q.x, z.x, fmaf(-q.y, z.y, acc[c]));
                }
                z = cmul(z, st);
            }
        }
#pragma unroll
        for (int c = 0; c < NM; ++c) {
            if (c >= nm) break;
            for (int f = 0; f < a.n_frames_out; ++f) {
                float* dst = a.rf + (((int64_t)(a.frame0 + fr + f) * a.n_angles_total + an) * a.n_elem + m0 + c) * a.T_len + t;
                *dst = a.accumulate ? *dst + acc[c] : acc[c];
            }
        }
    }
}

using FdFn = void (*)(const FdArgs);
template <int NA>
FdFn fd_fn(bool tx, int na) {
    if constexpr (NA > AG) {
        return nullptr;
    } else {
        if (na == NA) return tx ? fd_tx_kernel<NA> : fd_rx_kernel<NA>;
        return fd_fn<NA + 1>(tx, na);
    }
}

// Elements of an inverse-transform workgroup: they share the stepped exponential, so as many as
// leave IDFT_WG workgroups (a launch, 1500 samples: 32 elements, 6 transmits at 8 483 us, at 1
// 124; 16 x 16 elements, 9 transmits at 8 564, at 2 375).
int idft_elements(int E, int K, int64_t transmits) {
    int nm = K <= MC_MAX_K ? MC : 2;
    while (nm > 1 && (E + nm - 1) / nm * transmits < IDFT_WG) nm /= 2;
    return nm;
}
FdFn idft_fn(int nm) {
    return nm == 8 ? fd_idft_kernel<8> : nm == 4 ? fd_idft_kernel<4> : nm == 2 ? fd_idft_kernel<2> : fd_idft_kernel<1>;
}

__global__ void fd_weights_kernel(float* w, int K, int j_lo, int N, double df, double fc, double sig) {
    const int kk = blockIdx.x * blockDim.x + threadIdx.x;
    if (kk >= K) return;
    const int j = j_lo + kk;
    const double f = j * df;
    const double aa = 2.0 * 3.141592653589793 * 3.141592653589793 * sig * sig;
    const double S = sig * 2.5066282746310002 / 2.0 * (exp(-aa * (f - fc) * (f - fc)) + exp(-aa * (f + fc) * (f + fc)));
    const double q = (j == 0 || 2 * j == N) ? 0.5 : 1.0;
    w[kk] = (float)(2.0 * q * S * df);
}

struct FdPlan {
    int N, j_lo, K, chunks;
    size_t off_T;      // the weights come first
    size_t bytes;      // what the size query asks for
};

double spectrum(double f, double fc, double sig) {
    const double aa = 2.0 * M_PI * M_PI * sig * sig;
    return sig * std::sqrt(2.0 * M_PI) / 2.0 * (std::exp(-aa * (f - fc) * (f - fc)) + std::exp(-aa * (f + fc) * (f + fc)));
}

size_t field_bytes(int K, int64_t nsb, int na) { return round_up(sizeof(float2) * (size_t)K * nsb * na, 256); }

FdPlan plan(const fq_probe& p, const fq_pulse& pl, const fq_fd_params& fd, int n_samples, int64_t nsb) {
    FdPlan r{};
    const double sig = pl.n_cycles / (2.0 * std::sqrt(2.0 * std::log(2.0)) * p.fc_hz);
    r.N = n_samples + 2 * (int)std::ceil(6.0 * sig * p.fs_hz);
    const double df = p.fs_hz / r.N;
    double smax = 0.0;
    for (int j = 0; j <= r.N / 2; ++j) smax = std::max(smax, spectrum(j * df, p.fc_hz, sig));
    int lo = -1, hi = -1;
    for (int j = 0; j <= r.N / 2; ++j) {
        if (spectrum(j * df, p.fc_hz, sig) >= fd.spectral_floor * smax) {
            if (lo < 0) lo = j;
            hi = j;
        }
    }
    r.j_lo = lo;
    r.K = hi - lo + 1;
    r.chunks = (r.K + KC - 1) / KC;
    const int E = p.nx_el * p.ny_el;
    // one frame's buffers for AG transmits and up to 8 echo splits
    const int wg0 = ((E + FD_THREADS - 1) / FD_THREADS) * ((r.K + 3) / 4);
    const int nsplit = (int)std::max<int64_t>(1, std::min<int64_t>({(int64_t)8, (1024 + wg0 - 1) / wg0, (nsb + 63) / 64}));
    r.off_T = round_up(sizeof(float) * r.K, 256);
    r.bytes = r.off_T + field_bytes(r.K, nsb, AG) + round_up(sizeof(float2) * (size_t)nsplit * r.K * E * AG, 256);
    return r;
}

int check_fd(const fq_probe* probe, const fq_tx* tx, const fq_pulse* pulse, const fq_fd_params* fd, int n_samples) {
    int st = check_probe_tx(probe, tx);
    if (st != FQ_OK) return st;
    FQ_REQUIRE(pulse && fd, "pulse / fd parameters must not be NULL");
    FQ_REQUIRE(pulse->n_cycles > 0 && pulse->r_ref_m > 0, "bad pulse parameters");
    FQ_REQUIRE(fd->n_sub_x >= 1 && fd->n_sub_y >= 1 && fd->n_sub_x * fd->n_sub_y <= 64, "sub-elements must be 1..64");
    FQ_REQUIRE(fd->elem_width_x >= 0 && fd->elem_width_y >= 0 && fd->elem_width_x <= probe->pitch_x * 4 &&
                   fd->elem_width_y <= probe->pitch_y * 4,
               "bad element size");
    FQ_REQUIRE(fd->atten_db_cm_mhz >= 0 && fd->atten_db_cm_mhz < 100, "bad attenuation");
    FQ_REQUIRE(fd->spectral_floor > 0 && fd->spectral_floor < 1, "spectral_floor must be in (0, 1)");
    FQ_REQUIRE(n_samples >= 1 && n_samples <= 16384, "bad n_samples");
    return FQ_OK;
}

}  // namespace
}  // namespace fq

using namespace fq;

extern "C" size_t fd_workspace_size(const fq_probe* probe, const fq_tx* tx, const fq_pulse* pulse,
                                    const fq_fd_params* fd, int32_t n_samples, int64_t scatterers_per_block) {
    if (check_fd(probe, tx, pulse, fd, n_samples) != FQ_OK) return 0;
    return plan(*probe, *pulse, *fd, n_samples, std::max<int64_t>(FD_MIN_BLOCK, scatterers_per_block)).bytes;
}

extern "C" int fd_synth(const fq_probe* probe, const fq_tx* tx, const fq_pulse* pulse, const fq_fd_params* fd,
                        int32_t n_frames, int64_t n_scat, const float* pos, int32_t pos_static, const float* amp,
                        const float* apod, int32_t n_samples, int32_t accumulate, void* ws, size_t ws_bytes, float* rf,
                        void* stream) {
    int st = check_fd(probe, tx, pulse, fd, n_samples);
    if (st != FQ_OK) return st;
    FQ_REQUIRE(n_frames >= 1 && n_scat >= 0, "bad n_frames / n_scat");
    FQ_REQUIRE(rf && aligned16(rf) && ws && aligned16(ws), "null or misaligned rf / ws");
    FQ_REQUIRE(n_scat == 0 || (pos && amp), "pos/amp must not be NULL");
    const int E = probe->nx_el * probe->ny_el;
    const int A = tx->n_angles;
    hipStream_t s = as_stream(stream);
    if (n_scat == 0) return accumulate ? FQ_OK : zero_async(rf, sizeof(float) * (size_t)n_frames * A * E * n_samples, s);
    // largest scatterer block whose buffers fit the workspace (memory partition)
    const int64_t want = n_scat;
    FdPlan pl = plan(*probe, *pulse, *fd, n_samples, FD_MIN_BLOCK);
    if (ws_bytes < pl.bytes) {
        set_error("workspace too small: %zu < %zu bytes", ws_bytes, pl.bytes);
        return FQ_E_WORKSPACE;
    }
    int64_t lo = FD_MIN_BLOCK, hi = std::max<int64_t>(FD_MIN_BLOCK, want);
    if (plan(*probe, *pulse, *fd, n_samples, hi).bytes <= ws_bytes) {
        lo = hi;
    } else {
        while (hi - lo > 1) {
            const int64_t mid = (lo + hi) / 2;
            if (plan(*probe, *pulse, *fd, n_samples, mid).bytes <= ws_bytes) lo = mid; else hi = mid;
        }
    }
    const int64_t nsb = lo;
    FQ_REQUIRE(pl.K >= 1 && pl.K <= FD_MAX_K, "frequency band of %d samples (limit %d)", pl.K, FD_MAX_K);
    char* w = reinterpret_cast<char*>(ws);
    const TxHost th = make_tx(*probe, *tx);
    const double sig = pulse->n_cycles / (2.0 * std::sqrt(2.0 * std::log(2.0)) * probe->fc_hz);
    const double df = probe->fs_hz / pl.N;

    FdArgs a{};
    a.apod = apod;
    a.T = reinterpret_cast<float2*>(w + pl.off_T);
    a.w = reinterpret_cast<const float*>(w);
    a.rf = rf;
    a.amp = amp;
    a.nsb = nsb;
    a.n_elem = E;
    a.nx_el = probe->nx_el;
    a.K = pl.K;
    a.j_lo = pl.j_lo;
    a.N = pl.N;
    a.vx = fd->n_sub_x;
    a.vy = fd->n_sub_y;
    a.chunks = pl.chunks;
    a.dir = fd->elem_width_x > 0 || fd->elem_width_y > 0;
    a.pos_stride = pos_static ? 0 : 3 * n_scat;
    a.pitch_x = probe->pitch_x;
    a.pitch_y = probe->pitch_y;
    a.hx = 0.5 * (probe->nx_el - 1) * probe->pitch_x;
    a.hy = 0.5 * (probe->ny_el - 1) * probe->pitch_y;
    a.wx = fd->elem_width_x;
    a.wy = fd->elem_width_y;
    a.df = df;
    a.df_c = df / probe->c_mps;
    a.bx_df_c = 0.5 * fd->elem_width_x / fd->n_sub_x * df / probe->c_mps;
    a.by_df_c = 0.5 * fd->elem_width_y / fd->n_sub_y * df / probe->c_mps;
    a.alpha2_df = fd->atten_db_cm_mhz / (20.0 * std::log10(2.0)) * 100.0 * df / 1e6;
    a.r_ref = (float)pulse->r_ref_m;
    a.inv_c = 1.0 / probe->c_mps;
    a.T_len = n_samples;
    a.n_angles_total = A;
    a.accumulate = accumulate ? 1 : 0;

    hipLaunchKernelGGL(fd_weights_kernel, dim3((pl.K + 255) / 256), dim3(256), 0, s,
                       reinterpret_cast<float*>(w), pl.K, pl.j_lo, pl.N, df, probe->fc_hz, sig);
    FQ_LAUNCH_CHECK();
    const int nfr = pos_static ? 1 : n_frames;
    const int rx_lanes = std::min(FD_THREADS, (E + 63) / 64 * 64), rx_blocks = (E + rx_lanes - 1) / rx_lanes;
    a.rx_groups = FD_THREADS / rx_lanes;
    const int rx_threads = rx_lanes * a.rx_groups;
    const int groups = (A + AG - 1) / AG;
    for (int a0 = 0; a0 < A; a0 += a.na) {
        a.a0 = a0;
        a.na = (A + groups - 1) / groups;   // groups of equal size
        if (a0 + a.na > A) a.na = A - a0;
        for (int g = 0; g < a.na; ++g) {
            a.ux[g] = th.ux[a0 + g];
            a.uy[g] = th.uy[a0 + g];
            a.t0[g] = th.t0[a0 + g];
        }
        // Frames per batch: what the workspace holds (one if the scatterers come in blocks).
        // Echo splits: enough for about 16 wavefronts a compute unit, again if there is room.
        const bool both = a.na <= BOTH_NA && E <= BOTH_MAX_E;
        const size_t t_bytes = both ? 0 : field_bytes(pl.K, nsb, a.na), p_bytes = sizeof(float2) * (size_t)pl.K * E * a.na;
        const size_t room = ws_bytes - pl.off_T;
        int64_t batch = both || nsb >= n_scat ? std::min<int64_t>(nfr, room / (t_bytes + p_bytes)) : 1;
        batch = std::max<int64_t>(1, std::min<int64_t>(batch, 2048));
        batch = (nfr + (nfr + batch - 1) / batch - 1) / ((nfr + batch - 1) / batch);
        const int both_threads = (E + 63) / 64 * 64;
        const int64_t waves = (int64_t)(both ? both_threads / 64 : rx_blocks * (rx_threads / 64)) * pl.chunks * batch;
        a.nsplit = (int)std::max<int64_t>(1, std::min<int64_t>({(int64_t)16, (4096 + waves - 1) / waves, (nsb + SB - 1) / SB,
                                                                (int64_t)((room / batch - t_bytes) / p_bytes)}));
        a.P = reinterpret_cast<float2*>(w + pl.off_T + batch * t_bytes);
        for (int f = 0; f < nfr; f += (int)batch) {
            const unsigned nb = (unsigned)std::min<int64_t>(batch, nfr - f);
            a.pos = pos + (int64_t)f * a.pos_stride;
            if (both) {   // (all scatterers at once: no field to hold)
                a.s0 = 0;
                a.ns = n_scat;
                auto fn = a.na == 1 ? fd_both_kernel<1> : a.na == 2 ? fd_both_kernel<2> : fd_both_kernel<3>;
                const size_t lds = a.na == 1 ? both_lds<1>(both_threads) : a.na == 2 ? both_lds<2>(both_threads) : both_lds<3>(both_threads);
                hipLaunchKernelGGL(fn, dim3(pl.chunks, a.nsplit, nb), dim3(both_threads), lds, s, a);
                FQ_LAUNCH_CHECK();
            }
            for (int64_t s0 = 0; s0 < n_scat && !both; s0 += nsb) {
                a.s0 = s0;
                a.ns = std::min<int64_t>(nsb, n_scat - s0);
                a.p_acc = s0 > 0 ? 1 : 0;
                hipLaunchKernelGGL(fd_fn<1>(true, a.na), dim3((unsigned)((a.ns + 63) / 64), pl.chunks, nb),
                                   dim3(FD_THREADS), 0, s, a);
                FQ_LAUNCH_CHECK();
                hipLaunchKernelGGL(fd_fn<1>(false, a.na), dim3(rx_blocks, pl.chunks, nb * a.nsplit), dim3(rx_threads), 0,
                                   s, a);
                FQ_LAUNCH_CHECK();
            }
            a.frame0 = f;
            a.n_frames_out = pos_static ? n_frames : 1;
            const int nm = idft_elements(E, pl.K, (int64_t)a.na * nb);
            hipLaunchKernelGGL(idft_fn(nm), dim3((E + nm - 1) / nm, a.na, nb), dim3(FD_THREADS),
                               sizeof(float2) * (size_t)pl.K * nm, s, a);
            FQ_LAUNCH_CHECK();
        }
    }
    return FQ_OK;
}
