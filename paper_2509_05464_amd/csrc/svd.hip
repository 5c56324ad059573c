// svd_clutter_filter / hermitian_eig / power_doppler (gfx950).
//
// The clutter filter needs every eigenvalue of the N_t x N_t Hermitian Gram G = S^H S
// (the singular-value curve, the knee) but only the K <= 64 leading eigenvectors (the
// tissue subspace).  Its FP64 eigensolver therefore runs:
//  1. tridiagonalisation (one workgroup up to 128 frames, one launch a step beyond): for
//     k = 0 .. n-2 a Householder reflector
//     H_k = I - tau_k v_k v_k^H (v_k[k+1] = 1) maps column k below the diagonal to
//     beta_k e_1 with beta_k real, and the trailing block is updated two-sided,
//     A22 <- H^H A22 H = A22 - (v w^H + w v^H),  w = tau A22 v - |tau|^2 (v^H A22 v) v / 2.
//     G = Q T Q^H with Q = H_0 H_1 ... and T real symmetric tridiagonal (d, e = beta).
//  2. eigenvalues of T by multisection on Sturm counts: the number of negative pivots of
//     the LDL^T factorisation of T - x I is the number of eigenvalues below x (Sylvester's
//     law of inertia); one wavefront per eigenvalue evaluates the count at 64 points of
//     its bracket at once and keeps the sub-interval where the count passes the
//     eigenvalue's index (a 65-fold narrowing per round), on T scaled to unit size;
//  3. the rank K (fixed, or the knee of the dB spectrum);
//  4. eigenvectors of T for the K leading eigenvalues by inverse iteration: a few solves
//     of (T - lambda I) z = x with a tridiagonal LU factorisation with partial pivoting,
//     one workgroup per eigenvalue, all in parallel; the vectors of eigenvalues closer
//     than 1e-6 of ||T|| (a cluster) are then made orthogonal by Gram-Schmidt, twice;
//  5. back-transformation of the K columns, V_K = Q Z_K, one wavefront per column.
// hermitian_eig (every eigenvector) keeps the implicit QL iteration with Wilkinson shifts
// (the EISPACK tql2 recurrence, Bowdler, Martin, Reinsch & Wilkinson 1968) on T, logging
// each plane rotation, and replays the log on the identity to form all of Z.
// Eigenvalues are clamped at zero (round-off of a PSD matrix).
//
// The projection S_f = S - (S V_K) V_K^H and the power Doppler are fused: one wavefront per 16
// voxels forms their K projections on the matrix cores, reads the series again to subtract them
// and accumulates |S_f|^2.  Power Doppler alone takes one read of S up to K = 16.
#include "fq_common.hpp"

namespace fq {
namespace {

constexpr int KMAX = 64;
constexpr int QL_MAX_ITER = 60;       // QL iterations per eigenvalue
constexpr int ROT_PER_N2 = 8;         // rotation log capacity, in units of n^2 (typical use ~1.2)
// The knee rule reads the dB spectrum down to -60 dB: the cutoff is marked by eye on the
// singular-value curve (Section 3.2) and power Doppler is shown over 60 dB (Sections 3.1,
// 3.3); eigen-energies further below the leading one are treated as one flat floor.
constexpr double KNEE_FLOOR = 1e-6;
constexpr int EV_THREADS = 256;       // four eigenvalues (one per wavefront) per workgroup
constexpr int EV_ROUNDS = 16;         // multisection rounds (65-fold narrowing each)
constexpr double CLUSTER_TOL = 1e-6;  // eigenvalues of the unit-scaled T this close form a cluster
constexpr int INVIT_ITERS = 4;        // inverse-iteration solves per eigenvector
constexpr double DBL_TINY = 2.2250738585072014e-308;

__device__ __forceinline__ double2 zmul(double2 a, double2 b) {
    return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ double2 zconj(double2 a) { return make_double2(a.x, -a.y); }
// a * conj(b)
__device__ __forceinline__ double2 zmulc(double2 a, double2 b) {
    return make_double2(a.x * b.x + a.y * b.y, a.y * b.x - a.x * b.y);
}

// ------------------------------------------------------------------ 1. tridiagonalisation
struct TriArgs {
    const double2* G;   // [n][n]
    double2* A;         // [n][n] work copy
    double2* vh;        // [n][n]: v_k in row k, entries k+1 .. n-1
    double2* tau;       // [n]
    double* d;          // [n]
    double* e;          // [n]
    double2* p;         // [2][n] (tridiag_row_kernel)
    int n;
};

__device__ __forceinline__ void rt_block(int b, int nbr, int& I, int& J) {
    I = J = -1;
    for (int jj = nbr - 1; jj >= 0; --jj) {
        const int cnt = nbr - jj;
        if (b < cnt) {
            J = jj;
            I = jj + b;
            return;
        }
        b -= cnt;
    }
}

// Lane exchanges inside a row of 16 lanes on the VALU (DPP), for FP64 values:
// row_ror:n gives lane x the value of lane (x - n) mod 16 of its row; quad_perm swaps.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
    const long long u = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)u, CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, 0xF, 0xF, true);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
constexpr int DPP_XOR1 = 0xB1;       // quad_perm [1, 0, 3, 2]
constexpr int DPP_XOR2 = 0x4E;       // quad_perm [2, 3, 0, 1]
constexpr int DPP_ROR4 = 0x124, DPP_ROR8 = 0x128, DPP_ROR12 = 0x12C;

// value of lane l (l uniform), the same in every lane
__device__ __forceinline__ double lane_f64(double x, int l) {
    const long long u = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_readlane((int)u, l), hi = __builtin_amdgcn_readlane((int)(u >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
// x + x(lane ^ 16) and x + x(lane ^ 32), the same value in both lanes of each pair: the
// gfx950 row swaps (permlane16_swap of x with itself gives the even rows' values in the first
// result and the odd rows' in the second, permlane32_swap the lower and upper halves')
template <bool HALVES>
__device__ __forceinline__ double swap_sum(double x) {
    const long long u = __double_as_longlong(x);
    const int lo = (int)u, hi = (int)(u >> 32);
    auto l = HALVES ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false) : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    auto h = HALVES ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false) : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    const double a = __longlong_as_double(((long long)h[0] << 32) | (unsigned int)l[0]);
    const double b = __longlong_as_double(((long long)h[1] << 32) | (unsigned int)l[1]);
    return a + b;
}
// sums over a full wavefront, the same values in every lane: each row of 16 lanes summed by DPP
// (quad swaps, then rotations by 4 and 8; every lane has its source, so the bound control only
// saves clearing the destination), then the rows by the swaps.  Several at once hide each
// other's latency.
template <int N>
__device__ __forceinline__ void wave_totals(double (&x)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] += dpp_f64<DPP_XOR1>(x[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] += dpp_f64<DPP_XOR2>(x[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] += dpp_f64<DPP_ROR4>(x[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] += dpp_f64<DPP_ROR8>(x[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = swap_sum<false>(x[i]);
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = swap_sum<true>(x[i]);
}
__device__ __forceinline__ double wave_total(double x) {
    double t[1] = {x};
    wave_totals(t);
    return t[0];
}
__device__ __forceinline__ double2 wave_total(double2 x) {
    double t[2] = {x.x, x.y};
    wave_totals(t);
    return make_double2(t[0], t[1]);
}

// Householder reflector of a column with first entry alpha and sum of squares sigma below it:
// (alpha, x) -> beta, v = (1, scale x)
__device__ __forceinline__ void reflector(double2 alpha, double sigma, double& beta, double2& tau, double2& scale) {
    beta = alpha.x;
    tau = scale = make_double2(0.0, 0.0);
    if (sigma > 0.0 || alpha.y != 0.0) {
        // square root and its reciprocal from one estimate, two Newton steps each (correct to
        // the last place or two); the other reciprocal likewise
        const double s2 = alpha.x * alpha.x + alpha.y * alpha.y + sigma;
        double y = __builtin_amdgcn_rsq(s2);
        y = fma(0.5 * y, fma(-s2 * y, y, 1.0), y);
        y = fma(0.5 * y, fma(-s2 * y, y, 1.0), y);
        double nrm = s2 * y;
        nrm = fma(fma(-nrm, nrm, s2), 0.5 * y, nrm);
        beta = alpha.x >= 0.0 ? -nrm : nrm;
        const double ib = alpha.x >= 0.0 ? -y : y;
        tau = make_double2((beta - alpha.x) * ib, -alpha.y * ib);
        const double2 den = make_double2(alpha.x - beta, alpha.y);   // 1 / (alpha - beta)
        const double d2 = den.x * den.x + den.y * den.y;
        double idd = __builtin_amdgcn_rcp(d2);
        idd = fma(idd, fma(-d2, idd, 1.0), idd);
        idd = fma(idd, fma(-d2, idd, 1.0), idd);
        scale = make_double2(den.x * idd, -den.y * idd);
    }
}

// p = A22 v is summed in LDS by FP64 atomics from the blocks of every wavefront in the order
// they arrive.  Each contribution is first rounded to a multiple of delta = 1/scale: the
// contributions to p_i are the block pieces of one row of the Hermitian trailing matrix times v,
// so by Cauchy-Schwarz every partial sum of them is at most ||A_i|| ||v|| <= sqrt(2) ||A||_F
// (||v||^2 <= 2; the trailing block keeps ||A||_F), below 2^53 delta for the scale chosen; every
// FP64 addition is then exact and the sums do not depend on the order, so the reduction is
// deterministic.  delta <= 2^-51 ||A||_F, a few units in the last place of the products' sums.
__device__ __forceinline__ double quantize(double x, double scale, double inv_scale) {
    return rint(x * scale) * inv_scale;
}

// row sums d[2 q + part] and column sums cs of a block, added into p
__device__ __forceinline__ void rt_reduce(const double (&d)[8], double2 cs, int i0, int j, int n, int c, int lane, bool diag,
                                          double2* p, double scale, double inv_scale) {
    // row sums over the 16 lanes of this row group: halving butterfly on c, partners c ^ 8,
    // c ^ 4, c ^ 2, c ^ 1 (the row's lanes, exchanged by DPP: c ^ 8 is a rotation by 8, c ^ 4
    // a rotation by 4 for the lanes with bit 2 set and by 12 for the others)
    const bool b3 = c & 8, b2 = c & 4, b1 = c & 2;
    double e4[4], e2[2];
#pragma unroll
    for (int m = 0; m < 4; ++m) e4[m] = (b3 ? d[4 + m] : d[m]) + dpp_f64<DPP_ROR8>(b3 ? d[m] : d[4 + m]);
#pragma unroll
    for (int m = 0; m < 2; ++m) {
        const double snd = b2 ? e4[m] : e4[2 + m];
        const double a4 = dpp_f64<DPP_ROR4>(snd), a12 = dpp_f64<DPP_ROR12>(snd);
        e2[m] = (b2 ? e4[2 + m] : e4[m]) + (b2 ? a4 : a12);
    }
    double e1 = (b1 ? e2[1] : e2[0]) + dpp_f64<DPP_XOR2>(b1 ? e2[0] : e2[1]);
    e1 += dpp_f64<DPP_XOR1>(e1);
    if ((c & 1) == 0) {   // value 4 b3 + 2 b2 + b1: row q = 2 b3 + b2, part b1
        const int idx = (b3 ? 4 : 0) + (b2 ? 2 : 0) + (b1 ? 1 : 0);
        atomicAdd(reinterpret_cast<double*>(p + i0 + (idx >> 1)) + (idx & 1), quantize(e1, scale, inv_scale));
    }
    if (diag) return;
    // column sums over the block's 4 row groups
    cs.x = swap_sum<true>(swap_sum<false>(cs.x));
    cs.y = swap_sum<true>(swap_sum<false>(cs.y));
    if (lane < 16 && j < n) {
        atomicAdd(&p[j].x, quantize(cs.x, scale, inv_scale));
        atomicAdd(&p[j].y, quantize(cs.y, scale, inv_scale));
    }
}

// Up to TRI_ONE frames the lower block triangle of A (the Hermitian matrix) is held in the
// registers of one workgroup for the whole reduction, so a step reads and writes no global
// memory.  It is cut into 16x16 blocks (I >= J; the diagonal blocks are held whole, both
// triangles), listed by block column J descending and I ascending and dealt to the wavefronts in
// turn (a wavefront keeps blocks across the whole matrix, so the shrinking trailing block stays
// spread over all of them); in a block, lane l holds rows 4(l/16) .. 4(l/16)+3 of column l%16.
// Step k, with one barrier:
//   1. every wavefront forms w = tau p - |tau|^2 (v^H p) v / 2 of step k-1, takes its rank-2
//      update off column k (held in LDS as step k-2 left it), and forms the reflector v, tau of
//      column k, all redundantly: the vectors are one or two values a lane, and the chain (two
//      wavefront sums, a square root, a division) would otherwise need a barrier at each end
//      for the one wavefront that computes it;
//   2. the update of step k-1 and p = A22 v in one pass over the blocks: each stored A_ij adds
//      A_ij v_j to p_i and, in the blocks below the diagonal, conj(A_ij) v_i to p_j; row sums are
//      reduced over the block's 16 columns by a halving butterfly (each exchange halves the
//      values a lane carries), column sums over its 4 row groups, both added into p with LDS
//      atomics (each contribution rounded to a grid on which the FP64 sums are exact: the
//      reduction is deterministic).  The owners of column k+1 put it in LDS;
//   3. the barrier: p and column k+1 are complete.
// v and w are zero on the rows already reduced and on rows past n, which so stay as they are.
// All wavefronts write the same v and w to the same words (each reads back its own or an equal
// value); v and the column alternate between two buffers, p between three, so that a wavefront
// one step ahead writes nothing that another still reads.
// 20 frames: 33 us, 64: 134, 128: 436 (54, 180, 521 with three barriers a step).
// step 2 on one block (rows i0 .. i0+3 of column j in this lane): A -= v1 w^H + w v1^H, then its
// part of A v; a diagonal block holds both triangles and adds its row sums only.  get and put
// move the lane's element of row q.
template <class Get, class Put>
__device__ __forceinline__ void rt_block_step(Get get, Put put, int i0, int j, int n, int c, int lane, bool diag,
                                              const double2* v1, const double2* w, const double2* v, double2* p,
                                              double scale, double inv_scale) {
    const double2 v1j = v1[j], wj = w[j], vj = v[j];
    double d[8];
    double2 cs = make_double2(0.0, 0.0);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        double2 x = get(q);
        const double2 u1 = zmulc(v1[i0 + q], wj), u2 = zmulc(w[i0 + q], v1j);
        x.x -= u1.x + u2.x;
        x.y -= u1.y + u2.y;
        put(q, x);
        const double2 r = zmul(x, vj);
        d[2 * q] = r.x;
        d[2 * q + 1] = r.y;
        const double2 t = zmul(zconj(x), v[i0 + q]);
        cs.x += t.x;
        cs.y += t.y;
    }
    rt_reduce(d, cs, i0, j, n, c, lane, diag, p, scale, inv_scale);
}

template <int RN, int W>
__global__ void __launch_bounds__(64 * W) tridiag_step_kernel(const TriArgs a) {
    constexpr int NBLK = (RN / 16) * (RN / 16 + 1) / 2;
    constexpr int BPW = (NBLK + W - 1) / W;   // blocks per wavefront
    __shared__ double2 scol[2][RN], sv[2][RN], sw[RN], sp[3][RN];
    __shared__ double fro2_w[W];
    const int n = a.n, tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: block bookkeeping in scalars
    const int nbr = (n + 15) / 16;
    const int c = lane & 15, rb = (lane >> 4) * 4;
    for (int i = tid; i < RN; i += (64 * W)) {
        scol[0][i] = scol[1][i] = sv[0][i] = sv[1][i] = sw[i] = sp[0][i] = sp[1][i] = sp[2][i] = make_double2(0.0, 0.0);
    }
    int bI[BPW], bJ[BPW];
    double2 A[BPW][4];
    double fro2 = 0.0;   // this lane's part of ||A||_F^2
#pragma unroll
    for (int s = 0; s < BPW; ++s) {
        rt_block(wv + W * s, nbr, bI[s], bJ[s]);
        const int j = 16 * bJ[s] + c;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int i = 16 * bI[s] + rb + q;
            double2 x = make_double2(0.0, 0.0);
            if (bI[s] >= 0 && i < n && j < n) {
                // Hermitian part of the input (the Gram is Hermitian up to its own rounding)
                const double2 g = a.G[(size_t)i * n + j], gt = a.G[(size_t)j * n + i];
                x = i == j ? make_double2(g.x, 0.0) : make_double2(0.5 * (g.x + gt.x), 0.5 * (g.y - gt.y));
                fro2 += (bI[s] == bJ[s] ? 1.0 : 2.0) * (x.x * x.x + x.y * x.y);
            }
            A[s][q] = x;
        }
    }
    fro2 = wave_total(fro2);
    if (lane == 0) fro2_w[wv] = fro2;
    __syncthreads();
    // element (i, j) of the blocks into LDS if it belongs to column k, rows k .. n-1
    auto put_col = [&](int i, int j, int k, double2 x) {
        if (j == k && i >= k && i < n) scol[k & 1][i] = x;
    };
#pragma unroll
    for (int s = 0; s < BPW; ++s)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (bJ[s] == 0) put_col(16 * bI[s] + rb + q, c, 0, A[s][q]);
    // scale 2^(51 - e) with ||A||_F < 2^(e+1): partial sums of p_i below sqrt(2) 2^(e+1) + 13 delta
    // < 2^52.6 delta
    double fro = 0.0;
#pragma unroll
    for (int w = 0; w < W; ++w) fro += fro2_w[w];
    fro = sqrt(fro);
    const int fe = __builtin_amdgcn_readfirstlane(fro > 0.0 ? max(ilogb(fro), -900) : 0);
    const double scale = ldexp(1.0, 51 - fe), inv_scale = ldexp(1.0, fe - 51);
    __syncthreads();
    constexpr int VL = (RN + 63) / 64;   // values of a vector per lane: i = lane + 64 t
    double2 tau = make_double2(0.0, 0.0);   // of the step before
    auto at = [&](const double2 (&x)[VL], int i) {   // element i, i uniform
        double2 r = make_double2(0.0, 0.0);
#pragma unroll
        for (int t = 0; t < VL; ++t)
            if ((i >> 6) == t) r = make_double2(lane_f64(x[t].x, i & 63), lane_f64(x[t].y, i & 63));
        return r;
    };
    int pk = 0;   // k mod 3
    for (int k = 0; k < n; ++k) {
        const int pn = pk == 2 ? 0 : pk + 1;
        const double2* p1 = sp[pn == 2 ? 0 : pn + 1];   // of step k - 1
        double2* p = sp[pk];
        // 1. w of step k-1, column k, its reflector
        const double2* v1 = sv[(k & 1) ^ 1];
        double2* v = sv[k & 1];
        double2 vl[VL], wl[VL], col[VL];
        double pr = 0.0;
#pragma unroll
        for (int t = 0; t < VL; ++t) {
            const int i = lane + 64 * t;
            vl[t] = wl[t] = make_double2(0.0, 0.0);
            if (64 * t < n && i < RN) {
                vl[t] = v1[i];
                wl[t] = p1[i];
            }
            pr += vl[t].x * wl[t].x + vl[t].y * wl[t].y;
        }
        pr = wave_total(pr);
        const double hw = 0.5 * (tau.x * tau.x + tau.y * tau.y) * pr;
#pragma unroll
        for (int t = 0; t < VL; ++t) {
            const double2 tp = zmul(tau, wl[t]);
            const bool live = lane + 64 * t >= k;   // (p_i of a reduced row holds partial sums)
            wl[t] = make_double2(live ? tp.x - hw * vl[t].x : 0.0, live ? tp.y - hw * vl[t].y : 0.0);
        }
        const double2 wk = at(wl, k), vk = at(vl, k);
        double ps = 0.0;
#pragma unroll
        for (int t = 0; t < VL; ++t) {
            const int i = lane + 64 * t;
            col[t] = make_double2(0.0, 0.0);
            if (64 * t < n && i < RN) {
                col[t] = scol[k & 1][i];
                sw[i] = wl[t];
            }
            const double2 u1 = zmulc(vl[t], wk), u2 = zmulc(wl[t], vk);
            col[t].x -= u1.x + u2.x;
            col[t].y -= u1.y + u2.y;
            if (lane + 64 * t >= k + 2) ps += col[t].x * col[t].x + col[t].y * col[t].y;
        }
        const double dk = at(col, k).x;
        if (k == n - 1) {
            if (tid == 0) {
                a.d[k] = dk;
                a.e[k] = 0.0;
            }
            break;
        }
        const double sigma = wave_total(ps);
        const double2 alpha = at(col, k + 1);
        double2 scl;
        double beta;
        reflector(alpha, sigma, beta, tau, scl);
        if (tid == 0) {
            a.tau[k] = tau;
            a.e[k] = beta;
            a.d[k] = dk;
        }
#pragma unroll
        for (int t = 0; t < VL; ++t) {
            const int i = lane + 64 * t;
            double2 vi = make_double2(0.0, 0.0);
            if (i == k + 1) vi = make_double2(1.0, 0.0);
            else if (i > k + 1) vi = zmul(col[t], scl);
            if (64 * t < n && i < RN) {
                v[i] = vi;
                if (wv == t && i > k && i < n) a.vh[(size_t)k * n + i] = vi;
            }
        }
        for (int i = tid; i < n; i += (64 * W)) sp[pn][i] = make_double2(0.0, 0.0);
        __builtin_amdgcn_wave_barrier();
        // 2. the update of step k-1 and p = A22 v (blocks with a column beyond k)
#pragma unroll
        for (int s = 0; s < BPW; ++s) {
            // (opaque: addresses kept for all blocks through the whole reduction would not leave
            // the registers for the blocks)
            int I = bI[s], J = bJ[s];
            asm volatile("" : "+s"(I), "+s"(J));
            if (I < 0 || 16 * J + 15 <= k) continue;
            const int j = 16 * J + c, i0 = 16 * I + rb;
            rt_block_step(
                [&](int q) { return A[s][q]; },
                [&](int q, double2 x) {
                    A[s][q] = x;
                    put_col(i0 + q, j, k + 1, x);
                },
                i0, j, n, c, lane, I == J, v1, sw, v, p, scale, inv_scale);
        }
        pk = pn;
        __syncthreads();
    }
}

// Beyond TRI_ONE frames one launch a step, the launch being the barrier, and one wavefront a row
// of the trailing block (A is kept as a full Hermitian matrix in the workspace).  Step k: every
// wavefront forms w of step k-1 and the reflector of column k itself (its lanes hold the vectors
// in the columns they handle, so nothing goes through LDS), applies the update of step k-1 to
// its row i, stores it and writes p_i = (A22 v)_i.  Row k, which gives column k, is only read in
// step k; p alternates between two buffers; v_{k-1} is row k-1 of vh.  The wavefront of row
// k+1 writes what leaves the step.  CT chunks of 64 columns from column k & ~63 on.
// A step is latency: a launch, one round of loads, two wavefront sums, a square root and three
// divisions; 3.3 us at 200 frames, 4.7 at 400, where one workgroup for the whole matrix takes 7
// and 28 (registers and LDS hold 208 frames; beyond, every step streams the trailing block
// through one compute unit).  Whole filter of 4096 voxels: 130 frames 886 -> 670 us, 200: 1775
// -> 1015, 209: 3103 -> 1050, 400: 12131 -> 2220, 512: 21413 -> 3030.  At 1, 2, 4, 8 rows a
// workgroup 400 frames take 2226, 2220, 2265, 2589 us and 200 frames 1014, 1041, 1055, 1175.
// The line stands where the launches' cost to the calling thread does: on the GPU they win from
// about 90 frames on (80 frames 400 us, one workgroup 373; 100: 490, 535; 128: 618, 698), but 128
// launches hold the caller for 0.3 ms, half the filter's time, and one hardly at all; from
// 129 frames on the GPU's gain (886 -> 670 us at 130) outgrows what the caller pays.
constexpr int TRI_ONE = 128;
template <int CT, bool FIRST>
__global__ void __launch_bounds__(64) tridiag_row_kernel(const TriArgs a, int k) {
    const int n = a.n, lane = threadIdx.x, gw = blockIdx.x;
    const int i = k + 1 + gw, ir = min(i, n - 1);
    const int base = k & ~63, ko = k - base;
    const double2* p0 = a.p + (k & 1) * n;         // A22 v of step k-1
    double2* p1 = a.p + ((k + 1) & 1) * n;
    auto at = [&](int r, int c) {
        if (!FIRST) return a.A[(size_t)r * n + c];
        // Hermitian part of the input (the Gram is Hermitian up to its own rounding)
        const double2 g = a.G[(size_t)r * n + c], gt = a.G[(size_t)c * n + r];
        return r == c ? make_double2(g.x, 0.0) : make_double2(0.5 * (g.x + gt.x), 0.5 * (g.y - gt.y));
    };
    // every load ahead of the first use, without a branch (columns past n read column n - 1)
    double2 x[CT], y[CT], v1[CT], w[CT];
#pragma unroll
    for (int t = 0; t < CT; ++t) {
        const int j = min(base + lane + 64 * t, n - 1);
        x[t] = at(k, j);
        if (!FIRST) {
            v1[t] = a.vh[(size_t)(k - 1) * n + j];
            w[t] = p0[j];
        }
    }
#pragma unroll
    for (int t = 0; t < CT; ++t) y[t] = at(ir, min(base + lane + 64 * t, n - 1));
    const double2 zero = make_double2(0.0, 0.0);
    double2 v1i = zero, wi = zero;
    if (!FIRST) {
        v1i = a.vh[(size_t)(k - 1) * n + ir];
        wi = p0[ir];
        const double2 tau1 = a.tau[k - 1];
        double pr = 0.0;
#pragma unroll
        for (int t = 0; t < CT; ++t) {
            const int j = base + lane + 64 * t;
            if (j < k || j >= n) v1[t] = w[t] = zero;
            pr += v1[t].x * w[t].x + v1[t].y * w[t].y;
        }
        // r = v^H p (real for Hermitian A22); w = tau p - |tau|^2 r v / 2
        const double hw = 0.5 * (tau1.x * tau1.x + tau1.y * tau1.y) * wave_total(pr);
        auto to_w = [&](double2 p, double2 v) {
            const double2 tp = zmul(tau1, p);
            return make_double2(tp.x - hw * v.x, tp.y - hw * v.y);
        };
#pragma unroll
        for (int t = 0; t < CT; ++t) w[t] = to_w(w[t], v1[t]);
        wi = to_w(wi, v1i);
    }
    // column k = conj(row k), less the update of step k-1 (v_k of that step is 1)
    const double2 wk = FIRST ? zero : make_double2(lane_f64(w[0].x, ko), lane_f64(w[0].y, ko));
    double ps = 0.0;
#pragma unroll
    for (int t = 0; t < CT; ++t) {
        const int j = base + lane + 64 * t;
        x[t] = zconj(x[t]);
        if (!FIRST) {
            const double2 u = zmulc(v1[t], wk);
            x[t].x -= u.x + w[t].x;
            x[t].y -= u.y + w[t].y;
        }
        if (j >= k + 2 && j < n) ps += x[t].x * x[t].x + x[t].y * x[t].y;
    }
    const double dk = lane_f64(x[0].x, ko);
    if (k == n - 1) {
        if (gw == 0 && lane == 0) {
            a.d[k] = dk;
            a.e[k] = 0.0;
        }
        return;
    }
    const double sigma = wave_total(ps);
    const bool over = CT > 1 && ko == 63;   // row k+1 starts the second chunk
    const int al = (ko + 1) & 63;
    const double2 xa = over ? x[CT > 1 ? 1 : 0] : x[0];
    const double2 alpha = make_double2(lane_f64(xa.x, al), lane_f64(xa.y, al));
    double2 tau, scale;
    double beta;
    reflector(alpha, sigma, beta, tau, scale);
    double2 acc = zero;
#pragma unroll
    for (int t = 0; t < CT; ++t) {
        const int j = base + lane + 64 * t;
        double2 v = zmul(x[t], scale);
        if (j == k + 1) v = make_double2(1.0, 0.0);
        if (j <= k || j >= n) v = zero;
        double2 u = y[t];
        if (!FIRST) {
            const double2 u1 = zmulc(v1i, w[t]), u2 = zmulc(wi, v1[t]);
            u.x -= u1.x + u2.x;
            u.y -= u1.y + u2.y;
        }
        if (i < n && j > k && j < n) {
            a.A[(size_t)i * n + j] = u;
            acc.x += u.x * v.x - u.y * v.y;
            acc.y += u.x * v.y + u.y * v.x;
        }
        if (gw == 0 && j > k && j < n) a.vh[(size_t)k * n + j] = v;
    }
    acc = wave_total(acc);
    if (lane == 0 && i < n) {
        p1[i] = acc;
        if (gw == 0) {
            a.tau[k] = tau;
            a.e[k] = beta;
            a.d[k] = dk;
        }
    }
}

// ------------------------------------------------------------------ 2. QL on T
struct QlArgs {
    const double* d;
    const double* e;
    int* rot_i;         // rotation log: plane (i, i+1), cos, sin
    double* rot_c;
    double* rot_s;
    int* rot_n;
    int cap;
    double* lam;        // [n] descending, clamped at 0
    double* sigma;      // [n] or null
    int* perm;          // [n]: column of Z holding the eigenvalue of rank j
    int* status;        // or null
    int n;
};

__global__ void __launch_bounds__(64) ql_kernel(const QlArgs a) {
    __shared__ double d[FQ_MAX_NT], e[FQ_MAX_NT];
    __shared__ double s_sc;
    const int n = a.n, l0 = threadIdx.x;
    for (int i = l0; i < n; i += 64) {
        d[i] = a.d[i];
        e[i] = a.e[i];
    }
    __syncthreads();
    if (l0 == 0) {
        // scale T to unit size (no overflow in squares, scale-free tolerances)
        double sc = 0.0;
        for (int i = 0; i < n; ++i) sc = fmax(sc, fabs(d[i]) + fabs(e[i]));
        const double isc = sc > 0.0 ? 1.0 / sc : 0.0;
        for (int i = 0; i < n; ++i) {
            d[i] *= isc;
            e[i] *= isc;
        }
        e[n - 1] = 0.0;
        s_sc = sc;
    }
    __syncthreads();
    const double eps = 2.220446049250313e-16;
    // The wave runs the iteration in lockstep: the search for the deflation point is
    // wave-parallel, each sweep of rotations runs on lane 0 (a dependent chain).
    int cnt = 0, bad = 0;
    for (int l = 0; l < n && !bad; ++l) {
        for (int it = 0;; ++it) {
            // m = the first index >= l with a negligible off-diagonal e[m], n - 1 if none
            int m = n - 1;
            for (int m0 = l; m0 < n - 1; m0 += 64) {
                const int mm = m0 + l0;
                bool small = false;
                if (mm < n - 1) small = fabs(e[mm]) <= eps * (fabs(d[mm]) + fabs(d[mm + 1]));
                const uint64_t b = __ballot(small);
                if (b) {
                    m = m0 + __ffsll((unsigned long long)b) - 1;
                    break;
                }
            }
            if (m == l) break;
            if (it >= QL_MAX_ITER || cnt + (m - l) > a.cap) {
                bad = 1;
                break;
            }
            int split = 0;
            if (l0 == 0) {
                // Wilkinson shift from the leading 2x2 block
                double g = (d[l + 1] - d[l]) / (2.0 * e[l]);
                double r = sqrt(g * g + 1.0);
                g = d[m] - d[l] + e[l] / (g + (g >= 0.0 ? r : -r));
                double s = 1.0, c = 1.0, p = 0.0;
                int i = m - 1;
                // d[i], d[i+1], e[i] of the current plane; the next plane's e and d are
                // read one step ahead (this step writes only e[i+1] and d[i+1])
                double ei = e[i], di = d[i], dip1 = d[i + 1];
                for (; i >= l; --i) {
                    const int inx = i > 0 ? i - 1 : 0;   // clamped: read unconditionally
                    const double e_nx = e[inx], d_nx = d[inx];
                    const double f = s * ei, b = c * ei;
                    const double x = f * f + g * g;
                    if (x == 0.0) {   // e[i] vanished: the block splits, restart
                        e[i + 1] = 0.0;
                        d[i + 1] = dip1 - p;
                        e[m] = 0.0;
                        split = 1;
                        break;
                    }
                    // 1/sqrt(x) from the hardware estimate and two Newton steps
                    double y = __builtin_amdgcn_rsq(x);
                    y = y * fma(-0.5 * x * y, y, 1.5);
                    y = y * fma(-0.5 * x * y, y, 1.5);
                    e[i + 1] = x * y;
                    s = f * y;
                    c = g * y;
                    g = dip1 - p;
                    r = (di - g) * s + 2.0 * c * b;
                    p = s * r;
                    d[i + 1] = g + p;
                    g = c * r - b;
                    a.rot_i[cnt] = i;
                    a.rot_c[cnt] = c;
                    a.rot_s[cnt] = s;
                    ++cnt;
                    ei = e_nx;
                    dip1 = di;
                    di = d_nx;
                }
                if (!split) {
                    d[l] -= p;
                    e[l] = g;
                    e[m] = 0.0;
                }
            }
            cnt = __shfl(cnt, 0);
            __syncthreads();   // lane 0's updates of d and e before the next search
        }
    }
    if (l0 == 0) {
        const double sc = s_sc;
        for (int i = 0; i < n; ++i) d[i] *= sc;
        *a.rot_n = cnt;
        if (a.status) *a.status = bad ? FQ_E_NUMERIC : FQ_OK;
    }
    __syncthreads();
    // rank: descending, ties by index
    for (int i = l0; i < n; i += 64) {
        const double li = d[i];
        int rank = 0;
        for (int j = 0; j < n; ++j) rank += (d[j] > li) || (d[j] == li && j < i);
        const double lc = li > 0.0 ? li : 0.0;
        a.lam[rank] = lc;
        if (a.sigma) a.sigma[rank] = sqrt(lc);
        a.perm[rank] = i;
    }
}

// ------------------------------------------------------------------ 2'. eigenvalues by multisection
struct EigvalArgs {
    const double* d;      // [n] diagonal of T
    const double* e;      // [n] off-diagonal: e[i] couples i and i+1 (e[n-1] = 0)
    double* ev;           // [n] eigenvalues of T / scale, descending, unclamped
    double* scale;        // [1] the scale: infinity norm of T
    double* lam;          // [n] eigenvalues of T, descending, clamped at 0
    double* sigma;        // [n] sqrt(lam), or null
    int* status;          // or null
    int n;
};

// Number of eigenvalues of the scaled T below x: the negative pivots of the LDL^T
// factorisation of T - x I.  A pivot smaller than pmin in magnitude is replaced by -pmin
// (the count of a nearby matrix; no division by zero).
// The division is the chain: e2 / q is e2 times the hardware's reciprocal of q (relative error
// up to 2^-24.3 over 10^8 mantissas), corrected by one third-order step, y (1 + r + r^2) with r = 1 - q y, which leaves
// r^3 < 2^-72 before rounding.  pmin <= |q| < 2^1022, so y and r stay finite.
// 20 frames: 20 -> 13 us for the kernel, 200: 151 -> 81, 400: 286 -> 157 (before: the IEEE division).
__device__ __forceinline__ int sturm_count(const double* d, const double* e2, int n, double x, double pmin) {
    double q = d[0] - x;
    if (fabs(q) < pmin) q = -pmin;
    int c = q < 0.0;
#pragma unroll 8
    for (int i = 1; i < n; ++i) {
        const double y = __builtin_amdgcn_rcp(q), r = fma(-q, y, 1.0);
        q = fma(-e2[i - 1], fma(y, fma(r, r, r), y), d[i] - x);
        if (fabs(q) < pmin) q = -pmin;
        c += q < 0.0;
    }
    return c;
}

__device__ __forceinline__ double wave_max(double v) {
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o));
    return v;
}
__device__ __forceinline__ double wave_min(double v) {
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o));
    return v;
}
__device__ __forceinline__ double wave_sum(double v) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

__global__ void __launch_bounds__(EV_THREADS) eigval_kernel(const EigvalArgs a) {
    constexpr int NW = EV_THREADS / 64;
    __shared__ double sd[FQ_MAX_NT], se2[FQ_MAX_NT];
    __shared__ double red[3][NW];
    const int n = a.n, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    // infinity norm of T
    double nrm = 0.0;
    for (int i = tid; i < n; i += EV_THREADS)
        nrm = fmax(nrm, fabs(a.d[i]) + fabs(a.e[i]) + (i > 0 ? fabs(a.e[i - 1]) : 0.0));
    nrm = wave_max(nrm);
    if (lane == 0) red[0][w] = nrm;
    __syncthreads();
    double sc = 0.0;
#pragma unroll
    for (int k = 0; k < NW; ++k) sc = fmax(sc, red[0][k]);
    const double isc = sc > 0.0 ? 1.0 / sc : 0.0;
    // scaled T in LDS and its Gershgorin interval
    double glo = 0.0, ghi = 0.0, emax = 0.0;
    for (int i = tid; i < n; i += EV_THREADS) {
        const double di = a.d[i] * isc, ei = i + 1 < n ? a.e[i] * isc : 0.0;
        const double em = i > 0 ? a.e[i - 1] * isc : 0.0;
        sd[i] = di;
        se2[i] = ei * ei;
        const double r = fabs(ei) + fabs(em);
        glo = fmin(glo, di - r);
        ghi = fmax(ghi, di + r);
        emax = fmax(emax, ei * ei);
    }
    glo = wave_min(glo);
    ghi = wave_max(ghi);
    emax = wave_max(emax);
    __syncthreads();
    if (lane == 0) {
        red[0][w] = glo;
        red[1][w] = ghi;
        red[2][w] = emax;
    }
    __syncthreads();
    double gl = red[0][0], gu = red[1][0], e2max = red[2][0];
#pragma unroll
    for (int k = 1; k < NW; ++k) {
        gl = fmin(gl, red[0][k]);
        gu = fmax(gu, red[1][k]);
        e2max = fmax(e2max, red[2][k]);
    }
    const double eps = 2.220446049250313e-16;
    const double pmin = DBL_TINY * fmax(1.0, e2max);
    const double widen = 2.1 * eps * n * fmax(fabs(gl), fabs(gu)) + 4.0 * pmin;
    gl -= widen;
    gu += widen;
    if (blockIdx.x == 0 && tid == 0) {
        *a.scale = sc;
        if (a.status) *a.status = FQ_OK;
    }
    const int j = blockIdx.x * NW + w;   // index in ascending order
    if (j >= n) return;
    // bracket [lo, hi) with count(lo) <= j < count(hi), narrowed 65-fold per round
    double lo = gl, hi = gu;
    for (int r = 0; r < EV_ROUNDS; ++r) {
        const double x = lo + (hi - lo) * ((double)(lane + 1) * (1.0 / 65.0));
        const int c = sturm_count(sd, se2, n, x, pmin);
        const uint64_t b = __ballot(c > j);
        const int f = b ? __ffsll((unsigned long long)b) - 1 : 64;
        const double xf = __shfl(x, f < 64 ? f : 63);
        const double xp = __shfl(x, f > 0 ? f - 1 : 0);
        if (f > 0) lo = xp;
        if (f < 64) hi = xf;
        if (hi - lo <= fmax(2.0 * eps * fmax(fabs(lo), fabs(hi)), 1e-20)) break;
    }
    if (lane == 0) {
        const double ev = 0.5 * (lo + hi);
        const int rk = n - 1 - j;
        a.ev[rk] = ev;
        const double l = ev > 0.0 ? ev * sc : 0.0;
        a.lam[rk] = l;
        if (a.sigma) a.sigma[rk] = sqrt(l);
    }
}

// ------------------------------------------------------------------ 4'. inverse iteration
struct InvitArgs {
    const double* d;
    const double* e;
    const double* ev;       // [n] eigenvalues of T / scale, descending
    const double* scale;    // [1]
    const int* k_dev;       // vectors wanted (device word), or null: k_const
    int k_const;
    double* Z;              // [KMAX][n]: Z[j * n + i] = component i of the eigenvector of ev[j]
    int* status;            // or null
    int n;
};

// deterministic pseudo-random start vector in [-1, 1)
__device__ __forceinline__ double start_component(int i, int j) {
    uint32_t h = (uint32_t)i * 0x9E3779B1u ^ ((uint32_t)j * 0x85EBCA77u + 0x27D4EB2Fu);
    h ^= h >> 15;
    h *= 0x2C1B3C6Du;
    h ^= h >> 12;
    h *= 0x297A2D39u;
    h ^= h >> 15;
    return (double)h * (2.0 / 4294967296.0) - 1.0;
}

// One workgroup (one wavefront) per wanted eigenvalue.  T - lambda I is factorised by
// Gaussian elimination with partial pivoting (rows i, i+1 exchanged when the sub-diagonal
// entry is the larger): U has a diagonal, a super-diagonal and a second super-diagonal
// (created by exchanges); pivots below eps of the unit-scaled T are raised to +-eps, which
// is what makes the nearly singular solve amplify the wanted eigenvector.  The serial
// factorisation and solves run on lane 0; the solves load the operands of IB rows at a time,
// ahead of the chain (LDS would otherwise answer once a row); normalisation is wave-parallel.
// 200 frames: 98 -> 87 us, of which the factorisation's divisions are the larger part.
// Vectors of eigenvalues closer than CLUSTER_TOL are made orthogonal afterwards
// (orth_kernel); farther apart, inverse iteration leaves them orthogonal to ~eps/gap.
constexpr int IB = 8;
__global__ void __launch_bounds__(64) invit_kernel(const InvitArgs a) {
    __shared__ double sd[FQ_MAX_NT], se[FQ_MAX_NT];
    __shared__ double ua[FQ_MAX_NT], ub[FQ_MAX_NT], uc[FQ_MAX_NT], lf[FQ_MAX_NT + IB];
    __shared__ unsigned char sw[FQ_MAX_NT + IB];
    __shared__ double x[FQ_MAX_NT + IB + 1];
    const int n = a.n, lane = threadIdx.x, j = blockIdx.x;
    const int K = a.k_dev ? *a.k_dev : a.k_const;
    if (j >= K) return;
    const double sc = *a.scale, isc = sc > 0.0 ? 1.0 / sc : 0.0;
    const double lam = a.ev[j];
    for (int i = lane; i < n; i += 64) {
        sd[i] = a.d[i] * isc - lam;
        se[i] = i + 1 < n ? a.e[i] * isc : 0.0;
        x[i] = start_component(i, j);
    }
    __syncthreads();
    const double tiny = 2.220446049250313e-16;
    if (lane == 0) {
        // elimination; (p, q) = diagonal and super-diagonal of the current row
        double p = sd[0], q = se[0];
        for (int i = 0; i + 1 < n; ++i) {
            const double sub = se[i];                           // entry (i+1, i)
            const double dn = sd[i + 1];                        // entry (i+1, i+1)
            const double en = i + 2 < n ? se[i + 1] : 0.0;      // entry (i+1, i+2)
            if (fabs(p) >= fabs(sub)) {
                const double l = sub / (p != 0.0 ? p : tiny);
                lf[i] = l;
                sw[i] = 0;
                ua[i] = p;
                ub[i] = q;
                uc[i] = 0.0;
                p = dn - l * q;
                q = en;
            } else {
                const double l = p / sub;
                lf[i] = l;
                sw[i] = 1;
                ua[i] = sub;
                ub[i] = dn;
                uc[i] = en;
                p = q - l * dn;
                q = -l * en;
            }
        }
        ua[n - 1] = p;
        ub[n - 1] = 0.0;
        uc[n - 1] = 0.0;
    }
    __syncthreads();
    for (int i = lane; i < n; i += 64) {
        const double p = ua[i];
        ua[i] = 1.0 / (fabs(p) >= tiny ? p : (p < 0.0 ? -tiny : tiny));
    }
    __syncthreads();
    int bad = 0;
    for (int it = 0; it < INVIT_ITERS; ++it) {
        if (lane == 0) {
            // L y = P x: the carried value is x[i] as updated by step i-1
            double c = x[0], f[IB], g[IB], h[IB], y[IB], fn[IB], gn[IB];
            int m[IB], mn[IB];
            const int nb = (n - 1) / IB * IB;   // rows in whole batches
            auto get = [&](int i0) {            // reads at most x[nb + IB] and lf, sw[nb + IB - 1]
#pragma unroll
                for (int u = 0; u < IB; ++u) {
                    fn[u] = x[i0 + u + 1];
                    gn[u] = lf[i0 + u];
                    mn[u] = sw[i0 + u];
                }
            };
            get(0);
            for (int i0 = 0; i0 < nb; i0 += IB) {
#pragma unroll
                for (int u = 0; u < IB; ++u) {
                    f[u] = fn[u];
                    g[u] = gn[u];
                    m[u] = mn[u];
                }
                get(i0 + IB);
#pragma unroll
                for (int u = 0; u < IB; ++u) {
                    y[u] = m[u] ? f[u] : c;
                    c = m[u] ? fma(-g[u], f[u], c) : fma(-g[u], c, f[u]);
                }
#pragma unroll
                for (int u = 0; u < IB; ++u) x[i0 + u] = y[u];
            }
            for (int i = nb; i + 1 < n; ++i) {
                const double nx = x[i + 1], l = lf[i];
                x[i] = sw[i] ? nx : c;
                c = sw[i] ? fma(-l, nx, c) : fma(-l, c, nx);
            }
            x[n - 1] = c;
            // U z = y
            double z1 = 0.0, z2 = 0.0;   // z[i+1], z[i+2]
            int i = n - 1;
            for (; i + 1 > n / IB * IB; --i) {
                const double zi = fma(-ub[i], z1, fma(-uc[i], z2, x[i])) * ua[i];
                x[i] = zi;
                z2 = z1;
                z1 = zi;
            }
            for (; i >= 0; i -= IB) {
                double a[IB];
#pragma unroll
                for (int u = 0; u < IB; ++u) {
                    f[u] = x[i - u];
                    g[u] = ub[i - u];
                    h[u] = uc[i - u];
                    a[u] = ua[i - u];
                }
#pragma unroll
                for (int u = 0; u < IB; ++u) {
                    const double zi = fma(-g[u], z1, fma(-h[u], z2, f[u])) * a[u];
                    y[u] = zi;
                    z2 = z1;
                    z1 = zi;
                }
#pragma unroll
                for (int u = 0; u < IB; ++u) x[i - u] = y[u];
            }
        }
        __syncthreads();
        double ss = 0.0;
        for (int i = lane; i < n; i += 64) ss += x[i] * x[i];
        ss = wave_total(ss);
        const bool ok = ss > 0.0 && ss < 1.0 / 0.0;
        bad |= !ok;
        const double inv = ok ? 1.0 / sqrt(ss) : 0.0;
        for (int i = lane; i < n; i += 64) x[i] = ok ? x[i] * inv : start_component(i, j + it + 1);
        __syncthreads();
    }
    for (int i = lane; i < n; i += 64) a.Z[(size_t)j * n + i] = x[i];
    if (bad && lane == 0 && a.status) *a.status = FQ_E_NUMERIC;
}

// Orthogonalisation inside clusters: modified Gram-Schmidt over the wanted vectors of each
// cluster, applied twice (after the first sweep the vectors are near orthonormal whatever
// their condition, the second makes them so to rounding), every vector normalised.
// One workgroup holds all vectors in registers, four per wavefront.  When a vector is
// final its wavefront puts it into LDS and every wavefront takes its component off the
// later vectors it holds, so a step costs one barrier and one dot product: the spatial-
// similarity cutoff's 64 vectors of 200 frames, one cluster of noise modes, took 937 us
// where each vector in turn was reduced against all earlier ones out of global memory,
// and take 86 us here.
constexpr int ORTH_THREADS = 1024;
constexpr int ORTH_WAVES = ORTH_THREADS / 64;
constexpr int ORTH_PER_WAVE = KMAX / ORTH_WAVES;

template <int PL>   // components per lane: n <= 64 PL
__device__ __forceinline__ void orth_clusters(const InvitArgs& a, int K, uint64_t starts, double (*zs)[FQ_MAX_NT]) {
    const int n = a.n, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    double z[ORTH_PER_WAVE][PL];   // vectors wv, wv + ORTH_WAVES, ...
    int first[ORTH_PER_WAVE];      // first vector of its cluster
#pragma unroll
    for (int q = 0; q < ORTH_PER_WAVE; ++q) {
        const int k = wv + q * ORTH_WAVES;
        first[q] = 63 - __clzll((long long)(starts & (~0ull >> (63 - k))));
#pragma unroll
        for (int t = 0; t < PL; ++t) {
            const int i = lane + 64 * t;
            z[q][t] = k < K && i < n ? a.Z[(size_t)k * n + i] : 0.0;
        }
    }
    bool bad = false;
    int turn = 0;
    for (int sweep = 0; sweep < 2; ++sweep) {
#pragma unroll
        for (int qj = 0; qj < ORTH_PER_WAVE; ++qj) {
            for (int wj = 0; wj < ORTH_WAVES; ++wj) {
                const int j = wj + qj * ORTH_WAVES;
                if (j >= K) break;
                // a cluster of one stays as inverse iteration left it
                const bool single = ((starts >> j) & 1) && (j + 1 >= K || ((starts >> (j + 1)) & 1));
                if (single) continue;
                double* zj = zs[turn];
                turn ^= 1;   // the array of the last step may still be read
                if (wv == wj) {
                    double ss = 0.0;
#pragma unroll
                    for (int t = 0; t < PL; ++t) ss += z[qj][t] * z[qj][t];
                    ss = wave_sum(ss);
                    const bool ok = ss > 0.0 && ss < 1.0 / 0.0;
                    bad |= !ok;
                    const double inv = ok ? 1.0 / sqrt(ss) : 0.0;
#pragma unroll
                    for (int t = 0; t < PL; ++t) {
                        z[qj][t] *= inv;
                        zj[lane + 64 * t] = z[qj][t];
                    }
                }
                __syncthreads();
                double dot[ORTH_PER_WAVE] = {}, v[PL];
#pragma unroll
                for (int t = 0; t < PL; ++t) v[t] = zj[lane + 64 * t];
#pragma unroll
                for (int q = qj; q < ORTH_PER_WAVE; ++q)
#pragma unroll
                    for (int t = 0; t < PL; ++t) dot[q] += v[t] * z[q][t];
#pragma unroll
                for (int q = qj; q < ORTH_PER_WAVE; ++q) {
                    const int k = wv + q * ORTH_WAVES;
                    const double d = wave_total(dot[q]);
                    if (k > j && first[q] <= j) {
#pragma unroll
                        for (int t = 0; t < PL; ++t) z[q][t] -= d * v[t];
                    }
                }
            }
        }
    }
#pragma unroll
    for (int q = 0; q < ORTH_PER_WAVE; ++q) {
        const int k = wv + q * ORTH_WAVES;
#pragma unroll
        for (int t = 0; t < PL; ++t) {
            const int i = lane + 64 * t;
            if (k < K && i < n) a.Z[(size_t)k * n + i] = z[q][t];
        }
    }
    if (bad && lane == 0 && a.status) *a.status = FQ_E_NUMERIC;
}

__global__ void __launch_bounds__(ORTH_THREADS) orth_kernel(const InvitArgs a) {
    __shared__ double zs[2][FQ_MAX_NT];
    const int lane = threadIdx.x & 63;
    const int K = a.k_dev ? *a.k_dev : a.k_const;
    // bit j: vector j starts a cluster
    const bool start = lane == 0 || lane >= K || a.ev[lane - 1] - a.ev[lane] > CLUSTER_TOL;
    const uint64_t starts = __ballot(start);
    if (starts == ~0ull) return;
    if (a.n <= 64) orth_clusters<1>(a, K, starts, zs);
    else if (a.n <= 128) orth_clusters<2>(a, K, starts, zs);
    else if (a.n <= 256) orth_clusters<4>(a, K, starts, zs);
    else orth_clusters<8>(a, K, starts, zs);
}

// ------------------------------------------------------------------ 3. replay of the log
struct ReplayArgs {
    const int* rot_i;
    const double* rot_c;
    const double* rot_s;
    const int* rot_n;
    const int* perm;
    double* Zs;         // [n][n], columns in rank order
    int n, rows;        // rows per workgroup (= threads)
};

// Each lane owns one row of Z, stored column-major in LDS (word col * rows + lane).  The
// rotation log is staged through LDS in chunks and read two rotations ahead.  A QL sweep
// applies rotations on planes i, i-1, i-2, ...: the column shared by consecutive planes
// stays in a register, and the next plane's other column is loaded before the current
// plane's result is stored (it is a different column), so the LDS latency is off the
// dependency chain.
constexpr int RCH = 1024;   // rotations per staged chunk

__global__ void __launch_bounds__(64) replay_kernel(const ReplayArgs a) {
    extern __shared__ double zl[];
    __shared__ int ri_s[RCH + 2];   // two sentinel planes (-1) after the chunk
    __shared__ double rc_s[RCH + 2], rs_s[RCH + 2];
    const int n = a.n, R = a.rows, lane = threadIdx.x;
    const int row = blockIdx.x * R + lane;
    const bool live = lane < R && row < n;
    if (lane < R)
        for (int col = 0; col < n; ++col) zl[col * R + lane] = (col == row) ? 1.0 : 0.0;
    const int cnt = *a.rot_n;
    double* z = zl + (lane < R ? lane : 0);
    for (int base = 0; base < cnt; base += RCH) {
        const int nch = min(RCH, cnt - base);
        __syncthreads();
        for (int t = lane; t < nch + 2; t += 64) {
            const bool in = t < nch;
            ri_s[t] = in ? a.rot_i[base + t] : -1;
            rc_s[t] = in ? a.rot_c[base + t] : 1.0;
            rs_s[t] = in ? a.rot_s[base + t] : 0.0;
        }
        __syncthreads();
        if (lane >= R) continue;
        int i = ri_s[0];
        double c = rc_s[0], s = rs_s[0];
        int i1 = ri_s[1];
        double c1 = rc_s[1], s1 = rs_s[1];
        double av = z[i * R], bv = z[(i + 1) * R];
        for (int k = 0; k < nch; ++k) {
            // rotation k+2 is fetched now (sentinels past the end), k+1 is in registers
            const int i2 = ri_s[k + 2];
            const double c2 = rc_s[k + 2], s2 = rs_s[k + 2];
            const int i1c = i1 > 0 ? i1 : 0;
            const double pre = z[i1c * R];   // column i-1 when the sweep continues (untouched here)
            const double na = c * av - s * bv;
            const double nb = s * av + c * bv;
            z[(i + 1) * R] = nb;
            z[i * R] = na;
            if (i1 == i - 1) {   // same sweep: plane i-1 shares column i
                bv = na;
                av = pre;
            } else if (i1 >= 0) {   // new sweep: read both columns after the stores above
                av = z[i1 * R];
                bv = z[(i1 + 1) * R];
            }
            i = i1;
            c = c1;
            s = s1;
            i1 = i2;
            c1 = c2;
            s1 = s2;
        }
    }
    __syncthreads();
    if (live)
        for (int j = 0; j < n; ++j) a.Zs[(size_t)row * n + j] = zl[a.perm[j] * R + lane];
}

// ------------------------------------------------------------------ 4. back-transformation
struct BackArgs {
    const double* Z;      // eigenvectors of T: component i of vector j at Z[i * zr + j * zc]
    int zr, zc;
    const double2* vh;    // [n][n]
    const double2* tau;   // [n]
    double2* V;           // [n][n], columns j < K written
    const int* k_dev;     // K (device word), or null: k_const
    int k_const;
    int n;
};

constexpr int BT_AHEAD = 4;   // reflectors in flight
// One wavefront a column; its chain of n - 1 reflectors is bound by the latency of the loads
// (covered by BT_AHEAD of them in flight) and of the sums: 200 frames 131 -> 71 us, 400: 255 -> 212
// (before: one reflector ahead, its loads behind per-lane branches).  Two reflectors a round of
// sums (with v1^H v0 added) took 83 and 262.

template <int CT>
__global__ void __launch_bounds__(64) back_kernel(const BackArgs a) {
    __shared__ double2 st[FQ_MAX_NT];
    const int n = a.n, j = blockIdx.x, lane = threadIdx.x;
    if (j >= (a.k_dev ? *a.k_dev : a.k_const)) return;
    double2 z[CT];
#pragma unroll
    for (int t = 0; t < CT; ++t) {
        const int i = lane + 64 * t;
        z[t] = make_double2(i < n ? a.Z[(size_t)i * a.zr + (size_t)j * a.zc] : 0.0, 0.0);
    }
    // tau and v of the next BT_AHEAD reflectors; entries outside rows k+1 .. n-1 become zero at
    // use, so that the loads need no branch
    double2 vn[BT_AHEAD][CT], taun[BT_AHEAD];
    for (int i = lane; i < n; i += 64) st[i] = a.tau[i];   // (scalar loads would be waited for all at once)
    __syncthreads();
    auto fetch = [&](double2 (&v)[CT], double2& tau, int k) {
        k = max(k, 0);
        tau = st[k];
#pragma unroll
        for (int t = 0; t < CT; ++t) v[t] = a.vh[(size_t)k * n + min(lane + 64 * t, n - 1)];
    };
    if (n < 2) {
        if (lane == 0) a.V[j] = z[0];
        return;
    }
#pragma unroll
    for (int u = 0; u < BT_AHEAD; ++u) fetch(vn[u], taun[u], n - 2 - u);
    for (int k0 = n - 2; k0 >= 0; k0 -= BT_AHEAD) {
#pragma unroll
        for (int u = 0; u < BT_AHEAD; ++u) {
            const int k = k0 - u;
            double2 v[CT];
#pragma unroll
            for (int t = 0; t < CT; ++t) {
                const int i = lane + 64 * t;
                v[t] = i > k && i < n ? vn[u][t] : make_double2(0.0, 0.0);
            }
            const double2 tau = k >= 0 ? taun[u] : make_double2(0.0, 0.0);
            fetch(vn[u], taun[u], k - BT_AHEAD);
            if (tau.x == 0.0 && tau.y == 0.0) continue;
            double2 dot = make_double2(0.0, 0.0);   // v^H z over rows k+1 .. n-1
#pragma unroll
            for (int t = 0; t < CT; ++t) {
                dot.x += v[t].x * z[t].x + v[t].y * z[t].y;
                dot.y += v[t].x * z[t].y - v[t].y * z[t].x;
            }
            const double2 td = zmul(tau, wave_total(dot));
#pragma unroll
            for (int t = 0; t < CT; ++t) {
                const double2 w = zmul(v[t], td);
                z[t].x -= w.x;
                z[t].y -= w.y;
            }
        }
    }
#pragma unroll
    for (int t = 0; t < CT; ++t) {
        const int i = lane + 64 * t;
        if (i < n) a.V[(size_t)i * n + j] = z[t];
    }
}

// K selection by one wavefront: the knee's candidates spread over its lanes (one thread for all
// of them: 30 us at 200 frames, 62 at 400, now 5 and 7).
struct RankArgs {
    const double* lam;
    int* k_used;
    int* status;           // may be null
    int n, cutoff;
};

__global__ void __launch_bounds__(64) rank_kernel(const RankArgs a) {
    const int n = a.n, lane = threadIdx.x;
    int K;
    if (a.cutoff >= 0) {
        K = a.cutoff;
    } else if (a.cutoff == FQ_CUTOFF_SSM) {
        K = *a.k_used;   // written by the spatial-similarity pass
    } else if (n < 4 || !(a.lam[0] > 0.0)) {
        K = 1;
    } else {
        // chord rule on the dB spectrum (k is 1-based in the description): the first k of the
        // largest gap
        const double l1 = a.lam[0];
        const double d1 = 0.0;
        const double dN = 10.0 * log10(fmax(a.lam[n - 1], KNEE_FLOOR * l1) / l1);
        int best_k = 2;
        double best = -1.0 / 0.0;
        for (int k = 2 + lane; k <= n / 2; k += 64) {
            const double dk = 10.0 * log10(fmax(a.lam[k - 1], KNEE_FLOOR * l1) / l1);
            const double chord = d1 + (dN - d1) * (double)(k - 1) / (double)(n - 1);
            const double gap = chord - dk;
            if (gap > best) {
                best = gap;
                best_k = k;
            }
        }
        for (int o = 32; o > 0; o >>= 1) {
            const double g = __shfl_xor(best, o);
            const int k = __shfl_xor(best_k, o);
            if (g > best || (g == best && k < best_k)) {
                best = g;
                best_k = k;
            }
        }
        K = min(max(best_k - 1, 1), n / 2 - 1);
        if (K > KMAX) {
            K = KMAX;
            if (a.status && lane == 0) *a.status = FQ_E_NUMERIC;
        }
    }
    if (lane == 0) *a.k_used = K;
}

// FP32 copy of V_K [n][KMAX] and FP64 copy of its first KN columns [n][KN], both zero
// beyond column K (the projections run whole size classes).
constexpr int KN = 16;
__global__ void vk_kernel(const double2* vecs, const int* k_used, float2* vk, double2* vk64, int n) {
    const int K = *k_used;
    for (int idx = blockIdx.x * blockDim.x + threadIdx.x; idx < n * KMAX; idx += gridDim.x * blockDim.x) {
        const int f = idx / KMAX, k = idx % KMAX;
        double2 d = make_double2(0.0, 0.0);
        if (k < K) d = vecs[(size_t)f * n + k];
        vk[idx] = make_float2((float)d.x, (float)d.y);
        if (k < KN) vk64[f * KN + k] = d;
    }
}

// Power Doppler alone (no filtered IQ) for K <= 16: V_K has orthonormal columns, so the
// filtered energy of a voxel's row s of S is ||s - s V_K V_K^H||^2 = ||s||^2 - ||s V_K||^2
// (Pythagoras), formed in FP64 (the clutter energy it cancels is up to ~1e6 times the
// result) from one read of S.
// One voxel per thread; V_K rows are uniform across the wavefront (scalar loads).  The
// difference is clamped at zero, the value it rounds around when K removes every mode.
struct PdNormArgs {
    const float2* iq;     // [nt][nv]
    const double2* vk64;  // [nt][KN]
    const int* k_used;
    float* pd;            // [nv]
    int64_t nv;
    int nt;
    int k_lo;             // this instantiation serves k_lo < K <= KM
};

// Each K up to 8 (and even K up to 16) has its own sums: with classes of 4, 8 and 16 columns the
// FP64 products of zero columns cost as much as the memory traffic.  200 frames x 2097152 voxels:
// K = 3 663 -> 627 us, 5 755 -> 656, 8 750 (4.5 TB/s), 12 1088 -> 930; x 262144, K = 5: 108 -> 88.
// Two voxels a lane, or 2 or 8 frames ahead instead of 4, are within 5 % either way.
constexpr int PN_AHEAD = 4;   // frames loaded ahead
template <int KM>
__device__ __forceinline__ void pd_norm(const PdNormArgs& a, int64_t v) {
    double cr[KM], ci[KM], nx = 0.0;
#pragma unroll
    for (int k = 0; k < KM; ++k) cr[k] = ci[k] = 0.0;
    const float2* sv = a.iq + v;
    auto add = [&](int f, float2 x) {
        const double xr = x.x, xi = x.y;
        nx = fma(xr, xr, fma(xi, xi, nx));
        const double2* w = a.vk64 + f * KN;
#pragma unroll
        for (int k = 0; k < KM; ++k) {
            const double2 u = w[k];   // c_k = sum_f s_f V[f][k] (s V_K for the row s of S)
            cr[k] = fma(u.x, xr, fma(-u.y, xi, cr[k]));
            ci[k] = fma(u.x, xi, fma(u.y, xr, ci[k]));
        }
    };
    const int nb = a.nt / PN_AHEAD * PN_AHEAD;
    float2 nxt[PN_AHEAD];
#pragma unroll
    for (int u = 0; u < PN_AHEAD; ++u) nxt[u] = sv[(int64_t)min(u, a.nt - 1) * a.nv];
    for (int f = 0; f < nb; f += PN_AHEAD) {
        float2 cur[PN_AHEAD];
#pragma unroll
        for (int u = 0; u < PN_AHEAD; ++u) cur[u] = nxt[u];
#pragma unroll
        for (int u = 0; u < PN_AHEAD; ++u) nxt[u] = sv[(int64_t)min(f + PN_AHEAD + u, a.nt - 1) * a.nv];
#pragma unroll
        for (int u = 0; u < PN_AHEAD; ++u) add(f + u, cur[u]);
    }
    for (int f = nb; f < a.nt; ++f) add(f, sv[(int64_t)f * a.nv]);
    double c2 = 0.0;
#pragma unroll
    for (int k = 0; k < KM; ++k) c2 = fma(cr[k], cr[k], fma(ci[k], ci[k], c2));
    a.pd[v] = (float)(fmax(nx - c2, 0.0) / a.nt);
}

template <int KM>   // 8 or 16
__global__ void __launch_bounds__(256) pd_norm_kernel(const PdNormArgs a) {
    const int K = *a.k_used;
    if (K <= a.k_lo || K > KM) return;
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= a.nv) return;
    if (KM == 8) {
        if (K <= 2) pd_norm<2>(a, v);
        else if (K == 3) pd_norm<3>(a, v);
        else if (K == 4) pd_norm<4>(a, v);
        else if (K == 5) pd_norm<5>(a, v);
        else if (K == 6) pd_norm<6>(a, v);
        else if (K == 7) pd_norm<7>(a, v);
        else pd_norm<8>(a, v);
    } else {
        if (K <= 10) pd_norm<10>(a, v);
        else if (K <= 12) pd_norm<12>(a, v);
        else if (K <= 14) pd_norm<14>(a, v);
        else pd_norm<16>(a, v);
    }
}

struct PdArgs {
    const float2* iq;     // [nt][nv]
    const float2* vk;     // [nt][KMAX]
    const int* k_used;
    float2* out;          // [nt][nv] or null
    float* pd;            // [nv] or null
    int64_t nv;
    int nt;
    int k_lo;             // this instantiation serves k_lo < K <= KM (device-side dispatch)
    float inv_nt;
    bool stream;          // store out past the caches
};

// Projection and power Doppler on the matrix cores.  A workgroup of four wavefronts
// stages V_K (FP32 copy, zero beyond column K and frame n_t) in LDS once; each wavefront
// then owns 16 voxels: P = S V_K (16 x KM) with v_mfma_f32_16x16x4_f32 over the frames
// (the four real products of the complex product, S read straight from HBM as MFMA
// operands), P staged in LDS, and R = S - P V_K^H formed 16 frames at a time with the
// same MFMA over the K columns, subtracted from S (read again: the wavefront's 16-voxel
// slice was just fetched, so this read is served by the L2), squared and summed per voxel.
// MFMA 16x16x4 (FP32) lane layout: lane l supplies A[l%16][l/16] and B[l/16][l%16] and
// holds D[4(l/16) + r][l%16], r = 0..3.
typedef float floatx4 __attribute__((ext_vector_type(4)));
// two samples of a row of the ensemble: rows of an odd number of voxels start on 8 bytes
typedef float samples2 __attribute__((ext_vector_type(4), aligned(8)));
constexpr int PV = 16;             // voxels per wavefront
constexpr int PW = 4;              // wavefronts per workgroup
// At most four workgroups a compute unit, V_K staged once for all of a workgroup's voxels.  A
// filtered ensemble larger than the 256 MB last-level cache is stored past it, so that S's second
// read still hits there, if every wavefront's 16 voxels are a whole 128-byte line (partial lines
// written past the caches cost more than they save).  200 frames x 2097152 voxels, filtered
// ensemble and power Doppler: K = 5 3506 -> 2450 us (2826 with cached stores), K = 24 4875 -> 2670,
// K = 50 9166 -> 4560; power Doppler alone: K = 24 4050 -> 2116, K = 50 8041 -> 4220; x 65536, K = 5:
// 99 -> 84 (91 stored past the caches); 400 x 1000001, K = 12: 3864 -> 2620 (4068).
constexpr int PGRID = 1024;
constexpr int64_t PSTREAM = (int64_t)256 << 20;

__host__ __device__ inline int vk_stride(int km) { return km + 2; }   // LDS row stride of V_K (float2)

// VL: V_K staged in LDS (when it fits beside the P staging), else read from the
// L2-resident table (rows beyond n_t are then masked).
template <int KM, bool VL>
__global__ void __launch_bounds__(64 * PW) project_mfma_kernel(const PdArgs a) {
    extern __shared__ float2 sm2[];
    const int K = *a.k_used;
    if (K <= a.k_lo || K > KM) return;
    constexpr int NKT = KM / 16;
    constexpr int VS = VL ? KM + 2 : KMAX;
    constexpr int PS = KM + 1;
    const int nt = a.nt, ntp = (nt + 15) & ~15;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    float* Pr = reinterpret_cast<float*>(sm2 + (VL ? ntp * VS : 0)) + wv * 2 * PV * PS;   // [PV][PS]
    float* Pi = Pr + PV * PS;
    if (VL) {
        for (int idx = threadIdx.x; idx < ntp * KM; idx += 64 * PW) {
            const int f = idx / KM, k = idx % KM;
            sm2[f * VS + k] = f < nt ? a.vk[f * KMAX + k] : make_float2(0.f, 0.f);
        }
    }
    const float2* V = VL ? sm2 : a.vk;   // [ntp or n_t][VS]
    __syncthreads();
    const int li = lane & 15, lk = lane >> 4;
    const int64_t step = (int64_t)gridDim.x * PW * PV;
    for (int64_t v0 = ((int64_t)blockIdx.x * PW + wv) * PV; v0 < a.nv; v0 += step) {
        const bool full = v0 + PV <= a.nv;
        const float2* S = a.iq;
        // P = S V_K: A[i][k] = S[voxel i][frame f0 + k], B[k][j] = V[frame f0 + k][column 16t + j]
        floatx4 rr[NKT], ii[NKT], ri[NKT], ir[NKT];
#pragma unroll
        for (int t = 0; t < NKT; ++t)
            for (int r = 0; r < 4; ++r) rr[t][r] = ii[t][r] = ri[t][r] = ir[t][r] = 0.f;
        // loads run 16 frames ahead, without a branch (past the last frame and voxel they repeat it)
        const int64_t vi = v0 + li < a.nv ? v0 + li : a.nv - 1;
        auto get1 = [&](float2 (&x)[4], int f0) {
#pragma unroll
            for (int u = 0; u < 4; ++u) x[u] = S[(int64_t)min(f0 + 4 * u + lk, nt - 1) * a.nv + vi];
        };
        float2 xn[4];
        get1(xn, 0);
        for (int f0 = 0; f0 < ntp; f0 += 16) {
            float2 xc[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const bool in = f0 + 4 * u + lk < nt;
                xc[u] = make_float2(in ? xn[u].x : 0.f, in ? xn[u].y : 0.f);
            }
            if (f0 + 16 < ntp) get1(xn, f0 + 16);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int f = f0 + 4 * u + lk;
                const float2 x = xc[u];
#pragma unroll
                for (int t = 0; t < NKT; ++t) {
                    const float2 w = (VL || f < nt) ? V[f * VS + 16 * t + li] : make_float2(0.f, 0.f);
                    rr[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x, w.x, rr[t], 0, 0, 0);
                    ii[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.y, w.y, ii[t], 0, 0, 0);
                    ri[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.x, w.y, ri[t], 0, 0, 0);
                    ir[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.y, w.x, ir[t], 0, 0, 0);
                }
            }
        }
        float2 sn[4];
        auto get2 = [&](int f0) {
            const float2* row = S + (int64_t)min(f0 + li, nt - 1) * a.nv;
            if (full) {
                const samples2* sp = reinterpret_cast<const samples2*>(row + v0 + 4 * lk);
                const samples2 s0 = sp[0], s1 = sp[1];
                sn[0] = make_float2(s0.x, s0.y);
                sn[1] = make_float2(s0.z, s0.w);
                sn[2] = make_float2(s1.x, s1.y);
                sn[3] = make_float2(s1.z, s1.w);
            } else {
#pragma unroll
                for (int r = 0; r < 4; ++r) sn[r] = row[min(v0 + 4 * lk + r, a.nv - 1)];
            }
        };
        get2(0);
        // P[voxel 4 lk + r][column 16 t + li]
#pragma unroll
        for (int t = 0; t < NKT; ++t)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                Pr[(4 * lk + r) * PS + 16 * t + li] = rr[t][r] - ii[t][r];
                Pi[(4 * lk + r) * PS + 16 * t + li] = ri[t][r] + ir[t][r];
            }
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        // R = S - P V_K^H, 16 frames at a time: A[i][k] = P[voxel i][k0 + k],
        // B[k][j] = conj(V[frame f0 + j][k0 + k]); lane holds R[voxel 4 lk + r][frame f0 + li]
        float pacc[4] = {0.f, 0.f, 0.f, 0.f};
        for (int f0 = 0; f0 < ntp; f0 += 16) {
            const int f = f0 + li;
            float2 sv[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) sv[r] = make_float2(f < nt ? sn[r].x : 0.f, f < nt ? sn[r].y : 0.f);
            if (f0 + 16 < ntp) get2(f0 + 16);
            floatx4 qa, qb, qc, qd;
            for (int r = 0; r < 4; ++r) qa[r] = qb[r] = qc[r] = qd[r] = 0.f;
#pragma unroll
            for (int k0 = 0; k0 < KM; k0 += 4) {
                const float pr = Pr[li * PS + k0 + lk], pi = Pi[li * PS + k0 + lk];
                const float2 w = (VL || f < nt) ? V[f * VS + k0 + lk] : make_float2(0.f, 0.f);
                qa = __builtin_amdgcn_mfma_f32_16x16x4f32(pr, w.x, qa, 0, 0, 0);
                qb = __builtin_amdgcn_mfma_f32_16x16x4f32(pi, w.y, qb, 0, 0, 0);
                qc = __builtin_amdgcn_mfma_f32_16x16x4f32(pi, w.x, qc, 0, 0, 0);
                qd = __builtin_amdgcn_mfma_f32_16x16x4f32(pr, w.y, qd, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                // P conj(V) = (Pr Vr + Pi Vi) + i (Pi Vr - Pr Vi)
                const float xr = sv[r].x - (qa[r] + qb[r]);
                const float xi = sv[r].y - (qc[r] - qd[r]);
                pacc[r] = fmaf(xr, xr, fmaf(xi, xi, pacc[r]));
                sv[r] = make_float2(xr, xi);
            }
            if (a.out && f < nt) {
                float2* op = a.out + (int64_t)f * a.nv + v0 + 4 * lk;
                if (full) {
                    const samples2 o0{sv[0].x, sv[0].y, sv[1].x, sv[1].y}, o1{sv[2].x, sv[2].y, sv[3].x, sv[3].y};
                    samples2* o = reinterpret_cast<samples2*>(op);
                    if (a.stream) {
                        __builtin_nontemporal_store(o0, o);
                        __builtin_nontemporal_store(o1, o + 1);
                    } else {
                        o[0] = o0;
                        o[1] = o1;
                    }
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
                        if (v0 + 4 * lk + r < a.nv) op[r] = sv[r];
                }
            }
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            float x = pacc[r];
            for (int o = 1; o < 16; o <<= 1) x += __shfl_xor(x, o);
            pacc[r] = x;
        }
        if (li == 0 && a.pd) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t v = v0 + 4 * lk + r;
                if (v < a.nv) a.pd[v] = pacc[r] * a.inv_nt;
            }
        }
        // (the next voxels' P overwrites this one's: the wavefront's own LDS, in order)
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    }
}

constexpr size_t PROJ_LDS_MAX = 150 * 1024;

size_t project_mfma_lds(int nt, int km, bool vl) {
    const int ntp = (nt + 15) & ~15;
    return (vl ? sizeof(float2) * (size_t)ntp * vk_stride(km) : 0) + sizeof(float) * 2 * PW * PV * (size_t)(km + 1);
}
bool project_vl(int nt, int km) { return project_mfma_lds(nt, km, true) <= PROJ_LDS_MAX; }

__global__ void __launch_bounds__(256) pd_kernel(const float2* iq, int64_t nv, int nt, float inv_nt, float* pd) {
    const int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (v >= nv) return;
    float acc = 0.f;
    for (int f = 0; f < nt; ++f) {
        const float2 s = iq[(int64_t)f * nv + v];
        acc = fmaf(s.x, s.x, fmaf(s.y, s.y, acc));
    }
    pd[v] = acc * inv_nt;
}

using BackFn = void (*)(const BackArgs);
BackFn back_fn(int n) {
    return n <= 64 ? back_kernel<1> : n <= 128 ? back_kernel<2> : n <= 256 ? back_kernel<4> : back_kernel<FQ_MAX_NT / 64>;
}
using TriRowFn = void (*)(const TriArgs, int);
template <bool FIRST>
TriRowFn tri_row_fn(int chunks) {
    static const TriRowFn fn[FQ_MAX_NT / 64] = {
        tridiag_row_kernel<1, FIRST>, tridiag_row_kernel<2, FIRST>, tridiag_row_kernel<3, FIRST>,
        tridiag_row_kernel<4, FIRST>, tridiag_row_kernel<5, FIRST>, tridiag_row_kernel<6, FIRST>,
        tridiag_row_kernel<7, FIRST>, tridiag_row_kernel<8, FIRST>};
    return fn[chunks - 1];
}

struct SvdWs {
    size_t off_A, off_vh, off_tau, off_d, off_e, off_ri, off_rc, off_rs, off_rn, off_perm, off_Zs;
    size_t off_lam, off_vecs, off_vk, off_vk64, off_k, off_ev, off_sc, off_zt, total;
    int cap;
};

SvdWs svd_layout(int n) {
    SvdWs w{};
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o += round_up(bytes, 256);
        return at;
    };
    const size_t nn = (size_t)n * n;
    w.cap = ROT_PER_N2 * n * n + 64;
    w.off_A = take(sizeof(double2) * nn);
    w.off_vh = take(sizeof(double2) * nn);
    w.off_tau = take(sizeof(double2) * n);
    w.off_d = take(sizeof(double) * n);
    w.off_e = take(sizeof(double) * n);
    w.off_ri = take(sizeof(int) * (size_t)w.cap);
    w.off_rc = take(sizeof(double) * (size_t)w.cap);
    w.off_rs = take(sizeof(double) * (size_t)w.cap);
    w.off_rn = take(sizeof(int));
    w.off_perm = take(sizeof(int) * n);
    w.off_Zs = take(sizeof(double) * nn);
    w.off_lam = take(sizeof(double) * n);
    w.off_vecs = take(sizeof(double2) * nn);
    w.off_vk = take(sizeof(float2) * (size_t)n * KMAX);
    w.off_vk64 = take(sizeof(double2) * (size_t)n * KN);
    w.off_k = take(sizeof(int));
    w.off_ev = take(sizeof(double) * n);
    w.off_sc = take(sizeof(double));
    w.off_zt = take(sizeof(double) * (size_t)n * KMAX);
    w.total = o;
    return w;
}

// One workgroup up to TRI_ONE frames, one launch a step beyond.
int launch_tridiag(const double* gram, int n, char* ws, const SvdWs& L, hipStream_t s) {
    const TriArgs a{reinterpret_cast<const double2*>(gram), reinterpret_cast<double2*>(ws + L.off_A),
                    reinterpret_cast<double2*>(ws + L.off_vh), reinterpret_cast<double2*>(ws + L.off_tau),
                    reinterpret_cast<double*>(ws + L.off_d), reinterpret_cast<double*>(ws + L.off_e),
                    reinterpret_cast<double2*>(ws + L.off_Zs), n};   // Zs is written by later kernels only
    if (n <= TRI_ONE) {
        if (n <= 64) hipLaunchKernelGGL((tridiag_step_kernel<64, 4>), dim3(1), dim3(256), 0, s, a);
        else hipLaunchKernelGGL((tridiag_step_kernel<TRI_ONE, 8>), dim3(1), dim3(512), 0, s, a);
        FQ_LAUNCH_CHECK();
        return FQ_OK;
    }
    for (int k = 0; k < n; ++k) {
        const int chunks = (n - (k & ~63) + 63) / 64;
        const TriRowFn kern = k ? tri_row_fn<false>(chunks) : tri_row_fn<true>(chunks);
        hipLaunchKernelGGL(kern, dim3(std::max(1, n - 1 - k)), dim3(64), 0, s, a, k);
        FQ_LAUNCH_CHECK();
    }
    return FQ_OK;
}

// Every eigenpair by QL (hermitian_eig): eigenvalues (descending, clamped) into lam/sigma;
// the leading ncols eigenvectors into vecs ([n][n] complex128, columns in rank order)
// unless vecs is null.
int launch_eig(const double* gram, int n, char* ws, const SvdWs& L, double* lam, double* sigma, double* vecs,
               int ncols, int* status, hipStream_t s) {
    double2* vh = reinterpret_cast<double2*>(ws + L.off_vh);
    double2* tau = reinterpret_cast<double2*>(ws + L.off_tau);
    double* d = reinterpret_cast<double*>(ws + L.off_d);
    double* e = reinterpret_cast<double*>(ws + L.off_e);
    int* ri = reinterpret_cast<int*>(ws + L.off_ri);
    double* rc = reinterpret_cast<double*>(ws + L.off_rc);
    double* rs = reinterpret_cast<double*>(ws + L.off_rs);
    int* rn = reinterpret_cast<int*>(ws + L.off_rn);
    int* perm = reinterpret_cast<int*>(ws + L.off_perm);
    double* Zs = reinterpret_cast<double*>(ws + L.off_Zs);

    const int st = launch_tridiag(gram, n, ws, L, s);
    if (st != FQ_OK) return st;
    QlArgs qa{d, e, ri, rc, rs, rn, L.cap, lam, sigma, perm, status, n};
    hipLaunchKernelGGL(ql_kernel, dim3(1), dim3(64), 0, s, qa);
    FQ_LAUNCH_CHECK();
    if (!vecs || ncols < 1) return FQ_OK;
    const int rows = n <= 256 ? 64 : 32;   // LDS: rows x n doubles <= 128 KiB
    ReplayArgs pa{ri, rc, rs, rn, perm, Zs, n, rows};
    hipLaunchKernelGGL(replay_kernel, dim3((n + rows - 1) / rows), dim3(64), sizeof(double) * (size_t)rows * n, s, pa);
    FQ_LAUNCH_CHECK();
    BackArgs ba{Zs, n, 1, vh, tau, reinterpret_cast<double2*>(vecs), nullptr, std::min(ncols, n), n};
    hipLaunchKernelGGL(back_fn(n), dim3(std::min(ncols, n)), dim3(64), 0, s, ba);
    FQ_LAUNCH_CHECK();
    return FQ_OK;
}

// The clutter filter's eigensolver, first half: tridiagonalisation and every eigenvalue
// (lam, sigma, and the unit-scaled ev for the vectors).
int launch_eigvals(const double* gram, int n, char* ws, const SvdWs& L, double* lam, double* sigma, int* status,
                   hipStream_t s) {
    const int st = launch_tridiag(gram, n, ws, L, s);
    if (st != FQ_OK) return st;
    EigvalArgs ea{reinterpret_cast<const double*>(ws + L.off_d), reinterpret_cast<const double*>(ws + L.off_e),
                  reinterpret_cast<double*>(ws + L.off_ev), reinterpret_cast<double*>(ws + L.off_sc), lam, sigma,
                  status, n};
    constexpr int per_block = EV_THREADS / 64;
    hipLaunchKernelGGL(eigval_kernel, dim3((n + per_block - 1) / per_block), dim3(EV_THREADS), 0, s, ea);
    FQ_LAUNCH_CHECK();
    return FQ_OK;
}

// Second half: the K leading eigenvectors (K from the device word k_dev, else k_const),
// by inverse iteration on T and back-transformation, into vecs columns 0 .. K-1.
int launch_eigvecs(int n, char* ws, const SvdWs& L, const int* k_dev, int k_const, double* vecs, int* status,
                   hipStream_t s) {
    double* zt = reinterpret_cast<double*>(ws + L.off_zt);
    const int grid = k_dev ? KMAX : k_const;
    if (grid < 1) return FQ_OK;
    InvitArgs ia{reinterpret_cast<const double*>(ws + L.off_d), reinterpret_cast<const double*>(ws + L.off_e),
                 reinterpret_cast<const double*>(ws + L.off_ev), reinterpret_cast<const double*>(ws + L.off_sc),
                 k_dev, k_const, zt, status, n};
    hipLaunchKernelGGL(invit_kernel, dim3(grid), dim3(64), 0, s, ia);
    FQ_LAUNCH_CHECK();
    hipLaunchKernelGGL(orth_kernel, dim3(1), dim3(ORTH_THREADS), 0, s, ia);
    FQ_LAUNCH_CHECK();
    BackArgs ba{zt, 1, n, reinterpret_cast<const double2*>(ws + L.off_vh),
                reinterpret_cast<const double2*>(ws + L.off_tau), reinterpret_cast<double2*>(vecs), k_dev, k_const, n};
    hipLaunchKernelGGL(back_fn(n), dim3(grid), dim3(64), 0, s, ba);
    FQ_LAUNCH_CHECK();
    return FQ_OK;
}

using PdFn = void (*)(const PdArgs);
PdFn pd_fn(int k, bool vl) {
    if (k <= 16) return vl ? project_mfma_kernel<16, true> : project_mfma_kernel<16, false>;
    if (k <= 32) return vl ? project_mfma_kernel<32, true> : project_mfma_kernel<32, false>;
    return vl ? project_mfma_kernel<64, true> : project_mfma_kernel<64, false>;
}

}  // namespace
}  // namespace fq

using namespace fq;

extern "C" size_t svd_workspace_size(int64_t n_vox, int32_t n_t) {
    if (n_t < 1 || n_vox < 1) return 0;
    return svd_layout(n_t).total + ssm_bytes(n_vox, n_t);
}

extern "C" int hermitian_eig(const double* gram, int32_t n_t, void* ws, size_t ws_bytes, double* lam, double* vecs,
                             int32_t* status, void* stream) {
    FQ_REQUIRE(n_t >= 1 && n_t <= FQ_MAX_NT, "n_t must be 1..%d", FQ_MAX_NT);
    FQ_REQUIRE(gram && ws && lam && aligned16(gram) && aligned16(ws), "null or misaligned pointer");
    const SvdWs L = svd_layout(n_t);
    if (ws_bytes < L.total) {
        set_error("workspace too small: %zu < %zu bytes", ws_bytes, L.total);
        return FQ_E_WORKSPACE;
    }
    return launch_eig(gram, n_t, reinterpret_cast<char*>(ws), L, lam, nullptr, vecs, n_t, status, as_stream(stream));
}

// The filter's last stage on the V_K (FP32 and FP64 copies) and K that the eigendecomposition
// left in the workspace: the filtered IQ and/or the power Doppler.
static int launch_apply(const float* iq, int64_t n_vox, int n_t, char* w, const SvdWs& L, int cutoff,
                        const int32_t* k_used, float* iq_filt, float* pd, hipStream_t s) {
    PdArgs pa{};
    pa.iq = reinterpret_cast<const float2*>(iq);
    pa.vk = reinterpret_cast<const float2*>(w + L.off_vk);
    pa.k_used = k_used;
    pa.out = reinterpret_cast<float2*>(iq_filt);
    pa.pd = pd;
    pa.nv = n_vox;
    pa.nt = n_t;
    pa.inv_nt = 1.0f / (float)n_t;
    pa.stream = iq_filt && n_vox % 16 == 0 && (uintptr_t)iq_filt % 128 == 0 &&
                (int64_t)sizeof(float2) * n_vox * n_t > PSTREAM;
    const unsigned blocks = (unsigned)std::min<int64_t>((n_vox + PV * PW - 1) / (PV * PW), PGRID);
    if (!iq_filt) {
        // power Doppler alone: the FP64 norm difference up to K = 16, the explicit
        // projection above; all but the class holding K return at once
        PdNormArgs na{pa.iq, reinterpret_cast<const double2*>(w + L.off_vk64), k_used, pd, n_vox, n_t, -1};
        const unsigned nb = (unsigned)((n_vox + 255) / 256);
        const int bounds[5] = {-1, 8, 16, 32, 64};
        for (int c = 0; c < 4; ++c) {
            if (cutoff >= 0 && !(cutoff > bounds[c] && cutoff <= bounds[c + 1])) continue;
            if (c < 2) {
                na.k_lo = bounds[c];
                auto kern = c == 0 ? pd_norm_kernel<8> : pd_norm_kernel<16>;
                hipLaunchKernelGGL(kern, dim3(nb), dim3(256), 0, s, na);
            } else {
                pa.k_lo = bounds[c];
                const bool vl = project_vl(n_t, bounds[c + 1]);
                hipLaunchKernelGGL(pd_fn(bounds[c + 1], vl), dim3(blocks), dim3(64 * PW),
                                   project_mfma_lds(n_t, bounds[c + 1], vl), s, pa);
            }
            FQ_LAUNCH_CHECK();
        }
        return FQ_OK;
    }
    if (cutoff >= 0) {
        const int km = cutoff <= 16 ? 16 : (cutoff <= 32 ? 32 : 64);
        pa.k_lo = -1;
        const bool vl = project_vl(n_t, km);
        hipLaunchKernelGGL(pd_fn(km, vl), dim3(blocks), dim3(64 * PW), project_mfma_lds(n_t, km, vl), s, pa);
        FQ_LAUNCH_CHECK();
    } else {
        // the knee's K is only known on the device: every size class is launched and
        // all but the one holding K return at once
        const int bounds[4] = {-1, 16, 32, 64};
        for (int c = 0; c < 3; ++c) {
            pa.k_lo = bounds[c];
            const bool vl = project_vl(n_t, bounds[c + 1]);
            hipLaunchKernelGGL(pd_fn(bounds[c + 1], vl), dim3(blocks), dim3(64 * PW),
                               project_mfma_lds(n_t, bounds[c + 1], vl), s, pa);
            FQ_LAUNCH_CHECK();
        }
    }
    return FQ_OK;
}

extern "C" int svd_clutter_filter(const float* iq, int64_t n_vox, int32_t n_t, const double* gram, int32_t cutoff,
                                  void* ws, size_t ws_bytes, float* iq_filt, float* pd, double* sigma,
                                  int32_t* k_used, int32_t* status, void* stream) {
    FQ_REQUIRE(n_t >= 1 && n_t <= FQ_MAX_NT, "n_t must be 1..%d", FQ_MAX_NT);
    FQ_REQUIRE(n_vox >= 1, "n_vox must be >= 1");
    FQ_REQUIRE(cutoff >= FQ_CUTOFF_SSM && cutoff <= n_t, "cutoff must be -2 (SSM), -1 (knee) or 0..n_t");
    FQ_REQUIRE(cutoff != FQ_CUTOFF_SSM || n_t >= 2, "the SSM cutoff needs n_t >= 2");
    FQ_REQUIRE(cutoff <= KMAX, "fixed cutoff above %d is not supported", KMAX);
    FQ_REQUIRE(iq && gram && ws && sigma && k_used && aligned16(iq) && aligned16(gram) && aligned16(ws),
               "null or misaligned pointer");
    FQ_REQUIRE(!iq_filt || aligned16(iq_filt), "misaligned iq_filt");
    const SvdWs L = svd_layout(n_t);
    const size_t need = L.total + (cutoff == FQ_CUTOFF_SSM ? ssm_bytes(n_vox, n_t) : 0);
    if (ws_bytes < need) {
        set_error("workspace too small: %zu < %zu bytes", ws_bytes, need);
        return FQ_E_WORKSPACE;
    }
    hipStream_t s = as_stream(stream);
    char* w = reinterpret_cast<char*>(ws);
    double* lam = reinterpret_cast<double*>(w + L.off_lam);
    double* vecs = reinterpret_cast<double*>(w + L.off_vecs);
    int st = launch_eigvals(gram, n_t, w, L, lam, sigma, status, s);
    if (st != FQ_OK) return st;
    RankArgs ra{lam, k_used, status, n_t, cutoff};
    if (cutoff == FQ_CUTOFF_SSM) {
        // the rank is read from the leading min(n_t, 64) spatial modes
        const int M = std::min(n_t, FQ_SSM_MAX_MODES);
        st = launch_eigvecs(n_t, w, L, nullptr, M, vecs, status, s);
        if (st != FQ_OK) return st;
        st = launch_ssm(iq, n_vox, n_t, vecs, M, w + L.total, nullptr, k_used, s);
        if (st != FQ_OK) return st;
        hipLaunchKernelGGL(rank_kernel, dim3(1), dim3(64), 0, s, ra);
        FQ_LAUNCH_CHECK();
    } else {
        hipLaunchKernelGGL(rank_kernel, dim3(1), dim3(64), 0, s, ra);
        FQ_LAUNCH_CHECK();
        st = launch_eigvecs(n_t, w, L, k_used, 0, vecs, status, s);
        if (st != FQ_OK) return st;
    }
    hipLaunchKernelGGL(vk_kernel, dim3((n_t * KMAX + 255) / 256), dim3(256), 0, s,
                       reinterpret_cast<const double2*>(vecs), static_cast<const int*>(k_used),
                       reinterpret_cast<float2*>(w + L.off_vk), reinterpret_cast<double2*>(w + L.off_vk64), n_t);
    FQ_LAUNCH_CHECK();
    if (!iq_filt && !pd) return FQ_OK;
    return launch_apply(iq, n_vox, n_t, w, L, cutoff, k_used, iq_filt, pd, s);
}

extern "C" int svd_filter_apply(const float* iq, int64_t n_vox, int32_t n_t, const void* ws, size_t ws_bytes,
                                const int32_t* k_used, float* iq_filt, float* pd, void* stream) {
    FQ_REQUIRE(n_t >= 1 && n_t <= FQ_MAX_NT, "n_t must be 1..%d", FQ_MAX_NT);
    FQ_REQUIRE(n_vox >= 1, "n_vox must be >= 1");
    FQ_REQUIRE(iq && ws && k_used && aligned16(iq) && aligned16(ws), "null or misaligned pointer");
    FQ_REQUIRE(iq_filt || pd, "nothing to compute: iq_filt and pd are both null");
    FQ_REQUIRE(!iq_filt || aligned16(iq_filt), "misaligned iq_filt");
    const SvdWs L = svd_layout(n_t);
    if (ws_bytes < L.total) {
        set_error("workspace too small: %zu < %zu bytes", ws_bytes, L.total);
        return FQ_E_WORKSPACE;
    }
    return launch_apply(iq, n_vox, n_t, reinterpret_cast<char*>(const_cast<void*>(ws)), L, -1, k_used, iq_filt, pd,
                        as_stream(stream));
}

extern "C" int power_doppler(const float* iq, int64_t n_vox, int32_t n_t, float* pd, void* stream) {
    FQ_REQUIRE(n_t >= 1 && n_vox >= 1, "bad sizes");
    FQ_REQUIRE(iq && pd && aligned16(iq), "null or misaligned pointer");
    const unsigned blocks = (unsigned)((n_vox + 255) / 256);
    hipLaunchKernelGGL(pd_kernel, dim3(blocks), dim3(256), 0, as_stream(stream), reinterpret_cast<const float2*>(iq),
                       n_vox, n_t, 1.0f / (float)n_t, pd);
    FQ_LAUNCH_CHECK();
    return FQ_OK;
}
