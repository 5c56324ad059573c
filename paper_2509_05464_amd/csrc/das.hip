// das_beamform: RF -> IQ demodulation and 3-D delay-and-sum with coherent compounding (gfx950).
//
// Frames are processed in blocks of FB <= 8: the F frames of a call are divided evenly over
// ceil(F / 8) blocks, so a call of 3 frames sums 3 and one of 20 sums 3 x 7.
//
// Stage 1, rf2iq: one workgroup per (frame block, angle, element) stages the FB RF traces in
// LDS and writes the baseband in a frame-blocked layout
//     bb[fblock][angle][element][sample][FB frames]   (complex64)
// so that one delay tap of one (angle, element) for all frames of a block is a single row of
// FB values.  b[n] = exp(-i w n) sum_k c_k rf[n-k] with precomputed complex taps
// c_k = 2 h_k exp(i w k), w = 2 pi fc/fs.
//
// Stage 2, DAS (das_kernel.hpp): one workgroup per (tile of 512 voxels, frame block).  The
// per-(voxel, element) work (FP64 receive distance, its phase) is shared by all angles and
// the per-(voxel, element, angle) work by the frames of the block, as the paper does by
// building the delay operator once and applying it to every frame.
#include "das_kernel.hpp"

namespace fq {
namespace {

// The tile that das_window_rows describes; its window also decides which grids are refused.
constexpr int TILE_X = 16, TILE_Y = 16, TILE_Z = 2;
constexpr int FIR_HALF = 16;
constexpr int IQ_THREADS = 256;
constexpr int IQ_RUN = 4;       // consecutive samples per thread
constexpr size_t DAS_LDS_BUDGET = 64 * 1024;

// --------------------------------------------------------------------------- rf2iq
struct IqArgs {
    const float* rf;       // [F][A][E][T]
    float2* bb;            // [nfb][A][E][TR][FB]
    int F, A, E, T, TR;
    int FB;                // frames per block
    int fb0;               // first global frame block of this launch
    int stride;            // LDS floats per trace
    double fc_fs;          // fc / fs
    float2 taps[2 * FIR_HALF + 1];
};

// A thread forms IQ_RUN consecutive samples of one frame: the 36 inputs they share are read
// from LDS once (9 reads a sample instead of 33).
__global__ void __launch_bounds__(IQ_THREADS) rf2iq_kernel(const IqArgs a) {
    extern __shared__ float sh[];          // [FB][stride]
    const int e = blockIdx.x, an = blockIdx.y, fbl = blockIdx.z;
    const int fb = a.fb0 + fbl;
    for (int fl = 0; fl < a.FB; ++fl) {
        const int f = fb * a.FB + fl;
        const float* src = a.rf + (((int64_t)f * a.A + an) * a.E + e) * a.T - FIR_HALF;
        for (int i = threadIdx.x; i < a.stride; i += IQ_THREADS)
            sh[fl * a.stride + i] = f < a.F && i >= FIR_HALF && i < a.T + FIR_HALF ? src[i] : 0.0f;
    }
    __syncthreads();
    float2* out = a.bb + (((int64_t)fbl * a.A + an) * a.E + e) * (int64_t)a.TR * a.FB;
    const int runs = (a.TR + IQ_RUN - 1) / IQ_RUN;
    for (int i = threadIdx.x; i < a.FB * runs; i += IQ_THREADS) {
        const int run = i / a.FB, fl = i - run * a.FB, n0 = run * IQ_RUN;
        const float* row = sh + fl * a.stride + n0;   // inputs n0 - FIR_HALF ..
        float x[IQ_RUN + 2 * FIR_HALF];
#pragma unroll
        for (int k = 0; k < IQ_RUN + 2 * FIR_HALF; ++k) x[k] = row[k];
#pragma unroll
        for (int m = 0; m < IQ_RUN; ++m) {
            const int n = n0 + m;
            float re = 0.0f, im = 0.0f;
#pragma unroll
            for (int k = -FIR_HALF; k <= FIR_HALF; ++k) {
                const float v = x[m + FIR_HALF - k];
                re = fmaf(a.taps[k + FIR_HALF].x, v, re);
                im = fmaf(a.taps[k + FIR_HALF].y, v, im);
            }
            const float2 rot = cis_cycles(-(double)n * a.fc_fs);
            // row T of an odd-length trace is zero, like every sample outside the record
            if (n < a.TR) out[(int64_t)n * a.FB + fl] = n < a.T ? cmul(rot, make_float2(re, im)) : make_float2(0.f, 0.f);
        }
    }
}

DasFn das_fn(int fb, int at, int interp, bool wide, int groups) {
    switch (fb) {
        case 1: return das_fn1(at, interp, wide, groups);
        case 2: return das_fn2(at, interp, wide, groups);
        case 3: return das_fn3(at, interp, wide, groups);
        case 4: return das_fn4(at, interp, wide, groups);
        case 5: return das_fn5(at, interp, wide, groups);
        case 6: return das_fn6(at, interp, wide, groups);
        case 7: return das_fn7(at, interp, wide, groups);
        default: return das_fn8(at, interp, wide, groups);
    }
}

// Low-pass taps: Hann(33)-windowed sinc with cutoff fc, unit DC gain; folded with the
// carrier as c_k = 2 h_k exp(i 2 pi fc k / fs).
void make_taps(double fc, double fs, float2* taps) {
    double h[2 * FIR_HALF + 1], sum = 0.0;
    for (int k = -FIR_HALF; k <= FIR_HALF; ++k) {
        const double w = 0.5 * (1.0 + std::cos(M_PI * k / (FIR_HALF + 1)));
        const double x = 2.0 * fc * k / fs;
        const double sn = k == 0 ? 1.0 : std::sin(M_PI * x) / (M_PI * x);
        h[k + FIR_HALF] = w * sn;
        sum += w * sn;
    }
    for (int k = -FIR_HALF; k <= FIR_HALF; ++k) {
        const double hk = 2.0 * h[k + FIR_HALF] / sum;
        const double ph = 2.0 * M_PI * fc * k / fs;
        taps[k + FIR_HALF] = make_float2((float)(hk * std::cos(ph)), (float)(hk * std::sin(ph)));
    }
}

// Upper bound on the delay-window rows that a tile of nx x ny x nz voxels can touch for one
// (angle, element): receive-distance spread <= tile diameter, transmit spread <= |u|.extent,
// plus the interpolation taps and the integer row bases' margins.
int window_rows(const fq_grid& g, const TxHost& th, double fs_c, int nx, int ny, int nz) {
    const double Lx = (nx - 1) * g.dx, Ly = (ny - 1) * g.dy, Lz = (nz - 1) * g.dz;
    const double diam = std::sqrt(Lx * Lx + Ly * Ly + Lz * Lz);
    double txr = 0.0;
    for (int j = 0; j < th.n; ++j)
        txr = std::max(txr, std::fabs(th.ux[j]) * Lx + std::fabs(th.uy[j]) * Ly + th.uz[j] * Lz);
    const int w = (int)std::floor((diam + txr) * fs_c) + 8;
    return (int)round_up((size_t)w, 8);
}

size_t block_bytes(int A, int E, int T, int fb) { return (size_t)A * E * T * fb * sizeof(float2); }

// Frames per block, and the rows kept for a trace.  An even division over ceil(F / 8) blocks
// computes at most one unused frame per block; a fixed 8 computed 8 for a call of 3 frames
// (five plane waves, 100^3 voxels, 1024 elements: 24.2 ms, with 3 frames per block 10.5 ms).
// Rows of an odd number of frames are copied in 16-byte pieces, so their traces have an even
// number of rows; a block never takes more room than the 8 frames the workspace sizes count.
void frame_blocks(int F, int T, int& nfb, int& fb, int& TR) {
    nfb = (F + DAS_MAX_FB - 1) / DAS_MAX_FB;
    fb = (F + nfb - 1) / nfb;
    TR = T + (fb & T & 1);
    if (fb * TR > DAS_MAX_FB * T) {
        fb = DAS_MAX_FB;
        TR = T;
    }
}

// Voxel tile (log2 of its threads per axis), angles per pass, window rows, element groups.
struct DasTile {
    int sx, sy, sz, W, WB, at, groups;
    bool wide;
    double cost;
    int64_t ntx, nty, ntz;
};

// The tile with the least work: every tile costs its 512 voxels, padding included, and its
// staging, which grows with the window (about 15% of a 64-row tile's time); a second pass
// over the elements for more angles than the LDS arrays hold repeats the receive geometry.
// 128^3 voxels take 16 x 16 x 2 tiles or 8 x 8 x 8 ones; 35 x 33 x 61 voxels are padded to
// 1.30 times their number by 8 x 2 x 32 where 16 x 16 x 2 made it 2.03.
bool choose_tile(const fq_grid& g, const TxHost& th, double fs_c, int A, int fb, int groups, DasTile& best) {
    const int bits = groups == 1 ? 8 : groups == 4 ? 8 : 6, vz = das_vz(groups);
    bool found = false;
    for (int sx = 0; sx <= 6; ++sx)
        for (int sy = 0; sy <= 6 && sx + sy <= bits; ++sy) {
            DasTile t{};
            t.sx = sx;
            t.sy = sy;
            t.sz = bits - sx - sy;
            t.groups = groups;
            const int tx = 1 << t.sx, ty = 1 << t.sy, tz = vz << t.sz;
            t.ntx = (g.nx + tx - 1) / tx;
            t.nty = (g.ny + ty - 1) / ty;
            t.ntz = (g.nz + tz - 1) / tz;
            t.W = window_rows(g, th, fs_c, std::min(tx, g.nx), std::min(ty, g.ny), std::min(tz, g.nz));
            t.WB = (int)round_up((size_t)t.W * das_row_lds(fb) + DAS_SLACK, 16);
            t.wide = t.W > DAS_W_NARROW;
            if (t.wide && groups > 1) continue;
            const int bytes = das_rows(groups, t.wide, fb) * das_row_lds(fb);
            int at = std::min(t.wide ? 2 : DAS_MAX_AT, 2 * (bytes / t.WB));
            if (at < 1) continue;
            const int passes = (A + at - 1) / at;
            t.at = (A + passes - 1) / passes;
            t.cost = (1.0 + 0.15 * t.W / 64.0) * (1.0 + 0.3 * (passes - 1));
            if (!found || t.cost * (t.ntx * t.nty * t.ntz) < best.cost * (best.ntx * best.nty * best.ntz)) {
                found = true;
                best = t;
            }
        }
    return found;
}

// Tile and element groups by the time of a launch, in that of one wavefront's voxels over all
// elements.  Unsplit, a compute unit takes its workgroups in rounds of the three it holds, and
// one, two or three of them take 5.7, 6.7 or 7.5 (one wavefront a SIMD waits most of its time);
// split, it takes one at a time, 16 wavefronts on a half or an eighth of the voxels.  Measured
// on 45 calls of 4000 to 500000 voxels, 1 to 61 frames, 64 to 1024 elements: the choice is
// within 4% of the best of the three on average.  34 x 16 x 14 voxels, 4 frames, 576
// elements, 5 transmits: 1125 us unsplit, 379 with 4 groups, 122 with 16; 35 x 33 x 61, 20
// frames, cubic: 1209, 881, 997; 107 x 72 x 91, 2 frames: 247, 422, 896.
// Below 64 elements the 6 us that a split workgroup takes to set up and to add its sums count, 44
// elements' worth with one transmit: 64 x 48 x 7 voxels, 33 frames, 16 elements, 1 transmit: 31
// us unsplit, 33 with 4 groups, 61 with 16.
bool choose_launch(const fq_grid& g, const TxHost& th, double fs_c, int A, int E, int fb, int nfb, int interp, DasTile& best) {
    static const double unsplit[4] = {0.0, 5.7, 6.7, 7.5};
    // (little work per row of a window: the staging shows)
    const double split4 = interp ? 1.5 : fb * A <= 9 ? 2.1 : 1.75, split16 = 0.6;
    const double fixed = E < 64 ? 44.0 / (E * A) : 0.0;
    bool found = false;
    double best_time = 0.0;
    for (int groups : {1, 4, 16}) {
        DasTile t{};
        if (!choose_tile(g, th, fs_c, A, fb, groups, t)) continue;
        // (a launch holds 2^32 threads: beyond, one group's 256 a tile are the fewest)
        if (groups > 1 && t.ntx * t.nty * t.ntz * nfb * DAS_SPLIT_THREADS >= (1LL << 32)) continue;
        const double per_cu = (double)(t.ntx * t.nty * t.ntz) * nfb / 256.0;
        double time;
        if (groups == 1) {
            const int n = (int)std::min(1e6, std::ceil(per_cu));
            time = n > 6 ? per_cu * unsplit[3] / 3.0 : n / 3 * unsplit[3] + unsplit[n % 3];
        } else {
            time = std::ceil(per_cu) * ((groups == 4 ? split4 : split16) + fixed);
        }
        time *= t.cost;
        if (!found || time < best_time) {
            found = true;
            best_time = time;
            best = t;
        }
    }
    return found;
}

}  // namespace
}  // namespace fq

using namespace fq;

extern "C" size_t das_workspace_size(const fq_probe* probe, const fq_tx* tx, int32_t n_frames, int32_t n_samples,
                                     int32_t minimum) {
    if (!probe || !tx || n_frames < 1 || n_samples < 1 || tx->n_angles < 1) return 0;
    const int nfb = (n_frames + DAS_MAX_FB - 1) / DAS_MAX_FB;
    const size_t b = block_bytes(tx->n_angles, probe->nx_el * probe->ny_el, n_samples, DAS_MAX_FB);
    return minimum ? b : b * nfb;
}

extern "C" int das_window_rows(const fq_probe* probe, const fq_tx* tx, const fq_grid* grid) {
    if (check_probe_tx(probe, tx) != FQ_OK) return -1;
    if (!grid || grid->nx < 1 || grid->ny < 1 || grid->nz < 1 || !(grid->dx > 0) || !(grid->dy > 0) ||
        !(grid->dz > 0)) {
        set_error("bad grid");
        return -1;
    }
    return window_rows(*grid, make_tx(*probe, *tx), probe->fs_hz / probe->c_mps, TILE_X, TILE_Y, TILE_Z);
}

extern "C" int das_launch_shape(const fq_probe* probe, const fq_tx* tx, const fq_grid* grid, int32_t n_frames,
                                int32_t n_samples, int32_t interp, int64_t* shape) {
    const int st = check_probe_tx(probe, tx);
    if (st != FQ_OK) return st;
    FQ_REQUIRE(grid && grid->nx > 0 && grid->ny > 0 && grid->nz > 0 && grid->dx > 0 && grid->dy > 0 && grid->dz > 0,
               "bad grid");
    FQ_REQUIRE(n_frames >= 1 && n_samples >= 2 && shape, "bad n_frames / n_samples / shape");
    const TxHost th = make_tx(*probe, *tx);
    int nfb, fb, TR;
    frame_blocks(n_frames, n_samples, nfb, fb, TR);
    DasTile t{};
    FQ_REQUIRE(choose_launch(*grid, th, probe->fs_hz / probe->c_mps, th.n, probe->nx_el * probe->ny_el, fb, nfb, interp, t),
               "voxel spacing too coarse for the on-chip delay window");
    shape[0] = fb;
    shape[1] = t.at;
    shape[2] = t.groups;
    shape[3] = t.wide ? 1 : 0;
    shape[4] = t.ntx * t.nty * t.ntz;
    return FQ_OK;
}

namespace fq {
namespace {

struct DasPlan {
    IqArgs ia;
    DasArgs da;
    DasTile tile;
    TxHost th;
    int A, E, T, nfb, fb;
    size_t bblk;       // workspace bytes of one block
    size_t full;       // workspace bytes that the whole baseband is asked to have
    size_t iq_lds;
    double fs_c;
};

int das_prepare(const fq_probe* probe, const fq_tx* tx, const fq_grid* grid, int32_t n_frames, int32_t n_samples,
                const float* rf, int32_t interp, void* ws, size_t ws_bytes, float* iq, DasPlan& P) {
    int st = check_probe_tx(probe, tx);
    if (st != FQ_OK) return st;
    FQ_REQUIRE(grid && grid->nx > 0 && grid->ny > 0 && grid->nz > 0 && grid->dx > 0 && grid->dy > 0 && grid->dz > 0,
               "bad grid");
    FQ_REQUIRE(grid->z0 > 0, "the voxel grid must lie in front of the array (z0 > 0)");
    FQ_REQUIRE(n_frames >= 1 && n_samples >= 2 && n_samples <= (1 << 20), "bad n_frames / n_samples");
    FQ_REQUIRE(interp == FQ_INTERP_LINEAR || interp == FQ_INTERP_HERMITE, "bad interp");
    FQ_REQUIRE(ws && aligned16(ws), "null or misaligned workspace");
    FQ_REQUIRE((!rf || aligned16(rf)) && (!iq || aligned16(iq)), "misaligned pointer");
    P.A = tx->n_angles;
    P.E = probe->nx_el * probe->ny_el;
    P.T = n_samples;
    const size_t bmax = block_bytes(P.A, P.E, P.T, DAS_MAX_FB);
    if (ws_bytes < bmax) {
        set_error("workspace too small: %zu < %zu bytes", ws_bytes, bmax);
        return FQ_E_WORKSPACE;
    }
    P.th = make_tx(*probe, *tx);
    P.fs_c = probe->fs_hz / probe->c_mps;
    const int W0 = window_rows(*grid, P.th, P.fs_c, TILE_X, TILE_Y, TILE_Z);
    int TR = P.T;
    frame_blocks(n_frames, P.T, P.nfb, P.fb, TR);
    P.bblk = block_bytes(P.A, P.E, TR, P.fb);
    P.full = bmax * P.nfb;
    FQ_REQUIRE((size_t)W0 * das_row_lds(DAS_MAX_FB) <= DAS_LDS_BUDGET &&
                   choose_launch(*grid, P.th, P.fs_c, P.A, P.E, P.fb, P.nfb, interp, P.tile),
               "voxel spacing too coarse for the on-chip delay window (%d rows)", W0);

    IqArgs& ia = P.ia;
    ia = IqArgs{};
    ia.rf = rf;
    ia.bb = reinterpret_cast<float2*>(ws);
    ia.F = n_frames;
    ia.A = P.A;
    ia.E = P.E;
    ia.T = P.T;
    ia.TR = TR;
    ia.FB = P.fb;
    // Room for the inputs of every sample, odd (frames fall in different banks).  The samples of a
    // last run past the record read up to IQ_RUN - 1 values into the next trace, or behind the
    // last one, and are not stored: with rows of whole runs 8 frames of 5085 to 5087 samples
    // would not fit.
    ia.stride = (TR + 2 * FIR_HALF) | 1;
    ia.fc_fs = probe->fc_hz / probe->fs_hz;
    make_taps(probe->fc_hz, probe->fs_hz, ia.taps);
    P.iq_lds = sizeof(float) * (P.fb * (size_t)ia.stride + IQ_RUN - 1);
    // (one limit for every number of frames: that of a block of 8)
    FQ_REQUIRE(P.iq_lds <= 160 * 1024 && sizeof(float) * DAS_MAX_FB * (size_t)(P.T + 2 * FIR_HALF + 1) <= 160 * 1024,
               "n_samples too large for on-chip demodulation");

    DasArgs& da = P.da;
    da = DasArgs{};
    da.bb = reinterpret_cast<const char*>(ws);
    da.iq = reinterpret_cast<float2*>(iq);
    da.nx = grid->nx;
    da.ny = grid->ny;
    da.nz = grid->nz;
    da.sx = P.tile.sx;
    da.sy = P.tile.sy;
    da.sz = P.tile.sz;
    da.ntx = (int)P.tile.ntx;
    da.nty = (int)P.tile.nty;
    da.x0 = grid->x0;
    da.y0 = grid->y0;
    da.z0 = grid->z0;
    da.dx = grid->dx;
    da.dy = grid->dy;
    da.dz = grid->dz;
    da.nx_el = probe->nx_el;
    da.pitch_x = probe->pitch_x;
    da.pitch_y = probe->pitch_y;
    da.fs_c = P.fs_c;
    da.fc_fs = probe->fc_hz / probe->fs_hz;
    da.A = P.A;
    da.E = P.E;
    da.TR = TR;
    da.F = n_frames;
    da.W = P.tile.W;
    da.WB = P.tile.WB;
    da.inv_A = 1.0f / (float)P.A;
    const int64_t n_tiles = P.tile.ntx * P.tile.nty * P.tile.ntz;
    FQ_REQUIRE(n_tiles < (1LL << 31), "grid too large");
    da.ntiles = (int)n_tiles;
    return FQ_OK;
}

int launch_demod(DasPlan& P, int fb0, int nb, hipStream_t s) {
    P.ia.fb0 = fb0;
    hipLaunchKernelGGL(rf2iq_kernel, dim3(P.E, P.A, nb), dim3(IQ_THREADS), P.iq_lds, s, P.ia);
    FQ_LAUNCH_CHECK();
    return FQ_OK;
}

int launch_das(DasPlan& P, int fb0, int nb, int interp, const fq_grid* grid, double fs_hz, hipStream_t s) {
    DasArgs& da = P.da;
    da.fb0 = fb0;
    da.nwork = (int64_t)da.ntiles * nb;
    const int threads = P.tile.groups == 1 ? DAS_THREADS : DAS_SPLIT_THREADS;
    FQ_REQUIRE(da.nwork * threads < (1LL << 32), "grid too large");
    for (int a0 = 0; a0 < P.A; a0 += P.tile.at) {
        const int na = std::min(P.tile.at, P.A - a0);
        da.a0 = a0;
        da.accumulate = a0 > 0;
        for (int j = 0; j < na; ++j) {
            const int an = a0 + j;
            da.ux[j] = P.th.ux[an];
            da.uy[j] = P.th.uy[an];
            da.uz[j] = P.th.uz[an];
            da.t0s[j] = P.th.t0[an] * fs_hz;
            const double step = P.th.uz[an] * grid->dz * P.fs_c;     // samples per z step
            // (a narrow window holds a step below 2^8 rows; a single plane or voxel takes none)
            const double rows = P.tile.wide ? std::floor(step) : 0.0;
            const bool steps = grid->nz > 1 && P.tile.groups == 1;
            da.dzr[j] = steps ? (int)rows : 0;
            da.dzs[j] = steps ? (uint32_t)std::floor((step - rows) * (1 << 24) + 0.5) : 0u;
            const double cyc = step * da.fc_fs;
            const double fr = cyc - std::floor(cyc);
            da.zeta[j] = make_float2((float)std::cos(2 * M_PI * fr), (float)std::sin(2 * M_PI * fr));
        }
        hipLaunchKernelGGL(das_fn(P.fb, na, interp, P.tile.wide, P.tile.groups), dim3((unsigned)da.nwork),
                           dim3(threads), P.tile.wide ? 2 * (size_t)da.WB : 0, s, da);
        FQ_LAUNCH_CHECK();
    }
    return FQ_OK;
}

}  // namespace
}  // namespace fq

extern "C" int das_beamform(const fq_probe* probe, const fq_tx* tx, const fq_grid* grid, int32_t n_frames,
                            int32_t n_samples, const float* rf, int32_t interp, void* ws, size_t ws_bytes,
                            float* iq, void* stream) {
    FQ_REQUIRE(rf && iq, "rf and iq must not be NULL");
    DasPlan P;
    int st = das_prepare(probe, tx, grid, n_frames, n_samples, rf, interp, ws, ws_bytes, iq, P);
    if (st != FQ_OK) return st;
    hipStream_t s = as_stream(stream);
    const int per_launch = (int)std::min<size_t>(P.nfb, ws_bytes / P.bblk);
    for (int fb0 = 0; fb0 < P.nfb; fb0 += per_launch) {
        const int nb = std::min(per_launch, P.nfb - fb0);
        if ((st = launch_demod(P, fb0, nb, s)) != FQ_OK) return st;
        if ((st = launch_das(P, fb0, nb, interp, grid, probe->fs_hz, s)) != FQ_OK) return st;
    }
    return FQ_OK;
}

extern "C" int das_demodulate(const fq_probe* probe, const fq_tx* tx, int32_t n_frames, int32_t n_samples,
                              const float* rf, void* ws, size_t ws_bytes, void* stream) {
    FQ_REQUIRE(rf, "rf must not be NULL");
    fq_grid g{1, 1, 1, 0.0, 0.0, 1.0, 1e-4, 1e-4, 1e-4};
    DasPlan P;
    int st = das_prepare(probe, tx, &g, n_frames, n_samples, rf, 0, ws, ws_bytes, nullptr, P);
    if (st != FQ_OK) return st;
    if (ws_bytes < P.full) {
        set_error("das_demodulate needs the full workspace (%zu bytes)", P.full);
        return FQ_E_WORKSPACE;
    }
    return launch_demod(P, 0, P.nfb, as_stream(stream));
}

extern "C" int das_delay_sum(const fq_probe* probe, const fq_tx* tx, const fq_grid* grid, int32_t n_frames,
                             int32_t n_samples, int32_t interp, const void* ws, size_t ws_bytes, float* iq,
                             void* stream) {
    FQ_REQUIRE(iq, "iq must not be NULL");
    DasPlan P;
    int st = das_prepare(probe, tx, grid, n_frames, n_samples, nullptr, interp, const_cast<void*>(ws), ws_bytes, iq, P);
    if (st != FQ_OK) return st;
    if (ws_bytes < P.full) {
        set_error("das_delay_sum needs the full workspace (%zu bytes)", P.full);
        return FQ_E_WORKSPACE;
    }
    return launch_das(P, 0, P.nfb, interp, grid, probe->fs_hz, as_stream(stream));
}
