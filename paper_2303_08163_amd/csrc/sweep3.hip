// sweep3.hip -- host side of the two-step D3Q27 sweeps and blocks
// (kernels_sweep3.hpp): which domains take them, their geometry and launches.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "kernels_sweep3.hpp"
#include "lbm_internal.hpp"

namespace lbm {

// Tiles of 64 or 32 own columns (whole 128-byte lines, so that no line is
// written in two parts: 150 x 131 x 120 FP64 with 32 own columns 281 us per
// launch, with 30 316), the own rows and planes of a workgroup by the least
// estimated time.  A sweep takes planes + 2 iterations of about T0 + T1 own us
// (own = own nodes per plane; FP32 64 x 7 own 5.5, 64 x 8 6.5, 64 x 9 6.9, 32 x 13
// 5.6, 32 x 16 7.0, 32 x 19 7.4; FP64 64 x 4 5.8, 64 x 5 7.2, 32 x 8 6.3, 32 x 13
// 9.5), one workgroup to each of the 256 compute units.  Fewer of them hardly
// speed an iteration up, and in a single round the workgroups stay together,
// so that neighbours find their halo in L2: one full round of long sweeps
// wins (256^3, us per step: FP32 64 x 8 x 128 planes, 256 workgroups, 433; 64 x 9 x
// 128, 232, 485; 64 x 9 x 24, 1276, 457; FP64 64 x 4 x 256, 256, 742; 32 x 13 x 32,
// 1280, 810; 32 x 13 x 256, 160, 1023).
static Sweep3Geom sweep3_geom(int64_t nx, int64_t ny, int64_t nz, size_t elem, double *us) {
    Sweep3Geom best{};
    double best_cost = -1.0;
    const double T1 = elem == 4 ? 0.0102 : 0.0203;
    for (int W : {66, 34}) {
        const double T0 = elem == 4 ? (W == 66 ? 1.3 : 1.8) : (W == 66 ? 0.8 : 1.0);
        const int64_t tiles_x = (nx + W - 3) / (W - 2);
        int64_t last_ty = 0;
        for (int oy = sweep3_columns(elem) / W - 2; oy >= 1; --oy) {
            const int64_t tiles_y = (ny + oy - 1) / oy;
            if (tiles_y == last_ty)
                continue;  // more rows a tile, the same tiles
            last_ty = tiles_y;
            const int64_t rows = (ny + tiles_y - 1) / tiles_y;
            const double it = T0 + T1 * (double)(W - 2) * (double)rows;
            // every chunk count c once, with the fewest planes that give it
            for (int64_t most = nz, planes; most >= 1; most = planes - 1) {
                const int64_t c = (nz + most - 1) / most;
                planes = (nz + c - 1) / c;
                const int64_t wgs = tiles_x * tiles_y * c, rest = wgs % 256;
                const double rounds =
                    (double)(wgs / 256) + (rest ? 0.8 + 0.2 * (double)rest / 256.0 : 0.0);
                const double cost = (double)(planes + 2) * it * rounds * (wgs > 256 ? 1.03 : 1.0);
                if (best_cost < 0.0 || cost < best_cost) {
                    best_cost = cost;
                    best.w = W;
                    best.rows = (int)rows;
                    best.planes = (int)planes;
                }
            }
        }
    }
    *us = best_cost;
    return best;
}

// One step per launch, us.  Within the last-level cache: the launch, the stored
// nodes (row padding included), and the wavefronts of a SIMD, lanes outside the
// domain and vector lanes counted.  Beyond it, and for the vector kernel, whose
// accesses pass the cache by: one read and one write at 5.3 bytes per ns.  (110
// domains from 64 x 40 x 100 to 130 x 256^2: within 8 %, rows of 256 nodes and more
// up to 1.3 times slower.)
static double one_step3_us(const lbm_config *cfg, const Layout &L) {
    const double bytes = 2.0 * (double)L.buf_bytes, stored = (double)L.buf_bytes / (27.0 * (double)L.elem);
    if (L.npt > 1 || bytes > (double)(256 << 20))
        return bytes / 5.3e6;
    const int64_t tiles =
        (cfg->nx + L.block_x - 1) / L.block_x * ((cfg->ny + L.block_y - 1) / L.block_y) * cfg->nz;
    const double waves = std::ceil((double)(tiles * (L.block_x * L.block_y / 64)) / 1024.0);
    return L.elem == 4 ? 2.85 + 0.0175e-3 * stored + 0.69 * waves : 3.11 + 0.040e-3 * stored + 0.80 * waves;
}

// Whether sweeps of this geometry (and estimate, us per launch) beat one step per launch.
// The estimate holds for full tiles and many planes; the first two of a sweep's
// planes + 2 iterations take no second step, and neither do the lanes outside the
// domain: both taken into account, it is within 15 % of 136 domains of 16 x 128 x 128
// to 150 x 256^2 nodes.  us per step, sweeps / one step: FP32 16 x 4 x 25,000 129 / 74,
// 16 x 8 x 12,500 95 / 76, 16 x 256^2 43 / 34, 1000^2 x 1 45 / 32, 600^2 x 2 28 / 24,
// 128 x 64^2 18.2 / 17.2, 33 x 128^2 22 / 27, 20 x 256^2 65 / 86; FP64 16 x 4 x 25,000
// 140 / 129, 35 x 86 x 57 18.7 / 16.2, 16 x 256^2 70 / 88, 64^3 15.7 / 17.5.
static bool sweep3_pays(const lbm_config *cfg, const Layout &L, const Sweep3Geom &g, double us) {
    const int64_t own_x = (cfg->nx + g.w - 3) / (g.w - 2) * (g.w - 2),
                  own_y = (cfg->ny + g.rows - 1) / g.rows * g.rows;
    const double used = (double)cfg->nx / (double)own_x * ((double)cfg->ny / (double)own_y);
    const double step = us / 2 * (g.planes + 0.7) / (g.planes + 2) * (0.5 + 0.5 * used);
    return step < 0.965 * one_step3_us(cfg, L);
}

// Block of k_block3 with the least estimated time, and that time in us per
// launch: a fixed part, a part for each round of workgroups that share the
// compute units, and for each workgroup of a compute unit its wavefronts in
// step 1 and step 2 and the 128-byte lines of its row runs.  (Fitted to 20^3 ..
// 56^3; the block it picks is within 7 % of the best one measured there: 32^3
// FP32 16 x 2 x 4 own 6.8, 48^3 FP32 12 x 6 x 6 11.8, 48^3 FP64 16 x 4 x 4 16.2.)
static Block3Geom block3_geom(int64_t nx, int64_t ny, int64_t nz, size_t elem, double *us) {
    const bool f32 = elem == 4;
    const double fixed = f32 ? 3.2 : 2.4, per_round = f32 ? 1.3 : 1.95, wave1 = 0.145, wave2 = f32 ? 0.40 : 0.575,
                 line = 0.0205;
    Block3Geom best{};
    *us = -1.0;
    for (int ox : {8, 12, 16, 20, 24, 32, 48})
        for (int oy = 1; oy <= 12; ++oy)
            for (int oz = 1; oz <= 12; ++oz) {
                const int threads = ((ox + 2) * (oy + 2) * (oz + 2) + 63) / 64 * 64;
                if (threads > block3_threads(elem) || oy > ny || oz > nz)
                    continue;
                const int64_t wgs = ((nx + ox - 1) / ox) * ((ny + oy - 1) / oy) * ((nz + oz - 1) / oz);
                const double rounds = (double)((wgs + 255) / 256);
                const int share = std::max(1, std::min((int)(163840 / block3_lds_bytes(threads, elem)),
                                                       (f32 ? 2048 : 1280) / threads));
                const double lines = (double)((oy + 2) * (oz + 2) * ((ox + 10 + 31) / 32));
                const double t = fixed + per_round * std::ceil(rounds / share) +
                                 rounds * (wave1 * (threads / 64) + wave2 * ((ox * oy * oz + 63) / 64) + line * lines);
                if (*us < 0.0 || t < *us) {
                    *us = t;
                    best = Block3Geom{ox, oy, oz, threads};
                }
            }
    return best;
}

// Which form the runs of a D3Q27 domain take: sweeps, blocks (small domains), or
// one step per launch.  us per step, one step per launch against sweeps: FP32 64^3
// 10.2 / 12.0, 80^3 19.2 / 18.0, 128^3 86 / 60, 256^3 630 / 435; FP64 64^3 17.6 /
// 15.9, 128^3 164 / 98, 256^3 1267 / 736.
void plan3(const lbm_config *cfg, Layout &L) {
    if (L.dim != 3 || L.zhalo || L.layout != LBM_LAYOUT_ROWS ||
        (cfg->dtype != LBM_FP64 && cfg->dtype != LBM_FP32_DEV))
        return;
    // byte offsets inside a plane (a block: inside the buffer) are 32-bit
    double us;
    if (2 * L.buf_bytes > kSweep3Bytes && cfg->nx >= 16 && cfg->ny >= 4 &&
        L.plane * (int64_t)L.elem < ((int64_t)1 << 31)) {
        const Sweep3Geom g = sweep3_geom(cfg->nx, cfg->ny, cfg->nz, L.elem, &us);
        if (sweep3_pays(cfg, L, g, us)) {
            L.sweep3 = g;
            L.deep = 2;
        }
    } else if (L.n <= kBlock3Nodes) {
        // one step per launch took about (us) 3.2 + 0.034 n / 1000 with FP32 storage,
        // 4.0 + 0.056 n / 1000 with FP64 (16^3 3.7 / 4.2, 40^3 5.5 / 7.5, 56^3 9.2 / 14.5)
        double one = L.elem == 4 ? 3.2 + 0.034e-3 * (double)L.n : 4.0 + 0.056e-3 * (double)L.n;
        // That is high for FP32 rows that fill their padding and their wavefronts: of 2700
        // ragged domains of up to 200,000 nodes that took blocks by it, 69 ran up to 1.24
        // times slower than with one step per launch (us per step, blocks / one:
        // 147 x 5 x 40 4.6 / 3.7, 108 x 23 x 19 5.2 / 4.3, 111 x 20 x 22 5.0 / 4.3; 48^3 5.9 /
        // 6.9).  By the lower of the two estimates 22 do, at most 1.12 times.  (The vector
        // kernel is the slower one there: 256 x 16^2 4.9 / 7.3.)
        if (L.elem == 4 && L.npt == 1)
            one = std::min(one, one_step3_us(cfg, L));
        const Block3Geom g = block3_geom(cfg->nx, cfg->ny, cfg->nz, L.elem, &us);
        if (us > 0.0 && us / 2 < 0.86 * one) {  // (the estimate runs up to 15 % low)
            L.block3 = g;
            L.deep = 2;
        }
    }
}

template <int DT, int EQ, bool CORR>
static void (*sweep3_w(int w, bool back))(Sweep3Args) {
    return back ? (w == 66 ? k_sweep3<DT, CORR, EQ, 66, true> : k_sweep3<DT, CORR, EQ, 34, true>)
                : (w == 66 ? k_sweep3<DT, CORR, EQ, 66, false> : k_sweep3<DT, CORR, EQ, 34, false>);
}
template <int DT, int EQ>
static void (*sweep3_corr(bool corr, int w, bool back))(Sweep3Args) {
    return corr ? sweep3_w<DT, EQ, true>(w, back) : sweep3_w<DT, EQ, false>(w, back);
}
template <int DT>
static void (*sweep3_kernel(int eq, bool corr, int w, bool back))(Sweep3Args) {
    return eq == LBM_EQ_POLY2     ? sweep3_corr<DT, kEqPoly2>(corr, w, back)
           : eq == LBM_EQ_PRODUCT ? sweep3_corr<DT, kEqProduct>(corr, w, back)
                                  : sweep3_corr<DT, kEqEntropic>(corr, w, back);
}

int launch_sweep3(const Layout &L, const StepArgs &s, int dtype, bool corr, bool back, hipStream_t stream) {
    const Sweep3Geom &g = L.sweep3;
    Sweep3Args a{};
    a.src = s.src;
    a.dst = s.dst;
    a.nx = s.nx;
    a.ny = s.ny;
    a.nz = s.nz;
    a.own_y = g.rows;
    a.planes = g.planes;
    a.tiles_x = (s.nx + g.w - 3) / (g.w - 2);
    a.tiles_y = (s.ny + g.rows - 1) / g.rows;
    a.ps = L.ps;
    a.rs = L.rs;
    a.relax = s.relax;
    a.flag = s.flag;
    void (*fn)(Sweep3Args) = dtype == kF64 ? sweep3_kernel<kF64>(L.eq, corr, g.w, back)
                                           : sweep3_kernel<kDevF64>(L.eq, corr, g.w, back);
    const int64_t wgs = (int64_t)a.tiles_x * a.tiles_y * ((s.nz + g.planes - 1) / g.planes);
    const unsigned threads = (unsigned)((g.w * (g.rows + 2) + 63) / 64 * 64);
    hipLaunchKernelGGL(fn, dim3((unsigned)wgs), dim3(threads), 0, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return hip_fail(e, "sweep launch");
    return LBM_OK;
}

template <int DT>
static void (*block3_kernel(int eq, bool corr))(Block3Args) {
    switch (eq) {
    case LBM_EQ_POLY2:
        return corr ? k_block3<DT, true, kEqPoly2> : k_block3<DT, false, kEqPoly2>;
    case LBM_EQ_PRODUCT:
        return corr ? k_block3<DT, true, kEqProduct> : k_block3<DT, false, kEqProduct>;
    default:
        return corr ? k_block3<DT, true, kEqEntropic> : k_block3<DT, false, kEqEntropic>;
    }
}

int launch_block3(const Layout &L, const StepArgs &s, int dtype, bool corr, hipStream_t stream) {
    const Block3Geom &g = L.block3;
    const int tx = (s.nx + g.own_x - 1) / g.own_x, ty = (s.ny + g.own_y - 1) / g.own_y,
              tz = (s.nz + g.own_z - 1) / g.own_z;
    const Block3Args a{s.src, s.dst, s.nx, s.ny, s.nz, g.own_x, g.own_y, g.own_z, tx, ty, L.ps, L.rs, s.relax, s.flag};
    void (*fn)(Block3Args) = dtype == kF64 ? block3_kernel<kF64>(L.eq, corr) : block3_kernel<kDevF64>(L.eq, corr);
    hipLaunchKernelGGL(fn, dim3((unsigned)(tx * ty * tz)), dim3((unsigned)g.threads),
                       (unsigned)block3_lds_bytes(g.threads, L.elem), stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return hip_fail(e, "block launch");
    return LBM_OK;
}

}  // namespace lbm
