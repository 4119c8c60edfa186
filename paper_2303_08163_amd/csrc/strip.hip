// strip.hip -- host side of the register-strip kernels (kernels_strip.hpp):
// which domains take them, their geometry and launches.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels_strip.hpp"
#include "kernels_t2.hpp"
#include "lbm_internal.hpp"

namespace lbm {

constexpr double kLaunchUs = 2.6;  // from one launch of a small kernel to the next

// Registers of k_strip2 and so the wavefronts a SIMD holds: FP32 storage takes
// 4 steps in at most 168 registers (three wavefronts), FP64 4 steps (three)
// or 6 (240 registers, two).
constexpr int strip2_occupancy(int dtype, int K) { return dtype == kF64 && K == 6 ? 2 : 3; }

// Own rows per wavefront of k_strip2: the row chunks with the least estimated
// time, and that time in us per launch.  A sweep over R own rows takes
// R + 2 K - 2 iterations, and an iteration with w wavefronts on every SIMD about
// 0.54 + 0.77 w us (1024^2, 4 steps: 1.32 us with one, 2.09 with two, 2.86 with
// three; one wavefront alone waits for its own results).  More chunks than fit
// at once run in rounds.
static int strip2_rows(int64_t nx, int64_t ny, int dtype, int K, double *us) {
    const int64_t own = 64 - 2 * (K - 1), strips = (nx + own - 1) / own;
    const int occ = strip2_occupancy(dtype, K);
    int64_t best_c = 1;
    double best = -1.0;
    for (int64_t c = 1; c <= std::max<int64_t>(1, ny / 4); c += 1 + c / 64) {
        const int64_t R = (ny + c - 1) / c, waves = strips * ((ny + R - 1) / R);
        const int64_t slots = 1024 * occ, full = waves / slots, rest = waves % slots;
        const double cost = (double)(R + 2 * K - 2) * ((double)full * (0.54 + 0.77 * occ) +
                                                       (rest ? 0.54 + 0.77 * (double)((rest + 1023) / 1024) : 0.0));
        if (best < 0.0 || cost < best) {
            best = cost;
            best_c = c;
        }
    }
    *us = kLaunchUs + best;
    return (int)((ny + best_c - 1) / best_c);
}

// Rows that the busiest SIMD of a k_block2 workgroup collides in K steps: the
// halo shrinks by a row on each side every step, wavefront w runs on SIMD w mod 4.
static int block2_rows(int K, int rpt, int waves, int own) {
    int sum = 0;
    for (int halo = K - 1; halo >= 0; --halo) {
        int rows[4] = {0, 0, 0, 0};
        for (int r = 0; r < waves * rpt; ++r)
            if (r - (K - 1) >= -halo && r - (K - 1) < own + halo)
                ++rows[r / rpt % 4];
        sum += std::max(std::max(rows[0], rows[1]), std::max(rows[2], rows[3]));
    }
    return sum;
}

// Tiling of k_block2 for K steps per launch: rows per wavefront and wavefronts
// with the least estimated time, and that time in us per launch.  Fitted to 182
// tilings of 64^2 to 512^2 that run in one round: 3.15 us, 0.115 for every step
// and 0.27 for every row that a SIMD collides, within 0.6 us; several workgroups
// per compute unit take 1.1 times their sum.
static Block2Geom block2_geom(int64_t nx, int64_t ny, int K, double *us) {
    Block2Geom g{};
    const int own = 64 - 2 * (K - 1);
    const int64_t tiles_x = (nx + own - 1) / own;
    *us = -1.0;
    for (int rpt : {1, 2})
        for (int waves = 4; waves <= block_waves(rpt); ++waves) {
            const int rows = waves * rpt - 2 * (K - 1);
            if (rows < 1)
                continue;
            const int64_t tiles_y = (ny + rows - 1) / rows, wgs = tiles_x * tiles_y, q = (wgs + 255) / 256;
            const int own_y = (int)((ny + tiles_y - 1) / tiles_y);
            const double t =
                3.15 + 0.115 * K + 0.27 * (q > 1 ? 1.1 * (double)q : 1.0) * block2_rows(K, rpt, waves, own_y);
            if (*us < 0.0 || t < *us - 1e-9 || (t < *us + 1e-9 && wgs < (int64_t)g.tiles_x * g.tiles_y)) {
                *us = t;
                g.rpt = rpt;
                g.waves = waves;
                g.tiles_x = (int)tiles_x;
                g.tiles_y = (int)tiles_y;
            }
        }
    g.own_x = (int)((nx + g.tiles_x - 1) / g.tiles_x);
    g.own_y = (int)((ny + g.tiles_y - 1) / g.tiles_y);
    return g;
}

// One step per launch, us: the launch, and one read and one write of both
// buffers (row padding included) at the rate measured within and beyond the
// last-level cache (24 shapes from 1 x 3000 to 12 million nodes, within 25 % for rows of
// 8 nodes and more; shorter rows run slower than this).
static double one_step2_us(const Layout &L) {
    const double bytes = 2.0 * (double)L.buf_bytes, launch = L.elem == 4 ? 2.65 : 2.8;
    const double rate = bytes > (double)(256 << 20) ? 5.85e6 : L.elem == 4 ? 6.8e6 : 8.0e6;  // bytes per us
    return launch + bytes / rate;
}

// Which form the runs of a D2Q9 domain take: strips of 4 steps per launch (FP32)
// or 6 and 4 (FP64), blocks of 5 or 4, by the estimated time per step, or neither.
// FP32 strips are bound by the FP64 arithmetic at 4 steps already (4096^2, us
// per step: 3 steps 101.5, 4 steps 89.6, 6 steps 98.4 with one wavefront per
// SIMD less); FP64 by HBM until 6 (4 steps 131.8, 5 112.6, 6 96.6, 8 118.6 with
// one wavefront per SIMD).  Blocks are best with 5 steps (us per step, FP64 3 / 4 / 5 /
// 6 / 8 steps: 64^2 - / 1.25 / 1.13 / 1.23 / 1.22, 300^2 1.95 / 1.87 / 1.65 / 1.94 /
// 1.83), FP32 with several per compute unit 4 (512^2 3.35, 5 steps 3.43).  They win
// below about 700^2 (us per step, FP64 blocks / strips: 512^2 3.2 / 4.2, 700 x 600 3.9 /
// 5.1; 1024^2 with four steps 9.2 / 8.3).
// Both spend 64 lanes a row and collide halo rows again, so narrow and flat domains
// run sooner with time_block steps per launch (us per step, strip or block / one: FP32
// 8 x 375,000 98 / 32, 16 x 187,500 50 / 31, 24 x 125,000 35 / 44, 16 x 18,750 7.9 / 5.5,
// 24 x 12,500 5.6 / 6.3, 3,000,000 x 1 52 / 33, 600,000 x 5 26 / 33; FP64 4 x 750,000 162 /
// 102, 12 x 250,000 57 / 85, 8 x 37,500 11.1 / 8.3, 16 x 18,750 6.8 / 8.0).  The FP64
// estimates run low there, blocks by up to 1.5, strips by up to 1.25: hence `low`.
void plan2(const lbm_config *cfg, Layout &L) {
    if (L.dim != 2 || L.layout != LBM_LAYOUT_ROWS || (cfg->dtype != LBM_FP64 && cfg->dtype != LBM_FP32_DEV))
        return;
    if (cfg->nx > (1 << 28))  // byte offsets inside a row are 32-bit
        return;
    const bool six = cfg->dtype == LBM_FP64;
    double us4, us6, usb;
    L.strip_rows[0] = strip2_rows(cfg->nx, cfg->ny, cfg->dtype, 4, &us4);
    if (six)
        L.strip_rows[1] = strip2_rows(cfg->nx, cfg->ny, cfg->dtype, 6, &us6);
    const double strips = six ? us6 / 6 : us4 / 4;
    int K = 5;
    Block2Geom g = block2_geom(cfg->nx, cfg->ny, K, &usb);
    if (!six && (int64_t)g.tiles_x * g.tiles_y > 256)
        g = block2_geom(cfg->nx, cfg->ny, K = 4, &usb);
    const bool blocks = L.tblock == 1 && usb / K < strips;
    const double low = !six ? 1.0 : blocks ? 1.3 : 1.2;
    if (low * (blocks ? usb / K : strips) >= one_step2_us(L))
        return;
    if (blocks)
        L.block2 = g;
    L.deep = blocks ? K : six ? 6 : 4;
}

template <int DT, int K, int EQ, bool BACK>
static void (*strip2_corr(bool corr))(StripArgs) {
    constexpr int W = strip2_occupancy(DT, K);
    return corr ? k_strip2<DT, true, EQ, K, W, BACK> : k_strip2<DT, false, EQ, K, W, BACK>;
}
template <int DT, int K, bool BACK>
static void (*strip2_eq(int eq, bool corr))(StripArgs) {
    return eq == LBM_EQ_POLY2     ? strip2_corr<DT, K, kEqPoly2, BACK>(corr)
           : eq == LBM_EQ_PRODUCT ? strip2_corr<DT, K, kEqProduct, BACK>(corr)
                                  : strip2_corr<DT, K, kEqEntropic, BACK>(corr);
}
template <int DT, int K>
static void (*strip2_kernel(int eq, bool corr, bool back))(StripArgs) {
    return back ? strip2_eq<DT, K, true>(eq, corr) : strip2_eq<DT, K, false>(eq, corr);
}

int launch_strip2(const Layout &L, const StepArgs &s, int dtype, bool corr, int K, bool back, hipStream_t stream) {
    StripArgs a{};
    a.src = s.src;
    a.dst = s.dst;
    a.nx = s.nx;
    a.ny = s.ny;
    a.K = K;
    a.h = K - 1;
    a.tx = 64 - 2 * a.h;
    a.strips = (s.nx + a.tx - 1) / a.tx;
    a.rows = L.strip_rows[K == 6];
    a.chunks = (s.ny + a.rows - 1) / a.rows;
    a.ps = L.ps;
    a.rs = L.rs;
    a.relax = s.relax;
    a.flag = s.flag;
    void (*fn)(StripArgs) = dtype == kF64 ? (K == 6 ? strip2_kernel<kF64, 6>(L.eq, corr, back)
                                                    : strip2_kernel<kF64, 4>(L.eq, corr, back))
                                          : strip2_kernel<kDevF64, 4>(L.eq, corr, back);
    const int64_t waves = (int64_t)a.strips * a.chunks;
    constexpr int per_wg = kStripThreads / 64;
    hipLaunchKernelGGL(fn, dim3((unsigned)((waves + per_wg - 1) / per_wg)), dim3(kStripThreads), 0, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return hip_fail(e, "strip launch");
    return LBM_OK;
}

template <int DT, int EQ, int RPT>
static void (*block2_corr(bool corr))(BlockArgs) {
    return corr ? k_block2<DT, true, EQ, RPT> : k_block2<DT, false, EQ, RPT>;
}
template <int DT, int RPT>
static void (*block2_kernel(int eq, bool corr))(BlockArgs) {
    return eq == LBM_EQ_POLY2     ? block2_corr<DT, kEqPoly2, RPT>(corr)
           : eq == LBM_EQ_PRODUCT ? block2_corr<DT, kEqProduct, RPT>(corr)
                                  : block2_corr<DT, kEqEntropic, RPT>(corr);
}

// K <= L.deep steps (fewer leave more halo than they need).
int launch_block2(const Layout &L, const StepArgs &s, int dtype, bool corr, int K, hipStream_t stream) {
    const Block2Geom &g = L.block2;
    const BlockArgs a{s.src, s.dst, s.nx, s.ny, K, g.own_x, g.own_y, g.tiles_x, L.ps, L.rs, s.relax, s.flag};
    void (*fn)(BlockArgs) = dtype == kF64 ? (g.rpt == 1 ? block2_kernel<kF64, 1>(L.eq, corr)
                                                        : block2_kernel<kF64, 2>(L.eq, corr))
                                          : (g.rpt == 1 ? block2_kernel<kDevF64, 1>(L.eq, corr)
                                                        : block2_kernel<kDevF64, 2>(L.eq, corr));
    hipLaunchKernelGGL(fn, dim3((unsigned)((int64_t)g.tiles_x * g.tiles_y)), dim3(64u * (unsigned)g.waves), 0, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return hip_fail(e, "block launch");
    return LBM_OK;
}

// D1Q3.  Many columns per lane leave little halo, few keep short rows spread
// over the chip (K = 8 with the correction, us per launch: 2^20 nodes FP32 2
// columns 24.5, 4 24.7, 8 29.2; 2^27 FP32 2580, 2377, 2314; FP64 4 columns
// 2516, 8 2667).
template <int DT, int EQ, int NC, bool NT>
static void (*strip1_corr(bool corr))(StripArgs) {
    return corr ? k_strip1<DT, true, EQ, NC, NT> : k_strip1<DT, false, EQ, NC, NT>;
}
template <int DT, int EQ>
static void (*strip1_nc(bool corr, bool wide, bool nt))(StripArgs) {
    constexpr int NC = DT == kF64 ? 4 : 8;
    if (!wide)  // (short rows fit the caches, and full lines gain nothing: plain stores)
        return strip1_corr<DT, EQ, 2, false>(corr);
    return nt ? strip1_corr<DT, EQ, NC, true>(corr) : strip1_corr<DT, EQ, NC, false>(corr);
}
template <int DT>
static void (*strip1_kernel(int eq, bool corr, bool wide, bool nt))(StripArgs) {
    return eq == LBM_EQ_POLY2     ? strip1_nc<DT, kEqPoly2>(corr, wide, nt)
           : eq == LBM_EQ_PRODUCT ? strip1_nc<DT, kEqProduct>(corr, wide, nt)
                                  : strip1_nc<DT, kEqEntropic>(corr, wide, nt);
}

// Launches of few steps on doubles are bound by their bytes.  Two or three steps: lanes
// of two columns, whose stores fill whole lines, beat four (us per launch of two steps
// with the correction, four columns / two: 2^27 nodes 1657 / 1168, 2^24 211 / 148, 2^22
// 31.9 / 30.4).
static bool strip1_wide(int64_t nx, int dtype, int K) { return nx >= kStrip1Wide && !(dtype == kF64 && K < 4); }
static int strip1_halo(int K) { return (K + 7) / 8 * 8; }

// Columns a wavefront owns with K steps per launch.
int strip1_cols(int64_t nx, int dtype, int K) {
    return 64 * (strip1_wide(nx, dtype, K) ? (dtype == kF64 ? 4 : 8) : 2) - 2 * strip1_halo(K);
}

// Most steps per launch of a run: long rows 8 (with more the halo's share grows
// and the arithmetic is what bounds them), short rows, bound by the launch and
// the latency of a step, 16 to 32: as long as a SIMD holds at most two of the
// wavefronts of 64 own columns, 32 (us per step FP64, 16 / 24 / 32 / 40 steps: 3000 nodes
// 0.34 / 0.29 / 0.27 / 0.27, 100,000 0.48 / 0.44 / 0.42 / 0.58, 200,000 0.65 / 0.61 / 0.75,
// 400,000 1.00 / 0.93 / 1.19, 2^20 1.95 / 2.18 / 2.56; FP32 alike).
int strip1_steps(int64_t nx) {
    return nx >= kStrip1Wide ? 8 : nx > 400000 ? 16 : nx > 2 * 1024 * 64 ? 24 : 32;
}

int launch_strip1(const Layout &L, const StepArgs &s, int dtype, bool corr, int K, hipStream_t stream) {
    StripArgs a{};
    a.src = s.src;
    a.dst = s.dst;
    a.nx = s.nx;
    a.ny = 1;
    a.K = K;
    a.h = strip1_halo(K);
    a.tx = strip1_cols(s.nx, dtype, K);
    a.rows = a.chunks = 1;
    a.strips = (int)((s.nx + (int64_t)a.tx - 1) / a.tx);
    a.ps = L.ps;
    a.rs = L.rs;
    a.relax = s.relax;
    a.flag = s.flag;
    // (a lane's four doubles go in two stores, each of half lines, which non-temporal stores
    // do not join: four steps 1656 us with them, 1310 without; eight 2188 and 2204)
    const bool wide = strip1_wide(s.nx, dtype, K), nt = t2_nt_stores(L.buf_bytes) && !(dtype == kF64 && K < 8);
    void (*fn)(StripArgs) = dtype == kF64 ? strip1_kernel<kF64>(L.eq, corr, wide, nt)
                                          : strip1_kernel<kDevF64>(L.eq, corr, wide, nt);
    constexpr int per_wg = kStripThreads / 64;
    hipLaunchKernelGGL(fn, dim3((unsigned)((a.strips + per_wg - 1) / per_wg)), dim3(kStripThreads), 0, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return hip_fail(e, "strip launch");
    return LBM_OK;
}

// D1Q3 rows in one workgroup.
template <int DT, bool CORR, int EQ>
static void (*row1_kernel(bool one, bool energy))(RowArgs) {
    return one ? (energy ? k_row1<DT, CORR, EQ, true, true> : k_row1<DT, CORR, EQ, true, false>)
               : (energy ? k_row1<DT, CORR, EQ, false, true> : k_row1<DT, CORR, EQ, false, false>);
}
template <int DT, bool CORR>
static void (*row1_eq(int eq, bool one, bool energy))(RowArgs) {
    return eq == LBM_EQ_POLY2     ? row1_kernel<DT, CORR, kEqPoly2>(one, energy)
           : eq == LBM_EQ_PRODUCT ? row1_kernel<DT, CORR, kEqProduct>(one, energy)
                                  : row1_kernel<DT, CORR, kEqEntropic>(one, energy);
}

// One compute unit against the strips' whole chip: a row up to one wavefront per
// SIMD is bound by the latency of a step either way and spares the launches,
// beyond two the unit's arithmetic is slower.  us per step of a long run with
// the correction, strips and row: FP64 64 nodes 0.33 and 0.19, 256 0.33 and 0.25, 512
// 0.34 and 0.37, 1024 0.34 and 0.60.
int row1_plan(int64_t nx) { return nx <= 256 ? 1 : nx <= kRowMax ? 2 : 0; }

// A history also spares the energy's launch, which longer rows pay back for a few
// steps between readings (us per reading, strips and row: FP64 512 nodes every 32
// steps 14.1 and 12.6, every 64 24.8 and 24.8; 768 every 20 10.9 and 10.4, every 24 12.0
// and 12.4; 1024 every 10 8.3 and 6.6, every 16 9.9 and 10.3).
bool row1_history(int64_t nx, int64_t every) {
    return every <= kRowSteps &&
           (row1_plan(nx) == 1 || (row1_plan(nx) == 2 && (nx <= 512 ? every <= 64 : every * nx <= 15 * 1024)));
}

int launch_row1(const Layout &L, const StepArgs &s, int dtype, bool corr, int steps, const RowEnergy *e,
                hipStream_t stream) {
    RowArgs a{};
    a.src = s.src;
    a.dst = s.dst;
    a.nx = s.nx;
    a.steps = steps;
    a.ps = L.ps;
    a.relax = s.relax;
    a.flag = s.flag;
    a.rho_ref = 1.0;
    if (e) {
        a.every = e->every;
        a.first = e->first;
        a.out = e->out;
        a.rho_ref = e->rho_ref;
        a.U[0] = e->U;
    }
    const int waves = (s.nx + 63) / 64;
    const bool one = waves == 1;
    void (*fn)(RowArgs) = dtype == kF64 ? (corr ? row1_eq<kF64, true>(L.eq, one, e) : row1_eq<kF64, false>(L.eq, one, e))
                                        : (corr ? row1_eq<kDevF64, true>(L.eq, one, e)
                                                : row1_eq<kDevF64, false>(L.eq, one, e));
    hipLaunchKernelGGL(fn, dim3(1), dim3(64u * (unsigned)waves), 0, stream, a);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess)
        return hip_fail(err, "row launch");
    return LBM_OK;
}

}  // namespace lbm
