// sweep3.hip -- host side of the two-step D3Q27 sweep (kernels_sweep3.hpp): which
// domains take it, its geometry and launches.
#include <hip/hip_runtime.h>

#include <algorithm>

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
Sweep3Geom sweep3_geom(int64_t nx, int64_t ny, int64_t nz, size_t elem) {
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
    return best;
}

// Whether runs of a domain take two steps per launch (us per step, one step per
// launch against two: FP32 64^3 10.2 / 12.0, 80^3 19.2 / 18.0, 128^3 86 / 60, 256^3
// 630 / 435; FP64 64^3 17.6 / 15.9, 128^3 164 / 98, 256^3 1267 / 736).
bool sweep3_takes(const lbm_config *cfg, const Layout &L) {
    if (L.dim != 3 || L.zhalo || L.layout != LBM_LAYOUT_ROWS ||
        (cfg->dtype != LBM_FP64 && cfg->dtype != LBM_FP32_DEV))
        return false;
    // byte offsets inside a plane are 32-bit
    if (L.plane * (int64_t)L.elem >= ((int64_t)1 << 31))
        return false;
    return cfg->nx >= 16 && cfg->ny >= 4 && 2 * L.buf_bytes > kSweep3Bytes;
}

template <int DT, int EQ, bool CORR>
static void (*sweep3_w(int w))(Sweep3Args) {
    return w == 66 ? k_sweep3<DT, CORR, EQ, 66> : k_sweep3<DT, CORR, EQ, 34>;
}
template <int DT, int EQ>
static void (*sweep3_corr(bool corr, int w))(Sweep3Args) {
    return corr ? sweep3_w<DT, EQ, true>(w) : sweep3_w<DT, EQ, false>(w);
}
template <int DT>
static void (*sweep3_kernel(int eq, bool corr, int w))(Sweep3Args) {
    return eq == LBM_EQ_POLY2     ? sweep3_corr<DT, kEqPoly2>(corr, w)
           : eq == LBM_EQ_PRODUCT ? sweep3_corr<DT, kEqProduct>(corr, w)
                                  : sweep3_corr<DT, kEqEntropic>(corr, w);
}

int launch_sweep3(const Layout &L, const StepArgs &s, int dtype, bool corr, hipStream_t stream) {
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
    void (*fn)(Sweep3Args) = dtype == kF64 ? sweep3_kernel<kF64>(L.eq, corr, g.w)
                                           : sweep3_kernel<kDevF64>(L.eq, corr, g.w);
    const int64_t wgs = (int64_t)a.tiles_x * a.tiles_y * ((s.nz + g.planes - 1) / g.planes);
    const unsigned threads = (unsigned)((g.w * (g.rows + 2) + 63) / 64 * 64);
    hipLaunchKernelGGL(fn, dim3((unsigned)wgs), dim3(threads), 0, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return hip_fail(e, "sweep launch");
    return LBM_OK;
}

}  // namespace lbm
