// strip.hip -- host side of the register-strip kernels (kernels_strip.hpp):
// which domains take them, their geometry and launches.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "kernels_strip.hpp"
#include "kernels_t2.hpp"
#include "lbm_internal.hpp"

namespace lbm {

// Registers of k_strip2 and so the wavefronts a SIMD holds: FP32 storage takes
// 4 steps in at most 168 registers (three wavefronts), FP64 4 steps (three)
// or 6 (240 registers, two).
constexpr int strip2_occupancy(int dtype, int K) { return dtype == kF64 && K == 6 ? 2 : 3; }

// D2Q9: steps per launch of the longest strip launch, 0 for none.  FP32
// storage is bound by the FP64 arithmetic at 4 steps already (4096^2, us per
// step: 3 steps 101.5, 4 steps 89.6, 6 steps 98.4 with one wavefront per SIMD
// less); FP64 storage by HBM until 6 (4 steps 131.8, 5 112.6, 6 96.6, 8 118.6
// with one wavefront per SIMD).
int strip2_steps(const lbm_config *cfg, const Layout &L) {
    if (L.dim != 2 || L.layout != LBM_LAYOUT_ROWS || (cfg->dtype != LBM_FP64 && cfg->dtype != LBM_FP32_DEV))
        return 0;
    // byte offsets inside a row are 32-bit; below 64 nodes most columns of a wavefront are copies
    if (cfg->nx < 64 || cfg->nx > (1 << 28) || L.n < kStrip2Nodes)
        return 0;
    return cfg->dtype == LBM_FP64 ? 6 : 4;
}

// Own rows per wavefront of k_strip2: the row chunks with the least estimated
// time.  A sweep
// over R own rows takes R + 2 K - 2 iterations, and an iteration with w
// wavefronts on every SIMD about 0.7 + w units (1024^2, 4 steps: 1.32 us with
// one, 2.09 with two, 2.86 with three; one wavefront alone waits for its own
// results).  More chunks than fit at once run in rounds.
int strip2_rows(int64_t nx, int64_t ny, int dtype, int K) {
    const int64_t strips = (nx + 63 - 2 * K) / (64 - 2 * K);
    const int occ = strip2_occupancy(dtype, K);
    int64_t best_c = 1;
    double best = -1.0;
    for (int64_t c = 1; c <= std::max<int64_t>(1, ny / 4); c += 1 + c / 64) {
        const int64_t R = (ny + c - 1) / c, waves = strips * ((ny + R - 1) / R);
        const int64_t slots = 1024 * occ, full = waves / slots, rest = waves % slots;
        const double cost =
            (double)(R + 2 * K - 2) * ((double)full * (0.7 + occ) + (rest ? 0.7 + (double)((rest + 1023) / 1024) : 0.0));
        if (best < 0.0 || cost < best) {
            best = cost;
            best_c = c;
        }
    }
    return (int)((ny + best_c - 1) / best_c);
}

template <int DT, int K, int EQ, bool NT>
static void (*strip2_corr(bool corr))(StripArgs) {
    constexpr int W = strip2_occupancy(DT, K);
    return corr ? k_strip2<DT, true, EQ, K, 1, NT, W> : k_strip2<DT, false, EQ, K, 1, NT, W>;
}
template <int DT, int K>
static void (*strip2_kernel(int eq, bool corr, bool nt))(StripArgs) {
    switch (eq) {
    case LBM_EQ_POLY2:
        return nt ? strip2_corr<DT, K, kEqPoly2, true>(corr) : strip2_corr<DT, K, kEqPoly2, false>(corr);
    case LBM_EQ_PRODUCT:
        return nt ? strip2_corr<DT, K, kEqProduct, true>(corr) : strip2_corr<DT, K, kEqProduct, false>(corr);
    default:
        return nt ? strip2_corr<DT, K, kEqEntropic, true>(corr) : strip2_corr<DT, K, kEqEntropic, false>(corr);
    }
}

int launch_strip2(const Layout &L, const StepArgs &s, int dtype, bool corr, int K, hipStream_t stream) {
    StripArgs a{};
    a.src = s.src;
    a.dst = s.dst;
    a.nx = s.nx;
    a.ny = s.ny;
    a.K = K;
    a.h = K;
    a.tx = 64 - 2 * K;
    a.strips = (s.nx + a.tx - 1) / a.tx;
    a.rows = L.strip_rows[K == 6];
    a.chunks = (s.ny + a.rows - 1) / a.rows;
    a.ps = L.ps;
    a.rs = L.rs;
    a.relax = s.relax;
    a.flag = s.flag;
    const bool nt = t2_nt_stores(L.buf_bytes);
    void (*fn)(StripArgs) = dtype == kF64 ? (K == 6 ? strip2_kernel<kF64, 6>(L.eq, corr, nt)
                                                    : strip2_kernel<kF64, 4>(L.eq, corr, nt))
                                          : strip2_kernel<kDevF64, 4>(L.eq, corr, nt);
    const int64_t waves = (int64_t)a.strips * a.chunks;
    constexpr int per_wg = kStripThreads / 64;
    hipLaunchKernelGGL(fn, dim3((unsigned)((waves + per_wg - 1) / per_wg)), dim3(kStripThreads), 0, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return hip_fail(e, "strip launch");
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
    if (!wide)  // (short rows fit the caches: plain stores)
        return strip1_corr<DT, EQ, 2, false>(corr);
    return nt ? strip1_corr<DT, EQ, NC, true>(corr) : strip1_corr<DT, EQ, NC, false>(corr);
}
template <int DT>
static void (*strip1_kernel(int eq, bool corr, bool wide, bool nt))(StripArgs) {
    return eq == LBM_EQ_POLY2     ? strip1_nc<DT, kEqPoly2>(corr, wide, nt)
           : eq == LBM_EQ_PRODUCT ? strip1_nc<DT, kEqProduct>(corr, wide, nt)
                                  : strip1_nc<DT, kEqEntropic>(corr, wide, nt);
}

static bool strip1_wide(int64_t nx) { return nx >= kStrip1Wide; }
static int strip1_halo(int K) { return (K + 7) / 8 * 8; }

// Columns a wavefront owns with K steps per launch.
int strip1_cols(int64_t nx, int dtype, int K) {
    return 64 * (strip1_wide(nx) ? (dtype == kF64 ? 4 : 8) : 2) - 2 * strip1_halo(K);
}

// Most steps per launch of a run: long rows 8 (with more the halo's share grows
// and the arithmetic is what bounds them), short rows, bound by the launch and
// the latency of a step, 16.
int strip1_steps(int64_t nx) { return strip1_wide(nx) ? 8 : 16; }

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
    const bool wide = strip1_wide(s.nx), nt = t2_nt_stores(L.buf_bytes);
    void (*fn)(StripArgs) = dtype == kF64 ? strip1_kernel<kF64>(L.eq, corr, wide, nt)
                                          : strip1_kernel<kDevF64>(L.eq, corr, wide, nt);
    constexpr int per_wg = kStripThreads / 64;
    hipLaunchKernelGGL(fn, dim3((unsigned)((a.strips + per_wg - 1) / per_wg)), dim3(kStripThreads), 0, stream, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return hip_fail(e, "strip launch");
    return LBM_OK;
}

}  // namespace lbm
