// kernels_strip.hpp -- several LBGK steps per launch with the intermediate
// states in registers: K steps on D2Q9 (k_strip2, and k_block2 for small
// domains) and on D1Q3 (k_strip1).
//
// A wavefront owns a strip of columns.  Its 64 lanes hold 64 NC consecutive
// columns (NC per lane), of which the outer H on each side are halo: a
// population moves one node per step, so the columns that are still exact
// shrink by one on each side and step, and the inner tx = 64 NC - 2 H >= 1 are
// the strip's own after H >= K steps.  Neighbouring strips compute the halo
// columns again with the same per-node code, so the results are bitwise those
// of K one-step launches.  The x neighbours come from the lanes beside by a
// wavefront shift (one lane move per 32 bits, no LDS and no barrier).
//
// Domain flags are taken from the strip's own columns only: every node is
// some strip's own at every step.
#pragma once

#include "kernels.hpp"

namespace lbm {

// Value of the lane above / below (0 past the end of the wavefront: those
// columns are halo that no later step uses).
template <bool UP, typename T>
__device__ __forceinline__ T lane_move(T v) {
    return dpp_move<UP ? 0x130 : 0x138>(v);
}
// g[k] <- the value that the population with c_x = cx - 1 pulls into column k (cx 0 or 2).
template <typename T, int NC>
__device__ __forceinline__ void pull_columns(const T (&f)[NC], int cx, T (&g)[NC]) {
    if (cx == 2) {
        const T left = lane_move<false>(f[NC - 1]);
#pragma unroll
        for (int k = NC - 1; k > 0; --k)
            g[k] = f[k - 1];
        g[0] = left;
    } else {
        const T right = lane_move<true>(f[0]);
#pragma unroll
        for (int k = 0; k < NC - 1; ++k)
            g[k] = f[k + 1];
        g[NC - 1] = right;
    }
}

struct StripArgs {
    const void *src;  // f*(t), row-interleaved layout
    void *dst;        // f*(t + K)
    int nx, ny;
    int K;            // steps per launch (k_strip1; a template parameter of k_strip2)
    int tx, h;        // own columns per strip, halo columns on each side
    int rows;         // own rows per wavefront (k_strip2)
    int strips, chunks;
    int64_t ps, rs;
    Relax relax;
    int *flag;
};

constexpr int kStripThreads = 256;

template <typename T, int N>
struct StripVec {
    typedef T type __attribute__((ext_vector_type(N)));
};
template <typename T>
struct StripVec<T, 1> {
    typedef T type;
};

// One D2Q9 wavefront: the strip's own columns of the rows [y0, y0 + R), swept
// in y.  Sweep iteration s computes step 1 at row y0 - (K - 1) + s from HBM and,
// behind it, step j + 1 at the row below step j's (j = 1 .. K - 1): with step j's
// row b just computed, step j + 1 at row b - 1 pulls the populations with
// c_y = -1 from row b, c_y = 0 from row b - 1 and c_y = +1 from row b - 2, so a
// level keeps three populations of one row and three of two rows, nine values a
// column, in registers.  Step j + 1 starts at s = 2 j.  With BACK the sweep goes from
// the last row down and c_y = +1 and -1 change places: every second launch does, and
// finds in the last-level cache the rows that the one before touched last (us per
// step, always forward / alternating: FP64 2048^2 28.8 / 27.8, 3000 x 2001 40.5 / 40.1,
// FP32 2048^2 23.4 / 23.0; 4096^2 the same within 0.5 %).  Step 1 loads each
// population at its own source column, so K - 1 halo columns do.
//
// Bound: the FP64 arithmetic of the collisions with float storage (4096^2, four
// steps: 148 VALU instructions per node update, 1.14 times the collisions for the
// halo included, at 71 % of the issue rate and the vector units busy for 76 % of
// the time, three wavefronts per SIMD), arithmetic and HBM alike with double (six
// steps).  us per step at 4096^2, against the two-step sweep
// through LDS: FP32 117 -> 88, FP64 212 -> 95.  Two columns per lane spill
// (543 us per launch against 358); more than 168 / 256 registers a lane would
// be needed for five (FP32) or eight (FP64) steps at the same occupancy.  A
// barrier per row that keeps a workgroup's strips together gave 2 % on 4096^2 FP32
// and cost up to 10 % where a SIMD holds one wavefront (1024^2 FP64).
template <int DT, bool CORR, int EQ, int K, int WPE, bool BACK>
__global__ __launch_bounds__(kStripThreads) __attribute__((amdgpu_waves_per_eu(WPE))) void k_strip2(StripArgs a) {
    using T = store_t<DT>;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lane = (int)threadIdx.x & 63;
    const int w = xcd_tile((int)blockIdx.x, (int)gridDim.x) * (kStripThreads / 64) + wave;
    const int strip = w % a.strips, chunk = w / a.strips;
    if (chunk >= a.chunks)  // uniform per wavefront; no barrier follows
        return;
    // (global address space from the start: a uniform base and a 32-bit lane offset
    // then stay a scalar register pair and one vector register)
    typedef const __attribute__((address_space(1))) char *Gin;
    typedef __attribute__((address_space(1))) char *Gout;
    const Gin src = (Gin)a.src;
    const Gout dst = (Gout)a.dst;
    const int nx = a.nx, ny = a.ny;
    const int x0 = strip * a.tx;
    const int y0 = chunk * a.rows, R = min(a.rows, ny - y0);
    int x = (x0 - a.h + lane) % nx;  // this lane's column, wrapped
    x = x < 0 ? x + nx : x;
    // byte offsets of its source columns x - c_x
    uint32_t xb[3] = {(uint32_t)(x + 1 == nx ? 0 : x + 1) * (uint32_t)sizeof(T), (uint32_t)x * (uint32_t)sizeof(T),
                      (uint32_t)(x == 0 ? nx - 1 : x - 1) * (uint32_t)sizeof(T)};
    const int own = lane - a.h;
    const bool mine = own >= 0 && own < a.tx && x0 + own < nx;
    const int64_t psb = a.ps * (int64_t)sizeof(T), rsb = a.rs * (int64_t)sizeof(T);  // strides in bytes

    // the nine runs of a step-1 row: c_y = -1 from the row above, 0, +1 from below
    int yl;  // wrapped row of the next load's c_y = 0 runs
    // (an empty asm on the lane's byte offsets, here and at the stores: their
    // widening to 64 bits then stays beside the access, which so takes a scalar base
    // and a 32-bit vector offset instead of a 64-bit vector address of its own)
    auto load_row = [&](T (&f)[9]) {
        const int yp = yl + 1 == ny ? 0 : yl + 1, ym = yl == 0 ? ny - 1 : yl - 1;
        const Gin base[3] = {src + (int64_t)yp * rsb, src + (int64_t)yl * rsb, src + (int64_t)ym * rsb};
#pragma unroll
        for (int k = 0; k < 3; ++k)
            asm("" : "+v"(xb[k]));
#pragma unroll
        for (int i = 0; i < 9; ++i)
            f[i] = *(const __attribute__((address_space(1))) T *)(base[i / 3] + i * psb + xb[i % 3]);
        yl = BACK ? ym : yp;
    };

    const int S = R + 2 * K - 2;  // sweep iterations
    T A[K - 1][3];                // level j's last row, c_y = 0
    T B[K - 1][2][3];             // level j's last two rows, c_y = +1 (BACK: -1), by iteration parity
    bool bad_any = false;
    int ys = BACK ? y0 + R - 1 : y0;  // next row to store
    auto iteration = [&](T (&in)[9], int s, auto pp) {
        constexpr int P = decltype(pp)::value;
        T o[9];
#pragma unroll
        for (int i = 0; i < 9; ++i)
            o[i] = in[i];
        bad_any |= collide_dt<2, DT, CORR, EQ>(o, a.relax);
        if (s + 1 < S)  // the next row's loads, in flight during the steps below
            load_row(in);
#pragma unroll
        for (int j = 0; j < K - 1; ++j) {
            // inputs of step j + 2 from step j + 1's rows; its last rows move on
            T g[9];
#pragma unroll
            for (int cx = 0; cx < 3; ++cx) {
                auto pull = [&](T v) { return cx == 1 ? v : (cx == 2 ? lane_move<false>(v) : lane_move<true>(v)); };
                // the populations that wait two rows, and those that do not wait
                constexpr int far = BACK ? 0 : 6, near = 6 - far;
                g[near + cx] = pull(o[near + cx]);
                g[3 + cx] = pull(A[j][cx]);
                g[far + cx] = pull(B[j][P][cx]);
                A[j][cx] = o[3 + cx];
                B[j][P][cx] = o[far + cx];
            }
            if (s < 2 * (j + 1))  // uniform: the next level has not started
                return;
#pragma unroll
            for (int i = 0; i < 9; ++i)
                o[i] = g[i];
            bad_any |= collide_dt<2, DT, CORR, EQ>(o, a.relax);
        }
        const Gout row = dst + (int64_t)ys * rsb;
        ys += BACK ? -1 : 1;
        if (mine) {
            asm("" : "+v"(xb[1]));
#pragma unroll
            for (int i = 0; i < 9; ++i)
                *(__attribute__((address_space(1))) T *)(row + i * psb + xb[1]) = o[i];
        }
    };

    yl = (BACK ? y0 + R - 1 + (K - 1) : y0 - (K - 1)) % ny;
    yl = yl < 0 ? yl + ny : yl;
    T in[9];
    load_row(in);
    for (int s = 0;;) {
        iteration(in, s, std::integral_constant<int, 0>{});
        if (++s >= S)
            break;
        iteration(in, s, std::integral_constant<int, 1>{});
        if (++s >= S)
            break;
    }
    raise_flag(a.flag, bad_any && mine);
}

// D2Q9 block: K steps of a small block, for domains too small to fill the chip
// with strips.  A workgroup holds 64 columns (one per lane) of RPT rows per
// wavefront, every row at once: the rows' x neighbours come by lane moves, the y
// neighbours inside a wavefront from its registers and between wavefronts
// through LDS (three populations of the first and of the last row, two buffers
// used in turn, one barrier a step).  Step 1 pulls from HBM, so the block has
// K - 1 halo columns and rows on each side and 64 - 2 (K - 1) own columns.
//
// Bound: the gap between launches (2.6 us) and the latency of a step's chain of
// FP64 operations, about 0.27 us for each row a SIMD collides; rows that no later
// step needs are left out.  One step per launch paid the gap every step (us per
// step, one step per launch / five: 64^2 FP64 2.84 / 1.10, 200 x 150 3.03 / 1.30, 300^2
// 4.50 / 1.64, 500 x 333 FP32 with the correction 4.23 / 2.24; four steps with every
// row to the end 1.29, 1.59, 2.00 and 2.84).
struct BlockArgs {
    const void *src;  // f*(t), row-interleaved layout
    void *dst;        // f*(t + K)
    int nx, ny;
    int K;
    int own_x, own_y;  // own columns and rows per workgroup
    int tiles_x;
    int64_t ps, rs;
    Relax relax;
    int *flag;
};

// most wavefronts of a workgroup: 128 registers a lane with one row, 168 with two
__host__ __device__ constexpr int block_waves(int rpt) { return rpt == 1 ? 16 : 12; }

// NW: most wavefronts; NB: exchange buffers (1 for a single exchange, K = 2).
template <int DT, bool CORR, int EQ, int RPT, int NW = block_waves(RPT), int NB = 2>
__device__ __forceinline__ void block2_tile(const BlockArgs &a, int tile) {
    using T = store_t<DT>;
    __shared__ T edge[NB][NW][6][64];
    typedef const __attribute__((address_space(1))) char *Gin;
    typedef __attribute__((address_space(1))) char *Gout;
    const Gin src = (Gin)a.src;
    const Gout dst = (Gout)a.dst;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), waves = (int)blockDim.x >> 6;
    const int lane = (int)threadIdx.x & 63;
    const int nx = a.nx, ny = a.ny, h = a.K - 1;
    const int x0 = (tile % a.tiles_x) * a.own_x, y0 = (tile / a.tiles_x) * a.own_y;
    int x = (x0 - h + lane) % nx;
    x = x < 0 ? x + nx : x;
    const uint32_t xb[3] = {(uint32_t)(x + 1 == nx ? 0 : x + 1) * (uint32_t)sizeof(T), (uint32_t)x * (uint32_t)sizeof(T),
                            (uint32_t)(x == 0 ? nx - 1 : x - 1) * (uint32_t)sizeof(T)};  // x - c_x
    const int64_t psb = a.ps * (int64_t)sizeof(T), rsb = a.rs * (int64_t)sizeof(T);
    const int r0 = wave * RPT - h;  // the wavefront's first row within the own rows
    T f[RPT][9];
    {
        int y = (y0 + r0) % ny;
        y = y < 0 ? y + ny : y;
#pragma unroll
        for (int j = 0; j < RPT; ++j) {
            const int yp = y + 1 == ny ? 0 : y + 1, ym = y == 0 ? ny - 1 : y - 1;
            const Gin base[3] = {src + yp * rsb, src + y * rsb, src + ym * rsb};
#pragma unroll
            for (int i = 0; i < 9; ++i)
                f[j][i] = *(const __attribute__((address_space(1))) T *)(base[i / 3] + i * psb + xb[i % 3]);
            y = yp;
        }
    }
    // own rows and columns; the domain flag is taken from them at every step
    const bool own_col = lane >= h && lane < h + a.own_x && x0 + lane - h < nx;
    bool bad = false;
    // `halo` rows on each side are still needed (uniform; the others' values are unused)
    auto relax_rows = [&](int halo) {
#pragma unroll
        for (int j = 0; j < RPT; ++j)
            if (r0 + j >= -halo && r0 + j < a.own_y + halo) {
                const bool b = collide_dt<2, DT, CORR, EQ>(f[j], a.relax);
                const bool own_row = r0 + j >= 0 && r0 + j < a.own_y && y0 + r0 + j < ny;
                bad |= b && own_row;
            }
    };
    relax_rows(h);
    for (int k = 1; k < a.K; ++k) {
        T(*e)[6][64] = edge[k % NB];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            e[wave][q][lane] = f[0][q];                // to the row below the first
            e[wave][3 + q][lane] = f[RPT - 1][6 + q];  // to the row above the last
        }
        __syncthreads();
        // (the block's outermost rows have no neighbour there: halo rows no later step uses)
        const int up = wave + 1 < waves ? wave + 1 : wave, down = wave > 0 ? wave - 1 : wave;
        T in[2][3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            in[0][q] = e[up][q][lane];
            in[1][q] = e[down][3 + q][lane];
        }
        // row j pulls c_y = -1 from row j + 1 and c_y = +1 from row j - 1
        T g[RPT][9];
#pragma unroll
        for (int j = 0; j < RPT; ++j)
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const T v = i < 3 ? (j + 1 < RPT ? f[j + 1 < RPT ? j + 1 : j][i] : in[0][i])
                                  : (i < 6 ? f[j][i] : (j > 0 ? f[j > 0 ? j - 1 : j][i] : in[1][i - 6]));
                g[j][i] = i % 3 == 1 ? v : (i % 3 == 2 ? lane_move<false>(v) : lane_move<true>(v));
            }
#pragma unroll
        for (int j = 0; j < RPT; ++j)
#pragma unroll
            for (int i = 0; i < 9; ++i)
                f[j][i] = g[j][i];
        relax_rows(h - k);
    }
    raise_flag(a.flag, bad && own_col);
    if (!own_col)
        return;
#pragma unroll
    for (int j = 0; j < RPT; ++j) {
        if (r0 + j >= 0 && r0 + j < a.own_y && y0 + r0 + j < ny) {  // uniform
            const Gout row = dst + (int64_t)(y0 + r0 + j) * rsb;
#pragma unroll
            for (int i = 0; i < 9; ++i)
                *(__attribute__((address_space(1))) T *)(row + i * psb + xb[1]) = f[j][i];
        }
    }
}

template <int DT, bool CORR, int EQ, int RPT>
__global__ __launch_bounds__(64 * block_waves(RPT)) void k_block2(BlockArgs a) {
    block2_tile<DT, CORR, EQ, RPT>(a, xcd_tile((int)blockIdx.x, (int)gridDim.x));
}

// One D1Q3 wavefront: K steps (1 .. h) of the strip's own columns.  h and tx are
// multiples of NC and of the vector width.
//
// Bound: VALU issue.  2^27 nodes with the correction, float storage, eight steps: 69
// instructions per node update, halo included, 79 % of the issue rate and the
// vector units busy for 90 % of the time in a call of 64 steps (2384 us per launch),
// 86 and 98 % in one of 200.
template <int DT, bool CORR, int EQ, int NC, bool NT>
__global__ __launch_bounds__(kStripThreads) void k_strip1(StripArgs a) {
    using T = store_t<DT>;
    constexpr int VW = NC * sizeof(T) < 16 ? NC : 16 / (int)sizeof(T);
    using V = typename StripVec<T, VW>::type;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int lane = (int)threadIdx.x & 63;
    const int strip = xcd_tile((int)blockIdx.x, (int)gridDim.x) * (kStripThreads / 64) + wave;
    if (strip >= a.strips)
        return;
    const T *__restrict__ src = static_cast<const T *>(a.src);
    T *__restrict__ dst = static_cast<T *>(a.dst);
    const int nx = a.nx;
    const int x0 = strip * a.tx;
    const bool inside = x0 >= a.h && x0 - a.h + 64 * NC <= nx;  // uniform
    const int xl = x0 - a.h + lane * NC;                        // first column of the lane
    T f[3][NC];
    if (inside) {
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int k = 0; k < NC; k += VW) {
                const V v = *reinterpret_cast<const V *>(src + i * a.ps + xl + k);
#pragma unroll
                for (int q = 0; q < VW; ++q)
                    f[i][k + q] = v[q];
            }
    } else {
        int x = xl % nx;
        x = x < 0 ? x + nx : x;
#pragma unroll
        for (int k = 0; k < NC; ++k) {
#pragma unroll
            for (int i = 0; i < 3; ++i)
                f[i][k] = src[i * a.ps + x];
            x = x + 1 == nx ? 0 : x + 1;
        }
    }
    bool bad = false;
    for (int j = 0; j < a.K; ++j) {
        T g0[NC], g2[NC];
        pull_columns<T, NC>(f[0], 0, g0);
        pull_columns<T, NC>(f[2], 2, g2);
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            T v[3] = {g0[k], f[1][k], g2[k]};
            bad |= collide_dt<1, DT, CORR, EQ>(v, a.relax);
            f[0][k] = v[0];
            f[1][k] = v[1];
            f[2][k] = v[2];
        }
    }
    const int own = lane * NC - a.h;
    const bool mine = own >= 0 && own < a.tx;
    raise_flag(a.flag, bad && mine);
    if (!mine)
        return;
    if (inside) {
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
            for (int k = 0; k < NC; k += VW) {
                V v;
#pragma unroll
                for (int q = 0; q < VW; ++q)
                    v[q] = f[i][k + q];
                V *p = reinterpret_cast<V *>(dst + i * a.ps + xl + k);
                if constexpr (NT)
                    __builtin_nontemporal_store(v, p);
                else
                    *p = v;
            }
    } else {
#pragma unroll
        for (int k = 0; k < NC; ++k)
            if (x0 + own + k < nx)
#pragma unroll
                for (int i = 0; i < 3; ++i)
                    dst[i * a.ps + x0 + own + k] = f[i][k];
    }
}

// A whole short D1Q3 row in one workgroup, one node per thread: any number of
// steps in one launch, with the populations in registers, and the acoustic
// energies of a history on the way.
//
// Bound: the dependence chain of one collision (one wavefront per SIMD up to
// 256 nodes), 0.19 us per step within one wavefront, 0.25 with the exchange
// through LDS; launches of 32 steps cost the strips 0.33 us per step on such
// rows.
constexpr int kRowMax = 1024;  // nodes, one workgroup's threads

struct RowArgs {
    const void *src;
    void *dst;
    int nx;
    int steps;  // steps of this launch
    int every;  // steps between readings (energies only)
    bool first; // a reading before the first step
    int64_t ps;
    Relax relax;
    int *flag;
    double *out;  // energies (NULL: none), one per reading
    double rho_ref;
    double U[3];
};

// The neighbours' values come by a lane move (ONE: the row fits one wavefront,
// whose ends are read as scalars) or through LDS with one barrier per step.
// A reading's wavefront sums are folded after the next barrier; the order of
// the sum is k_energy's, so the energies are bitwise its.
template <int DT, bool CORR, int EQ, bool ONE, bool ENERGY>
__global__ __launch_bounds__(ONE ? 64 : kRowMax) void k_row1(RowArgs a) {
    using T = store_t<DT>;
    constexpr int N = ONE ? 1 : kRowMax;
    __shared__ T edge[2][2][N];
    __shared__ double sums[2][kRowMax / 64];
    const int x = (int)threadIdx.x, nx = a.nx;
    const bool in = x < nx;
    const int waves = (nx + 63) / 64;
    const int left = x == 0 ? nx - 1 : x - 1, right = x + 1 >= nx ? 0 : x + 1;
    T f[3];
#pragma unroll
    for (int i = 0; i < 3; ++i)
        f[i] = static_cast<const T *>(a.src)[i * a.ps + (in ? x : nx - 1)];
    const double half_cs2_over_rho = (1.0 / 6.0) / a.rho_ref;
    double *out = a.out;
    int slot = 0;
    // this wavefront's part of a reading / the whole of it, by thread 0
    auto put_energy = [&]() {
        const double v[3] = {(double)f[0], (double)f[1], (double)f[2]};
        const double e = node_energy<1>(v, DT == kF64 ? 0.0 : a.relax.rho0, a.rho_ref, half_cs2_over_rho, a.U);
        const double r = wave_sum(in ? e : 0.0);
        slot ^= 1;
        if ((x & 63) == 0)
            sums[slot][x >> 6] = r;
    };
    auto store_energy = [&]() {
        if (x == 0) {
            double part[4];  // sums of 256 nodes, as the workgroups of k_energy leave them
#pragma unroll
            for (int b = 0; b < 4; ++b) {
                part[b] = 4 * b < waves ? sums[slot][4 * b] : 0.0;
#pragma unroll
                for (int w = 1; w < 4; ++w)
                    part[b] += 4 * b + w < waves ? sums[slot][4 * b + w] : 0.0;
            }
            *out = (part[0] + part[1]) + (part[2] + part[3]);
        }
        ++out;
    };
    bool pending = false;  // a reading waits for the next barrier
    if (ENERGY && a.first) {
        put_energy();
        pending = true;
    }
    int to_reading = a.every;
    bool bad = false;
    for (int s = 0; s < a.steps; ++s) {
        T v[3] = {f[0], f[1], f[2]};
        if constexpr (ONE) {
            const T up = lane_move<true>(f[0]), down = lane_move<false>(f[2]);
            const T head = read_lane(f[0], 0), tail = read_lane(f[2], nx - 1);
            v[0] = right == 0 ? head : up;
            v[2] = x == 0 ? tail : down;
        } else {
            edge[s & 1][0][x] = f[0];
            edge[s & 1][1][x] = f[2];
            __syncthreads();
            v[0] = edge[s & 1][0][right];
            v[2] = edge[s & 1][1][left];
        }
        if (ENERGY && pending) {
            if (ONE)
                __syncthreads();
            store_energy();
            pending = false;
        }
        bad |= collide_dt<1, DT, CORR, EQ>(v, a.relax);
#pragma unroll
        for (int i = 0; i < 3; ++i)
            f[i] = v[i];
        if (ENERGY && --to_reading == 0) {
            to_reading = a.every;
            put_energy();
            pending = true;
        }
    }
    if (ENERGY && pending) {
        __syncthreads();
        store_energy();
    }
    raise_flag(a.flag, bad && in);
    if (in)
#pragma unroll
        for (int i = 0; i < 3; ++i)
            static_cast<T *>(a.dst)[i * a.ps + x] = f[i];
}

}  // namespace lbm
