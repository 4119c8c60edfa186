// kernels_sweep3.hpp -- two D3Q27 steps per launch (k_sweep3): one read and one
// write of every population for two steps.
//
// A workgroup owns a column block of (W - 2) x (H - 2) nodes in x and y and
// sweeps planes z0 - 1 .. z0 + R of its R own planes.  Its threads are the W x H
// columns with one column of halo around, x fastest.  At sweep plane p every
// thread
//   1. collides step 1 at (x, y, p), its 27 populations pulled from HBM one
//      plane ahead, puts the post-collision values (rounded to the storage
//      type, what a one-step launch would store) into LDS and starts the loads
//      of plane p + 1;
//   2. behind a barrier, pulls from LDS the values its column receives in x and
//      y.  Step 2 at plane p - 1 takes c_z = -1 from plane p, c_z = 0 from plane
//      p - 1 and c_z = +1 from plane p - 2: the pulled values of the last planes
//      wait in registers (9 of one plane, 9 of two), so LDS holds one plane
//      only.  The inner threads collide step 2 and store.
// With BACK the sweep runs from the last plane down, and c_z = +1 and -1 change
// places: every second launch does so, and starts with the planes that the one
// before left in the last-level cache (us per step, always forward / alternating:
// 112^3 FP32 44.1 / 42.2, FP64 73.8 / 68.7; 120 x 131 x 150 FP32 81.9 / 74.6; 256^3
// FP32 429 / 427).
//
// A population moves one node per step, so one halo column, row and plane on
// each side is all step 2 needs; the neighbouring workgroups compute the halo
// nodes too, with the same per-node code: results are bitwise those of two
// one-step launches.
//
// Bound: the access pattern.  At 256^3 FP32 the pattern without the collision
// takes 85-95 % of the launch, and it moves 1.2 times the bytes of one read and
// one write (the halo's lines), at about 5 TB/s; the FP64 arithmetic of 1.25
// times two collisions is 40 % of the VALU rate.  More columns per thread (two,
// or three: the tile's halo share falls) leave too few wavefronts or spill;
// two workgroups of half the size per compute unit and loads two planes ahead
// were not faster; non-temporal stores were slower (897 against 849 us), as
// were non-temporal loads (the halo loses its L2 reuse).
#pragma once

#include "kernels.hpp"

namespace lbm {

struct Sweep3Args {
    const void *src;  // f*(t), row-interleaved layout
    void *dst;        // f*(t + 2)
    int nx, ny, nz;
    int own_y, planes;  // own rows and planes per workgroup: W (own_y + 2) <= its threads
    int tiles_x, tiles_y;
    int64_t ps, rs;
    Relax relax;
    int *flag;
};

// LDS slots of the exchanged populations: all but the three with c_x = c_y = 0.
__host__ __device__ constexpr int sweep3_slot(int i) { return (i / 9) * 8 + (i % 9 < 4 ? i % 9 : i % 9 - 1); }
constexpr int kSweep3Slots = 24;
// Most threads of a workgroup, also the LDS stride of a slot: twelve wavefronts
// of at most 168 registers with float storage, eight of 256 with double.
__host__ __device__ constexpr int sweep3_columns(size_t elem) { return elem == 4 ? 768 : 512; }
__host__ __device__ constexpr size_t sweep3_lds_bytes(size_t elem) {
    return (size_t)kSweep3Slots * sweep3_columns(elem) * elem;
}

// W, the tile's width with the halo columns, is a constant of the kernel: the LDS
// offsets of the neighbouring columns are then part of the instructions; so is the
// direction (as an argument its selects cost 1-2 %).
template <int DT, bool CORR, int EQ, int W, bool BACK>
__global__ __launch_bounds__(sweep3_columns(sizeof(store_t<DT>)))
    __attribute__((amdgpu_waves_per_eu(DT == kF64 ? 2 : 3))) void k_sweep3(Sweep3Args a) {
    using T = store_t<DT>;
    constexpr int N = sweep3_columns(sizeof(T));
    __shared__ T lds[kSweep3Slots * N];
    typedef const __attribute__((address_space(1))) char *Gin;
    typedef __attribute__((address_space(1))) char *Gout;
    const Gin src = (Gin)a.src;
    const Gout dst = (Gout)a.dst;

    const int tile = xcd_tile((int)blockIdx.x, (int)gridDim.x);
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const int x0 = (tile % a.tiles_x) * (W - 2), y0 = (tile / a.tiles_x % a.tiles_y) * a.own_y;
    const int z0 = tile / (a.tiles_x * a.tiles_y) * a.planes;
    const int R = min(a.planes, nz - z0);
    const int t = (int)threadIdx.x;
    const int lx = t % W, ly = t / W;
    // an inner column whose node lies inside the grid and the workgroup's share
    const bool own = lx >= 1 && lx <= W - 2 && ly >= 1 && ly <= a.own_y && x0 + lx - 1 < nx && y0 + ly - 1 < ny;
    // the thread's column, wrapped (threads past the tile repeat a column)
    int x = (x0 + lx - 1) % nx, y = (y0 + ly - 1) % ny;
    x = x < 0 ? x + nx : x;
    y = y < 0 ? y + ny : y;
    const uint32_t rsb = (uint32_t)(a.rs * (int64_t)sizeof(T));
    const int64_t psb = a.ps * (int64_t)sizeof(T), plane = (int64_t)ny * a.rs * (int64_t)sizeof(T);
    // byte offsets of the sources x - c_x and y - c_y inside a plane
    const uint32_t xo[3] = {(uint32_t)(x + 1 == nx ? 0 : x + 1) * (uint32_t)sizeof(T), (uint32_t)x * (uint32_t)sizeof(T),
                            (uint32_t)(x == 0 ? nx - 1 : x - 1) * (uint32_t)sizeof(T)};
    const uint32_t yo[3] = {(uint32_t)(y + 1 == ny ? 0 : y + 1) * rsb, (uint32_t)y * rsb,
                            (uint32_t)(y == 0 ? ny - 1 : y - 1) * rsb};

    int zl;  // wrapped plane of the next load
    auto load_plane = [&](T (&f)[27]) {
        const int zp = zl + 1 == nz ? 0 : zl + 1, zm = zl == 0 ? nz - 1 : zl - 1;
        const Gin base[3] = {src + zp * plane, src + zl * plane, src + zm * plane};
#pragma unroll
        for (int cy = 0; cy < 3; ++cy)
#pragma unroll
            for (int cx = 0; cx < 3; ++cx) {
                uint32_t o = yo[cy] + xo[cx];
                asm("" : "+v"(o));  // (keeps the 32-bit lane offset beside the scalar base)
#pragma unroll
                for (int cz = 0; cz < 3; ++cz) {
                    const int i = cx + 3 * cy + 9 * cz;
                    f[i] = *(const __attribute__((address_space(1))) T *)(base[cz] + i * psb + o);
                }
            }
        zl = BACK ? zm : zp;
    };
    // the barriers order LDS only: loads and stores of the planes stay in flight across them
    auto lds_barrier = [&] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    // pulled in x and y from the plane's columns; a halo thread's neighbours may lie outside
    // the tile: it reads those of column (1, 1), whose values nobody uses there
    const T *at = lds + (own ? t : W + 1);
    auto pulled = [&](const T *from, int i) { return from[sweep3_slot(i) * N - (i % 3 - 1) - W * (i / 3 % 3 - 1)]; };
    // the populations that step 2 takes from the plane just computed, and those that wait two planes
    const T *now = at + (BACK ? sweep3_slot(18) * N : 0), *wait = at + (BACK ? 0 : sweep3_slot(18) * N);

    zl = BACK ? (z0 + R == nz ? 0 : z0 + R) : (z0 == 0 ? nz - 1 : z0 - 1);
    const int S = R + 2;
    T in[27], A[9], B[2][9];  // waiting values: c_z = 0 of the last plane, the others of the last two
    bool bad = false;
    auto iteration = [&](int s, auto pp) {
        constexpr int P = decltype(pp)::value;
        // step 1 at plane z0 - 1 + s (back: z0 + R - s)
        bad |= collide_dt<3, DT, CORR, EQ>(in, a.relax);
#pragma unroll
        for (int i = 0; i < 27; ++i)
            if (i % 9 != 4)
                lds[sweep3_slot(i) * N + t] = in[i];
        const T c0 = BACK ? in[22] : in[4], c1 = in[13], c2 = BACK ? in[4] : in[22];
        if (s + 1 < S)
            load_plane(in);
        lds_barrier();
        if (s >= 2 && own) {
            T g[27];
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                const T near = q == 4 ? c0 : pulled(now, q), far = B[P][q];
                g[q] = BACK ? far : near;
                g[9 + q] = A[q];
                g[18 + q] = BACK ? near : far;
            }
            bad |= collide_dt<3, DT, CORR, EQ>(g, a.relax);
            const Gout base = dst + (int64_t)(BACK ? z0 + R + 1 - s : z0 + s - 2) * plane;
            uint32_t o = yo[1] + xo[1];
            asm("" : "+v"(o));
#pragma unroll
            for (int i = 0; i < 27; ++i)
                *(__attribute__((address_space(1))) T *)(base + i * psb + o) = g[i];
        }
        // c_z = 0 waits one plane, the last of the others two (read only now: their registers held the
        // values step 2 has just used)
#pragma unroll
        for (int q = 0; q < 9; ++q) {
            A[q] = q == 4 ? c1 : pulled(at, 9 + q);
            B[P][q] = q == 4 ? c2 : pulled(wait, q);
        }
        lds_barrier();  // this plane's readers are done
    };
    load_plane(in);
    for (int s = 0;;) {  // S >= 3
        iteration(s, std::integral_constant<int, 0>{});
        if (++s >= S)
            break;
        iteration(s, std::integral_constant<int, 1>{});
        if (++s >= S)
            break;
    }
    raise_flag(a.flag, bad && own);
}

// Two steps of a small block, for domains too small for sweeps.  A workgroup
// takes a block of own_x x own_y x own_z nodes: its threads first collide step 1
// at the block's nodes with one layer of halo around (populations pulled from
// HBM) and put the values into LDS; behind the barrier the first own_x own_y
// own_z threads take one own node each, pull from LDS, collide step 2 and store.
//
// Bound: latency (the gap between launches, the pulls, two collisions of up to
// four wavefronts a SIMD); the halo makes two to three times the step-1
// collisions.  us per step, one step per launch / blocks: 16^3 FP32 3.7 / 2.7, 32^3
// FP64 5.0 / 3.8, 48^3 FP32 6.9 / 5.9, FP64 9.9 / 8.1; 64^3 FP32 10.2 / 11.2.
struct Block3Args {
    const void *src;
    void *dst;
    int nx, ny, nz;
    int own_x, own_y, own_z;  // (own_x + 2) (own_y + 2) (own_z + 2) <= the workgroup's threads
    int tiles_x, tiles_y;
    int64_t ps, rs;
    Relax relax;
    int *flag;
};

// most threads of a workgroup: 27 values each in LDS
__host__ __device__ constexpr int block3_threads(size_t elem) { return elem == 4 ? 1024 : 704; }
__host__ __device__ constexpr size_t block3_lds_bytes(int threads, size_t elem) { return (size_t)27 * threads * elem; }

template <int DT, bool CORR, int EQ>
__global__ __launch_bounds__(block3_threads(sizeof(store_t<DT>))) void k_block3(Block3Args a) {
    using T = store_t<DT>;
    extern __shared__ __align__(16) unsigned char block3_lds[];
    T *lds = reinterpret_cast<T *>(block3_lds);
    const int N = (int)blockDim.x, t = (int)threadIdx.x;
    const int tile = xcd_tile((int)blockIdx.x, (int)gridDim.x);
    const int x0 = tile % a.tiles_x * a.own_x, y0 = tile / a.tiles_x % a.tiles_y * a.own_y,
              z0 = tile / (a.tiles_x * a.tiles_y) * a.own_z;
    const int W = a.own_x + 2, WH = W * (a.own_y + 2);
    typedef const __attribute__((address_space(1))) char *Gin;
    typedef __attribute__((address_space(1))) char *Gout;
    const Gin src = (Gin)a.src;
    const Gout dst = (Gout)a.dst;
    const int64_t psb = a.ps * (int64_t)sizeof(T);
    const uint32_t rsb = (uint32_t)(a.rs * (int64_t)sizeof(T));  // the whole buffer is below 4 GiB
    bool bad = false;
    if (t < WH * (a.own_z + 2)) {
        const int lz = t / WH, r = t - lz * WH, ly = r / W, lx = r - ly * W;
        auto wrap = [](int v, int n) {
            v %= n;
            return v < 0 ? v + n : v;
        };
        const int x = wrap(x0 + lx - 1, a.nx), y = wrap(y0 + ly - 1, a.ny), z = wrap(z0 + lz - 1, a.nz);
        const uint32_t xo[3] = {(uint32_t)(x + 1 == a.nx ? 0 : x + 1) * (uint32_t)sizeof(T),
                                (uint32_t)x * (uint32_t)sizeof(T),
                                (uint32_t)(x == 0 ? a.nx - 1 : x - 1) * (uint32_t)sizeof(T)};  // x - c_x
        const int ys[3] = {y + 1 == a.ny ? 0 : y + 1, y, y == 0 ? a.ny - 1 : y - 1};           // y - c_y
        const int zs[3] = {z + 1 == a.nz ? 0 : z + 1, z, z == 0 ? a.nz - 1 : z - 1};           // z - c_z
        T f[27];
#pragma unroll
        for (int i = 0; i < 27; ++i) {
            const uint32_t o = (uint32_t)(zs[i / 9] * a.ny + ys[i / 3 % 3]) * rsb + xo[i % 3];
            f[i] = *(const __attribute__((address_space(1))) T *)(src + i * psb + o);
        }
        // (flags: step 1's own nodes are this or a neighbouring block's, all real nodes)
        bad = collide_dt<3, DT, CORR, EQ>(f, a.relax);
#pragma unroll
        for (int i = 0; i < 27; ++i)
            lds[i * N + t] = f[i];
    }
    __syncthreads();
    if (t < a.own_x * a.own_y * a.own_z) {
        const int oxy = a.own_x * a.own_y;
        const int lz = t / oxy, r = t - lz * oxy, ly = r / a.own_x, lx = r - ly * a.own_x;
        const int x = x0 + lx, y = y0 + ly, z = z0 + lz;
        if (x < a.nx && y < a.ny && z < a.nz) {
            const T *at = lds + (lz + 1) * WH + (ly + 1) * W + lx + 1;
            T g[27];
#pragma unroll
            for (int i = 0; i < 27; ++i)
                g[i] = at[i * N - (i / 9 - 1) * WH - (i / 3 % 3 - 1) * W - (i % 3 - 1)];
            bad |= collide_dt<3, DT, CORR, EQ>(g, a.relax);
            const uint32_t o = (uint32_t)(z * a.ny + y) * rsb + (uint32_t)x * (uint32_t)sizeof(T);
#pragma unroll
            for (int i = 0; i < 27; ++i)
                *(__attribute__((address_space(1))) T *)(dst + i * psb + o) = g[i];
        }
    }
    raise_flag(a.flag, bad);
}

}  // namespace lbm
