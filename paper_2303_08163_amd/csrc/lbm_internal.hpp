// lbm_internal.hpp -- host-side layout of a domain's workspace and shared
// helpers of the C-ABI implementation.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "kernels.hpp"
#include "lbm.h"

namespace lbm {

// Tile of a D3Q27 two-step sweep (sweep3.hip): width with halo columns, own
// rows and planes.
struct Sweep3Geom {
    int w, rows, planes;
};

// Block of a small D3Q27 domain (sweep3.hip): own nodes per axis (0: the domain
// takes no blocks) and threads of a workgroup.
struct Block3Geom {
    int own_x, own_y, own_z, threads;
};

// Tiling of a small D2Q9 domain's blocks (strip.hip): rows per wavefront (0: the
// domain takes no blocks), wavefronts, own columns and rows per workgroup.
struct Block2Geom {
    int rpt, waves, own_x, own_y, tiles_x, tiles_y;
};

// Workspace layout of one domain (all offsets in bytes, 256-byte aligned).
struct Layout {
    int dim, q;
    size_t elem;       // bytes per stored population
    int64_t n;         // nodes
    int layout;        // LBM_LAYOUT_ROWS or LBM_LAYOUT_PLANES
    int eq;            // LBM_EQ_* (kEq* in the device code)
    int64_t ps, rs;    // population and row strides (elements)
    int block_x, block_y;
    int npt;           // nodes per thread along x
    int flags;         // LBM_TUNE_* bits
    bool rowwave;      // one wavefront spans a whole row (vector kernels)
    int tblock;        // LBGK steps per launch (1; 2 on D2Q9; 2, 4 or 8 on D1Q3)
    int t2_tx, t2_rows;  // multi-step kernels: owned columns (nodes) and rows per workgroup
    int deep;          // steps of the longest launch of a run (strips, sweeps; 0: tblock)
    int row;           // 1: D1Q3 runs, 2: histories only, in one workgroup (k_row1)
    int strip_rows[2]; // D2Q9 strips: own rows per wavefront with 4 and with 6 steps
    Block2Geom block2; // D2Q9 blocks
    Sweep3Geom sweep3; // D3Q27 sweeps
    Block3Geom block3; // D3Q27 blocks
    bool zhalo;        // z-slab: each buffer holds halo planes -1 and nz around the nz planes
    int64_t plane;     // elements of one plane (rows layout: ny * rs)
    int red_blocks;    // workgroups of the moments reduction
    size_t buf_bytes;  // one population buffer
    size_t off_buf[2], off_flag, off_diag, off_partials, ws_bytes;
};

// One domain's state inside a workspace (owned by a handle or a pool slot).
struct DomainState {
    lbm_config cfg;
    Layout L;
    char *ws;
    void *buf[2];
    int cur;  // buffer holding the current state
    int *flag;
    double *diag_dev;
    double *partials;
    int64_t steps;
    Relax relax;
};

void set_error(const char *msg);
int hip_fail(hipError_t e, const char *what);
int validate_config(const lbm_config *cfg, const lbm_tuning *tun, Layout *out);
int launch_step(const Layout &L, const StepArgs &args, int dtype, bool corr, hipStream_t s, int nz,
                const HaloArgs *halo);
int launch_step2(const Layout &L, const StepArgs &args, int dtype, bool corr, hipStream_t s);

// Launches with the intermediate states in registers (strip.hip).
constexpr int64_t kStrip1Wide = 1 << 22;  // D1Q3 rows with many columns per lane
void plan2(const lbm_config *cfg, Layout &L);
int strip1_steps(int64_t nx);
int strip1_cols(int64_t nx, int dtype, int K);
int launch_strip1(const Layout &L, const StepArgs &args, int dtype, bool corr, int K, hipStream_t s);
// Short D1Q3 rows in one workgroup, with the readings of an energy history (NULL: none).
constexpr int kRowSteps = 16384;  // most steps per launch
struct RowEnergy {
    double *out;
    int every;
    bool first;  // a reading before the first step
    double rho_ref, U;
};
int row1_plan(int64_t nx);
bool row1_history(int64_t nx, int64_t every);  // of a row that row1_plan takes
int launch_row1(const Layout &L, const StepArgs &args, int dtype, bool corr, int steps, const RowEnergy *e,
                hipStream_t s);
int launch_strip2(const Layout &L, const StepArgs &args, int dtype, bool corr, int K, bool back, hipStream_t s);

int launch_block2(const Layout &L, const StepArgs &args, int dtype, bool corr, int K, hipStream_t s);

// Two-step D3Q27 sweeps and blocks (sweep3.hip).
constexpr size_t kSweep3Bytes = (size_t)96 << 20;  // sweeps: both population buffers from here on
constexpr int64_t kBlock3Nodes = 200000;           // blocks: domains up to here
void plan3(const lbm_config *cfg, Layout &L);
int launch_sweep3(const Layout &L, const StepArgs &args, int dtype, bool corr, bool back, hipStream_t s);
int launch_block3(const Layout &L, const StepArgs &args, int dtype, bool corr, hipStream_t s);

// Bind a domain to its workspace and enqueue f = f^eq(rho, u) plus the flag
// clear; the caller synchronises and reads the flag (domain_read_flag).
int domain_bind_and_init(DomainState &d, const lbm_config *cfg, const Layout &L, void *workspace,
                         const double *rho, const double *u, hipStream_t s);
// Synchronise the stream and return the domain flag (0/1) in *flag.
int domain_read_flag(const DomainState &d, hipStream_t s, int *flag);
// host: kHostBytes of pinned memory for the result, or NULL.  Synchronises s.
constexpr size_t kHostBytes = 256;
int domain_moments(DomainState &d, hipStream_t s, double *rho, double *u, lbm_diag *diag, double *host);
int domain_export(DomainState &d, hipStream_t s, double *out);
// Enqueue the acoustic energy about (rho_ref, U) into the device double *out.
int domain_energy(DomainState &d, hipStream_t s, const double *U, double rho_ref, double *out);

}  // namespace lbm
