// Internal interface between the C-ABI host code and the HIP kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <cstddef>
#include <cstdint>

namespace fvk {

// Compute units of an MI355X, which the rules on launch shapes count tiles
// against (a device with fewer takes the same shapes).
constexpr int CUS = 256;

// Device control block of one solve (lives in the caller's workspace).
struct Ctl {
    double t;             // simulated time
    long long step;       // completed steps
    int bad;              // a step produced an inadmissible cell: Bad bits, 0 = none
    int pad0;
    unsigned long long pad1[5];
};
static_assert(sizeof(Ctl) == 64, "control block layout");
// A launch that ends a step raises a bit of its kind and goes on as if it were
// not set, so that the whole step is stored, whichever workgroup fails first,
// and counted; every later launch finds a bit that is not its own, skips, and
// sets BAD_SKIP for those of the same kind behind it.  The kinds alternate: the
// first launch of a step in several (no bit of its own) or a step's copy
// (BAD_COPY) stands between two BAD_STEP or BAD_EVEN launches, and steps in
// pairs take BAD_EVEN and BAD_ODD in turn.
enum Bad { BAD_SKIP = 1, BAD_STEP = 2, BAD_EVEN = 4, BAD_ODD = 8, BAD_COPY = 16 };

// CFL rate slots.  Slot k holds RATE_SUB sub-slots, each the bits of a
// non-negative double reduced with atomicMax on the bit pattern (monotone for
// x >= 0).  Workgroups spread their atomics over the sub-slots, which sit
// RATE_STRIDE bytes apart so concurrent atomics land on different memory
// channels; readers load one sub-slot per lane and take a wave max.
constexpr int RATE_SUB = 64;
constexpr int RATE_STRIDE = 256;
constexpr size_t RATE_BYTES = 3 * RATE_SUB * RATE_STRIDE;
__host__ __device__ inline unsigned long long *rate_slot(unsigned long long *base, int k, int s)
{
    return base + ((size_t)(k * RATE_SUB + s) * RATE_STRIDE) / sizeof(unsigned long long);
}
constexpr size_t CTL_BYTES = 256;

struct StageDesc {
    int prec;   // 0 float, 1 double
    int eqn;    // 0 SWE, 1 Euler
    int bathy;  // bed present
    int flux;
    int recon;
    int nx, ny, bc_x, bc_y;
    double rdx, rdy, g, gamma;
    double h0;  // SWE reference depth of the pressure term (mean initial depth)
    double cfl, dt_fixed;
};

// One RK stage: out = a0*q0 + a1*(qs + dt*L(qs)); q0 is read only at the
// updated cell, so out may alias q0.  On the last stage the CFL rate of out
// is reduced into ctl->rate[rate_out] (rate_out >= 0), rate_clear is zeroed,
// admissibility is checked and time/step advance; own is the Bad bit it raises
// (0 on the others).
hipError_t launch_stage(const StageDesc &d, const void *qs, const void *q0, void *out, const void *bed,
                        double a0, double a1, Ctl *ctl, unsigned long long *rates, int rate_in, int rate_out,
                        int rate_clear, int own, hipStream_t st);

// A whole step of 1, 2 or 3 stages from src to dst (not the same buffer) in
// one launch, with the last stage's bookkeeping; own is BAD_EVEN or BAD_ODD.
hipError_t launch_step(const StageDesc &d, int stages, const void *src, void *dst, const void *bed, Ctl *ctl,
                       unsigned long long *rates, int rate_in, int rate_out, int rate_clear, int own, hipStream_t st);
// Has launch_step's kernels of a precision and system loaded on the current
// device, so that a later launch loads nothing (it may be under capture).
hipError_t load_step(int prec, int eqn);
// The end of a step whose BAD_EVEN launch went to another buffer than the
// state's: the result copied back, unless the launch skipped the step.
hipError_t launch_step_copy(const StageDesc &d, const void *src, void *dst, Ctl *ctl, hipStream_t st);
// The grids that step so.  One stage: no ring, and no copy back to the state
// (16 steps of 500^2 cells 86 us, with a launch and a copy 151, 1400^2 324 and
// 453): all.  FP32 Heun HLLE with MINMOD, in tiles of up to 12 rows: up to
// where the rings cost what the launches do (over a bed 760^2 272 us and 268
// with a launch per stage, 800^2 275 and 289, 1024^2 425 and 327, a flat bottom
// alike; Euler, with more work in a ring, 720^2 286 and 311, 760^2 351 and 318).
// The others, in 4 or 8 rows: while every tile has a CU of its own (FP32 Roe Heun
// 320^2 108 and 143, 500^2 189 and 183; FP64 Heun 320^2 160 and 201; FP64 Roe
// in three stages, 4 rows: 200^2 193 and 242, 250^2 352 and 245).
inline int step_rows(const StageDesc &d, int stages)  // most rows of a tile
{
    if (stages == 1 || (stages == 3 && d.prec == 1)) return 4;
    return stages == 2 && d.prec == 0 && d.flux == 0 && d.recon == 0 ? 12 : 8;
}
inline bool step_fits(const StageDesc &d, int stages)
{
    const int64_t cells = (int64_t)d.nx * d.ny;
    if (d.nx < 2 * stages || d.ny < 2 * stages) return false;
    const int rows = step_rows(d, stages), cols = 64 - 4 * (stages - 1);
    if (stages == 1) return true;
    if (rows == 12) return cells <= (d.eqn == 1 ? 540000 : 640000);
    return (int64_t)((d.nx + cols - 1) / cols) * ((d.ny + rows - 1) / rows) <= CUS;
}

// Batched FP32 Heun stages over many solves (serving).  BatchSolve is one
// solve's device descriptor; WorkItem one solve of a step's list: where its
// workgroups start in the launch and its CFL slots at that step.
struct BatchSolve {
    void *q, *s1;
    const void *bed;
    void *ctl, *rates;
    int nx, ny, bc_x, bc_y;
    double rdx, rdy, g, sqg, gamma, h0, cfl, dt_fixed;
};
struct WorkItem {
    int solve;
    int tile_begin;  // index of the solve's first workgroup in the launch (prefix sum of tiles)
    int tiles_x;     // tiles per row of the solve; tile = workgroup - tile_begin, row-major
    unsigned char ri, ro, rc, pad;
};
// Tile shapes of the stage kernels: 64 columns (one wave64 per row) by
// shape_rows rows, shape_rpw rows per wave.  A cell's arithmetic is the same
// in each, to the bit.  A small grid is bound by each wave's serial chain (load,
// barrier, faces, store) with most of the chip idle, so it takes the shape
// with the most and shortest waves; a large one is bound by vector-ALU issue,
// so it takes the one that shares the most work between a wave's rows (each
// row's face values formed once, one exchange per wave) while small
// workgroups keep loads and arithmetic of different tiles overlapping.
// Microseconds per shallow-water-over-a-bed step, shapes 4 x 1 / 8 x 1 /
// 16 x 2 / 16 x 4 (rows x rows per wave), and the 32 x 2 used before:
//   64^2   8.0 /  8.5 / 10.0 / 11.6, 12.4     256^2  8.2 /  8.5 / 10.4 / 11.8, 13.0
//   512^2 11.3 / 10.7 / 11.0 / 12.3, 13.5     768^2 16.8 / 16.5 / 17.0 / 17.8, 19.5
//   1000 x 700 18.0 (8 x 1) / 17.3 / 18.2, 19.9   1024^2 23.1 / 22.2 / 20.4 / 21.4, 20.1
//   2048^2 78.1 / 76.2 / 64.8 / 63.6, 69.5    4096^2  306 (8 x 1) / 269 / 265, 304
// Euler's order is the same.  Double precision (4 x 1 / 16 x 2, and the 8 x 2
// used before): 256^2 10.1 / 15.6, 12.3; 512^2 17.9 / 16.5, 17.1; 1024^2
// 49.8 / 43.8, 45.4.
constexpr int TILE_X = 64, NSHAPES = 4;
constexpr int shape_rows(int shape) { return shape == 0 ? 4 : shape == 1 ? 8 : 16; }
constexpr int shape_rpw(int shape) { return shape < 2 ? 1 : shape == 2 ? 2 : 4; }
// The shape for a launch over `cells` cells in all.
inline int stage_shape(int64_t cells, int prec = 0)
{
    if (prec == 1) return cells <= 150000 ? 0 : 2;
    return cells <= 160000 ? 0 : cells <= 640000 ? 1 : cells <= 3000000 ? 2 : 3;
}
inline int64_t stage_tiles(int nx, int ny, int shape)
{
    return (int64_t)((nx + TILE_X - 1) / TILE_X) * ((ny + shape_rows(shape) - 1) / shape_rows(shape));
}
// The work lists' shape, one for all of a server's rounds, since a captured
// launch keeps its kernel and a graph per shape would be captured for each.  Of
// the four this one is within 3 % of the best from half a million cells in a
// launch on, which a loaded server's rounds hold.
constexpr int LIST_SHAPE = 2;
// One workgroup per tile: grid = the list's tiles of LIST_SHAPE.  Shallow water
// has a bed.
hipError_t launch_batch_stage(int eqn, int stage, const BatchSolve *solves, const WorkItem *items, const int *nitems,
                              int grid, hipStream_t st);
// One solve, descriptor and list entry by value (it.tile_begin == 0): the
// launches of a single solve.
hipError_t launch_batch_stage_one(int eqn, int bathy, int stage, int shape, const BatchSolve &d, const WorkItem &it,
                                  int grid, hipStream_t st);
// The form recorded in graphs: wgs workgroups (a multiple of 8, set to
// xcd_grid(tiles) before each replay), the tile count read from the list
// header list = {items, tiles}.
hipError_t launch_batch_stage_list(int eqn, int stage, const BatchSolve *solves, const WorkItem *items, const int *list,
                                   int wgs, hipStream_t st);
// Grid of a tiled launch: the tiles padded to a multiple of the 8 XCDs.
__host__ __device__ inline int xcd_grid(int ntiles) { return (ntiles + 7) & ~7; }


// Reduce the CFL rate of q into ctl->rate[slot] and flag inadmissible cells.
hipError_t launch_rate(const StageDesc &d, const void *q, Ctl *ctl, unsigned long long *rates, int slot,
                       hipStream_t st);

// Deterministic double-precision totals (nvar sums + energy) into out_dev.
hipError_t launch_totals(const StageDesc &d, const void *q, double *partials, int max_blocks, double *out_dev,
                         hipStream_t st);

// Face fluxes of q (flat bottom): fx [nv][ny][nx+1], fy [nv][ny+1][nx].
hipError_t launch_face_fluxes(const StageDesc &d, const void *q, void *fx, void *fy, hipStream_t st);

constexpr int TOTALS_MAX_BLOCKS = 1024;

// Reset a solve's control block and CFL rate slots on the device (a kernel:
// nothing host-side, no memset node).
hipError_t launch_reset(Ctl *ctl, unsigned long long *rates, hipStream_t st);
// Copy a solve's simulated time, completed steps and inadmissible flag into
// the caller's device record {double t; int64 steps; int32 bad; int32 pad}.
hipError_t launch_report(const Ctl *ctl, void *info, hipStream_t st);

}  // namespace fvk
