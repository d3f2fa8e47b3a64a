// Finite-volume stage kernels for gfx950 (MI355X).
//
// One workgroup owns a tile of 64 columns (a wave64 per row) and 4, 8 or 16
// rows, one to four rows per wave; the launch's size picks the shape.
//  1. The tile plus a two-cell halo of every variable (and eta = h + b with a
//     bed) is staged into LDS, a wave loading whole rows, every load issued
//     before the first store; ghost cells are synthesised during the load
//     (periodic wrap or wall mirror with the normal momentum negated), the row
//     mapped in scalar registers and the column once per lane.
//  2. Every x face and y face of the tile is evaluated exactly once
//     (reconstruction, hydrostatic step, numerical flux), by the lane of its
//     high-side cell, and stays in registers: a cell's high x face comes from
//     the next lane by a DPP shift, its high y face from the lane's next row
//     (faces at a wave's edge go through LDS).
//  3. Each cell forms the flux divergence (eq 2.9 / eq 2.23), adds the bed
//     source, combines the Runge-Kutta stage (eq 2.19 / eq 2.20) and writes
//     its new value.  On the last stage the CFL rate of the new state is
//     reduced over the wave with DPP, then one atomicMax per wave into a
//     device sub-slot read by the next step, so Delta t never travels
//     through the host.
// On small grids one launch takes all stages of a step (step_kernels.hpp).
#include "stage_device.hpp"

namespace fvk {

__device__ __forceinline__ int map_index(int i, int n, int bc, bool &flip)
{
    if (i >= 0 && i < n) return i;
    if (bc == 0) return ((i % n) + n) % n;
    flip = true;
    int m = i < 0 ? -1 - i : 2 * n - 1 - i;
    return m < 0 ? 0 : (m >= n ? n - 1 : m);  // cells past the ghost layer are never used
}

// LDS of a tile of the given shape.
template <typename T, int EQN, bool BATHY, int SHAPE>
using ShapeLds = StageLds<T, EQN, BATHY, TILE_X, shape_rows(SHAPE), shape_rpw(SHAPE)>;

template <typename T, int EQN, bool BATHY, int FLUX, int RECON, int SHAPE>
__global__ __launch_bounds__((ShapeLds<T, EQN, BATHY, SHAPE>::NTH)) void stage_kernel(StageArgs<T> a, int tiles_x,
                                                                                 int ntiles)
{
    constexpr int TX = TILE_X, TY = shape_rows(SHAPE);
    const int tile = xcd_tile(blockIdx.x, gridDim.x);
    if (tile >= ntiles) return;
    const int ty = tile / tiles_x, tx = tile - ty * tiles_x;
    stage_tile<T, EQN, BATHY, FLUX, RECON, TX, TY, shape_rpw(SHAPE)>(a, tx * TX, ty * TY, tile, threadIdx.x);
}

// Batched stage over many solves: the step's list holds one item per solve
// (sorted by tile_begin); tile w of the launch belongs to the solve whose tile
// range contains it (binary search).  STAGE 1: S1 = q + dt L(q); STAGE 2:
// q = q/2 + (S1 + dt L(S1))/2 (Heun).
struct TileRef {
    int x0, y0, tile;
};

template <typename T, int STAGE, int SHAPE>
__device__ __forceinline__ TileRef batch_fill(const BatchSolve &d, const WorkItem &it, const int w, StageArgs<T> &a);

template <typename T, int STAGE, int SHAPE>
__device__ __forceinline__ TileRef batch_resolve(const BatchSolve *__restrict__ solves,
                                                 const WorkItem *__restrict__ items, const int *__restrict__ nitems,
                                                 const int w, StageArgs<T> &a)
{
    int lo = 0, hi = *nitems - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (items[mid].tile_begin <= w) lo = mid;
        else hi = mid - 1;
    }
    const WorkItem it = items[lo];
    return batch_fill<T, STAGE, SHAPE>(solves[it.solve], it, w, a);
}

// The stage arguments of workgroup w, whose solve is d with list entry it.
template <typename T, int STAGE, int SHAPE>
__device__ __forceinline__ TileRef batch_fill(const BatchSolve &d, const WorkItem &it, const int w, StageArgs<T> &a)
{
    constexpr int TX = TILE_X, TY = shape_rows(SHAPE);
    const int tile = w - it.tile_begin;
    a.qs = (const T *)(STAGE == 1 ? d.q : d.s1);
    a.q0 = (const T *)d.q;
    a.out = (T *)(STAGE == 1 ? d.s1 : d.q);
    a.bed = (const T *)d.bed;
    a.nx = d.nx;
    a.ny = d.ny;
    a.bc_x = d.bc_x;
    a.bc_y = d.bc_y;
    a.rdx = (T)d.rdx;
    a.rdy = (T)d.rdy;
    a.ph.g = (T)d.g;
    a.ph.sqg = (T)d.sqg;
    a.ph.gamma = (T)d.gamma;
    a.ph.h0 = (T)d.h0;
    a.a0 = STAGE == 1 ? T(0) : T(0.5);
    a.a1 = STAGE == 1 ? T(1) : T(0.5);
    a.cfl = d.cfl;
    a.dt_fixed = d.dt_fixed;
    a.ctl = (Ctl *)d.ctl;
    a.rates = (unsigned long long *)d.rates;
    a.rate_in = it.ri;
    a.rate_out = STAGE == 1 ? -1 : it.ro;
    a.rate_clear = STAGE == 1 ? -1 : it.rc;
    a.last = STAGE == 2;
    a.own = STAGE == 2 ? BAD_STEP : 0;
    const int ty = tile / it.tiles_x, tx = tile - ty * it.tiles_x;
    return TileRef{tx * TX, ty * TY, tile};
}

// One workgroup per tile.  ntiles > 0: the list holds ntiles tiles.
// ntiles == 0: the tile count is read from the list header (nitems[1]), so
// that a launch recorded in a graph serves whatever list is uploaded before
// each replay.  The grid is xcd_grid(tiles).  Eight waves per SIMD (at most
// 64 VGPRs); the shape with four rows per wave holds more values per lane and
// runs five.
constexpr int shape_waves(int shape) { return shape == 3 ? 5 : 8; }

template <typename T, int EQN, bool BATHY, int STAGE, int SHAPE>
__global__ __launch_bounds__((ShapeLds<T, EQN, BATHY, SHAPE>::NTH), shape_waves(SHAPE)) void batch_stage_kernel(
    const BatchSolve *__restrict__ solves, const WorkItem *__restrict__ items, const int *__restrict__ nitems,
    int ntiles)
{
    const int total = ntiles > 0 ? ntiles : nitems[1];
    const int w = xcd_tile(blockIdx.x, gridDim.x);
    if (w >= total) return;
    StageArgs<T> a;
    const TileRef t = batch_resolve<T, STAGE, SHAPE>(solves, items, nitems, w, a);
    stage_tile<T, EQN, BATHY, HLLE, MINMOD, TILE_X, shape_rows(SHAPE), shape_rpw(SHAPE)>(a, t.x0, t.y0, t.tile,
                                                                                        threadIdx.x);
}

// One solve, its descriptor and list entry passed by value: the halo loads
// wait for nothing but the arguments.  The same stage arguments, hence the
// same results, as the list form.
template <typename T, int EQN, bool BATHY, int STAGE, int SHAPE>
__global__ __launch_bounds__((ShapeLds<T, EQN, BATHY, SHAPE>::NTH), shape_waves(SHAPE)) void batch_stage_one_kernel(
    BatchSolve d, WorkItem it, int ntiles)
{
    const int w = xcd_tile(blockIdx.x, gridDim.x);
    if (w >= ntiles) return;
    StageArgs<T> a;
    const TileRef t = batch_fill<T, STAGE, SHAPE>(d, it, w, a);
    stage_tile<T, EQN, BATHY, HLLE, MINMOD, TILE_X, shape_rows(SHAPE), shape_rpw(SHAPE)>(a, t.x0, t.y0, t.tile,
                                                                                        threadIdx.x);
}

// ------------------------------------------------------------ CFL rate of q
template <typename T, int EQN>
__global__ __launch_bounds__(256) void rate_kernel(const T *q, int n, T rdx, T rdy, Phys<T> ph, Ctl *ctl,
                                                   unsigned long long *rates, int slot)
{
    __shared__ T s_red[4];
    constexpr int NV = EQN == SWE ? 3 : 4;
    T lmax = T(0);
    bool bad = false;
    for (int k = blockIdx.x * 256 + threadIdx.x; k < n; k += gridDim.x * 256) {
        T s[NV];
#pragma unroll
        for (int v = 0; v < NV; v++) s[v] = q[(size_t)v * n + k];
        T r;
        if (cell_rate_ok<T, EQN>(s, ph, rdx, rdy, r)) lmax = tmax(lmax, r);
        else bad = true;
    }
    if (bad) atomicExch(&ctl->bad, 1);
    T m = block_max256(lmax, s_red);
    if (threadIdx.x == 0) push_rate(rates, slot, (double)m, blockIdx.x);
}

// ----------------------------------------------------------------- totals
// Block b sums a fixed set of cells in a fixed order, then a fixed-order tree;
// a single block then adds the block partials in index order.
template <typename T, int EQN>
__global__ __launch_bounds__(256) void totals_partial_kernel(const T *q, int n, double dA, double g, double *partials)
{
    constexpr int NV = EQN == SWE ? 3 : 4;
    __shared__ double s[NV + 1][256];
    double acc[NV + 1];
#pragma unroll
    for (int v = 0; v <= NV; v++) acc[v] = 0.0;
    for (int k = blockIdx.x * 256 + threadIdx.x; k < n; k += gridDim.x * 256) {
        double c[NV];
#pragma unroll
        for (int v = 0; v < NV; v++) c[v] = (double)q[(size_t)v * n + k];
#pragma unroll
        for (int v = 0; v < NV; v++) acc[v] += c[v] * dA;
        double kin = 0.5 * (c[1] * c[1] + c[2] * c[2]) / c[0];
        acc[NV] += (EQN == SWE ? 0.5 * g * c[0] * c[0] + kin : kin) * dA;
    }
#pragma unroll
    for (int v = 0; v <= NV; v++) s[v][threadIdx.x] = acc[v];
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w)
#pragma unroll
            for (int v = 0; v <= NV; v++) s[v][threadIdx.x] += s[v][threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0)
#pragma unroll
        for (int v = 0; v <= NV; v++) partials[blockIdx.x * (NV + 1) + v] = s[v][0];
}

// One workgroup per output: thread t adds partials t, t+256, ... in order,
// then a fixed-order tree over the 256 threads.
__global__ __launch_bounds__(256) void totals_final_kernel(const double *partials, int nblocks, int nout, double *out)
{
    __shared__ double s[256];
    const int o = blockIdx.x;
    double acc = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += 256) acc += partials[b * nout + o];
    s[threadIdx.x] = acc;
    __syncthreads();
    for (int w = 128; w > 0; w >>= 1) {
        if (threadIdx.x < w) s[threadIdx.x] += s[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) out[o] = s[0];
}

// ------------------------------------------------------- solve reset/report
__global__ __launch_bounds__(256) void reset_kernel(Ctl *ctl, unsigned long long *rates)
{
    const int t = threadIdx.x;
    for (int k = t; k < (int)(RATE_BYTES / sizeof(unsigned long long)); k += 256) rates[k] = 0ull;
    if (t < (int)(sizeof(Ctl) / sizeof(unsigned long long))) ((unsigned long long *)ctl)[t] = 0ull;
}

struct RunInfo {
    double t;
    long long steps;
    int bad;
    int pad;
};

__global__ void report_kernel(const Ctl *ctl, RunInfo *info)
{
    if (threadIdx.x == 0) {
        info->t = ctl->t;
        info->steps = ctl->step;
        info->bad = ctl->bad != 0;
        info->pad = 0;
    }
}

hipError_t launch_reset(Ctl *ctl, unsigned long long *rates, hipStream_t st)
{
    hipLaunchKernelGGL(reset_kernel, dim3(1), dim3(256), 0, st, ctl, rates);
    return hipGetLastError();
}

hipError_t launch_report(const Ctl *ctl, void *info, hipStream_t st)
{
    hipLaunchKernelGGL(report_kernel, dim3(1), dim3(64), 0, st, ctl, (RunInfo *)info);
    return hipGetLastError();
}

// --------------------------------------------------------------- face export
template <typename T, int EQN, int FLUX, int RECON>
__global__ void face_kernel(const T *q, int nx, int ny, int bc_x, int bc_y, Phys<T> ph, T *fx, T *fy)
{
    constexpr int NV = EQN == SWE ? 3 : 4;
    const size_t plane = (size_t)nx * ny;
    const int nfx = (nx + 1) * ny, nfy = nx * (ny + 1);
    int f = blockIdx.x * blockDim.x + threadIdx.x;
    if (f >= nfx + nfy) return;
    int axis = f < nfx ? 0 : 1;
    int i, j;
    if (axis == 0) {
        j = f / (nx + 1);
        i = f - j * (nx + 1) - 1;  // face between cells i and i+1
    } else {
        int g = f - nfx;
        j = g / nx - 1;            // face between rows j and j+1
        i = g - (j + 1) * nx;
    }
    T st[NV][4];
    for (int k = 0; k < 4; k++) {
        int ci = axis == 0 ? i - 1 + k : i, cj = axis == 0 ? j : j - 1 + k;
        bool flx = false, fly = false;
        int ix = map_index(ci, nx, bc_x, flx), iy = map_index(cj, ny, bc_y, fly);
        for (int v = 0; v < NV; v++) {
            T val = q[v * plane + (size_t)iy * nx + ix];
            if ((v == 1 && flx) || (v == 2 && fly)) val = -val;
            st[v][k] = val;
        }
    }
    T Fl[NV];
    if (axis == 0) {
        face_flux<T, EQN, FLUX, RECON, 0>(st, ph, Fl);
        for (int v = 0; v < NV; v++) fx[(size_t)v * nfx + (size_t)j * (nx + 1) + i + 1] = Fl[v];
    } else {
        face_flux<T, EQN, FLUX, RECON, 1>(st, ph, Fl);
        for (int v = 0; v < NV; v++) fy[(size_t)v * nfy + (size_t)(j + 1) * nx + i] = Fl[v];
    }
}

// ----------------------------------------------------------------- dispatch

template <typename T, int EQN, bool BATHY, int FLUX, int RECON>
static hipError_t stage_t(const StageDesc &d, const void *qs, const void *q0, void *out, const void *bed, double a0,
                          double a1, Ctl *ctl, unsigned long long *rates, int ri, int ro, int rc, int own,
                          hipStream_t st)
{
    StageArgs<T> a = stage_args<T>(d, qs, q0, out, bed, ctl, rates, ri, ro, rc);
    a.a0 = (T)a0;
    a.a1 = (T)a1;
    a.last = own != 0;
    a.own = own;
    // the shapes with one and with two rows per wave serve every scheme, the
    // other two FP32 HLLE with MINMOD (the scheme of long runs)
    constexpr bool ALL = sizeof(T) == 4 && FLUX == HLLE && RECON == MINMOD;
    int shape = stage_shape((int64_t)d.nx * d.ny, d.prec);
    if (!ALL) shape = shape < 2 ? 0 : 2;
    // a cell's offset from its tile's first is 32 bits of bytes: fewer rows in
    // a tile of very long ones
    if ((uint64_t)(shape_rows(shape) + 4) * d.nx * sizeof(T) >> 32) shape = 0;
    const int tiles_x = (d.nx + TILE_X - 1) / TILE_X, ntiles = (int)stage_tiles(d.nx, d.ny, shape);
    const dim3 grid(xcd_grid(ntiles));
#define FV_GO(S)                                                                                       \
    hipLaunchKernelGGL((stage_kernel<T, EQN, BATHY, FLUX, RECON, S>), grid,                            \
                       dim3(ShapeLds<T, EQN, BATHY, S>::NTH), 0, st, a, tiles_x, ntiles)
    if (shape == 0) FV_GO(0);
    else if (shape == 2) FV_GO(2);
    if constexpr (ALL) {
        if (shape == 1) FV_GO(1);
        else if (shape == 3) FV_GO(3);
    }
#undef FV_GO
    return hipGetLastError();
}

template <typename T, int EQN, bool BATHY, int FLUX>
static hipError_t stage_r(const StageDesc &d, const void *qs, const void *q0, void *out, const void *bed, double a0,
                          double a1, Ctl *ctl, unsigned long long *rates, int ri, int ro, int rc, int own,
                          hipStream_t st)
{
    if (d.recon == FIRST)
        return stage_t<T, EQN, BATHY, FLUX, FIRST>(d, qs, q0, out, bed, a0, a1, ctl, rates, ri, ro, rc, own, st);
    return stage_t<T, EQN, BATHY, FLUX, MINMOD>(d, qs, q0, out, bed, a0, a1, ctl, rates, ri, ro, rc, own, st);
}

template <typename T, int EQN, bool BATHY>
static hipError_t stage_f(const StageDesc &d, const void *qs, const void *q0, void *out, const void *bed, double a0,
                          double a1, Ctl *ctl, unsigned long long *rates, int ri, int ro, int rc, int own,
                          hipStream_t st)
{
    switch (d.flux) {
    case RUSANOV: return stage_r<T, EQN, BATHY, RUSANOV>(d, qs, q0, out, bed, a0, a1, ctl, rates, ri, ro, rc, own, st);
    case ROE: return stage_r<T, EQN, BATHY, ROE>(d, qs, q0, out, bed, a0, a1, ctl, rates, ri, ro, rc, own, st);
    default: return stage_r<T, EQN, BATHY, HLLE>(d, qs, q0, out, bed, a0, a1, ctl, rates, ri, ro, rc, own, st);
    }
}

template <typename T>
static hipError_t stage_p(const StageDesc &d, const void *qs, const void *q0, void *out, const void *bed, double a0,
                          double a1, Ctl *ctl, unsigned long long *rates, int ri, int ro, int rc, int own,
                          hipStream_t st)
{
    if (d.eqn == EULER) return stage_f<T, EULER, false>(d, qs, q0, out, bed, a0, a1, ctl, rates, ri, ro, rc, own, st);
    if (d.bathy) return stage_f<T, SWE, true>(d, qs, q0, out, bed, a0, a1, ctl, rates, ri, ro, rc, own, st);
    return stage_f<T, SWE, false>(d, qs, q0, out, bed, a0, a1, ctl, rates, ri, ro, rc, own, st);
}

hipError_t launch_stage(const StageDesc &d, const void *qs, const void *q0, void *out, const void *bed, double a0,
                        double a1, Ctl *ctl, unsigned long long *rates, int rate_in, int rate_out, int rate_clear,
                        int own, hipStream_t st)
{
    if (d.prec == 1)
        return stage_p<double>(d, qs, q0, out, bed, a0, a1, ctl, rates, rate_in, rate_out, rate_clear, own, st);
    return stage_p<float>(d, qs, q0, out, bed, a0, a1, ctl, rates, rate_in, rate_out, rate_clear, own, st);
}

hipError_t launch_step(const StageDesc &d, int stages, const void *src, void *dst, const void *bed, Ctl *ctl,
                       unsigned long long *rates, int rate_in, int rate_out, int rate_clear, int own, hipStream_t st)
{
    if (stages < 1 || stages > 3 || d.nx < 2 * stages || d.ny < 2 * stages || src == dst) return hipErrorInvalidValue;
    auto go = [&](auto zero) {
        using T = decltype(zero);
        StageArgs<T> a = stage_args<T>(d, src, src, dst, bed, ctl, rates, rate_in, rate_out, rate_clear);
        a.own = own;
        return d.eqn == EULER ? step_go<T, EULER>(d, stages, a, st) : step_go<T, SWE>(d, stages, a, st);
    };
    return d.prec == 1 ? go(0.0) : go(0.0f);
}

hipError_t load_step(int prec, int eqn)
{
    if (eqn == EULER) return prec == 1 ? step_load<double, EULER>() : step_load<float, EULER>();
    return prec == 1 ? step_load<double, SWE>() : step_load<float, SWE>();
}

template <typename T>
__global__ __launch_bounds__(256) void step_copy_kernel(const T *__restrict__ src, T *__restrict__ dst, size_t n,
                                                        Ctl *ctl)
{
    const int bad = ctl->bad;
    if (bad & ~(BAD_EVEN | BAD_COPY)) return;
    if (bad && blockIdx.x == 0 && threadIdx.x == 0) atomicOr(&ctl->bad, BAD_COPY);
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) dst[i] = src[i];
}

hipError_t launch_step_copy(const StageDesc &d, const void *src, void *dst, Ctl *ctl, hipStream_t st)
{
    const size_t bytes = (size_t)(d.eqn == EULER ? 4 : 3) * d.nx * d.ny * (d.prec == 1 ? 8 : 4);
    auto go = [&](auto unit) {
        using U = decltype(unit);
        const size_t n = bytes / sizeof(U), blocks = (n + 255) / 256;
        hipLaunchKernelGGL(step_copy_kernel<U>, dim3((unsigned)(blocks < 65536 ? blocks : 65536)), dim3(256), 0, st,
                           (const U *)src, (U *)dst, n, ctl);
        return hipGetLastError();
    };
    // 16 bytes per lane where the caller's state allows it
    return (((uintptr_t)src | (uintptr_t)dst | bytes) & 15) ? go(0.0f) : go(float4{});
}

template <typename T>
static hipError_t rate_t(const StageDesc &d, const void *q, Ctl *ctl, unsigned long long *rates, int slot,
                         hipStream_t st)
{
    int n = d.nx * d.ny;
    int blocks = (n + 255) / 256;
    if (blocks > 2048) blocks = 2048;
    Phys<T> ph{(T)d.g, (T)__builtin_sqrt(d.g), (T)d.gamma, T(0)};
    if (d.eqn == EULER)
        hipLaunchKernelGGL((rate_kernel<T, EULER>), dim3(blocks), dim3(256), 0, st, (const T *)q, n, (T)d.rdx,
                           (T)d.rdy, ph, ctl, rates, slot);
    else
        hipLaunchKernelGGL((rate_kernel<T, SWE>), dim3(blocks), dim3(256), 0, st, (const T *)q, n, (T)d.rdx,
                           (T)d.rdy, ph, ctl, rates, slot);
    return hipGetLastError();
}

// A single solve's kernel in every shape; the lists' in theirs, with a bed
// under shallow water (a flat one is a bed of zeros).
template <int EQN, bool BATHY, int STAGE, int SHAPE> static const void *one_kernel(int *threads)
{
    *threads = ShapeLds<float, EQN, BATHY, SHAPE>::NTH;
    return (const void *)batch_stage_one_kernel<float, EQN, BATHY, STAGE, SHAPE>;
}
template <int EQN, bool BATHY, int STAGE> static const void *one_kernel_e(int shape, int *threads)
{
    switch (shape) {
    case 0: return one_kernel<EQN, BATHY, STAGE, 0>(threads);
    case 1: return one_kernel<EQN, BATHY, STAGE, 1>(threads);
    case 2: return one_kernel<EQN, BATHY, STAGE, 2>(threads);
    default: return one_kernel<EQN, BATHY, STAGE, 3>(threads);
    }
}

hipError_t launch_batch_stage_one(int eqn, int bathy, int stage, int shape, const BatchSolve &d, const WorkItem &it,
                                  int grid, hipStream_t st)
{
    if (grid <= 0) return hipSuccess;
    if (it.tile_begin != 0 || shape < 0 || shape >= NSHAPES) return hipErrorInvalidValue;
    int threads;
    const void *fn;
    if (eqn == EULER)
        fn = stage == 1 ? one_kernel_e<EULER, false, 1>(shape, &threads) : one_kernel_e<EULER, false, 2>(shape, &threads);
    else if (bathy)
        fn = stage == 1 ? one_kernel_e<SWE, true, 1>(shape, &threads) : one_kernel_e<SWE, true, 2>(shape, &threads);
    else
        fn = stage == 1 ? one_kernel_e<SWE, false, 1>(shape, &threads) : one_kernel_e<SWE, false, 2>(shape, &threads);
    void *args[] = {(void *)&d, (void *)&it, (void *)&grid};
    return hipLaunchKernel(fn, dim3(xcd_grid(grid)), dim3(threads), args, 0, st);
}

template <int EQN, bool BATHY>
static hipError_t go_list(int stage, const BatchSolve *solves, const WorkItem *items, const int *nitems, int ntiles,
                          int wgs, hipStream_t st)
{
    const dim3 grid(wgs), blk(ShapeLds<float, EQN, BATHY, LIST_SHAPE>::NTH);
    if (stage == 1)
        hipLaunchKernelGGL((batch_stage_kernel<float, EQN, BATHY, 1, LIST_SHAPE>), grid, blk, 0, st, solves, items,
                           nitems, ntiles);
    else
        hipLaunchKernelGGL((batch_stage_kernel<float, EQN, BATHY, 2, LIST_SHAPE>), grid, blk, 0, st, solves, items,
                           nitems, ntiles);
    return hipGetLastError();
}

hipError_t launch_batch_stage(int eqn, int stage, const BatchSolve *solves, const WorkItem *items, const int *nitems,
                              int grid, hipStream_t st)
{
    if (grid <= 0) return hipSuccess;
    return eqn == EULER ? go_list<EULER, false>(stage, solves, items, nitems, grid, xcd_grid(grid), st)
                        : go_list<SWE, true>(stage, solves, items, nitems, grid, xcd_grid(grid), st);
}

hipError_t launch_batch_stage_list(int eqn, int stage, const BatchSolve *solves, const WorkItem *items, const int *list,
                                   int wgs, hipStream_t st)
{
    if (wgs <= 0 || (wgs & 7)) return hipErrorInvalidValue;
    return eqn == EULER ? go_list<EULER, false>(stage, solves, items, list, 0, wgs, st)
                        : go_list<SWE, true>(stage, solves, items, list, 0, wgs, st);
}

hipError_t launch_rate(const StageDesc &d, const void *q, Ctl *ctl, unsigned long long *rates, int slot,
                       hipStream_t st)
{
    return d.prec == 1 ? rate_t<double>(d, q, ctl, rates, slot, st) : rate_t<float>(d, q, ctl, rates, slot, st);
}

template <typename T>
static hipError_t totals_t(const StageDesc &d, const void *q, double *partials, int max_blocks, double *out,
                           hipStream_t st)
{
    int n = d.nx * d.ny;
    int blocks = (n + 255) / 256;
    if (blocks > max_blocks) blocks = max_blocks;
    double dA = 1.0 / (d.rdx * d.rdy);
    int nv = d.eqn == EULER ? 4 : 3;
    if (d.eqn == EULER)
        hipLaunchKernelGGL((totals_partial_kernel<T, EULER>), dim3(blocks), dim3(256), 0, st, (const T *)q, n, dA,
                           d.g, partials);
    else
        hipLaunchKernelGGL((totals_partial_kernel<T, SWE>), dim3(blocks), dim3(256), 0, st, (const T *)q, n, dA,
                           d.g, partials);
    hipLaunchKernelGGL(totals_final_kernel, dim3(nv + 1), dim3(256), 0, st, partials, blocks, nv + 1, out);
    return hipGetLastError();
}

hipError_t launch_totals(const StageDesc &d, const void *q, double *partials, int max_blocks, double *out_dev,
                         hipStream_t st)
{
    return d.prec == 1 ? totals_t<double>(d, q, partials, max_blocks, out_dev, st)
                       : totals_t<float>(d, q, partials, max_blocks, out_dev, st);
}

template <typename T, int EQN, int FLUX>
static hipError_t face_r(const StageDesc &d, const void *q, void *fx, void *fy, hipStream_t st)
{
    int nf = (d.nx + 1) * d.ny + d.nx * (d.ny + 1);
    Phys<T> ph{(T)d.g, (T)__builtin_sqrt(d.g), (T)d.gamma, T(0)};  // exported fluxes carry the full pressure
    dim3 grid((nf + 255) / 256);
    if (d.recon == FIRST)
        hipLaunchKernelGGL((face_kernel<T, EQN, FLUX, FIRST>), grid, dim3(256), 0, st, (const T *)q, d.nx, d.ny,
                           d.bc_x, d.bc_y, ph, (T *)fx, (T *)fy);
    else
        hipLaunchKernelGGL((face_kernel<T, EQN, FLUX, MINMOD>), grid, dim3(256), 0, st, (const T *)q, d.nx, d.ny,
                           d.bc_x, d.bc_y, ph, (T *)fx, (T *)fy);
    return hipGetLastError();
}

template <typename T, int EQN>
static hipError_t face_f(const StageDesc &d, const void *q, void *fx, void *fy, hipStream_t st)
{
    switch (d.flux) {
    case RUSANOV: return face_r<T, EQN, RUSANOV>(d, q, fx, fy, st);
    case ROE: return face_r<T, EQN, ROE>(d, q, fx, fy, st);
    default: return face_r<T, EQN, HLLE>(d, q, fx, fy, st);
    }
}

template <typename T>
static hipError_t face_p(const StageDesc &d, const void *q, void *fx, void *fy, hipStream_t st)
{
    return d.eqn == EULER ? face_f<T, EULER>(d, q, fx, fy, st) : face_f<T, SWE>(d, q, fx, fy, st);
}

hipError_t launch_face_fluxes(const StageDesc &d, const void *q, void *fx, void *fy, hipStream_t st)
{
    return d.prec == 1 ? face_p<double>(d, q, fx, fy, st) : face_p<float>(d, q, fx, fy, st);
}

}  // namespace fvk
