// Steps in one launch.  Every system and precision is a file of its own: the
// runtime loads a file's kernels together when the first of them is asked for
// (a process's first solve, of a grid that does not step so, took 11.7 ms with
// all of them in one file with the stage kernels, 4.9 ms so).
#pragma once

#include "stage_device.hpp"

#include <type_traits>

namespace fvk {

// ---------------------------------------------------- a step in one launch
// All S stages of a tile of step_cols(S) x TY cells in one workgroup, from one
// buffer to another: stage k on the tile and its 2 (S - k)-cell ring (64
// columns in the first, a wave64 per row), its result in LDS as the next
// stage's halo tile.  Ghost cells of a result past a wall are mirrored from
// it, as the next stage's loads would mirror them; past a periodic border they
// are computed from the same values as their images.  The same arithmetic as
// a launch per stage, so the same bits.  A frozen solve's cells are carried
// over.  On small grids a launch is its chain (start, load, two barriers,
// store) and little work: 16 Heun steps over a bed, a launch per stage and
// one: 64^2 128 and 95 us, 256^2 131 and 103, 400^2 160 and 115, 600^2 192 and
// 143.
constexpr int step_cols(int s) { return 64 - 4 * (s - 1); }

// Stage K's results to LDS, all of them; q0 from the first stage's halo tile.
template <typename T, int K, typename L1, typename L2> struct RingIO {
    static constexpr bool GLOBAL = false;
    const L1 &from;
    L2 &to;
    __device__ __forceinline__ bool in(int, int) const { return true; }
    __device__ __forceinline__ T q0(int v, int cy, int lane) const
    {
        return from.q[v][cy + 2 * K][min(lane + 2 * K, L1::HX - 1)];
    }
    __device__ __forceinline__ void put(int v, int cy, int lane, T o) const { to.q[v][cy][lane] = o; }
    __device__ __forceinline__ void keep(int cy, int lane, const T *) const
    {
#pragma unroll
        for (int v = 0; v < L1::NV; v++) to.q[v][cy][lane] = T(0);
    }
};
// The last stage's (K of K).
template <typename T, int K, typename L1> struct StepIO {
    static constexpr bool GLOBAL = false;
    const StageArgs<T> &a;
    const L1 &from;
    int x0, y0;
    __device__ __forceinline__ bool in(int cy, int lane) const
    {
        return lane < step_cols(K) && x0 + lane < a.nx && y0 + cy < a.ny;
    }
    __device__ __forceinline__ T q0(int v, int cy, int lane) const
    {
        return from.q[v][cy + 2 * K][min(lane + 2 * K, L1::HX - 1)];
    }
    __device__ __forceinline__ void put(int v, int cy, int lane, T o) const
    {
        *st_off(a.out + v * ((size_t)a.nx * a.ny) + (size_t)y0 * a.nx + x0, (unsigned)(cy * a.nx + lane)) = o;
    }
    __device__ __forceinline__ void keep(int cy, int lane, const T *) const
    {
#pragma unroll
        for (int v = 0; v < L1::NV; v++) put(v, cy, lane, q0(v, cy, lane));
    }
};

// This lane's cell of a stage's region from (ox, oy): its image in the grid
// and the bed there.
template <typename T, bool BATHY> struct RingCell {
    int gx, gy;
    bool fx = false, fy = false;
    T bed = T(0);
    __device__ __forceinline__ void set(const StageArgs<T> &a, int ox, int oy, int wave, int lane)
    {
        gx = ghost_index(ox + lane, a.nx, a.bc_x, fx);
        gy = ghost_index(oy + wave, a.ny, a.bc_y, fy);
        if (BATHY) bed = ld_off(a.bed + (size_t)gy * a.nx, (unsigned)gx);
    }
};

// A stage's result in `to` (ROWS x 64 places from (ox, oy), a wave per row)
// made the next stage's halo tile: the free surface, and in a cell past a wall
// its image's values with the normal momentum negated.  Every wave calls it.
template <typename T, bool BATHY, int ROWS, typename L>
__device__ __forceinline__ void ring_close(const StageArgs<T> &a, const RingCell<T, BATHY> &r, L &to, int ox, int oy,
                                           int wave, int lane)
{
    constexpr int NV = L::NV;
    __syncthreads();
    T m[NV];
    if (wave < ROWS) {
        const int lx = r.fx ? min(max(r.gx - ox, 0), 63) : lane, ly = r.fy ? min(max(r.gy - oy, 0), ROWS - 1) : wave;
#pragma unroll
        for (int v = 0; v < NV; v++) m[v] = to.q[v][ly][lx];
        m[1] = r.fx ? -m[1] : m[1];
        m[2] = r.fy ? -m[2] : m[2];
        if constexpr (BATHY) to.q[NV][wave][lane] = m[0] + r.bed;
    }
    if ((a.bc_x != 0 || a.bc_y != 0) && !(ox >= 0 && oy >= 0 && ox + 64 <= a.nx && oy + ROWS <= a.ny)) {
        __syncthreads();  // a cell's image may be another wave's
        if (wave < ROWS) {
#pragma unroll
            for (int v = 0; v < NV; v++) to.q[v][wave][lane] = m[v];
        }
    }
    __syncthreads();
}

template <typename T, int EQN, bool BATHY, int FLUX, int RECON, int S, int TY>
__global__ __launch_bounds__(64 * (TY + 4 * (S - 1))) void step_kernel(StageArgs<T> a, int tiles_x, int ntiles)
{
    constexpr int R1 = TY + 4 * (S - 1);  // rows of the first stage, a wave each
    using L1 = StageLds<T, EQN, BATHY, 64, R1, 1>;
    __shared__ L1 s1;
    const int w = xcd_tile(blockIdx.x, gridDim.x);
    if (w >= ntiles) return;
    const int ty = w / tiles_x, tx = w - ty * tiles_x;
    const int x0 = tx * step_cols(S), y0 = ty * TY;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    auto weights = [&](double a0, double a1, int last) {
        StageArgs<T> b = a;
        b.a0 = (T)a0;
        b.a1 = (T)a1;
        b.last = last;
        return b;
    };
    const StageArgs<T> e1 = weights(0.0, 1.0, S == 1);
    const int o1 = 2 * (S - 1);  // the first stage's ring
    RingCell<T, BATHY> c1, c2;
    auto load = [&] {
        HaloRegs<T, EQN, BATHY, 64, R1, 1> r;
        if (inner_tile<64, R1>(x0 - o1, y0 - o1, a.nx, a.ny))
            halo_issue<T, EQN, BATHY, 64, R1, 1, false>(e1, x0 - o1, y0 - o1, tid, r);
        else
            halo_issue<T, EQN, BATHY, 64, R1, 1, true>(e1, x0 - o1, y0 - o1, tid, r);
        if (S > 1) c1.set(a, x0 - o1, y0 - o1, wave, lane);
        if (S > 2) c2.set(a, x0 - 2, y0 - 2, wave, lane);
        stage_dt(e1, tid, s1);
        halo_commit(r, s1, tid);
        __syncthreads();
    };
    if constexpr (S == 1) {
        load();
        stage_compute<T, EQN, BATHY, FLUX, RECON, 64, R1, 1>(e1, StepIO<T, 1, L1>{a, s1, x0, y0}, w, tid, s1);
    } else {
        using L2 = StageLds<T, EQN, BATHY, 64, R1 - 4, 1>;
        __shared__ L2 s2;
        if constexpr (S == 2) {
            load();
            if (tid == 0) s2.dt = s1.dt;
            stage_compute<T, EQN, BATHY, FLUX, RECON, 64, R1, 1>(e1, RingIO<T, 1, L1, L2>{s1, s2}, w, tid, s1);
            ring_close<T, BATHY, R1>(a, c1, s2, x0 - o1, y0 - o1, wave, lane);
            if (wave < TY)
                stage_compute<T, EQN, BATHY, FLUX, RECON, 64, TY, 1>(weights(0.5, 0.5, 1), StepIO<T, 2, L1>{a, s1, x0, y0},
                                                                     w, tid, s2);
            else
                __syncthreads();  // stage_compute's
        } else {
            using L3 = StageLds<T, EQN, BATHY, 64, TY, 1>;
            __shared__ L3 s3;
            load();
            if (tid == 0) s2.dt = s3.dt = s1.dt;
            stage_compute<T, EQN, BATHY, FLUX, RECON, 64, R1, 1>(e1, RingIO<T, 1, L1, L2>{s1, s2}, w, tid, s1);
            ring_close<T, BATHY, R1>(a, c1, s2, x0 - o1, y0 - o1, wave, lane);
            if (wave < R1 - 4)
                stage_compute<T, EQN, BATHY, FLUX, RECON, 64, R1 - 4, 1>(weights(0.75, 0.25, 0),
                                                                         RingIO<T, 2, L1, L3>{s1, s3}, w, tid, s2);
            else
                __syncthreads();
            ring_close<T, BATHY, R1 - 4>(a, c2, s3, x0 - 2, y0 - 2, wave, lane);
            if (wave < TY)
                stage_compute<T, EQN, BATHY, FLUX, RECON, 64, TY, 1>(weights(1.0 / 3.0, 2.0 / 3.0, 1),
                                                                     StepIO<T, 3, L1>{a, s1, x0, y0}, w, tid, s3);
            else
                __syncthreads();
        }
    }
}

// The tile rows of a step's launch: the fewest whose tiles all get a CU of
// their own, else the most (least of the earlier stages computed twice).
template <typename T, int EQN, bool BATHY, int FLUX, int RECON, int S>
static hipError_t step_s(const StageDesc &d, const StageArgs<T> &a, hipStream_t st)
{
    auto go = [&](auto rows) {
        constexpr int TY = decltype(rows)::value;
        const int tiles_x = (d.nx + step_cols(S) - 1) / step_cols(S), ntiles = tiles_x * ((d.ny + TY - 1) / TY);
        hipLaunchKernelGGL((step_kernel<T, EQN, BATHY, FLUX, RECON, S, TY>), dim3(xcd_grid(ntiles)),
                           dim3(64 * (TY + 4 * (S - 1))), 0, st, a, tiles_x, ntiles);
        return hipGetLastError();
    };
    const int most = step_rows(d, S);
    const int64_t cols = (d.nx + step_cols(S) - 1) / step_cols(S);
    const bool four = cols * ((d.ny + 3) / 4) <= CUS, eight = cols * ((d.ny + 7) / 8) <= CUS;
    if (four || most == 4) return go(std::integral_constant<int, 4>{});
    if constexpr (S == 2 || (S == 3 && sizeof(T) == 4)) {
        if constexpr (S == 2 && sizeof(T) == 4 && FLUX == HLLE && RECON == MINMOD)
            if (!eight) return go(std::integral_constant<int, 12>{});
        return go(std::integral_constant<int, 8>{});
    }
    return hipErrorInvalidValue;
}

template <typename T, int EQN, bool BATHY, int FLUX>
static hipError_t step_f(const StageDesc &d, int stages, const StageArgs<T> &a, hipStream_t st)
{
#define FV_STEP(RC)                                                                        \
    (stages == 1   ? step_s<T, EQN, BATHY, FLUX, RC, 1>(d, a, st)                          \
     : stages == 2 ? step_s<T, EQN, BATHY, FLUX, RC, 2>(d, a, st)                          \
                   : step_s<T, EQN, BATHY, FLUX, RC, 3>(d, a, st))
    return d.recon == FIRST ? FV_STEP(FIRST) : FV_STEP(MINMOD);
#undef FV_STEP
}

template <typename T, int EQN, bool BATHY>
static hipError_t step_e(const StageDesc &d, int stages, const StageArgs<T> &a, hipStream_t st)
{
    return d.flux == RUSANOV ? step_f<T, EQN, BATHY, RUSANOV>(d, stages, a, st)
           : d.flux == ROE   ? step_f<T, EQN, BATHY, ROE>(d, stages, a, st)
                             : step_f<T, EQN, BATHY, HLLE>(d, stages, a, st);
}

template <typename T, int EQN>
hipError_t step_go(const StageDesc &d, int stages, const StageArgs<T> &a, hipStream_t st)
{
    if constexpr (EQN == EULER) return step_e<T, EULER, false>(d, stages, a, st);
    else return d.bathy ? step_e<T, SWE, true>(d, stages, a, st) : step_e<T, SWE, false>(d, stages, a, st);
}

template <typename T, int EQN> hipError_t step_load()
{
    hipFuncAttributes at;
    return hipFuncGetAttributes(&at, (const void *)step_kernel<T, EQN, EQN == SWE, HLLE, MINMOD, 2, 4>);
}

}  // namespace fvk
