// Stage arithmetic of one tile, shared by the launch-per-stage and the
// step-per-launch kernels (fv_kernels.hip describes the split of the work).
#pragma once

#include "fv_device.hpp"
#include "fv_internal.hpp"

namespace fvk {

template <typename T> struct StageArgs {
    const T *qs;
    const T *q0;
    T *out;
    const T *bed;
    int nx, ny, bc_x, bc_y;
    T rdx, rdy;
    Phys<T> ph;
    T a0, a1;
    double cfl, dt_fixed;
    Ctl *ctl;
    unsigned long long *rates;
    int rate_in, rate_out, rate_clear, last;
    int own;  // the Bad bit that this launch raises (0: it does not end a step)
};

// Global-memory view of a pointer.  The batched kernels read their array
// pointers from a device descriptor, where the compiler cannot see that they
// address global memory; it would then emit flat accesses, which may alias
// LDS and so are ordered behind every LDS store.
template <typename T> using gmem = __attribute__((address_space(1))) T;
template <typename T> __device__ __forceinline__ const gmem<T> *gload(const T *p) { return (const gmem<T> *)p; }
template <typename T> __device__ __forceinline__ gmem<T> *gstore(T *p) { return (gmem<T> *)p; }
// base[i] for a wave-uniform base and a byte offset that fits in 32 bits:
// the address is then an SGPR pair plus a 32-bit VGPR offset, with no 64-bit
// arithmetic per element.
// The base goes through readfirstlane so that the compiler keeps it in
// SGPRs instead of folding a uniform offset into every lane's address.
template <typename T> __device__ __forceinline__ T *sbase(T *p)
{
    const unsigned long long u = (unsigned long long)p;
    const unsigned lo = __builtin_amdgcn_readfirstlane((unsigned)u);
    const unsigned hi = __builtin_amdgcn_readfirstlane((unsigned)(u >> 32));
    return (T *)(((unsigned long long)hi << 32) | lo);
}
template <typename T> __device__ __forceinline__ T ld_off(const T *base, unsigned i)
{
    return *(const gmem<T> *)((const char *)sbase(base) + i * (unsigned)sizeof(T));
}
template <typename T> __device__ __forceinline__ gmem<T> *st_off(T *base, unsigned i)
{
    return (gmem<T> *)((char *)sbase(base) + i * (unsigned)sizeof(T));
}

template <typename T> __device__ __forceinline__ T wave_max(T v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = tmax(v, __shfl_xor(v, off, 64));
    return v;
}

__device__ __forceinline__ void push_rate(unsigned long long *rates, int k, double m, int block_linear)
{
    atomicMax(rate_slot(rates, k, block_linear & (RATE_SUB - 1)), (unsigned long long)__double_as_longlong(m));
}

// Max over a wave of non-negative values, in every lane.  Non-negative
// floats order like their bit patterns, so the float path reduces unsigned
// integers with DPP row shifts (lane 15 of each 16-lane row ends with its
// row's max) and combines the four rows with lane reads.
template <int CTRL> __device__ __forceinline__ unsigned dpp_u(unsigned x)
{
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xf, 0xf, false);  // lanes with no source read 0
}
__device__ __forceinline__ float wave_max_nonneg(float v)
{
    unsigned x = __float_as_uint(v);
    x = max(x, dpp_u<0x111>(x));  // row_shr:1
    x = max(x, dpp_u<0x112>(x));  // row_shr:2
    x = max(x, dpp_u<0x114>(x));  // row_shr:4
    x = max(x, dpp_u<0x118>(x));  // row_shr:8
    const unsigned a = max((unsigned)__builtin_amdgcn_readlane((int)x, 15), (unsigned)__builtin_amdgcn_readlane((int)x, 31));
    const unsigned b = max((unsigned)__builtin_amdgcn_readlane((int)x, 47), (unsigned)__builtin_amdgcn_readlane((int)x, 63));
    return __uint_as_float(max(a, b));
}
// The same for non-negative doubles, as 64-bit patterns in two halves (no
// lane-index arithmetic, so nothing stays live across a workgroup's tiles).
template <int CTRL> __device__ __forceinline__ unsigned long long dpp_u64(unsigned long long x)
{
    return (unsigned long long)dpp_u<CTRL>((unsigned)(x >> 32)) << 32 | dpp_u<CTRL>((unsigned)x);
}
__device__ __forceinline__ unsigned long long readlane_u64(unsigned long long x, int l)
{
    return (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)(x >> 32), l) << 32 |
           (unsigned)__builtin_amdgcn_readlane((int)x, l);
}
__device__ __forceinline__ unsigned long long umax64(unsigned long long a, unsigned long long b) { return a > b ? a : b; }
__device__ __forceinline__ double wave_max_nonneg(double v)
{
    unsigned long long x = (unsigned long long)__double_as_longlong(v);
    x = umax64(x, dpp_u64<0x111>(x));
    x = umax64(x, dpp_u64<0x112>(x));
    x = umax64(x, dpp_u64<0x114>(x));
    x = umax64(x, dpp_u64<0x118>(x));
    const unsigned long long a = umax64(readlane_u64(x, 15), readlane_u64(x, 31));
    const unsigned long long b = umax64(readlane_u64(x, 47), readlane_u64(x, 63));
    return __longlong_as_double((long long)umax64(a, b));
}

// Largest CFL rate stored in slot k (max over its sub-slots, all >= 0),
// wave-uniform.
static_assert(RATE_SUB == 64, "one sub-slot per lane");
__device__ __forceinline__ double read_rate(unsigned long long *rates, int k, int lane)
{
    return wave_max_nonneg(__longlong_as_double(*gload(rate_slot(rates, k, lane))));
}

// Block-wide max of v (threads 0..255) -> returned in thread 0.
template <typename T> __device__ __forceinline__ T block_max256(T v, T *red)
{
    v = wave_max(v);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    T m = red[0];
#pragma unroll
    for (int w = 1; w < 4; w++) m = tmax(m, red[w]);
    return m;
}

// Lane l receives v from lane l + 1 of its wave (DPP wave shift); lane 63
// receives `edge`.  Every lane of the wave must be active.
__device__ __forceinline__ float from_right(float v, float edge)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(edge), __float_as_int(v), 0x130, 0xf, 0xf, false));
}
__device__ __forceinline__ double from_right(double v, double edge)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned long long e = (unsigned long long)__double_as_longlong(edge);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp((int)(unsigned)e, (int)(unsigned)b, 0x130, 0xf, 0xf, false);
    const unsigned hi =
        (unsigned)__builtin_amdgcn_update_dpp((int)(unsigned)(e >> 32), (int)(unsigned)(b >> 32), 0x130, 0xf, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// LDS of one stage tile: the halo tile of every variable (and eta), the
// faces handed between waves, and the step's Delta t.
template <typename T, int EQN, bool BATHY, int TX, int TY, int RPW_> struct StageLds {
    static constexpr int RPW = RPW_;          // tile rows per wave
    static constexpr int NW = TY / RPW;       // waves per workgroup
    static constexpr int NTH = 64 * NW;       // threads per workgroup
    static_assert(TX == 64 && TY % RPW == 0 && NW >= 2 && NW <= 16, "a tile row is one wave64; whole rows, 2..16 waves");
    static constexpr int NV = EQN == SWE ? 3 : 4;
    static constexpr int NL = NV + (BATHY ? 1 : 0);  // LDS planes: variables (+ eta)
    static constexpr int HX = TX + 4, HY = TY + 4;
    static constexpr int NIT = (HY + NW - 1) / NW;   // halo rows per wave
    // the waves that stage the last four columns: those without a last row if they are enough
    static constexpr int XT0 = 64 * (HY % NW) + 4 * HY <= NTH ? 64 * (HY % NW) : 0;
    static_assert(4 * HY <= NTH, "one pass stages the last four columns");
    T q[NL][HY][HX];
    T edge[NV][TY];         // right face of column TX-1, handed to that cell
    T low[NW - 1][NV][TX];  // low y face of wave w+1's first row, handed to wave w
    double dt;
};

// A tile whose two-cell halo lies inside the grid (all but the border tiles)
// loads without ghost synthesis.
template <int TX, int TY> __device__ __forceinline__ bool inner_tile(int x0, int y0, int nx, int ny)
{
    return x0 >= 2 && y0 >= 2 && x0 + TX + 2 <= nx && y0 + TY + 2 <= ny;
}

// The grid index of ghost or inner index i (i >= -2), and whether it is a
// wall's mirror image.  Indices past the ghost layer, in the last tile's
// overhang, give some index of the grid; their cells are never used.
__device__ __forceinline__ int ghost_index(int i, int n, int bc, bool &flip)
{
    flip = bc != 0 && (i < 0 || i >= n);
    const int lo = bc == 0 ? i + n : -1 - i;
    const int hi = bc == 0 ? min(i - n, n - 1) : max(2 * n - 1 - i, 0);
    return i < 0 ? lo : (i >= n ? hi : i);
}

// The halo tile's values held in registers between the issue of their loads
// and their store to LDS.
template <typename T, int EQN, bool BATHY, int TX, int TY, int RPW> struct HaloRegs {
    using L = StageLds<T, EQN, BATHY, TX, TY, RPW>;
    T row[L::NIT][L::NL];  // halo row wave + it * NW, column lane
    T tail[L::NL];         // one element of the last four columns
};

// Issue every load of the halo tile (no LDS access, no wait).  A wave loads
// whole rows, so a row's address is scalar and its column offset is the same
// in every pass; border tiles map the row (scalar) and the column (once per
// lane) to the wrapped or mirrored cell, and cost no further pass.
template <typename T, int EQN, bool BATHY, int TX, int TY, int RPW, bool BORDER>
__device__ __forceinline__ void halo_issue(const StageArgs<T> &a, const int x0, const int y0, const int tid,
                                           HaloRegs<T, EQN, BATHY, TX, TY, RPW> &r)
{
    using L = StageLds<T, EQN, BATHY, TX, TY, RPW>;
    const int nx = a.nx, ny = a.ny;
    const size_t plane = (size_t)nx * ny;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    bool fx = false, fy = false;
    const unsigned col = BORDER ? (unsigned)ghost_index(x0 - 2 + lane, nx, a.bc_x, fx) : (unsigned)lane;
#pragma unroll
    for (int it = 0; it < L::NIT; it++) {
        const int ly = wave + it * L::NW;
        if (L::HY % L::NW != 0 && it == L::NIT - 1 && ly >= L::HY) break;
        const int gy = y0 - 2 + ly;
        const size_t base = BORDER ? (size_t)ghost_index(gy, ny, a.bc_y, fy) * nx : (size_t)gy * nx + (x0 - 2);
#pragma unroll
        for (int v = 0; v < L::NV; v++) r.row[it][v] = ld_off(a.qs + v * plane + base, col);
        if constexpr (BATHY) r.row[it][L::NV] = ld_off(a.bed + base, col);
        if (BORDER) {
            r.row[it][1] = fx ? -r.row[it][1] : r.row[it][1];
            r.row[it][2] = fy ? -r.row[it][2] : r.row[it][2];
        }
    }
    const int te = tid - L::XT0;
    if (te >= 0 && te < 4 * L::HY) {
        const int ly = te >> 2, gx = x0 + TX - 2 + (te & 3);
        if (BORDER) {
            const size_t idx = (size_t)ghost_index(y0 - 2 + ly, ny, a.bc_y, fy) * nx + ghost_index(gx, nx, a.bc_x, fx);
#pragma unroll
            for (int v = 0; v < L::NV; v++) r.tail[v] = gload(a.qs)[v * plane + idx];
            if constexpr (BATHY) r.tail[L::NV] = gload(a.bed)[idx];
        } else {
            const size_t base = (size_t)(y0 - 2) * nx;
            const unsigned off = (unsigned)(ly * nx + gx);
#pragma unroll
            for (int v = 0; v < L::NV; v++) r.tail[v] = ld_off(a.qs + v * plane + base, off);
            if constexpr (BATHY) r.tail[L::NV] = ld_off(a.bed + base, off);
        }
        if (BORDER) {
            r.tail[1] = fx ? -r.tail[1] : r.tail[1];
            r.tail[2] = fy ? -r.tail[2] : r.tail[2];
        }
    }
}

template <typename T, int EQN, bool BATHY, int TX, int TY, int RPW>
__device__ __forceinline__ void halo_commit(const HaloRegs<T, EQN, BATHY, TX, TY, RPW> &r,
                                            StageLds<T, EQN, BATHY, TX, TY, RPW> &sh, const int tid)
{
    using L = StageLds<T, EQN, BATHY, TX, TY, RPW>;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
#pragma unroll
    for (int it = 0; it < L::NIT; it++) {
        const int ly = wave + it * L::NW;
        if (L::HY % L::NW != 0 && it == L::NIT - 1 && ly >= L::HY) break;
#pragma unroll
        for (int v = 0; v < L::NV; v++) sh.q[v][ly][lane] = r.row[it][v];
        if constexpr (BATHY) sh.q[L::NV][ly][lane] = r.row[it][0] + r.row[it][L::NV];
    }
    const int te = tid - L::XT0;
    if (te >= 0 && te < 4 * L::HY) {
#pragma unroll
        for (int v = 0; v < L::NV; v++) sh.q[v][te >> 2][TX + (te & 3)] = r.tail[v];
        if constexpr (BATHY) sh.q[L::NV][te >> 2][TX + (te & 3)] = r.tail[0] + r.tail[L::NV];
    }
}

// Delta t of the step = CFL / (max over the previous step's rate sub-slots),
// read by wave 1 into LDS.
template <typename T, int EQN, bool BATHY, int TX, int TY, int RPW>
__device__ __forceinline__ void stage_dt(const StageArgs<T> &a, const int tid,
                                         StageLds<T, EQN, BATHY, TX, TY, RPW> &sh)
{
    if ((tid >> 6) == 1) {
        const int lane = tid & 63;
        const double d = a.dt_fixed > 0.0 ? a.dt_fixed : a.cfl / read_rate(a.rates, a.rate_in, lane);
        if (lane == 0) sh.dt = d;
    }
}

// Where a stage's cells come from and go: the global arrays of its arguments.
template <typename T, int EQN> struct StageIO {
    static constexpr bool GLOBAL = true;
    const StageArgs<T> &a;
    int x0, y0;
    size_t tbase;
    __device__ __forceinline__ bool in(int cy, int lane) const { return x0 + lane < a.nx && y0 + cy < a.ny; }
    __device__ __forceinline__ T q0(int v, int cy, int lane) const
    {
        const unsigned off = in(cy, lane) ? (unsigned)(cy * a.nx + lane) : 0u;
        return ld_off(a.q0 + v * ((size_t)a.nx * a.ny) + tbase, off);
    }
    __device__ __forceinline__ void put(int v, int cy, int lane, T o) const
    {
        __builtin_nontemporal_store(o, st_off(a.out + v * ((size_t)a.nx * a.ny) + tbase, (unsigned)(cy * a.nx + lane)));
    }
    __device__ __forceinline__ void keep(int, int, const T *) const {}
};

// One RK stage on the TX x TY tile at (x0, y0) whose halo, faces and Delta t
// are staged in `sh` (after a barrier).  `tile_linear` is the tile's index
// within its solve; the tile with index 0 does the per-step bookkeeping of
// the solve.  Shared by every stage kernel, so a solve computes bit-identical
// results in all of them.
//
// Work split: lane = column, wave w owns tile rows RPW w .. RPW w + RPW - 1.
// Each lane evaluates the low x face and the low y face of each of its cells, so
// face results stay in registers: the high x face arrives from lane + 1 by a
// DPP shift, the high y face from the same lane's next row.  Faces with no
// owner inside the wave are the tile's right column (one lane per row, wave
// 0, through LDS), the tile's top row (last wave) and the low face of each
// wave's first row, which the wave below reads through LDS.
// Bound by vector-ALU issue and, a grid of one round of tiles, by the wait for
// its halos: 229 and 253 lane instructions per cell in the two stages of
// shallow water over a bed (270 and 299 before the faces shared their
// reconstruction and the flux was rearranged) keep the SIMDs busy for 62 % of
// the traced kernels at 1024^2; a wave waits 44 % of its time for loads and
// barriers.  1024^2 21.8 -> 20.6 us a step, 2048^2 76.2 -> 63.6, Euler 1000 x
// 700 26.6 -> 20.9; by latency on small grids (64^2 13.7 -> 8.1).
template <typename T, int EQN, bool BATHY, int FLUX, int RECON, int TX, int TY, int RPW, typename IO>
__device__ __forceinline__ void stage_compute(const StageArgs<T> &a, const IO &io, const int tile_linear, const int tid,
                                              StageLds<T, EQN, BATHY, TX, TY, RPW> &sh)
{
#pragma clang fp contract(off)
    using LD = StageLds<T, EQN, BATHY, TX, TY, RPW>;
    constexpr int NW = LD::NW;
    constexpr int NV = LD::NV, NL = LD::NL;
    constexpr int ES = BATHY ? NL - 1 : 0;  // plane of the free surface (flat bottom: the depth)
    auto &s_q = sh.q;
    auto &s_edge = sh.edge;
    auto &s_low = sh.low;

    // An earlier step failed: the state is frozen.  The flag is checked only
    // where something would be written, so its load is off the critical path.
    // Its bits but the launch's own do not change from none to some while the
    // launch runs: every workgroup and every stage of a step sees the same.
    const bool frozen = (gload(a.ctl)->bad & ~a.own) != 0;
    const int lane = tid & 63, wave = tid >> 6;
    const int r0 = wave * RPW;
    const T dt = (T)sh.dt;
    // stage weight times Delta t over the cell width, per axis
    const T cxs = a.a1 * dt * a.rdx, cys = a.a1 * dt * a.rdy;

    // 2. faces with no owner lane: the tile's right column
    if (wave == 0 && lane < TY) {
        T c[NL][4], F[NV], nr, slope;
#pragma unroll
        for (int v = 0; v < NL; v++)
#pragma unroll
            for (int k = 0; k < 4; k++) c[v][k] = s_q[v][lane + 2][TX + k];
        line_face<T, EQN, BATHY, FLUX, RECON, 0>(c, a.ph, F, nr, slope);
#pragma unroll
        for (int k = 0; k < NV; k++) s_edge[k][lane] = F[k];
    }

    // 3. y faces, from the wave's last row down: a cell's two face values are
    //    formed once, its low value kept for the face below it.  The last
    //    wave starts with the face above the tile.
    T Ly[RPW][NV];  // y flux difference; without the face above in the last row until the exchange
    {
        T qa[NL], qi[NL], d[NL];  // the row above, row i and their difference
        T lo[NL], sa[NL];         // low value and slope of the row above
        T top[NV];                // the face above the row above, seen from below
#pragma unroll
        for (int v = 0; v < NL; v++) {
            qa[v] = s_q[v][r0 + RPW + 2][lane + 2];
            qi[v] = s_q[v][r0 + RPW + 1][lane + 2];
            d[v] = qa[v] - qi[v];
        }
        if (wave == NW - 1) {
#pragma unroll
            for (int v = 0; v < NL; v++) {
                T x;
                cell_ends<T, RECON>(qa[v], d[v], s_q[v][TY + 3][lane + 2] - qa[v], lo[v], x, sa[v]);
            }
        }
#pragma unroll
        for (int i = RPW - 1; i >= -1; i--) {
            T qb[NL], db[NL], nlo[NL], hi[NL], s[NL];
#pragma unroll
            for (int v = 0; v < NL; v++) {
                qb[v] = s_q[v][r0 + i + 1][lane + 2];
                db[v] = qi[v] - qb[v];
                cell_ends<T, RECON>(qi[v], db[v], d[v], nlo[v], hi[v], s[v]);
            }
            if (i < RPW - 1 || wave == NW - 1) {
                T F[NV], nr;
                stage_face<T, EQN, BATHY, FLUX, 1>(hi, lo, qi, qa, face_jump<T, RECON>(d[ES], s[ES], sa[ES]), a.ph, F, nr);
                if (i < RPW - 1) {
                    // the face is the low face of row i + 1
                    T hs[NV];
#pragma unroll
                    for (int v = 0; v < NV; v++) hs[v] = v == 2 ? nr : F[v];
                    if constexpr (EQN == SWE) hs[2] = tfma(-(a.ph.g * qa[0]), sa[ES], hs[2]);
#pragma unroll
                    for (int v = 0; v < NV; v++)
                        Ly[i + 1][v] = i + 1 < RPW - 1 || wave == NW - 1 ? hs[v] - top[v] : hs[v];
                    if (i == -1 && wave > 0) {
#pragma unroll
                        for (int k = 0; k < NV; k++) s_low[wave - 1][k][lane] = F[k];
                    }
                }
#pragma unroll
                for (int k = 0; k < NV; k++) top[k] = F[k];
            }
#pragma unroll
            for (int v = 0; v < NL; v++) {
                qa[v] = qi[v];
                qi[v] = qb[v];
                d[v] = db[v];
                lo[v] = nlo[v];
                sa[v] = s[v];
            }
        }
    }
    __syncthreads();
    if (wave < NW - 1) {
#pragma unroll
        for (int v = 0; v < NV; v++) Ly[RPW - 1][v] -= s_low[wave][v][lane];
    }

    // 4. x faces, divergence, bed source, RK combine
    T lmax = T(0);
    bool bad = false;
#pragma unroll
    for (int j = 0; j < RPW; j++) {
        const int cy = r0 + j;
        T c[NL][4], F[NV], nr, slope, Lv[NV];
        // q0 is needed only in the combine: its latency hides behind the x face
        T q0r[NV];
        if (a.a0 != T(0)) {
#pragma unroll
            for (int v = 0; v < NV; v++) q0r[v] = io.q0(v, cy, lane);
        }
#pragma unroll
        for (int v = 0; v < NL; v++)
#pragma unroll
            for (int k = 0; k < 4; k++) c[v][k] = s_q[v][cy + 2][lane + k];
        line_face<T, EQN, BATHY, FLUX, RECON, 0>(c, a.ph, F, nr, slope);
#pragma unroll
        for (int v = 0; v < NV; v++) {
            const T rt = from_right(F[v], s_edge[v][cy]);
            T tr = v == 1 ? nr : F[v];
            if (EQN == SWE && v == 1) tr = tfma(-(a.ph.g * c[0][2]), slope, tr);
            Lv[v] = tr - rt;
        }
        const bool in = io.in(cy, lane);
        if (!IO::GLOBAL && in && frozen) io.keep(cy, lane, q0r);
        if (in && !frozen) {
            T qn[NV];
#pragma unroll
            for (int v = 0; v < NV; v++) {
                // out = a0 q0 + a1 (q + dt L), L = (x flux difference) / dx + (y flux difference) / dy;
                // the increment is summed first, so the result is rounded
                // twice at its own magnitude (once per added state)
                const T inc = tfma(cys, Ly[j][v], cxs * Lv[v]);
                T o = tfma(a.a1, c[v][2], inc);
                if (a.a0 != T(0)) o = tfma(a.a0, q0r[v], o);
                io.put(v, cy, lane, o);
                qn[v] = o;
            }
            if (a.last) {
                T r;
                if (cell_rate_ok<T, EQN>(qn, a.ph, a.rdx, a.rdy, r)) lmax = tmax(lmax, r);
                else bad = true;
            }
        }
    }
    if (frozen && tile_linear == 0 && tid == 0) atomicOr(&a.ctl->bad, BAD_SKIP);
    if (!a.last || frozen) return;
    if (bad) atomicOr(&a.ctl->bad, a.own);
    if (a.rate_out >= 0) {
        // one atomic per wave: no block-wide reduction, no further barrier
        const T m = wave_max_nonneg(lmax);
        if (lane == 0) push_rate(a.rates, a.rate_out, (double)m, tile_linear * NW + wave);
    }
    if (tile_linear == 0) {
        if (tid == 0) {
            a.ctl->t += sh.dt;
            a.ctl->step += 1;
        }
        if (a.rate_clear >= 0 && tid < RATE_SUB) *rate_slot(a.rates, a.rate_clear, tid) = 0ull;
    }
}

// One RK stage on one tile, loaded and computed by the calling workgroup.
// Every halo load is issued before the first LDS store and before the Delta t
// read, whose reduction would otherwise hold them back.
template <typename T, int EQN, bool BATHY, int FLUX, int RECON, int TX, int TY, int RPW>
__device__ __forceinline__ void stage_tile(const StageArgs<T> &a, const int x0, const int y0, const int tile_linear,
                                           const int tid)
{
    __shared__ StageLds<T, EQN, BATHY, TX, TY, RPW> sh;
    {
        HaloRegs<T, EQN, BATHY, TX, TY, RPW> r;
        if (inner_tile<TX, TY>(x0, y0, a.nx, a.ny)) halo_issue<T, EQN, BATHY, TX, TY, RPW, false>(a, x0, y0, tid, r);
        else halo_issue<T, EQN, BATHY, TX, TY, RPW, true>(a, x0, y0, tid, r);
        stage_dt(a, tid, sh);
        halo_commit(r, sh, tid);
    }
    __syncthreads();
    const StageIO<T, EQN> io{a, x0, y0, (size_t)y0 * a.nx + x0};
    stage_compute<T, EQN, BATHY, FLUX, RECON, TX, TY, RPW>(a, io, tile_linear, tid, sh);
}

// Workgroups are handed to the eight XCDs in turn (workgroup w runs on XCD
// w mod 8).  For a grid that is a multiple of 8, give XCD k the contiguous
// k-th eighth of the tiles, so that neighbouring tiles, which re-read each
// other's halo rows, share one L2.
__device__ __forceinline__ int xcd_tile(int w, int grid)
{
    return (grid & 7) ? w : (w & 7) * (grid >> 3) + (w >> 3);
}

template <typename T>
static StageArgs<T> stage_args(const StageDesc &d, const void *qs, const void *q0, void *out, const void *bed, Ctl *ctl,
                               unsigned long long *rates, int ri, int ro, int rc)
{
    StageArgs<T> a{};
    a.qs = (const T *)qs;
    a.q0 = (const T *)q0;
    a.out = (T *)out;
    a.bed = (const T *)bed;
    a.nx = d.nx;
    a.ny = d.ny;
    a.bc_x = d.bc_x;
    a.bc_y = d.bc_y;
    a.rdx = (T)d.rdx;
    a.rdy = (T)d.rdy;
    a.ph.g = (T)d.g;
    a.ph.sqg = (T)__builtin_sqrt(d.g);
    a.ph.gamma = (T)d.gamma;
    a.ph.h0 = (T)d.h0;
    a.cfl = d.cfl;
    a.dt_fixed = d.dt_fixed;
    a.ctl = ctl;
    a.rates = rates;
    a.rate_in = ri;
    a.rate_out = ro;
    a.rate_clear = rc;
    return a;
}

// A step's launch (step_kernels.hpp); d is of system EQN.
template <typename T, int EQN>
hipError_t step_go(const StageDesc &d, int stages, const StageArgs<T> &a, hipStream_t st);
template <typename T, int EQN> hipError_t step_load();

}  // namespace fvk
