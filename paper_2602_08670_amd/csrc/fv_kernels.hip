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
// On small grids one launch takes all stages of a step (step_kernel).
#include "fv_device.hpp"
#include "fv_internal.hpp"

#include <type_traits>

namespace fvk {

__device__ __forceinline__ int map_index(int i, int n, int bc, bool &flip)
{
    if (i >= 0 && i < n) return i;
    if (bc == 0) return ((i % n) + n) % n;
    flip = true;
    int m = i < 0 ? -1 - i : 2 * n - 1 - i;
    return m < 0 ? 0 : (m >= n ? n - 1 : m);  // cells past the ghost layer are never used
}

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
// Bound by vector-ALU issue where the chip is full: 228 lane instructions per
// cell and stage of shallow water over a bed (270 before the faces shared
// their reconstruction and the flux was rearranged), 1024^2 21.3 -> 20.4 us a
// step, 2048^2 76.2 -> 63.6, Euler 1000 x 700 26.6 -> 19.9; by latency on
// small grids (64^2 13.0 -> 8.0).
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

template <typename T, int EQN, bool BATHY, int FLUX, int RECON>
static hipError_t stage_t(const StageDesc &d, const void *qs, const void *q0, void *out, const void *bed, double a0,
                          double a1, Ctl *ctl, unsigned long long *rates, int ri, int ro, int rc, int last,
                          hipStream_t st)
{
    StageArgs<T> a = stage_args<T>(d, qs, q0, out, bed, ctl, rates, ri, ro, rc);
    a.a0 = (T)a0;
    a.a1 = (T)a1;
    a.last = last;
    a.own = last ? BAD_STEP : 0;
    // the shapes with one and with two rows per wave serve every scheme, the
    // other two FP32 HLLE with MINMOD (the scheme of long runs)
    constexpr bool ALL = sizeof(T) == 4 && FLUX == HLLE && RECON == MINMOD;
    int shape = stage_shape((int64_t)d.nx * d.ny, d.prec);
    if (!ALL) shape = shape < 2 ? 0 : 2;
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
                          double a1, Ctl *ctl, unsigned long long *rates, int ri, int ro, int rc, int last,
                          hipStream_t st)
{
    if (d.recon == FIRST)
        return stage_t<T, EQN, BATHY, FLUX, FIRST>(d, qs, q0, out, bed, a0, a1, ctl, rates, ri, ro, rc, last, st);
    return stage_t<T, EQN, BATHY, FLUX, MINMOD>(d, qs, q0, out, bed, a0, a1, ctl, rates, ri, ro, rc, last, st);
}

template <typename T, int EQN, bool BATHY>
static hipError_t stage_f(const StageDesc &d, const void *qs, const void *q0, void *out, const void *bed, double a0,
                          double a1, Ctl *ctl, unsigned long long *rates, int ri, int ro, int rc, int last,
                          hipStream_t st)
{
    switch (d.flux) {
    case RUSANOV: return stage_r<T, EQN, BATHY, RUSANOV>(d, qs, q0, out, bed, a0, a1, ctl, rates, ri, ro, rc, last, st);
    case ROE: return stage_r<T, EQN, BATHY, ROE>(d, qs, q0, out, bed, a0, a1, ctl, rates, ri, ro, rc, last, st);
    default: return stage_r<T, EQN, BATHY, HLLE>(d, qs, q0, out, bed, a0, a1, ctl, rates, ri, ro, rc, last, st);
    }
}

template <typename T>
static hipError_t stage_p(const StageDesc &d, const void *qs, const void *q0, void *out, const void *bed, double a0,
                          double a1, Ctl *ctl, unsigned long long *rates, int ri, int ro, int rc, int last,
                          hipStream_t st)
{
    if (d.eqn == EULER) return stage_f<T, EULER, false>(d, qs, q0, out, bed, a0, a1, ctl, rates, ri, ro, rc, last, st);
    if (d.bathy) return stage_f<T, SWE, true>(d, qs, q0, out, bed, a0, a1, ctl, rates, ri, ro, rc, last, st);
    return stage_f<T, SWE, false>(d, qs, q0, out, bed, a0, a1, ctl, rates, ri, ro, rc, last, st);
}

hipError_t launch_stage(const StageDesc &d, const void *qs, const void *q0, void *out, const void *bed, double a0,
                        double a1, Ctl *ctl, unsigned long long *rates, int rate_in, int rate_out, int rate_clear,
                        int last, hipStream_t st)
{
    if (d.prec == 1)
        return stage_p<double>(d, qs, q0, out, bed, a0, a1, ctl, rates, rate_in, rate_out, rate_clear, last, st);
    return stage_p<float>(d, qs, q0, out, bed, a0, a1, ctl, rates, rate_in, rate_out, rate_clear, last, st);
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
    const bool four = cols * ((d.ny + 3) / 4) <= 256, eight = cols * ((d.ny + 7) / 8) <= 256;
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

template <typename T>
static hipError_t step_p(const StageDesc &d, int stages, const StageArgs<T> &a, hipStream_t st)
{
    return d.eqn == EULER ? step_e<T, EULER, false>(d, stages, a, st)
           : d.bathy      ? step_e<T, SWE, true>(d, stages, a, st)
                          : step_e<T, SWE, false>(d, stages, a, st);
}

hipError_t launch_step(const StageDesc &d, int stages, const void *src, void *dst, const void *bed, Ctl *ctl,
                       unsigned long long *rates, int rate_in, int rate_out, int rate_clear, int own, hipStream_t st)
{
    if (stages < 1 || stages > 3 || d.nx < 2 * stages || d.ny < 2 * stages || src == dst) return hipErrorInvalidValue;
    auto go = [&](auto zero) {
        using T = decltype(zero);
        StageArgs<T> a = stage_args<T>(d, src, src, dst, bed, ctl, rates, rate_in, rate_out, rate_clear);
        a.own = own;
        return step_p<T>(d, stages, a, st);
    };
    return d.prec == 1 ? go(0.0) : go(0.0f);
}

template <typename T>
__global__ __launch_bounds__(256) void step_copy_kernel(const T *__restrict__ src, T *__restrict__ dst, size_t n,
                                                        Ctl *ctl)
{
    if (blockIdx.x == 0 && threadIdx.x == 0 && ctl->bad) atomicOr(&ctl->bad, BAD_SKIP);
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) dst[i] = src[i];
}

hipError_t launch_step_copy(const StageDesc &d, const void *src, void *dst, Ctl *ctl, hipStream_t st)
{
    const size_t n = (size_t)(d.eqn == EULER ? 4 : 3) * d.nx * d.ny, blocks = (n + 255) / 256;
    const dim3 grid((unsigned)(blocks < 8192 ? blocks : 8192));
    if (d.prec == 1)
        hipLaunchKernelGGL(step_copy_kernel<double>, grid, dim3(256), 0, st, (const double *)src, (double *)dst, n, ctl);
    else
        hipLaunchKernelGGL(step_copy_kernel<float>, grid, dim3(256), 0, st, (const float *)src, (float *)dst, n, ctl);
    return hipGetLastError();
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
