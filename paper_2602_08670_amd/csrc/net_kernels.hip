// Network pass over batches and large grids: all five 3x3 layers of a tile of
// tw x 8 output pixels in one workgroup, weights stationary in registers.
//
// Run layer by layer, a 32-channel network moves 128 bytes of activations per
// pixel and hidden layer and is bound by that traffic (3.9 TB/s at a million
// pixels) or, on few pixels, by its launches; with the weights in LDS an MFMA
// waits for two operand reads.  Here
//  - activations stay in LDS: layer l is computed on the tile grown by 4 - l
//    pixels on each side (only rows where the tile spans the periodic grid's
//    width), from and to one of two buffers;
//  - each of the eight waves has its share of every layer's weights in
//    registers (one of the two 16-channel output tiles of each hidden layer,
//    up to two of the last layer's), so an MFMA reads LDS for its pixels only;
//    the first two layers' stay there over all tiles of the workgroup, the
//    others' are loaded a layer or more ahead of their use;
//  - a wave walks down a column of 16 pixels with three rows of accumulators:
//    a fragment of an input row (one per column shift) is read once and used
//    by the three output rows it belongs to, three MFMAs per LDS read, below
//    the LDS rate at which the matrix cores would wait.
// Every output pixel accumulates its MFMAs in the order of the other network
// passes (taps 0..8, K slices within a tap) with the same bias, ReLU and
// rounding, so the bits are the same.
//
// LDS: activation buffers of 16 x 80 and 14 x 80 pixels x 64 bytes and the
// biases, one workgroup of eight waves per CU.  A pixel's four 16-byte channel
// octets are XOR-swizzled by column, so that the 16 lanes that read one octet
// of consecutive pixels hit distinct banks.
//
// Measured: 256 solves of 64^2 208 us layer by layer, 163 us here (302 MB of z
// alone take 60 us, the MFMAs with the halo rows' 56 us; a tile's cycles:
// staging 5 500, layer 0 4 700, hidden layers 17 000, last layer 15 000 to
// 20 000 with its stores); 64 x 80 x 64 81 and 66 us, 16 x 64^2 33 and 20 us;
// one tile per workgroup is bound by its chain of loads and layers, 11 us.
#include "cnn_internal.hpp"
#include "fv_internal.hpp"

#include <algorithm>
#include <type_traits>

namespace cnn {

typedef __bf16 bf16;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
typedef int i32x4 __attribute__((ext_vector_type(4), aligned(4)));
typedef int i32x2 __attribute__((ext_vector_type(2), aligned(8)));

namespace {

constexpr int TR = 8;                  // output rows of a tile
constexpr int NWAVE = 8, NTHR = 64 * NWAVE;
constexpr int MAXW = 64;               // most output columns of a tile within a row
constexpr int MAXWRAP = 80;            // and of a tile that spans it
constexpr int rows_of(int l) { return TR + 2 * (4 - l); }  // rows of layer l's region; l = -1: the states
static_assert(MAXWRAP >= MAXW + 8, "a tile within a row with its margin");
constexpr int LR = 4;                  // output rows of a last-layer unit
enum { OUT_Z, OUT_KEEP, OUT_LIST };

template <int C> struct Net {
    static constexpr int K0 = C == 3 ? 32 : 64;    // layer 0's padded K
    static constexpr int CO = C == 3 ? COUT : E_COUT;
    static constexpr int NT = (CO + 15) / 16;      // output tiles of the last layer
    static constexpr int BUF_A = rows_of(0) * MAXWRAP * 64, BUF_B = rows_of(1) * MAXWRAP * 64;
    static constexpr int LDS = BUF_A + BUF_B + (4 * 32 + NT * 16) * 4;
    // the staged states, channels innermost, and with three channels a second
    // copy one value later, so that any run of values starts 4-byte aligned in
    // one of them; then 16 zero bytes
    static constexpr int ST = (C * (rows_of(-1) * (MAXWRAP + 2) + 4) * 2 + 15) & ~15, COPIES = C == 3 ? 2 : 1;
    static_assert(COPIES * ST + 16 <= BUF_B, "states staged in buffer B");
    static_assert(LDS <= 160 * 1024, "LDS of a CU");
};

struct NetArgs {
    const float *q;          // [B][C][H][W]
    const char *P;           // packed weights
    unsigned w[NL], b[NL];   // byte offsets in P
    float mean[4], inv[4];
    int B, H, W, tw, wrap, txn, tyn, ntiles;
    float *z;                // [B][H][W][CO]
    bf16 *acts[4];           // OUT_KEEP: [B][H][W][32]
    // OUT_LIST: the listed solves' q or S1 -> their z
    const LSolve *tab;
    const LItem *items;
    const int *list;
    int stage;
};

// One column group of a layer: N output rows from input rows in, in + pitch,
// ... (N + 2 of them), off[dx] a lane's byte offset of its pixel shifted by
// dx, w the nine taps' weights.  done(j, acc) takes output row j.  Unrolled,
// so that a row's epilogue and the next row's reads run between MFMAs.
template <int N, typename Done>
__device__ __forceinline__ void walk(const char *in, const int pitch, const int (&off)[3], const bf16x8 (&w)[9],
                                     Done done)
{
    floatx4 acc[3];
    bf16x8 b[2][3];
    auto fetch = [&](bf16x8 (&f)[3]) {
#pragma unroll
        for (int d = 0; d < 3; d++) f[d] = *(const bf16x8 *)(in + off[d]);
        in += pitch;
    };
    fetch(b[0]);
#pragma unroll
    for (int i = 0; i < N + 2; i++) {
        // input row i: output row i - 2 ends, i - 1 goes on, i starts; the
        // next row's fragments are on their way meanwhile
        if (i + 1 < N + 2) fetch(b[(i + 1) & 1]);
        const bf16x8(&x)[3] = b[i & 1];
#pragma unroll
        for (int d = 0; d < 3; d++)
#pragma unroll
            for (int dy = 2; dy >= 0; dy--) {
                const int j = i - dy;
                if (j < 0 || j >= N) continue;
                floatx4 &s = acc[j % 3];
                s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[dy * 3 + d], x[d],
                                                            dy == 0 && d == 0 ? floatx4{0.f, 0.f, 0.f, 0.f} : s, 0, 0, 0);
            }
        if (i >= 2) done(i - 2, acc[(i - 2) % 3]);
    }
}

// byte offset of octet o of a pixel in column c of its row
__device__ __forceinline__ int px_off(int c, int o) { return c * 64 + ((o ^ (-(c >> 2) & 3)) << 4); }

// Where a tile lies.
struct Loc {
    const float *q;   // its solve's states
    float *z;         // and output
    size_t pix;       // first pixel of its solve in a batch's arrays
    int H, W, tw, grow, x0, y0;  // grow: growth of a layer's region per side (0: the tile spans the width)
};

template <int C, int OUT> __device__ __forceinline__ Loc locate(const NetArgs &a, int tile)
{
    Loc t;
    int tx, ty;
    if (OUT == OUT_LIST) {
        int lo = 0, hi = a.list[0] - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (a.items[mid].tb_h <= tile) lo = mid;
            else hi = mid - 1;
        }
        const LItem it = a.items[lo];
        const LSolve &d = a.tab[it.solve];
        t.H = d.ny;
        t.W = d.nx;
        t.tw = net_tile_cols(t.W);
        t.grow = t.tw < t.W;
        t.q = a.stage == 1 ? d.q : d.s1;
        t.z = d.z;
        t.pix = 0;
        const int txn = (t.W + t.tw - 1) / t.tw, k = tile - it.tb_h;
        ty = k / txn;
        tx = k - ty * txn;
    } else {
        t.H = a.H;
        t.W = a.W;
        t.tw = a.tw;
        t.grow = a.wrap ? 0 : 1;
        const int per = a.txn * a.tyn, bi = tile / per, k = tile - bi * per;
        ty = k / a.txn;
        tx = k - ty * a.txn;
        t.pix = (size_t)bi * t.H * t.W;
        t.q = a.q + C * t.pix;
        t.z = a.z + Net<C>::CO * t.pix;
    }
    // the last tile of a row or column overlaps the one before
    t.x0 = min(tx * t.tw, t.W - t.tw);
    t.y0 = min(ty * TR, t.H - TR);
    return t;
}

// A tile's states in registers between their loads and their rounding into
// LDS: columns x0 - 1 - 4 grow .. of rows y0 - 5 .. y0 + 12, [18][sp][C].  A
// wave takes whole rows; every load is unconditional (a lane past the row's
// end reads its last column).
template <int C> struct States {
    static constexpr int SR = C * rows_of(-1), IT = (SR + NWAVE - 1) / NWAVE;
    float v[IT][2];
    unsigned o[IT];  // rounded, the lane's two columns
    static __device__ __forceinline__ int pitch(const Loc &t) { return t.tw + 2 + 8 * t.grow; }
    __device__ __forceinline__ void load(const Loc &t, int wave, int lane)
    {
        const int sp = pitch(t);
        int x[2];
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const int xx = t.x0 - 1 - 4 * t.grow + min(64 * h + lane, sp - 1);
            x[h] = xx < 0 ? xx + t.W : (xx >= t.W ? xx - t.W : xx);
        }
#pragma unroll
        for (int k = 0; k < IT; k++) {
            const int rid = min(wave + k * NWAVE, SR - 1), ci = rid / rows_of(-1);
            int yy = t.y0 - 5 + rid - ci * rows_of(-1);
            yy = yy < 0 ? yy + t.H : (yy >= t.H ? yy - t.H : yy);
            const float *row = t.q + ((size_t)ci * t.H + yy) * t.W;
#pragma unroll
            for (int h = 0; h < 2; h++) v[k][h] = row[x[h]];
        }
    }
    // normalise and round (waits for the loads)
    __device__ __forceinline__ void round(const NetArgs &a, int wave)
    {
#pragma unroll
        for (int k = 0; k < IT; k++) {
            const int ci = min(wave + k * NWAVE, SR - 1) / rows_of(-1);
            float mean = a.mean[0], inv = a.inv[0];
#pragma unroll
            for (int c = 1; c < C; c++) {
                mean = ci == c ? a.mean[c] : mean;
                inv = ci == c ? a.inv[c] : inv;
            }
            const bf16 lo = (bf16)((v[k][0] - mean) * inv), hi = (bf16)((v[k][1] - mean) * inv);
            o[k] = __builtin_bit_cast(unsigned short, lo) | (unsigned)__builtin_bit_cast(unsigned short, hi) << 16;
            __asm__ volatile("" : "+v"(o[k]));  // here, not where it is stored
        }
    }
    template <typename N> __device__ __forceinline__ void store(char *s, const Loc &t, int wave, int lane) const
    {
        const int sp = pitch(t);
        if (wave == 0 && lane < 4) *(int *)(s + N::COPIES * N::ST + 4 * lane) = 0;
#pragma unroll
        for (int k = 0; k < IT; k++) {
            const int rid = min(wave + k * NWAVE, SR - 1), ci = rid / rows_of(-1);
#pragma unroll
            for (int h = 0; h < 2; h++)
                if (64 * h + lane < sp) {
                    const int i = ((rid - ci * rows_of(-1)) * sp + 64 * h + lane) * C + ci;
                    const unsigned short x = (unsigned short)(o[k] >> 16 * h);
                    *(unsigned short *)(s + 2 * i) = x;
                    if (C == 3) *(unsigned short *)(s + N::ST + 2 * i + 2) = x;
                }
        }
    }
};

template <int C, int OUT>
__global__ __launch_bounds__(NTHR, 2) void net_kernel(NetArgs a)
{
    using N = Net<C>;
    constexpr int CO = N::CO, NT = N::NT, KB0 = N::K0 / 32;
    __shared__ __align__(16) char smem[N::LDS];
    char *const bufA = smem, *const bufB = smem + N::BUF_A;
    float *const s_bias = (float *)(smem + N::BUF_A + N::BUF_B);
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int ntiles = OUT == OUT_LIST ? a.list[3] : a.ntiles;
    if ((int)blockIdx.x >= ntiles) return;

    Loc T = locate<C, OUT>(a, blockIdx.x);
    States<C> st;
    st.load(T, wave, threadIdx.x & 63);

    // nine taps' fragments of output tile t of layer l (whose blocks hold nt tiles)
    auto weights = [&](bf16x8 (&w)[9], int l, int nt, int t, int lane) {
#pragma unroll
        for (int tap = 0; tap < 9; tap++)
            w[tap] = *(const bf16x8 *)(a.P + a.w[l] + (((tap * nt + t) * 16 + (lane & 15)) * 32 + (lane >> 4) * 8) * 2);
    };
    // layers 0 and 1 stay in registers; layers 2 and 3 and the two last-layer
    // tiles that this wave's eighth of a pass touches are loaded per tile, a
    // layer or more ahead of their use
    const int cot = wave & 1;
    bf16x8 w0[2][KB0], w1[9], wa[9], wb[9];
    {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int t = 0; t < 2; t++)
#pragma unroll
            for (int k = 0; k < KB0; k++)
                w0[t][k] = *(const bf16x8 *)(a.P + a.w[0] + ((t * 16 + (lane & 15)) * N::K0 + k * 32 + (lane >> 4) * 8) * 2);
        weights(w1, 1, 2, cot, lane);
    }
    if (threadIdx.x < 4 * 32 + NT * 16) {
        const int tid = threadIdx.x, l = tid < 128 ? tid >> 5 : 4;
        s_bias[tid] = ((const float *)(a.P + a.b[l]))[tid < 128 ? tid & 31 : tid - 128];
    }

    // Over several rounds of tiles a quarter of the CUs each starts a quarter
    // of a tile later: all in step, their last layers wait for memory together
    // and leave it idle in between (256 x 64^2: 182 us in step, 163 so)
    if (OUT != OUT_LIST && ntiles >= 4 * (int)gridDim.x)
        for (int i = (blockIdx.x >> 3 & 3) * 8; i > 0; i--) __builtin_amdgcn_s_sleep(15);
    st.round(a, wave);
    for (int tile = blockIdx.x; tile < ntiles;) {
        // opaque: index arithmetic is redone per tile, not held in registers
        // that the weights need
        int tid = threadIdx.x;
        __asm__ volatile("" : "+v"(tid));
        const int lane = tid & 63, g = lane >> 4, px = lane & 15;
        const Loc cur = T;
        const int tw = cur.tw, grow = cur.grow, gw = tw >> 4;
        weights(wa, 2, 2, cot, lane);
        weights(wb, 3, 2, cot, lane);
        st.template store<N>(bufB, cur, wave, lane);
        __syncthreads();

        // a finished row piece: bias, ReLU, BF16 to its buffer
        // (lanes past the region's width compute and store its last column again)
        auto put = [&](char *out, const floatx4 &acc, const floatx4 &bias) {
            bf16x4 o;
#pragma unroll
            for (int i = 0; i < 4; i++) o[i] = (bf16)__builtin_fmaxf(acc[i] + bias[i], 0.0f);
            *(bf16x4 *)out = o;
            return o;
        };
        // and, for training, the tile's own pixels of layer l to memory: row
        // r and column col of its region
        auto keep = [&](const int l, const int r, const int col, const int t, const bf16x4 &o) {
            if (OUT != OUT_KEEP) return;
            const int m = 4 - l, ty = r - m, tx = col - m * grow;
            if (ty >= 0 && ty < TR && tx >= 0 && tx < tw)
                *(bf16x4 *)(a.acts[l] + (cur.pix + (size_t)(cur.y0 + ty) * cur.W + cur.x0 + tx) * 32 + t * 16 + 4 * g) = o;
        };

        {  // layer 0: states (buffer B) -> buffer A, both output tiles per wave
            const int cols = tw + 8 * grow, rows = rows_of(0), units = ((cols + 15) >> 4) * rows, sp = st.pitch(cur);
            floatx4 bias[2];
#pragma unroll
            for (int t = 0; t < 2; t++) bias[t] = *(const floatx4 *)(s_bias + t * 16 + 4 * g);
            // A lane's eight K values (tap * C + ci) of a pixel.  Three channels:
            // the nine values of a tap row are consecutive, so lane group g's
            // are the run from value {0, 8, 7, 6}[g] of tap row {0, 0, 1, 2}[g],
            // of which the first {8, 1, 2, 3}[g] count, then the start of the
            // next tap row (zeros for g = 3).  Four channels: taps 2 g and
            // 2 g + 1, and in the second K block tap 8 (g = 0) or zeros.
            const int zero = N::COPIES * N::ST;
            const int na = g == 0 ? 8 : g;
            i32x4 mask;
#pragma unroll
            for (int d = 0; d < 4; d++) mask[d] = (2 * d < na ? 0xffff : 0) | (2 * d + 1 < na ? (int)0xffff0000 : 0);
            auto at = [&](int i) { return C == 3 && (i & 1) ? N::ST + 2 * i + 2 : 2 * i; };
            // RQ rows of a column group at a time: their reads overlap
            constexpr int RQ = C == 3 ? 4 : 2;
            static_assert(rows_of(0) % RQ == 0, "whole groups of rows");
            const int quads = units / RQ, u1 = quads * (wave + 1) / NWAVE;
#pragma unroll 1
            for (int u = quads * wave / NWAVE; u < u1; u++) {
                const int k = u / (rows / RQ), r = (u - k * (rows / RQ)) * RQ;
                const int col = min(16 * k + px, cols - 1);
                const char *pa, *pb, *pc = bufB + zero;
                int stepb = sp * C * 2, stepc = 0;
                if (C == 3) {
                    const int e = (r * sp + col) * C, da = (g >> 1) * sp * C;
                    pa = bufB + at(e + (g < 2 ? 0 : da) + (g == 3 ? sp * C : 0) + (g == 0 ? 0 : 9 - g));
                    pb = bufB + (g == 3 ? zero : at(e + (g == 2 ? 2 : 1) * sp * C - (g == 0 ? 0 : g)));
                    if (g == 3) stepb = 0;
                } else {
                    const int ta = 2 * g, tb = 2 * g + 1;
                    pa = bufB + ((r + ta / 3) * sp + col + ta % 3) * C * 2;
                    pb = bufB + ((r + tb / 3) * sp + col + tb % 3) * C * 2;
                    if (g == 0) {
                        pc = bufB + ((r + 2) * sp + col + 2) * C * 2;
                        stepc = stepb;
                    }
                }
                bf16x8 x[RQ][KB0];
#pragma unroll
                for (int j = 0; j < RQ; j++) {
                    if (C == 3) {
                        const i32x4 va = *(const i32x4 *)pa, vb = *(const i32x4 *)pb;
                        x[j][0] = __builtin_bit_cast(bf16x8, (i32x4)((va & mask) | (vb & ~mask)));
                    } else {
                        const i32x2 va = *(const i32x2 *)pa, vb = *(const i32x2 *)pb, vc = *(const i32x2 *)pc;
                        x[j][0] = __builtin_bit_cast(bf16x8, i32x4{va[0], va[1], vb[0], vb[1]});
                        x[j][KB0 - 1] = __builtin_bit_cast(bf16x8, i32x4{vc[0], vc[1], 0, 0});
                    }
                    pa += sp * C * 2;
                    pb += stepb;
                    pc += stepc;
                }
                char *op = bufA + r * cols * 64 + px_off(col, g >> 1) + (g & 1) * 8;
                const int flip = px_off(col, 2 + (g >> 1)) - px_off(col, g >> 1);  // to the second output tile
#pragma unroll
                for (int j = 0; j < RQ; j++) {
#pragma unroll
                    for (int t = 0; t < 2; t++) {
                        floatx4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                        for (int kb = 0; kb < KB0; kb++)
                            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w0[t][kb], x[j][kb], acc, 0, 0, 0);
                        keep(0, r + j, col, t, put(op + t * flip, acc, bias[t]));
                    }
                    op += cols * 64;
                }
            }
        }
        __syncthreads();

        // a layer's input offsets of a lane in output column col
        auto shifts = [&](const int col, int (&off)[3]) {
#pragma unroll
            for (int d = 0; d < 3; d++) {
                int ic = col + d;
                if (!grow) {
                    ic -= 1;
                    ic = ic < 0 ? ic + tw : (ic >= tw ? ic - tw : ic);
                }
                off[d] = px_off(ic, g);
            }
        };
        // hidden layer l: its column halves dealt to the four pairs of waves
        auto hidden = [&](auto layer, const bf16x8 (&w)[9]) {
            constexpr int l = decltype(layer)::value, R = rows_of(l) / 2;
            const char *in = l & 1 ? bufA : bufB;
            char *out = l & 1 ? bufB : bufA;
            const int cols = tw + 2 * (4 - l) * grow, units = ((cols + 15) >> 4) * 2;
            const int pitch = (cols + 2 * grow) * 64;
            const floatx4 bias = *(const floatx4 *)(s_bias + l * 32 + cot * 16 + 4 * g);
            const int part = wave >> 1, u1 = units * (part + 1) / 4;
#pragma unroll 1
            for (int u = units * part / 4; u < u1; u++) {
                const int r = (u & 1) * R, col = min(16 * (u >> 1) + px, cols - 1);
                int off[3];
                shifts(col, off);
                char *op = out + r * cols * 64 + px_off(col, 2 * cot + (g >> 1)) + (g & 1) * 8;
                walk<R>(in + r * pitch, pitch, off, w, [&](const int j, const floatx4 &acc) {
                    keep(l, r + j, col, cot, put(op, acc, bias));
                    op += cols * 64;
                });
            }
        };
        // last layer: units of LR rows of a column group of an output tile, in that order
        const int per = gw * (TR / LR), units = NT * per, t0 = units * wave / NWAVE / per;
        hidden(std::integral_constant<int, 1>{}, w1);
        __syncthreads();
        hidden(std::integral_constant<int, 2>{}, wa);
        weights(wa, 4, NT, t0, lane);
        __syncthreads();
        // the next tile's states, and below the last layer's second tile of
        // weights: their arrival must not wait for the last layer's stores
        const int next = tile + gridDim.x;
        if (next < ntiles) {
            T = locate<C, OUT>(a, next);
            st.load(T, wave, lane);
        }
        hidden(std::integral_constant<int, 3>{}, wb);
        weights(wb, 4, NT, min(t0 + 1, NT - 1), lane);
        if (next < ntiles) st.round(a, wave);
        __syncthreads();

        // last layer: from buffer B, an eighth of the units per wave
        const int pitch = (tw + 2 * grow) * 64, u1 = units * (wave + 1) / NWAVE;
#pragma unroll 1
        for (int u = units * wave / NWAVE; u < u1; u++) {
            const int t = u / per, v = u - t * per, k = v / (TR / LR), r = (v - k * (TR / LR)) * LR;
            const int col = 16 * k + px, co0 = 16 * t + 4 * g;
            const floatx4 bias = *(const floatx4 *)(s_bias + 128 + co0);
            int off[3];
            shifts(col, off);
            float *op = cur.z + ((size_t)(cur.y0 + r) * cur.W + cur.x0 + col) * CO + co0;
            auto done = [&](const int j, const floatx4 &acc) {
                if (CO % 16 == 0 || co0 < CO) *(floatx4 *)op = acc + bias;
                op += cur.W * CO;
            };
            if (t == t0) walk<LR>(bufB + r * pitch, pitch, off, wa, done);
            else walk<LR>(bufB + r * pitch, pitch, off, wb, done);
        }
        __syncthreads();
        tile = next;
    }
}

template <int C, typename PK, typename NormT>
NetArgs net_args(const void *packed, const PK &pk, const NormT &nrm, const float *q, int B, int nx, int ny)
{
    NetArgs a{};
    a.q = q;
    a.P = (const char *)packed;
    for (int l = 0; l < NL; l++) {
        a.w[l] = (unsigned)pk.w[l];
        a.b[l] = (unsigned)pk.b[l];
    }
    for (int c = 0; c < C; c++) {
        a.mean[c] = nrm.mean[c];
        a.inv[c] = nrm.inv_std[c];
    }
    a.B = B;
    a.H = ny;
    a.W = nx;
    a.tyn = (ny + TR - 1) / TR;
    // Wider tiles recompute less, the whole row least; narrower ones fill more
    // CUs: the width with the fewest rounds of tiles, each the MFMAs of its
    // longest wave and what a tile costs besides (in MFMAs).  One 64^2 solve:
    // 13 us in 16 columns, 20 us in 64; 64 of them 51 us in 64.
    long best = 0;
    for (int tw = nx <= MAXWRAP ? nx : MAXW; tw >= 16; tw = (tw < nx ? tw : std::min(nx, MAXW + 16)) - 16) {
        const long grown = tw < nx, tiles = (long)B * a.tyn * ((nx + tw - 1) / tw), g = tw / 16;
        const long cost = (tiles + fvk::CUS - 1) / fvk::CUS * (750 + (g + grown + 1) / 2 * 2 * 36 * 18 + g * 8 * 9 * Net<C>::NT);
        if (!a.tw || cost < best) {
            best = cost;
            a.tw = tw;
        }
    }
    a.wrap = a.tw == nx;
    a.txn = (nx + a.tw - 1) / a.tw;
    a.ntiles = B * a.txn * a.tyn;
    return a;
}

}  // namespace

// One workgroup per CU (its LDS); fewer tiles take fewer.
int net_grid(int ntiles)
{
    static int cus = [] {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
            n = fvk::CUS;
        return n;
    }();
    return ntiles < cus ? ntiles : cus;
}

int net_tiles(int nx, int ny)
{
    const int tw = net_tile_cols(nx);
    return ((nx + tw - 1) / tw) * ((ny + TR - 1) / TR);
}

hipError_t launch_net(const void *packed, const Norm &nrm, const float *q, int B, int nx, int ny, void *const acts[4],
                      float *z, hipStream_t st)
{
    if (!net_takes(nx, ny)) return hipErrorInvalidValue;
    NetArgs a = net_args<CIN>(packed, packed_layout(), nrm, q, B, nx, ny);
    a.z = z;
    const dim3 grid(net_grid(a.ntiles)), blk(NTHR);
    if (acts) {
        for (int l = 0; l < 4; l++) a.acts[l] = (bf16 *)acts[l];
        hipLaunchKernelGGL((net_kernel<CIN, OUT_KEEP>), grid, blk, 0, st, a);
    } else {
        hipLaunchKernelGGL((net_kernel<CIN, OUT_Z>), grid, blk, 0, st, a);
    }
    return hipGetLastError();
}

hipError_t launch_net_euler(const void *packed, const ENorm &nrm, const float *q, int B, int nx, int ny,
                            void *const acts[4], float *z, hipStream_t st)
{
    if (!net_takes(nx, ny)) return hipErrorInvalidValue;
    NetArgs a = net_args<E_CIN>(packed, euler_packed_layout(), nrm, q, B, nx, ny);
    a.z = z;
    const dim3 grid(net_grid(a.ntiles)), blk(NTHR);
    if (acts) {
        for (int l = 0; l < 4; l++) a.acts[l] = (bf16 *)acts[l];
        hipLaunchKernelGGL((net_kernel<E_CIN, OUT_KEEP>), grid, blk, 0, st, a);
    } else {
        hipLaunchKernelGGL((net_kernel<E_CIN, OUT_Z>), grid, blk, 0, st, a);
    }
    return hipGetLastError();
}

hipError_t launch_net_list(int stage, const void *packed, const Norm &nrm, const LSolve *tab, const LItem *items,
                           const int *list, int tiles, hipStream_t st)
{
    if (tiles <= 0) return hipErrorInvalidValue;
    NetArgs a = net_args<CIN>(packed, packed_layout(), nrm, nullptr, 1, 16, 8);
    a.tab = tab;
    a.items = items;
    a.list = list;
    a.stage = stage;
    hipLaunchKernelGGL((net_kernel<CIN, OUT_LIST>), dim3(net_grid(tiles)), dim3(NTHR), 0, st, a);
    return hipGetLastError();
}

}  // namespace cnn
