// mlp_train.hpp -- the training step's gradient in two launches.
//
// k_train_rows carries TR rows of one member forward through all layers, through the
// loss, and backward to dz1 without leaving the work-group: activations and dz go from
// layer to layer through LDS, the pre-activations z stay in registers (FP32).  It writes
// the BF16 operands of the weight gradients as MFMA fragments with the rows along a
// lane's registers, so that k_train_wgrad loads a fragment as 1 KiB in a row (stored
// [feature][row] instead, the 16 rows of a fragment lie a power of two apart in the same
// few L2 channels: 16.6 us at 1024 rows), and per-group partial
// sums of the output layer's gradients.  k_train_wgrad forms dW2, dW3, their biases and
// the input layer's gradients, and adds those partials.
//
// Every gradient is a sum over the batch in one order that depends on the batch alone (the
// order of a layer-by-layer step: chunks of rows summed in ascending order, the chunks
// added one after another), so a seeded training run repeats bit for bit whatever the
// launch.  The rules are wgrad_split, bias_tile, HEAD_ROWS and column_rows below.
//
// What bounds a step of this size (5 members x 1024 rows: 4 GFLOP, 18 MB) is latency:
// one launch per layer and direction (13 of them, each 4 - 17 us, with z, a and dz in
// memory between them) took 97.6 us with the Adam step, 195.6 us at 4096 rows; the two
// launches take 25 + 10 us and 66 + 25 us, 36.7 and 90.2 us with the Adam step.  The
// arithmetic and the roundings are the layer-by-layer ones, bit for bit.
#pragma once

#include "mlp_kernels.hpp"

namespace bm {
namespace mlp {

constexpr int TRT = 2, TR = 16 * TRT;   // row tiles of 16 and rows per pass of a work-group
constexpr int TWAVES = 8, TBT = 64 * TWAVES;
constexpr int TLD = H + 8;              // LDS row of activations (bf16): 4 banks further per row
constexpr int TTL = 32 + 4;             // LDS row of a wave's transposed weight slice: 8 banks further per 4 rows
constexpr int HEAD_W = H + 2;           // partial record of the output layer: dW4[256], db4, sum e^2
constexpr int HEAD_ROWS = 16;           // rows of a record: four sums of four rows, added in order
constexpr int NV1 = IN + 1;             // sums of the input layer: dW1[o][0..4], db1[o]
static_assert(TWAVES * 32 == H, "a wave owns 32 features of a layer");

// Chunks of rows whose products with the 256 x 256 weight gradients are summed apart: the
// largest power of two <= min(8, B / 256) with B / split a multiple of 32.
__host__ __device__ constexpr int wgrad_split(int B)
{
    int ks = 1;
    while (ks < 8 && 2 * ks * 256 <= B && B % (2 * ks * 32) == 0) ks *= 2;
    return ks;
}
// The bias gradient of a chunk is four sums: of the q-th quarters of its tiles of this
// many rows.
__host__ __device__ constexpr int bias_tile(int chunk) { return chunk % 128 == 0 ? 128 : 32; }
// Rows of a partial sum of the input layer's gradients.
__host__ __device__ constexpr int column_rows(int B) { return B / 64 < 16 ? 16 : B / 64; }
constexpr int MAX_COLUMNS = 64;         // most partial sums: B / column_rows(B)

struct TrainArgs {
    const float *x, *t;                 // rows [.][5] and targets
    const uint32_t *idx;                // row of (member, r): idx[m * B + r], or r if null
    const bf16_t *wbf;
    const float *params;
    int B;                              // rows per member, a multiple of 64
    bf16_t *a1T, *a2T, *dz1T, *dz2T, *dz3T;   // [member][B / 32][16 feature tiles][64 lanes][8 rows]
    float *u;                           // normalised inputs [member][B][IN]
    float *hpart;                       // [member][B / HEAD_ROWS][HEAD_W]
    int members;
    int groups;                         // work-groups per member (gridDim.x of k_train_rows)
    float *grad, *loss;
};

// Four consecutive rows of one feature, rounded to BF16 (v_cvt_pk_bf16_f32: nearest even).
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));

// 16 or 8 bytes at `base` + `off` bytes: a wave-uniform base and a 32-bit lane offset, so
// that the many weight addresses of a lane share one register.
template <typename T> __device__ __forceinline__ T load_at(const bf16_t *base, uint32_t off)
{
    return *reinterpret_cast<const T *>(reinterpret_cast<const char *>(base) + off);
}

// Eight BF16 in LDS at an 8-byte aligned address.
__device__ __forceinline__ bf16x8 pair8(const bf16_t *p)
{
    struct P { uint2 a, b; } v{*reinterpret_cast<const uint2 *>(p), *reinterpret_cast<const uint2 *>(p + 4)};
    return __builtin_bit_cast(bf16x8, v);
}

// grid (groups, members): a group takes the row tiles blockIdx.x, + groups, ...  A wave
// owns 32 features of every layer: its weight fragments come from global memory (L2)
// straight into registers -- no other wave of the group needs them, so there is nothing
// to stage -- and only activations and dz pass through LDS.  The backward products need
// W with the contraction (the outputs) along a lane's registers: each wave transposes
// its own 32 columns in 32-wide slices through a private LDS tile, so no barrier.
// 5 members x 1024 rows put one group of 8 waves on 160 of the 256 CUs; a pass over 32
// rows takes some 46k cycles whatever the batch (25 us the first, 20 us each further one),
// 31k of them while the 4 x 128 KiB of weights come in: 17 B per cycle and CU, in pieces of
// 16 bytes (W) and 8 (its transpose).  The same matrices in rows of 1 KiB, turned into
// fragments through LDS, were measured on layer 2 only: 8.1k -> 4.4k cycles.  A pass of more
// rows would amortise better, but needs the registers that hold z and the weights of the
// next layer.
__global__ void __launch_bounds__(TBT, 2) k_train_rows(const TrainArgs a)
{
    __shared__ __align__(16) bf16_t sAct[2][TR * TLD];
    __shared__ __align__(16) bf16_t sTr[TWAVES][4][32 * TTL];
    __shared__ __align__(16) float sU[TR][8], sW1[H][8], sW4[H];
    __shared__ float sB[2][H];
    __shared__ float sTgt[TR], sDy[TR], sE[TR];
    const int tid = threadIdx.x;
    const int m = blockIdx.y, B = a.B;
    const bf16_t *WB = a.wbf + (uint64_t)m * NBF;
    const float *P = a.params + (uint64_t)m * NPARAM;
    const uint64_t mT = (uint64_t)m * H * B;

    // the small parameters, once, into LDS: loads return in order, so one waited for where
    // it is used would wait for the weights fetched ahead of their layer as well
    if (tid < H) {
#pragma unroll
        for (int j = 0; j < IN; ++j) sW1[tid][j] = bf2f(WB[BOFF_W1 + tid * IN + j]);
        sW1[tid][IN] = P[OFF_B1 + tid];
        sB[0][tid] = P[OFF_B2 + tid];
        sB[1][tid] = P[OFF_B3 + tid];
        sW4[tid] = bf2f(WB[BOFF_W4 + tid]);
    }
    const float b4 = P[OFF_B4];
    // inputs and target of one row per thread, fetched a tile ahead
    float xr[IN] = {}, tr = 0.0f;
    auto fetch = [&](int at) {
        if (tid < TR && at < B / TR) {
            const uint64_t r = (uint64_t)at * TR + tid;
            const uint64_t src = a.idx ? (uint64_t)a.idx[(uint64_t)m * B + r] : r;
#pragma unroll
            for (int j = 0; j < IN; ++j) xr[j] = a.x[src * IN + j];
            tr = a.t[src];
        }
    };
    int tile = blockIdx.x;
    fetch(tile);

    for (; tile < B / TR; tile += a.groups) {
        // The lane and a zero offset, opaque per tile: addresses are formed where they are
        // used.  Hoisted out of the loop they would spill, and loads return in order, so a
        // reload waits for all the weights fetched ahead of their layer.
        int id = threadIdx.x;
        uint32_t opaque = 0;
        asm volatile("" : "+v"(id), "+s"(opaque));
        const int lane = id & 63, wave = __builtin_amdgcn_readfirstlane(id >> 6), g = lane >> 4, c = lane & 15;
        const int f0 = 32 * wave + c;   // the lane's features: f0 and f0 + 16
        // fragments of W (row = output feature, k along the row)
        const uint32_t wofs = 2u * (uint32_t)(f0 * H + 8 * g);
        auto load_w = [&](int off, bf16x8 (&f)[2][8]) {
            const bf16_t *base = WB + off + opaque;
    #pragma unroll
            for (int t = 0; t < 2; ++t)
    #pragma unroll
                for (int s = 0; s < 8; ++s)
                    f[t][s] = load_at<bf16x8>(base, wofs + 2u * (16 * t * H + 32 * s));
        };
        // the wave's 32 columns of W, four consecutive output rows of four columns per lane and slice
        const int kq = lane >> 3, ng = lane & 7;
        const uint32_t wtofs = 2u * (uint32_t)(4 * kq * H + 32 * wave + 4 * ng);
        auto load_wt = [&](int off, uint2 (&r)[8][4]) {
            const bf16_t *base = WB + off + opaque;
    #pragma unroll
            for (int s = 0; s < 8; ++s)
    #pragma unroll
                for (int q = 0; q < 4; ++q)
                    r[s][q] = load_at<uint2>(base, wtofs + 2u * ((32 * s + q) * H));
        };
        // acc += A(LDS rows) x W^T fragments, k ascending
        auto forward = [&](const bf16_t *src, const bf16x8 (&f)[2][8], floatx4 (&acc)[TRT][2]) {
    #pragma unroll
            for (int rt = 0; rt < TRT; ++rt)
    #pragma unroll
                for (int t = 0; t < 2; ++t) acc[rt][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    #pragma unroll
            for (int s = 0; s < 8; ++s)
    #pragma unroll
                for (int rt = 0; rt < TRT; ++rt) {
                    const bf16x8 av = *reinterpret_cast<const bf16x8 *>(src + (16 * rt + c) * TLD + 32 * s + 8 * g);
    #pragma unroll
                    for (int t = 0; t < 2; ++t)
                        acc[rt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, f[t][s], acc[rt][t], 0, 0, 0);
                }
        };
        auto backward = [&](const bf16_t *src, const uint2 (&r)[8][4], floatx4 (&acc)[TRT][2]) {
    #pragma unroll
            for (int rt = 0; rt < TRT; ++rt)
    #pragma unroll
                for (int t = 0; t < 2; ++t) acc[rt][t] = floatx4{0.f, 0.f, 0.f, 0.f};
    #pragma unroll
            for (int h = 0; h < 2; ++h) {           // four slices transposed, then used
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4)
#pragma unroll
                    for (int i = 0; i < 4; ++i) {   // column 4 ng + i, rows 4 kq .. 4 kq + 3
                        const uint2 *v = r[4 * h + q4];
                        auto half = [&](int q) { return ((i < 2 ? v[q].x : v[q].y) >> (16 * (i & 1))) & 0xFFFFu; };
                        *reinterpret_cast<uint2 *>(&sTr[wave][q4][(4 * ng + i) * TTL + 4 * kq]) =
                            uint2{half(0) | (half(1) << 16), half(2) | (half(3) << 16)};
                    }
                // the wave's own LDS accesses complete in order; keep the compiler's order too
                asm volatile("" ::: "memory");
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    bf16x8 bv[2];
#pragma unroll
                    for (int t = 0; t < 2; ++t)
                        bv[t] = pair8(&sTr[wave][q4][(16 * t + c) * TTL + 8 * g]);
#pragma unroll
                    for (int rt = 0; rt < TRT; ++rt) {
                        const bf16x8 av = *reinterpret_cast<const bf16x8 *>(src + (16 * rt + c) * TLD +
                                                                            32 * (4 * h + q4) + 8 * g);
#pragma unroll
                        for (int t = 0; t < 2; ++t)
                            acc[rt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, bv[t], acc[rt][t], 0, 0, 0);
                    }
                }
                asm volatile("" ::: "memory");
            }
        };
        // BF16 values of rows 16 rt + 4 g + e, feature f0 + 16 t: into LDS; transposed to memory
        auto put = [&](int rt, int t, bf16x4 v, bf16_t *dst) {
            const uint2 p = __builtin_bit_cast(uint2, v);
    #pragma unroll
            for (int e = 0; e < 4; ++e)
                dst[(16 * rt + 4 * g + e) * TLD + f0 + 16 * t] = (bf16_t)((e < 2 ? p.x : p.y) >> (16 * (e & 1)));
        };
        auto store = [&](int rt, int t, bf16x4 v, bf16_t *gT) {
            bf16_t *p = gT + mT + ((uint64_t)tile * 16 + 2 * wave + t) * 512;
            *reinterpret_cast<uint2 *>(p + ((2 * rt + (g >> 1)) * 16 + c) * 8 + 4 * (g & 1)) = __builtin_bit_cast(uint2, v);
        };
        bf16x8 w[2][8];
        load_w(BOFF_W2, w);
        if (tid < TR) {
            float u[IN];
            normalise(xr, u);
#pragma unroll
            for (int j = 0; j < IN; ++j) {
                sU[tid][j] = u[j];
                a.u[((uint64_t)m * B + tile * TR + tid) * IN + j] = u[j];
            }
            sTgt[tid] = tr;
        }
        fetch(tile + a.groups);
        __syncthreads();
        // ---- forward ----
        float z2[TRT][2][4], z3[TRT][2][4];
        floatx4 acc[TRT][2];
        // layer 1; formed again for dz1 (cheaper than 16 registers held through the pass)
        auto input_layer = [&](auto use) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                float w1[IN + 1];
#pragma unroll
                for (int j = 0; j <= IN; ++j) w1[j] = sW1[f0 + 16 * t][j];
#pragma unroll
                for (int rt = 0; rt < TRT; ++rt) {
                    float z[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float *u = sU[16 * rt + 4 * g + e];
                        z[e] = w1[IN];
#pragma unroll
                        for (int j = 0; j < IN; ++j) z[e] = fmaf(w1[j], u[j], z[e]);
                    }
                    use(rt, t, z);
                }
            }
        };
        input_layer([&](int rt, int t, const float (&z)[4]) {
            bf16x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (__bf16)(gelu(z[e]));
            put(rt, t, v, sAct[0]);
            store(rt, t, v, a.a1T);
        });
        __syncthreads();
        forward(sAct[0], w, acc);
        asm volatile("" ::: "memory");
        load_w(BOFF_W3, w);
        auto finish = [&](const float *bias, float (&z)[TRT][2][4], bf16_t *dst, auto keep) {
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const float b = bias[f0 + 16 * t];
#pragma unroll
                for (int rt = 0; rt < TRT; ++rt) {
                    bf16x4 v;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        z[rt][t][e] = acc[rt][t][e] + b;
                        v[e] = (__bf16)(gelu(z[rt][t][e]));
                    }
                    put(rt, t, v, dst);
                    keep(rt, t, v);
                }
            }
        };
        finish(sB[0], z2, sAct[1], [&](int rt, int t, bf16x4 v) { store(rt, t, v, a.a2T); });
        __syncthreads();
        forward(sAct[1], w, acc);
        uint2 wt[8][4];
        asm volatile("" ::: "memory");
        load_wt(BOFF_W3, wt);
        finish(sB[1], z3, sAct[0], [](int, int, bf16x4) {});
        __syncthreads();
        // ---- output layer and loss: a wave per row, four features per lane ----
        constexpr int HR = TR / TWAVES;
        float y[HR], w4h[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) w4h[j] = sW4[lane * 4 + j];
#pragma unroll
        for (int rr = 0; rr < HR; ++rr) {
            const uint2 a3 = *reinterpret_cast<const uint2 *>(&sAct[0][(wave * HR + rr) * TLD + lane * 4]);
            y[rr] = fmaf(__uint_as_float(a3.x << 16), w4h[0], 0.0f);
            y[rr] = fmaf(__uint_as_float(a3.x & 0xFFFF0000u), w4h[1], y[rr]);
            y[rr] = fmaf(__uint_as_float(a3.y << 16), w4h[2], y[rr]);
            y[rr] = fmaf(__uint_as_float(a3.y & 0xFFFF0000u), w4h[3], y[rr]);
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1)     // the same sum in every lane, the rows side by side
#pragma unroll
            for (int rr = 0; rr < HR; ++rr) y[rr] += __shfl_xor(y[rr], off, 64);
#pragma unroll
        for (int rr = 0; rr < HR; ++rr) {
            const float e = (y[rr] + b4) - sTgt[wave * HR + rr];
            if (lane == 0) {
                sE[wave * HR + rr] = e;
                sDy[wave * HR + rr] = 2.0f * e / (float)B;
            }
        }
        __syncthreads();
        // ---- dz3, dW4, db4, loss ----
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const float w4 = sW4[f0 + 16 * t];
#pragma unroll
            for (int rt = 0; rt < TRT; ++rt) {
                bf16x4 v;
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = (__bf16)(sDy[16 * rt + 4 * g + e] * w4 * gelu_grad(z3[rt][t][e]));
                put(rt, t, v, sAct[1]);
                store(rt, t, v, a.dz3T);
            }
        }
        float *rec = a.hpart + ((uint64_t)m * (B / HEAD_ROWS) + tile * (TR / HEAD_ROWS)) * HEAD_W;
        if (tid < H) {
#pragma unroll
            for (int q = 0; q < TR / HEAD_ROWS; ++q) {
                float sw[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    sw[k] = 0.0f;
#pragma unroll
                    for (int rr = 0; rr < 4; ++rr) {
                        const int r = HEAD_ROWS * q + 4 * k + rr;
                        sw[k] = fmaf(sDy[r], bf2f(sAct[0][r * TLD + tid]), sw[k]);
                    }
                }
                rec[q * HEAD_W + tid] = ((sw[0] + sw[1]) + sw[2]) + sw[3];
            }
        } else if (tid < H + TR / 4) {          // four rows per lane
            const int r0 = 4 * (tid - H);
            float sb = 0.0f, se = 0.0f;
#pragma unroll
            for (int rr = 0; rr < 4; ++rr) {
                sb += sDy[r0 + rr];
                se = fmaf(sE[r0 + rr], sE[r0 + rr], se);
            }
            float b[4], e[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                b[k] = __shfl(sb, (lane & ~3) + k, 64);
                e[k] = __shfl(se, (lane & ~3) + k, 64);
            }
            if ((lane & 3) == 0) {
                rec[lane / 4 * HEAD_W + H] = ((b[0] + b[1]) + b[2]) + b[3];
                rec[lane / 4 * HEAD_W + H + 1] = ((e[0] + e[1]) + e[2]) + e[3];
            }
        }
        __syncthreads();
        // ---- dz2 and dz1 ----
        backward(sAct[1], wt, acc);
        asm volatile("" ::: "memory");
        load_wt(BOFF_W2, wt);
        auto gradient = [&](int rt, int t, const float (&z)[4]) {
            bf16x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (__bf16)(acc[rt][t][e] * gelu_grad(z[e]));
            return v;
        };
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int rt = 0; rt < TRT; ++rt) {
                const bf16x4 v = gradient(rt, t, z2[rt][t]);
                put(rt, t, v, sAct[0]);
                store(rt, t, v, a.dz2T);
            }
        __syncthreads();
        backward(sAct[0], wt, acc);
        input_layer([&](int rt, int t, const float (&z)[4]) { store(rt, t, gradient(rt, t, z), a.dz1T); });
        __syncthreads();                        // the next tile overwrites sU and sAct
    }
}

// Weight gradients dW[o][i] = sum_r dz[r][o] a[r][i] of the 256 x 256 layers from the
// fragments of k_train_rows, KS = wgrad_split(B): grid wg_blocks(WGM) members; a group of
// the first wg_tiles(WGM) members forms a WGM x 64 tile.  Its eight waves share the KS chunks
// of rows, 8 / KS waves to a chunk with as many 16 x 16 products of the tile each, so that a
// product is one accumulation over its chunk and all waves work at any batch; up to SL slices
// of 32 rows have their loads in flight.  The chunks are added in order through LDS, which
// needs no partials in memory.  The bias gradients are row sums of dz in the groups of the
// first column tile.  The last (COLUMN_BLOCKS + 1) members blocks form the gradients of the
// input layer and add the records of the output layer.
// 5 members: 9.8 us at 1024 rows and 24.9 us at 4096; slices dealt to the waves in turn (a
// quarter fewer loads at KS = 4, but sums in another order) took 10.4 and 24.0 us.
// At KS = 2 (a batch that is an odd multiple of 64, from 512 on) four waves share a chunk,
// with two products of a 32 x 64 tile each for three fragments, and the chunks are long: the
// loads count.  Where the tiles of 32 rows are more than the 256 CUs take at once, from five
// members on, tiles of 64 rows (four products for four fragments, half the groups) and the
// next slices fetched ahead take less: 5 members x 4032 rows 89 us a gradient against 99 (90
// with the slices in turn), but 3 members 68 against 62.
constexpr int CW = 16;                          // columns of the input layer per block
constexpr int COLUMN_BLOCKS = H / CW;
constexpr int WGN = 64;
constexpr int wg_tiles(int wgm) { return 2 * (H / wgm) * (H / WGN); }                  // per member
constexpr int wg_blocks(int wgm) { return wg_tiles(wgm) + COLUMN_BLOCKS + 1; }
constexpr uint32_t WGRAD_TALL = 256 / wg_tiles(32) + 1;   // members whose 32-row tiles exceed the CUs

// The value of lane I of this lane's row of 16.
template <int I> __device__ __forceinline__ float row_lane(float v)
{
    return __uint_as_float(__builtin_amdgcn_update_dpp(0u, __float_as_uint(v), 0x150 + I, 0xF, 0xF, true));
}

// 16 rows of dz1 in one column, and of the inputs: one row per lane of a row of lanes.
struct ColumnRows {
    bf16x8 d[2];
    float u[IN];
};

// Adds rows I .. 15 of `v` to the sums of the lane's column: those below n (the same in all
// lanes); with EDGES those from `first` on, n of them, as zeros elsewhere.
template <int I, bool EDGES>
__device__ __forceinline__ void add_rows(const ColumnRows &v, int first, int n, float (&s)[NV1])
{
    if constexpr (I < 16) {
        if (EDGES || I < n) {
            float d = (float)v.d[I >> 3][I & 7];
            if constexpr (EDGES) d = (uint32_t)(I - first) < (uint32_t)n ? d : 0.0f;
#pragma unroll
            for (int j = 0; j < IN; ++j) s[j] = fmaf(d, row_lane<I>(v.u[j]), s[j]);
            s[IN] += d;
        }
        add_rows<I + 1, EDGES>(v, first, n, s);
    }
}

// dW1[o][0..4] and db1[o] of 16 columns o: a partial sum over column_rows(B) rows per row
// of 16 lanes, a column per lane, then the partial sums in order.  16 batch rows at a time:
// lane i holds the inputs of row i, which reach the other lanes of its row by DPP (read by
// every lane for itself, from memory or LDS, the inputs are ten times dz's bytes).  Whole
// waves on one partial sum and 64 columns left 20 blocks of 5 members to work for 22 us at
// 1024 rows; these 80 end before the tiles do.
__device__ __forceinline__ void column_sums(const TrainArgs &a, int m, int f0, float (*part)[NV1][CW])
{
    const int tid = threadIdx.x, c = tid & 15;
    const int B = a.B, rows = column_rows(B), n = B / rows;
    const bf16_t *dz = a.dz1T + (uint64_t)m * H * B + (uint64_t)(f0 / 16) * 512 + c * 8;
    const float *um = a.u + (uint64_t)m * B * IN;
    auto eight = [&](int r) { return dz + (uint64_t)(r >> 5) * (32 * H) + ((r >> 3) & 3) * 128; };
    // rows r .. r + 15, r a multiple of 8; those from `end` on are not used
    auto load = [&](int r, int end) {
        ColumnRows v;
        v.d[0] = *reinterpret_cast<const bf16x8 *>(eight(r < end ? r : 0));
        v.d[1] = *reinterpret_cast<const bf16x8 *>(eight(r + 8 < end ? r + 8 : 0));
        const float *u = um + (uint64_t)(r + c < end ? r + c : 0) * IN;
#pragma unroll
        for (int j = 0; j < IN; ++j) v.u[j] = u[j];
        return v;
    };
    const bool aligned = rows % 8 == 0;             // else a partial sum may begin inside an eight
    for (int k = tid >> 4; k < n; k += TBT / 16) {
        const int lo = k * rows, hi = lo + rows, at = lo & ~7;
        const int span = aligned ? rows : rows + 7;
        float s[NV1];
#pragma unroll
        for (int q = 0; q < NV1; ++q) s[q] = 0.0f;
        ColumnRows v = load(at, hi);
        for (int r = 0; r < span; r += 16) {
            const ColumnRows next = load(at + r + 16, hi);
            if (aligned) add_rows<0, false>(v, 0, rows - r, s);
            else add_rows<0, true>(v, lo - at - r, rows, s);
            v = next;
        }
#pragma unroll
        for (int q = 0; q < NV1; ++q) part[k][q][c] = s[q];
    }
    __syncthreads();
    if (tid < NV1 * CW) {
        const int q = tid / CW, o = tid % CW;
        float s = 0.0f;
#pragma unroll 8
        for (int k = 0; k < n; ++k) s += part[k][q][o];
        float *g = a.grad + (uint64_t)m * NPARAM;
        if (q < IN) g[OFF_W1 + (f0 + o) * IN + q] = s;
        else g[OFF_B1 + f0 + o] = s;
    }
}

// Four slices' fragments, lane group e holding rows 8 e .. 8 e + 7 of each, transposed:
// lane group g then holds slice g, its rows 8 e .. in q[e].
__device__ __forceinline__ void slices_to_groups(bf16x8 (&q)[4])
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    u32x4 v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = __builtin_bit_cast(u32x4, q[k]);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
#pragma unroll
        for (int k = 0; k < 2; ++k) {           // the halves of slices k and k + 2
            const auto s = __builtin_amdgcn_permlane32_swap(v[k][d], v[k + 2][d], false, false);
            v[k][d] = s[0];
            v[k + 2][d] = s[1];
        }
#pragma unroll
        for (int k = 0; k < 4; k += 2) {        // the quarters
            const auto s = __builtin_amdgcn_permlane16_swap(v[k][d], v[k + 1][d], false, false);
            v[k][d] = s[0];
            v[k + 1][d] = s[1];
        }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) q[k] = __builtin_bit_cast(bf16x8, v[k]);
}

template <int KS, int WGM> __global__ void __launch_bounds__(TBT, 2) k_train_wgrad(const TrainArgs a)
{
    constexpr int WG_TILES = wg_tiles(WGM);
    constexpr int WC = TWAVES / KS;                             // waves of a chunk
    constexpr int PROD = (WGM / 16) * (WGN / 16) / WC;          // products of a wave: NI x NJ
    constexpr int NI = PROD >= 4 ? 2 : 1;
    constexpr int NJ = PROD / NI;
    constexpr bool AHEAD = WGM > 32;                            // the next slices are fetched ahead
    constexpr int SL = AHEAD || KS == 8 ? 4 : 8;                // slices in flight
    static_assert(NI * NJ * WC == (WGM / 16) * (WGN / 16) && SL % 4 == 0, "the waves of a chunk cover the tile");
    // the sums of the chunks, or the partial sums of the input layer
    __shared__ __align__(16) union {
        float red[KS][WGM * WGN];
        float part[MAX_COLUMNS][NV1][CW];
    } sm;
    __shared__ float redb[KS][WGM];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, c = lane & 15;
    const int nm = a.members, B = a.B;
    // Work-groups go to the 8 XCDs in turn.  XCD x takes layer 3 - x % 2 and the output
    // quarter x / 2 of every member, so its L2 reads a quarter of that layer's dz and its
    // activations once, instead of every operand (26.4 -> 24.1 us at 4096 rows).
    const int tiles = WG_TILES * nm, b = (int)blockIdx.x;
    if (b >= tiles) {
        const int m = (b - tiles) / (COLUMN_BLOCKS + 1), q = (b - tiles) % (COLUMN_BLOCKS + 1);
        if (q < COLUMN_BLOCKS) {
            column_sums(a, m, q * CW, sm.part);
        } else if (tid < HEAD_W) {
            float *grad = a.grad + (uint64_t)m * NPARAM;
            const int n = B / HEAD_ROWS;
            const float *p = a.hpart + (uint64_t)m * n * HEAD_W + tid;
            float s = 0.0f;
#pragma unroll 32
            for (int k = 0; k < n; ++k) s += p[(uint64_t)k * HEAD_W];
            if (tid < H) grad[OFF_W4 + tid] = s;
            else if (tid == H) grad[OFF_B4] = s;
            else if (a.loss) a.loss[m] = s / (float)B;
        }
        return;
    }
    const int m = b / WG_TILES;
    float *grad = a.grad + (uint64_t)m * NPARAM;
    const int x = b % 8, k8 = b % WG_TILES / 8;     // tile k8 of the quarter's, four to a row
    const bool l3 = x % 2 == 0;
    const int o0 = x / 2 * (H / 4) + k8 / 4 * WGM, i0 = k8 % 4 * WGN;
    // this wave's chunk and products: rows i = wi .. of the tile's, columns j = wj ..
    const int chunk = wave % KS, part = wave / KS;
    const int wi = part / (4 / NJ) * NI, wj = part % (4 / NJ) * NJ;
    const int ns = B / KS / 32;                     // slices of a chunk
    const uint64_t mT = (uint64_t)m * H * B + (uint64_t)chunk * ns * (32 * H);
    const bf16_t *dzc = (l3 ? a.dz3T : a.dz2T) + mT + (o0 / 16 + wi) * 512;
    const bf16_t *dz = dzc + lane * 8;
    const bf16_t *av = (l3 ? a.a2T : a.a1T) + mT + (i0 / 16 + wj) * 512 + lane * 8;
    // Bias: the sum of quarter g of every tile of bias_tile rows, for column c of each of
    // this wave's rows of products; the waves with wj = 0 of the first column tile.  A tile
    // of 32 rows has its quarters in the lane groups already; one of 128 has a slice each.
    const bool bias = i0 == 0 && wj == 0, wide = bias_tile(B / KS) == 128;
    floatx4 acc[NI][NJ];
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    float bs[NI] = {};
    if constexpr (AHEAD) {
        struct Slices {
            bf16x8 a[SL][NI], b[SL][NJ];
        } f0, f1;
        auto load = [&](int s0, Slices &f) {
#pragma unroll
            for (int k = 0; k < SL; ++k) {
                const int s = s0 + k;
                if (s < ns) {                   // wave-uniform
#pragma unroll
                    for (int i = 0; i < NI; ++i)
                        f.a[k][i] = *reinterpret_cast<const bf16x8 *>(dz + (uint64_t)s * (32 * H) + 512 * i);
#pragma unroll
                    for (int j = 0; j < NJ; ++j)
                        f.b[k][j] = *reinterpret_cast<const bf16x8 *>(av + (uint64_t)s * (32 * H) + 512 * j);
                }
            }
        };
        auto add = [&](int s0, const Slices &f) {
#pragma unroll
            for (int k = 0; k < SL; ++k)
                if (s0 + k < ns) {
#pragma unroll
                    for (int i = 0; i < NI; ++i)
#pragma unroll
                        for (int j = 0; j < NJ; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.a[k][i], f.b[k][j], acc[i][j], 0, 0, 0);
                }
            if (bias) {
#pragma unroll
                for (int k = 0; k < SL; k += 4) {
                    if (s0 + k >= ns) break;
#pragma unroll
                    for (int i = 0; i < NI; ++i) {
                        bf16x8 q[4] = {f.a[k][i], f.a[k + 1][i], f.a[k + 2][i], f.a[k + 3][i]};
                        if (wide) slices_to_groups(q);
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (s0 + k + e < ns) {
#pragma unroll
                                for (int j = 0; j < 8; ++j) bs[i] += (float)q[e][j];
                            }
                    }
                }
            }
        };
        load(0, f0);
        for (int s0 = 0; s0 < ns; s0 += 2 * SL) {
            load(s0 + SL, f1);
            add(s0, f0);
            load(s0 + 2 * SL, f0);
            add(s0 + SL, f1);
        }
    } else {
        for (int s0 = 0; s0 < ns; s0 += SL) {
            bf16x8 fa[SL][NI], fb[SL][NJ];
#pragma unroll
            for (int k = 0; k < SL; ++k) {
                const int s = s0 + k;
                if (s < ns) {                   // wave-uniform
#pragma unroll
                    for (int i = 0; i < NI; ++i)
                        fa[k][i] = *reinterpret_cast<const bf16x8 *>(dz + (uint64_t)s * (32 * H) + 512 * i);
#pragma unroll
                    for (int j = 0; j < NJ; ++j)
                        fb[k][j] = *reinterpret_cast<const bf16x8 *>(av + (uint64_t)s * (32 * H) + 512 * j);
                }
            }
#pragma unroll
            for (int k = 0; k < SL; ++k)
                if (s0 + k < ns) {
#pragma unroll
                    for (int i = 0; i < NI; ++i)
#pragma unroll
                        for (int j = 0; j < NJ; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[k][i], fb[k][j], acc[i][j], 0, 0, 0);
                }
            if (bias) {
#pragma unroll
                for (int k = 0; k < SL; k += 4) {
                    if (s0 + k >= ns) break;
#pragma unroll
                    for (int i = 0; i < NI; ++i) {
                        bf16x8 q[4] = {fa[k][i], fa[k + 1][i], fa[k + 2][i], fa[k + 3][i]};
                        if (wide) slices_to_groups(q);
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (s0 + k + e < ns) {
#pragma unroll
                                for (int j = 0; j < 8; ++j) bs[i] += (float)q[e][j];
                            }
                    }
                }
            }
        }
    }
    // acc[i][j][e] is dW[o0 + 16 (wi + i) + 4 g + e][i0 + 16 (wj + j) + c] of this chunk's rows
    if (bias) {
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            bs[i] += __shfl_xor(bs[i], 16, 64);
            bs[i] += __shfl_xor(bs[i], 32, 64);
            if (g == 0) redb[chunk][16 * (wi + i) + c] = bs[i];
        }
    }
#pragma unroll
    for (int i = 0; i < NI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                sm.red[chunk][(16 * (wi + i) + 4 * g + e) * WGN + 16 * (wj + j) + c] = acc[i][j][e];
    __syncthreads();
    float *gw = grad + (l3 ? OFF_W3 : OFF_W2);
#pragma unroll
    for (int k = 0; k < WGM * WGN / TBT; ++k) {
        const int q = k * TBT + tid;
        float s = 0.0f;
#pragma unroll
        for (int kc = 0; kc < KS; ++kc) s += sm.red[kc][q];
        gw[(uint64_t)(o0 + q / WGN) * H + i0 + q % WGN] = s;
    }
    if (i0 == 0 && tid < WGM) {
        float s = 0.0f;
#pragma unroll
        for (int kc = 0; kc < KS; ++kc) s += redb[kc][tid];
        grad[(l3 ? OFF_B3 : OFF_B2) + o0 + tid] = s;
    }
}

} // namespace mlp
} // namespace bm
