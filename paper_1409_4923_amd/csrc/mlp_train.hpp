// mlp_train.hpp -- the training step's gradient in two launches.
//
// k_train_rows carries TR rows of one member forward through all layers, through the
// loss, and backward to dz1 without leaving the work-group: activations and dz go from
// layer to layer through LDS, the pre-activations z stay in registers (FP32).  It writes
// the BF16 operands of the weight gradients as MFMA fragments with the rows along a
// lane's registers, so that k_train_wgrad loads a fragment as 1 KiB in a row (stored
// [feature][row] instead, the 16 rows of a fragment lie a power of two apart in the same
// few L2 channels: 16.6 us at 1024 rows), and per-group partial
// sums of the small layers' gradients.  k_train_wgrad forms dW2, dW3 and their biases and
// adds those partials.
//
// What bounds a step of this size (5 members x 1024 rows: 4 GFLOP, 18 MB) is latency:
// one launch per layer and direction (13 of them, each 4 - 17 us, with z, a and dz in
// memory between them) took 97 us with the Adam step, 197 us at 4096 rows; the two
// launches take 27 + 10.5 us and 72 + 24 us, 40 and 98 us with the Adam step.  The arithmetic per element is the layer-by-layer one in the same order up to dz1, so
// the BF16 roundings between the layers are the same.
#pragma once

#include "mlp_kernels.hpp"

namespace bm {
namespace mlp {

constexpr int TRT = 2, TR = 16 * TRT;   // row tiles of 16 and rows per pass of a work-group
constexpr int TWAVES = 8, TBT = 64 * TWAVES;
constexpr int TLD = H + 8;              // LDS row of activations (bf16): 4 banks further per row
constexpr int TTL = 32 + 4;             // LDS row of a wave's transposed weight slice: 8 banks further per 4 rows
constexpr int HEAD_W = H + 2;           // partial record of the output layer: dW4[256], db4, sum e^2
constexpr int NV1 = IN + 1;             // of the input layer: dW1[o][0..4], db1[o]
static_assert(TWAVES * 32 == H, "a wave owns 32 features of a layer");

struct TrainArgs {
    const float *x, *t;                 // rows [.][5] and targets
    const uint32_t *idx;                // row of (member, r): idx[m * B + r], or r if null
    const bf16_t *wbf;
    const float *params;
    int B;                              // rows per member, a multiple of 64
    bf16_t *a1T, *a2T, *dz2T, *dz3T;    // [member][B / 32][16 feature tiles][64 lanes][8 rows]
    float *hpart, *cpart;               // [member][group][HEAD_W], [member][group][NV1][H]
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
// rows takes 46k cycles whatever the batch, 31k of them where the 4 x 128 KiB of weights
// come in (13 B per cycle and CU, the limit of the L1 misses in flight), so a pass of
// more rows would amortise better, but needs the registers that hold z and the weights
// of the next layer.
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
    float sw = 0.0f, sb = 0.0f, se = 0.0f;      // dW4 (threads < 256), db4 and sum e^2 (lanes of wave 4)
    float s1[NV1];                              // dW1, db1 (threads >= 256)
#pragma unroll
    for (int q = 0; q < NV1; ++q) s1[q] = 0.0f;

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
            for (int j = 0; j < IN; ++j) sU[tid][j] = u[j];
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
        if (tid < H) {
#pragma unroll 8
            for (int r = 0; r < TR; ++r) sw = fmaf(sDy[r], bf2f(sAct[0][r * TLD + tid]), sw);
        } else if (tid < H + TR) {              // a row per lane, the lanes added at the end
            sb += sDy[tid - H];
            se = fmaf(sE[tid - H], sE[tid - H], se);
        }
        __syncthreads();
        // ---- dz2 and dz1 ----
        backward(sAct[1], wt, acc);
        asm volatile("" ::: "memory");
        load_wt(BOFF_W2, wt);
        auto gradient = [&](int rt, int t, const float (&z)[4], bf16_t *dst) {
            bf16x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (__bf16)(acc[rt][t][e] * gelu_grad(z[e]));
            put(rt, t, v, dst);
            return v;
        };
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int rt = 0; rt < TRT; ++rt) store(rt, t, gradient(rt, t, z2[rt][t], sAct[0]), a.dz2T);
        __syncthreads();
        backward(sAct[0], wt, acc);
        input_layer([&](int rt, int t, const float (&z)[4]) { gradient(rt, t, z, sAct[1]); });
        __syncthreads();
        if (tid >= H) {
            const int o = tid - H;
#pragma unroll 4
            for (int r = 0; r < TR; ++r) {
                const float d = bf2f(sAct[1][r * TLD + o]);
#pragma unroll
                for (int j = 0; j < IN; ++j) s1[j] = fmaf(d, sU[r][j], s1[j]);
                s1[IN] += d;
            }
        }
        __syncthreads();                        // the next tile overwrites sU and sAct
    }
    if (tid >> 6 == H / 64) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            sb += __shfl_xor(sb, off, 64);
            se += __shfl_xor(se, off, 64);
        }
    }
    const uint64_t blk = (uint64_t)m * a.groups + blockIdx.x;
    if (tid < H) {
        a.hpart[blk * HEAD_W + tid] = sw;
    } else {
        if (tid == H) {
            a.hpart[blk * HEAD_W + H] = sb;
            a.hpart[blk * HEAD_W + H + 1] = se;
        }
#pragma unroll
        for (int q = 0; q < NV1; ++q) a.cpart[(blk * NV1 + q) * H + tid - H] = s1[q];
    }
}

// Weight gradients dW[o][i] = sum_r dz[r][o] a[r][i] of the 256 x 256 layers from the
// fragments of k_train_rows: grid (64 + NV1 + 1) members; a group of the first 64 members
// forms a 32 x 64 tile.  The rows are dealt to the eight waves in
// slices of 32 (wave w: slices w, w + 8, ...), up to four slices' loads in flight, and the
// waves' sums are added in a fixed order through LDS: splitting the rows inside the group
// keeps the chip's 256 CUs busy at small batches without partials in memory.  The bias
// gradients are the row sums of the dz fragments of the first column tile.  The last
// (NV1 + 1) members blocks add the groups' partials of the input and the output layer in order.
constexpr int WG_TILES = 64;
constexpr int WG_BLOCKS = WG_TILES + NV1 + 1;   // per member
constexpr int WGM = 32, WGN = 64;

__global__ void __launch_bounds__(TBT, 2) k_train_wgrad(const TrainArgs a)
{
    __shared__ __align__(16) float red[TWAVES / 2][WGM * WGN];
    __shared__ float redb[TWAVES][WGM];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, c = lane & 15;
    const int nm = a.members, B = a.B;
    // Work-groups go to the 8 XCDs in turn.  XCD x takes layer 3 - x % 2 and the output
    // quarter x / 2 of every member, so its L2 reads a quarter of that layer's dz and its
    // activations once, instead of every operand (26.4 -> 24.1 us at 4096 rows).
    const int tiles = WG_TILES * nm, b = (int)blockIdx.x;
    const int m = b < tiles ? b / WG_TILES : (b - tiles) / (NV1 + 1);
    float *grad = a.grad + (uint64_t)m * NPARAM;
    if (b >= tiles) {
        const int q = (b - tiles) % (NV1 + 1);
        if (q < NV1) {
            if (tid >= H) return;
            const float *p = a.cpart + ((uint64_t)m * a.groups * NV1 + q) * H + tid;
            float s = 0.0f;
#pragma unroll 8
            for (int k = 0; k < a.groups; ++k) s += p[(uint64_t)k * NV1 * H];
            if (q < IN) grad[OFF_W1 + tid * IN + q] = s;
            else grad[OFF_B1 + tid] = s;
        } else if (tid < HEAD_W) {
            const float *p = a.hpart + (uint64_t)m * a.groups * HEAD_W + tid;
            float s = 0.0f;
#pragma unroll 8
            for (int k = 0; k < a.groups; ++k) s += p[(uint64_t)k * HEAD_W];
            if (tid < H) grad[OFF_W4 + tid] = s;
            else if (tid == H) grad[OFF_B4] = s;
            else if (a.loss) a.loss[m] = s / (float)B;
        }
        return;
    }
    const int x = b % 8, k8 = b % WG_TILES / 8;     // tile k8 of the 2 x 4 tiles of a quarter
    const bool l3 = x % 2 == 0;
    const int o0 = (x / 2 * 2 + k8 / 4) * WGM, i0 = k8 % 4 * WGN;
    const uint64_t mT = (uint64_t)m * H * B;
    const bf16_t *dz = (l3 ? a.dz3T : a.dz2T) + mT + o0 / 16 * 512 + lane * 8;
    const bf16_t *av = (l3 ? a.a2T : a.a1T) + mT + i0 / 16 * 512 + lane * 8;
    floatx4 acc[2][4];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    float bs[2] = {0.0f, 0.0f};
    constexpr int SL = 4;                       // slices in flight
    const int ns = B / 32;
    for (int s0 = wave; s0 < ns; s0 += SL * TWAVES) {
        bf16x8 fa[SL][2], fb[SL][4];
#pragma unroll
        for (int k = 0; k < SL; ++k) {
            const int s = s0 + k * TWAVES;
            if (s < ns) {                       // wave-uniform
#pragma unroll
                for (int i = 0; i < 2; ++i)
                    fa[k][i] = *reinterpret_cast<const bf16x8 *>(dz + (uint64_t)s * (32 * H) + 512 * i);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    fb[k][j] = *reinterpret_cast<const bf16x8 *>(av + (uint64_t)s * (32 * H) + 512 * j);
            }
        }
#pragma unroll
        for (int k = 0; k < SL; ++k) {
            if (s0 + k * TWAVES < ns) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[k][i], fb[k][j], acc[i][j], 0, 0, 0);
                if (i0 == 0) {
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 8; ++j) bs[i] += (float)fa[k][i][j];
                }
            }
        }
    }
    // acc[i][j][e] is dW[o0 + 16 i + 4 g + e][i0 + 16 j + c] of this wave's rows
    auto at = [&](int i, int j, int e) { return (16 * i + 4 * g + e) * WGN + 16 * j + c; };
    if (i0 == 0) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            bs[i] += __shfl_xor(bs[i], 16, 64);
            bs[i] += __shfl_xor(bs[i], 32, 64);
            if (g == 0) redb[wave][16 * i + c] = bs[i];
        }
    }
    if (wave >= TWAVES / 2) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) red[wave - TWAVES / 2][at(i, j, e)] = acc[i][j][e];
    }
    __syncthreads();
    if (wave < TWAVES / 2) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) red[wave][at(i, j, e)] += acc[i][j][e];
    }
    __syncthreads();
    float *gw = grad + (l3 ? OFF_W3 : OFF_W2);
#pragma unroll
    for (int k = 0; k < WGM * WGN / TBT; ++k) {
        const int q = k * TBT + tid;
        gw[(uint64_t)(o0 + q / WGN) * H + i0 + q % WGN] = (red[0][q] + red[1][q]) + (red[2][q] + red[3][q]);
    }
    if (i0 == 0 && tid < WGM) {
        float s = 0.0f;
#pragma unroll
        for (int w = 0; w < TWAVES; ++w) s += redb[w][tid];
        grad[(l3 ? OFF_B3 : OFF_B2) + o0 + tid] = s;
    }
}

} // namespace mlp
} // namespace bm
