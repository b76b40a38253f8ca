// mlp.hip -- ensemble MLP surrogate: inference, training (back-propagation of the
// mean squared error, Adam), ensemble statistics and the routing of uncertain
// queries to the Monte Carlo fallback.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>
#include <mutex>

#include "bmotor.h"
#include "common.hpp"
#include "host.hpp"
#include "mlp_kernels.hpp"
#include "mlp_train.hpp"

using namespace bm;
using namespace bm::host;
using namespace bm::mlp;

static_assert(NPARAM == BM_MLP_PARAMS, "parameter block differs from bmotor.h");
static_assert(NBF == BM_MLP_BF16, "BF16 block differs from bmotor.h");
static_assert(IN == BM_MLP_INPUTS && H == BM_MLP_HIDDEN, "shape differs from bmotor.h");

namespace {


// BF16 index of parameter p of a member, or -1 for biases.
__device__ __forceinline__ int bf_index(int p)
{
    if (p < OFF_B1) return BOFF_W1 + (p - OFF_W1);
    if (p >= OFF_W2 && p < OFF_B2) return BOFF_W2 + (p - OFF_W2);
    if (p >= OFF_W3 && p < OFF_B3) return BOFF_W3 + (p - OFF_W3);
    if (p >= OFF_W4 && p < OFF_B4) return BOFF_W4 + (p - OFF_W4);
    return -1;
}

__global__ void __launch_bounds__(256) k_cast(const float *params, bf16_t *wbf, uint64_t total)
{
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    const uint64_t m = i / NPARAM;
    const int p = (int)(i - m * NPARAM);
    const int b = bf_index(p);
    if (b >= 0) wbf[m * NBF + b] = f2bf(params[i]);
}

// Adam (Kingma & Ba) with bias-corrected moments, then the BF16 weight copy.
__global__ void __launch_bounds__(256) k_adam(float *params, const float *grad, float *mo, float *ve, bf16_t *wbf,
                                              uint64_t total, float lr, float b1, float b2, float eps, float c1,
                                              float c2)
{
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    const float g = grad[i];
    const float m = b1 * mo[i] + (1.0f - b1) * g;
    const float v = b2 * ve[i] + (1.0f - b2) * g * g;
    mo[i] = m;
    ve[i] = v;
    const float p = params[i] - lr * (m * c1) / (sqrtf(v * c2) + eps);
    params[i] = p;
    const uint64_t mem = i / NPARAM;
    const int b = bf_index((int)(i - mem * NPARAM));
    if (b >= 0) wbf[mem * NBF + b] = f2bf(p);
}

// Initial parameters U(-1/sqrt(fan_in), 1/sqrt(fan_in)) from Philox (tag 4).
__global__ void __launch_bounds__(256) k_init_params(float *params, uint64_t total, uint32_t k0, uint32_t k1)
{
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= total) return;
    const uint64_t m = i / NPARAM;
    const int p = (int)(i - m * NPARAM);
    const U4 q = philox4x32_10((uint32_t)p, (uint32_t)m, 0u, 4u, k0, k1);
    const float u = (float)(q.x >> 8) * 0x1p-24f * 2.0f - 1.0f;
    const float fan = (p < OFF_W2) ? (float)IN : (float)H;
    params[i] = u / sqrtf(fan);
}

// Mean and population std of the members' predictions of row b; true if the row is
// routed to the fallback.
__device__ __forceinline__ bool row_stats(const float *y, int members, uint64_t B, uint64_t b, float thr, float *mean,
                                          float *stdv)
{
    float s = 0.0f;
    for (int m = 0; m < members; ++m) s += y[(uint64_t)m * B + b];
    const float mu = s / (float)members;
    float v = 0.0f;
    for (int m = 0; m < members; ++m) {
        const float d = y[(uint64_t)m * B + b] - mu;
        v = fmaf(d, d, v);
    }
    const float sd = sqrtf(v / (float)members);
    mean[b] = mu;
    stdv[b] = sd;
    return !(sd <= thr);                        // NaN std also falls back
}

// Rank of this thread's flag among the flags of its work-group (cnt: a counter per wave),
// and their number.
__device__ __forceinline__ uint32_t flag_rank(bool flag, uint32_t *cnt, uint32_t &total)
{
    const unsigned long long bal = __ballot(flag);
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) cnt[w] = (uint32_t)__popcll(bal);
    __syncthreads();
    uint32_t before = 0;
    total = 0;
    for (int i = 0; i < (int)(blockDim.x >> 6); ++i) {
        before += i < w ? cnt[i] : 0u;
        total += cnt[i];
    }
    return before + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
}

// A query of at most ROUTE_ROWS rows in one work-group: statistics, routing flags and the
// ordered compaction (three launches' work; 9 us of a 28 us query of 100 rows).
constexpr int ROUTE_ROWS = 1024;

__global__ void __launch_bounds__(ROUTE_ROWS) k_route_small(const float *y, int members, uint32_t B, float thr,
                                                            float *mean, float *stdv, uint32_t *out, uint32_t *count)
{
    __shared__ uint32_t cnt[ROUTE_ROWS / 64];
    const uint32_t b = threadIdx.x;
    const bool flag = b < B && row_stats(y, members, B, b, thr, mean, stdv);
    uint32_t total;
    const uint32_t rank = flag_rank(flag, cnt, total);
    if (flag) out[rank] = b;
    if (b == 0) *count = total;
}

// Statistics of 256 rows per work-group and the number of routed ones; grid over rows.
__global__ void __launch_bounds__(256) k_stats(const float *y, int members, uint64_t B, float thr, float *mean,
                                               float *stdv, uint32_t *blk_count)
{
    const uint64_t b = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    const bool flag = b < B && row_stats(y, members, B, b, thr, mean, stdv);
    __shared__ uint32_t cnt[4];
    uint32_t total;
    (void)flag_rank(flag, cnt, total);
    if (threadIdx.x == 0) blk_count[blockIdx.x] = total;
}

// Exclusive scan of the block counts (one block, sequential chunks) and the total.
__global__ void __launch_bounds__(256) k_scan_counts(uint32_t *blk, uint64_t nblk, uint32_t *total)
{
    __shared__ uint32_t part[256];
    const uint64_t per = (nblk + 255) / 256;
    const uint64_t lo = per * threadIdx.x, hi = lo + per < nblk ? lo + per : nblk;
    uint32_t s = 0;
    for (uint64_t i = lo; i < hi; ++i) s += blk[i];
    part[threadIdx.x] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t acc = 0;
        for (int i = 0; i < 256; ++i) { const uint32_t c = part[i]; part[i] = acc; acc += c; }
        *total = acc;
    }
    __syncthreads();
    uint32_t acc = part[threadIdx.x];
    for (uint64_t i = lo; i < hi; ++i) { const uint32_t c = blk[i]; blk[i] = acc; acc += c; }
}

// Scatter the flagged row indices in increasing order.  blk: the work-groups' counts
// scanned by k_scan_counts (SCANNED), or as k_stats left them: each group then adds up
// those before it, and the last one writes the total.
template <bool SCANNED>
__global__ void __launch_bounds__(256) k_compact(const float *stdv, uint64_t B, float thr, const uint32_t *blk,
                                                 uint32_t *out, uint32_t *count)
{
    const uint64_t b = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    const bool flag = b < B && !(stdv[b] <= thr);
    __shared__ uint32_t cnt[4], sum[4];
    uint32_t base = 0;
    if constexpr (SCANNED) {
        base = blk[blockIdx.x];
    } else {
        uint32_t s = 0;
#pragma unroll 8
        for (uint32_t i = threadIdx.x; i < blockIdx.x; i += 256) s += blk[i];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) s += __shfl_xor(s, off, 64);
        if ((threadIdx.x & 63) == 0) sum[threadIdx.x >> 6] = s;
    }
    uint32_t total;
    const uint32_t rank = flag_rank(flag, cnt, total);       // its barrier publishes sum as well
    if constexpr (!SCANNED) {
        base = (sum[0] + sum[1]) + (sum[2] + sum[3]);
        if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) *count = base + total;
    }
    if (flag) out[base + rank] = (uint32_t)b;
}

// ---------------------------------------------------------------------------
// Workspace layout
// ---------------------------------------------------------------------------
size_t up(size_t v) { return (v + 255) & ~(size_t)255; }

struct MlpLayout {
    size_t a1, a2, dz1, dz2, dz3, u, hpart, y, blk, total;
};

// Work-groups per member of the training pass: one per 32 rows, but no more in all than
// the 256 CUs take at once (a group then takes several row tiles, in as many passes as the
// fullest group needs).
int train_groups(uint32_t nm, uint64_t batch)
{
    const int tiles = (int)(batch / TR);
    const int most = (int)(256 / nm);
    const int passes = (tiles + most - 1) / most;
    return (tiles + passes - 1) / passes;
}

MlpLayout mlp_layout(uint32_t nm, uint64_t batch, bool training)
{
    MlpLayout L{};
    const uint64_t R = batch;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o += up(bytes); return at; };
    if (training) {                    // operands of the gradients, records of the output layer
        L.a1 = take(nm * R * H * 2);
        L.a2 = take(nm * R * H * 2);
        L.dz1 = take(nm * R * H * 2);
        L.dz2 = take(nm * R * H * 2);
        L.dz3 = take(nm * R * H * 2);
        L.u = take(nm * R * IN * 4);
        L.hpart = take(nm * (R / HEAD_ROWS) * HEAD_W * 4);
    } else {                           // inference keeps its activations in registers
        L.y = take(nm * batch * 4);
        L.blk = take(((batch + 255) / 256) * 4 + 4);
    }
    L.total = o;
    return L;
}

int check_members(uint32_t nm)
{
    if (nm < 1 || nm > BM_MLP_MAX_MEMBERS)
        return fail(BM_ERR_INVALID_ARG, "n_members must be in [1, %d]", BM_MLP_MAX_MEMBERS);
    return BM_OK;
}

int check_ws(const MlpLayout &L, void *d_ws, size_t ws_bytes)
{
    if (!d_ws || ((uintptr_t)d_ws & 255u)) return fail(BM_ERR_WORKSPACE, "workspace NULL or not 256-byte aligned");
    if (ws_bytes < L.total) return fail(BM_ERR_WORKSPACE, "workspace %zu B < %zu B needed", ws_bytes, L.total);
    return BM_OK;
}

// ---------------------------------------------------------------------------
// Fused inference: one work-group runs 128 rows of one member through all four
// layers; activations never leave the registers.  The 256 x 256 layers are
// computed transposed, Z^T = W A^T, with W as the MFMA A operand and the
// activations as the B operand: a 16 x 16 output tile leaves lane (g = lane/16,
// c = lane%16) holding features 4g..4g+3 of row c, which is exactly the B-operand
// slot of the next layer if its contraction index is permuted -- k-step s, slot j
// of lane group g stands for feature 32 s + 4 g + j (j < 4) or 32 s + 16 + 4 g +
// (j - 4) (j >= 4), and the W fragments are read from LDS in that order.
// The contraction runs outermost: each wave keeps the accumulators of all 16 output
// tiles of its 32 rows (128 registers) and walks the 8 k-steps of a layer, so W is
// staged one 32-wide k slice (all 256 output rows) at a time and the GELU epilogue
// runs once per layer.  256 registers per lane give two waves per SIMD (two
// work-groups per CU), so one group's epilogue overlaps the other's MFMAs.
// ---------------------------------------------------------------------------
constexpr int FROWS = 128;             // rows per work-group
constexpr int INFER_RT = 2;            // row tiles of 16 per wave
constexpr int INFER_BT = 256;          // 4 waves per work-group
constexpr int SK = 32;                 // row of a staged k slice (bf16), 16-byte pairs swizzled
constexpr int NSLICE = 16;             // k slices of the two 256 x 256 layers

__device__ __forceinline__ __bf16 to_bf(float f) { return (__bf16)f; }   // v_cvt_pk_bf16_f32 (RNE)

__device__ __forceinline__ int perm_feature(int s, int g, int j)
{
    return 32 * s + (j < 4 ? 4 * g + j : 16 + 4 * g + (j - 4));
}

__global__ void __launch_bounds__(INFER_BT, 2) k_mlp_infer(const float *x, uint64_t rows, const bf16_t *wbf,
                                                           const float *params, float *y, uint64_t y_stride)
{
    constexpr int RT = INFER_RT, BT = INFER_BT;
    static_assert(BT == H, "thread t fills the small tables' entries of feature t");
    static_assert(BT / 64 * 16 * RT == FROWS, "the waves cover the group's rows");
    __shared__ __align__(16) bf16_t sW[3][H * SK];
    __shared__ __align__(16) float sL1[H * 8];          // per feature: W1[f][0..4], b1[f], pad
    __shared__ __align__(16) float sB[2][H];
    __shared__ float sW4[H];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6, g = lane >> 4, c = lane & 15;
    const int m = blockIdx.y;
    const float *P = params + (uint64_t)m * NPARAM;
    const bf16_t *WB = wbf + (uint64_t)m * NBF;
#pragma unroll
    for (int j = 0; j < IN; ++j) sL1[t * 8 + j] = bf2f(WB[BOFF_W1 + t * IN + j]);
    sL1[t * 8 + 5] = P[OFF_B1 + t];
    sB[0][t] = P[OFF_B2 + t];
    sB[1][t] = P[OFF_B3 + t];
    sW4[t] = bf2f(WB[BOFF_W4 + t]);

    // slice T: layer 2 + T / 8, k columns 32 (T % 8) .. + 31 of all 256 rows, in
    // 16-byte units: unit u = t + i BT is row u / 4, columns 8 (u % 4) .. + 7
    constexpr int UNITS = H * 32 / 8 / BT;
    auto load_slice = [&](int T, uint4 (&v)[UNITS]) {
        const bf16_t *W = WB + (T < 8 ? BOFF_W2 : BOFF_W3) + 32 * (T & 7);
#pragma unroll
        for (int i = 0; i < UNITS; ++i) {
            const int u = t + i * BT;
            v[i] = *reinterpret_cast<const uint4 *>(W + (uint64_t)(u >> 2) * H + (u & 3) * 8);
        }
    };
    // In LDS a slice row holds four 16-byte pairs: pair p is 8-byte unit p (k columns
    // 4p .. 4p + 3) followed by unit p + 4, which is exactly one lane group's A
    // fragment (one 16-byte read, no register shuffling), and it sits at position
    // p ^ ((r >> 1) & 3) of row r, so the 8 lanes a read serves at a time hit
    // different banks.  Inside the k loop a slice is staged in two halves of
    // UNITS / 2 units per thread.
    auto load_half = [&](int T, int hf, uint4 (&v)[UNITS / 2]) {
        const bf16_t *W = WB + (T < 8 ? BOFF_W2 : BOFF_W3) + 32 * (T & 7);
#pragma unroll
        for (int i = 0; i < UNITS / 2; ++i) {
            const int u = t + (i + hf * UNITS / 2) * BT;
            v[i] = *reinterpret_cast<const uint4 *>(W + (uint64_t)(u >> 2) * H + (u & 3) * 8);
        }
    };
    auto store_half = [&](int buf, int hf, const uint4 (&v)[UNITS / 2]) {
#pragma unroll
        for (int i = 0; i < UNITS / 2; ++i) {
            const int u = t + (i + hf * UNITS / 2) * BT;
            const int r = u >> 2, q = u & 3, f = (r >> 1) & 3;
            const int p0 = (2 * q) & 3, p1 = (2 * q + 1) & 3, hf = q >> 1;   // units 2q, 2q + 1
            *reinterpret_cast<uint2 *>(&sW[buf][r * SK + (p0 ^ f) * 8 + 4 * hf]) = uint2{v[i].x, v[i].y};
            *reinterpret_cast<uint2 *>(&sW[buf][r * SK + (p1 ^ f) * 8 + 4 * hf]) = uint2{v[i].z, v[i].w};
        }
    };
    auto store_slice = [&](int buf, const uint4 (&v)[UNITS]) {
#pragma unroll
        for (int i = 0; i < UNITS; ++i) {
            const int u = t + i * BT;
            const int r = u >> 2, q = u & 3, f = (r >> 1) & 3;
            const int p0 = (2 * q) & 3, p1 = (2 * q + 1) & 3, hf = q >> 1;   // units 2q, 2q + 1
            *reinterpret_cast<uint2 *>(&sW[buf][r * SK + (p0 ^ f) * 8 + 4 * hf]) = uint2{v[i].x, v[i].y};
            *reinterpret_cast<uint2 *>(&sW[buf][r * SK + (p1 ^ f) * 8 + 4 * hf]) = uint2{v[i].z, v[i].w};
        }
    };
    uint4 pv[UNITS];
    load_slice(0, pv);
    store_slice(0, pv);
    load_slice(1, pv);
    store_slice(1, pv);
    __syncthreads();

    // ---- layer 1 (5 -> 256, FP32 FMA on the BF16 weights) into B operands; each
    //      weight row read from LDS once for both row tiles ----
    const uint64_t base = (uint64_t)blockIdx.x * FROWS + (uint64_t)wave * 16 * RT;
    bf16x8 act[RT][8];
    float u[RT][IN];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        const uint64_t r = base + 16 * rt + c;
        normalise(x + (r < rows ? r : 0) * IN, u[rt]);
    }
#pragma unroll
    for (int s = 0; s < 8; ++s) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float *w = &sL1[perm_feature(s, g, j) * 8];
            const float4 w03 = *reinterpret_cast<const float4 *>(w);
            const float2 w45 = *reinterpret_cast<const float2 *>(w + 4);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                float z = w45.y;
                z = fmaf(w03.x, u[rt][0], z);
                z = fmaf(w03.y, u[rt][1], z);
                z = fmaf(w03.z, u[rt][2], z);
                z = fmaf(w03.w, u[rt][3], z);
                z = fmaf(w45.x, u[rt][4], z);
                act[rt][s][j] = to_bf(gelu(z));
            }
        }
    }

    // ---- layers 2 and 3 on MFMA, k slice by k slice ----
    // Slice T lives in LDS buffer T % 3; slice T + 2 is fetched from global memory
    // during iteration T, half after half, and stored into the buffer slice T - 1
    // used, which every wave finished reading before the barrier that ended iteration
    // T - 1.  That barrier also published slice T + 1 before iteration T + 1 reads it.
    floatx4 acc[16][RT];
#pragma unroll
    for (int T = 0; T < NSLICE; ++T) {
        const int s = T & 7;
        uint4 ph[UNITS / 2];
        if (T + 2 < NSLICE) load_half(T + 2, 0, ph);
        // The MFMA block runs at raised wave priority, so the scheduler keeps the
        // matrix cores fed from this wave while the other group's wave on the SIMD
        // works through its VALU epilogue.
        __builtin_amdgcn_s_setprio(1);
        // lane (g, c) reads pair g (units g and 4 + g) of rows 16 ft + c
        const bf16_t *sfr = &sW[T % 3][c * SK + 8 * (g ^ ((c >> 1) & 3))];
#pragma unroll
        for (int ft = 0; ft < 16; ++ft) {
            if (ft == 8 && T + 2 < NSLICE) {
                store_half((T + 2) % 3, 0, ph);
                load_half(T + 2, 1, ph);
            }
            const bf16x8 a = *reinterpret_cast<const bf16x8 *>(sfr + 16 * ft * SK);
            // the accumulators start at the bias of their output features
            const floatx4 bias = *reinterpret_cast<const floatx4 *>(&sB[T >> 3][16 * ft + 4 * g]);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
                acc[ft][rt] =
                    __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, act[rt][s], s == 0 ? bias : acc[ft][rt], 0, 0, 0);
        }
        __builtin_amdgcn_s_setprio(0);
        if (s == 7) {
            // epilogue: acc[ft][rt][i] = Z^T[16 ft + 4 g + i][row c of tile rt] -> the
            // next layer's slot (k-step ft / 2, j = 4 (ft % 2) + i)
#pragma unroll
            for (int ft = 0; ft < 16; ++ft)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int i = 0; i < 4; ++i) act[rt][ft >> 1][4 * (ft & 1) + i] = to_bf(gelu(acc[ft][rt][i]));
        }
        if (T + 2 < NSLICE) store_half((T + 2) % 3, 1, ph);
        __syncthreads();
    }

    // ---- layer 4 (256 -> 1): partial dot per lane group, then across the 4 groups ----
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
        float sum = 0.0f;
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
            for (int j = 0; j < 8; ++j) sum = fmaf((float)act[rt][s][j], sW4[perm_feature(s, g, j)], sum);
        sum += __shfl_xor(sum, 16, 64);
        sum += __shfl_xor(sum, 32, 64);
        const uint64_t r = base + 16 * rt + c;
        if (g == 0 && r < rows) y[(uint64_t)m * y_stride + r] = sum + P[OFF_B4];
    }
}

// ---------------------------------------------------------------------------
// Inference of few rows.  k_mlp_infer walks 16 weight slices one after another, a global
// load, an LDS write and a barrier each: about 20 us however few the rows.  Here a group
// of eight waves holds both 256 x 256 layers of a member in registers -- wave w the
// weights of features 32 w .. 32 w + 31, 128 registers per lane -- and activations pass
// between the waves through LDS, four barriers per tile of 32 rows.  The weights of a wave
// are 16 KiB in a row per layer: loaded 1 KiB at a time, all of them in flight, and
// turned into fragments through a private LDS tile (the fragments' own 8-byte pieces
// loaded directly took 13 us of the call, this 3 us).  100 rows x 5 members: 10 us against
// 20.5 us; 3264 rows (two tiles per group): 14 against 21 us.  Same fragments, accumulator start
// and element-wise order as k_mlp_infer, so a row's prediction does not depend on which of
// the two runs.
// ---------------------------------------------------------------------------
constexpr int SWAVES = 8, SBT = 64 * SWAVES;
constexpr int SRT = 2, SROWS = 16 * SRT;
// Most tiles of a group; beyond, k_mlp_infer is faster (5 members: 10.2 against 20.4 us with
// one tile per group, 14.0 and 20.3 with two, 18.0 and 20.3 with three, 22.0 and 20.6 with
// four; 1 and 16 members the same within 2 us).
constexpr int INFER_PASSES = 3;
constexpr int SLD = H + 8;             // LDS row (bf16): 4 banks further per row
static_assert(SWAVES * 32 == H, "wave w owns k-step w of the next layer");

__global__ void __launch_bounds__(SBT, 2) k_mlp_infer_rows(const float *x, uint64_t rows, const bf16_t *wbf,
                                                           const float *params, float *y, uint64_t y_stride)
{
    __shared__ __align__(16) bf16_t sAct[2][SROWS * SLD];
    __shared__ __align__(16) bf16_t sTile[SWAVES][16 * SLD];
    __shared__ __align__(16) float sL1[H * 8];           // per feature: W1[f][0..4], b1[f], pad
    __shared__ __align__(16) float sB[2][H];
    __shared__ __align__(16) float sW4[H];               // in the permuted order
    __shared__ __align__(16) float sU[SROWS * 8];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, c = lane & 15;
    const int m = blockIdx.y;
    const float *P = params + (uint64_t)m * NPARAM;
    const bf16_t *WB = wbf + (uint64_t)m * NBF;

    // inputs of a tile: a row per thread of the first SROWS
    float xr[IN] = {};
    auto fetch = [&](uint64_t tile) {
        const uint64_t r = tile * SROWS + tid;
        if (tid < SROWS) {
#pragma unroll
            for (int j = 0; j < IN; ++j) xr[j] = x[(r < rows ? r : 0) * IN + j];
        }
    };
    fetch(blockIdx.x);
    // the wave's rows of layer 2, then 3, 16 rows (8 KiB) at a time
    bf16x8 raw[4][8];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int i = 0; i < 8; ++i)
            raw[q][i] = *reinterpret_cast<const bf16x8 *>(WB + (q < 2 ? BOFF_W2 : BOFF_W3) +
                                                         (32 * wave + 16 * (q & 1)) * H + (64 * i + lane) * 8);
    if (tid < H) {
#pragma unroll
        for (int j = 0; j < IN; ++j) sL1[tid * 8 + j] = bf2f(WB[BOFF_W1 + tid * IN + j]);
        sL1[tid * 8 + 5] = P[OFF_B1 + tid];
    } else {
        const int f = tid - H, s = f >> 5, q = f & 31;
        sB[0][f] = P[OFF_B2 + f];
        sB[1][f] = P[OFF_B3 + f];
        // feature f's place in the permuted order of perm_feature
        sW4[32 * s + (q & 12) * 2 + (q & 3) + (q >> 4) * 4] = bf2f(WB[BOFF_W4 + f]);
    }
    const float b4 = P[OFF_B4];
    bf16x8 w[2][2][8];                       // [layer][feature tile][k-step]
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        bf16_t *t = sTile[wave];             // private: the wave's LDS accesses complete in order
#pragma unroll
        for (int i = 0; i < 8; ++i)
            *reinterpret_cast<bf16x8 *>(&t[(2 * i + (lane >> 5)) * SLD + (lane & 31) * 8]) = raw[q][i];
        asm volatile("" ::: "memory");
#pragma unroll
        for (int s = 0; s < 8; ++s) {
            struct Two { uint2 a, b; } v{*reinterpret_cast<const uint2 *>(&t[c * SLD + 32 * s + 4 * g]),
                                         *reinterpret_cast<const uint2 *>(&t[c * SLD + 32 * s + 16 + 4 * g])};
            w[q >> 1][q & 1][s] = __builtin_bit_cast(bf16x8, v);
        }
        asm volatile("" ::: "memory");
    }

    // eight values of row 16 rt + c: this wave's features, which are k-step `wave` of the
    // next layer, at the place of its fragment
    auto put = [&](bf16_t *dst, int rt, bf16x8 v) {
        *reinterpret_cast<bf16x8 *>(dst + (16 * rt + c) * SLD + 32 * wave + 8 * g) = v;
    };
    auto layer = [&](int l, const bf16_t *in, bf16_t *out) {
        floatx4 acc[2][SRT];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const floatx4 bias = *reinterpret_cast<const floatx4 *>(&sB[l][32 * wave + 16 * t + 4 * g]);
#pragma unroll
            for (int rt = 0; rt < SRT; ++rt) acc[t][rt] = bias;
        }
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
            for (int rt = 0; rt < SRT; ++rt) {
                const bf16x8 b = *reinterpret_cast<const bf16x8 *>(in + (16 * rt + c) * SLD + 32 * s + 8 * g);
#pragma unroll
                for (int t = 0; t < 2; ++t)
                    acc[t][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[l][t][s], b, acc[t][rt], 0, 0, 0);
            }
#pragma unroll
        for (int rt = 0; rt < SRT; ++rt) {
            bf16x8 v;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * t + e] = to_bf(gelu(acc[t][rt][e]));
            put(out, rt, v);
        }
    };

    const uint64_t tiles = (rows + SROWS - 1) / SROWS;
    for (uint64_t tile = blockIdx.x; tile < tiles; tile += gridDim.x) {
        if (tid < SROWS) {
            float u[IN];
            normalise(xr, u);
#pragma unroll
            for (int j = 0; j < IN; ++j) sU[tid * 8 + j] = u[j];
        }
        if (tile + gridDim.x < tiles) fetch(tile + gridDim.x);
        __syncthreads();
        // ---- layer 1 (5 -> 256, FP32 FMA on the BF16 weights) ----
        {
            bf16x8 v[SRT];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float *wr = &sL1[perm_feature(wave, g, j) * 8];
                const float4 w03 = *reinterpret_cast<const float4 *>(wr);
                const float2 w45 = *reinterpret_cast<const float2 *>(wr + 4);
#pragma unroll
                for (int rt = 0; rt < SRT; ++rt) {
                    const float *u = &sU[(16 * rt + c) * 8];
                    float z = w45.y;
                    z = fmaf(w03.x, u[0], z);
                    z = fmaf(w03.y, u[1], z);
                    z = fmaf(w03.z, u[2], z);
                    z = fmaf(w03.w, u[3], z);
                    z = fmaf(w45.x, u[4], z);
                    v[rt][j] = to_bf(gelu(z));
                }
            }
#pragma unroll
            for (int rt = 0; rt < SRT; ++rt) put(sAct[0], rt, v[rt]);
        }
        __syncthreads();
        layer(0, sAct[0], sAct[1]);
        __syncthreads();
        layer(1, sAct[1], sAct[0]);
        __syncthreads();
        // ---- layer 4 (256 -> 1): a wave per 16 rows, partial dot per lane group, then
        //      across the 4 groups ----
        if (wave < SRT) {
            const bf16_t *src = sAct[0] + (16 * wave + c) * SLD + 8 * g;
            float sum = 0.0f;
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const bf16x8 a = *reinterpret_cast<const bf16x8 *>(src + 32 * s);
#pragma unroll
                for (int j = 0; j < 8; ++j) sum = fmaf((float)a[j], sW4[32 * s + 8 * g + j], sum);
            }
            sum += __shfl_xor(sum, 16, 64);
            sum += __shfl_xor(sum, 32, 64);
            const uint64_t r = tile * SROWS + 16 * wave + c;
            if (g == 0 && r < rows) y[(uint64_t)m * y_stride + r] = sum + b4;
        }
        // the next tile writes sU (read by layer 1, two barriers ago) before its first
        // barrier and sAct[0] after it
    }
}

// Members' predictions y [nm][rows].
hipError_t launch_infer(uint32_t nm, const float *x, uint64_t rows, const bf16_t *wbf, const float *params, float *y,
                        hipStream_t s)
{
    const uint64_t tiles = (rows + SROWS - 1) / SROWS;
    const uint64_t most = 256 / nm;                  // groups of eight waves: one per CU
    if (tiles <= (uint64_t)INFER_PASSES * most) {
        hipLaunchKernelGGL(k_mlp_infer_rows, dim3((uint32_t)(tiles < most ? tiles : most), nm), dim3(SBT), 0, s, x, rows,
                           wbf, params, y, rows);
    } else {
        hipLaunchKernelGGL(k_mlp_infer, dim3((uint32_t)((rows + FROWS - 1) / FROWS), nm), dim3(INFER_BT), 0, s, x, rows,
                           wbf, params, y, rows);
    }
    return hipGetLastError();
}

} // namespace

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------
extern "C" int bm_mlp_workspace_size(uint32_t n_members, uint64_t batch, uint32_t training, size_t *bytes)
{
    int rc = check_members(n_members);
    if (rc) return rc;
    if (!bytes) return fail(BM_ERR_INVALID_ARG, "bytes must not be NULL");
    if (batch < 1 || batch > 0xFFFFFFFFull) return fail(BM_ERR_INVALID_ARG, "batch must be in [1, 2^32 - 1]");
    if (training && (batch % 64 != 0 || batch > 65536))
        return fail(BM_ERR_INVALID_ARG, "training batch must be a multiple of 64 and <= 65536");
    *bytes = mlp_layout(n_members, batch, training != 0).total;
    return ok();
}

extern "C" int bm_mlp_init(uint32_t n_members, uint64_t seed, float *d_params, void *stream)
{
    int rc = check_members(n_members);
    if (rc) return rc;
    if (!d_params) return fail(BM_ERR_INVALID_ARG, "d_params must not be NULL");
    int dev;
    rc = check_device(&dev);
    if (rc) return rc;
    const uint64_t total = (uint64_t)n_members * NPARAM;
    hipLaunchKernelGGL(k_init_params, dim3((uint32_t)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream,
                       d_params, total, (uint32_t)seed, (uint32_t)(seed >> 32));
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? ok() : hip_fail(e, "bm_mlp_init");
}

extern "C" int bm_mlp_cast(uint32_t n_members, const float *d_params, uint16_t *d_wbf, void *stream)
{
    int rc = check_members(n_members);
    if (rc) return rc;
    if (!d_params || !d_wbf) return fail(BM_ERR_INVALID_ARG, "NULL pointer");
    int dev;
    rc = check_device(&dev);
    if (rc) return rc;
    const uint64_t total = (uint64_t)n_members * NPARAM;
    hipLaunchKernelGGL(k_cast, dim3((uint32_t)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream, d_params,
                       (bf16_t *)d_wbf, total);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? ok() : hip_fail(e, "bm_mlp_cast");
}

extern "C" int bm_mlp_forward(uint32_t n_members, const float *d_params, const uint16_t *d_wbf, const float *d_x,
                              uint64_t batch, float *d_y, void *d_ws, size_t ws_bytes, void *stream)
{
    int rc = check_members(n_members);
    if (rc) return rc;
    if (!d_params || !d_wbf || !d_x || !d_y) return fail(BM_ERR_INVALID_ARG, "NULL pointer");
    if (batch < 1 || batch > 0xFFFFFFFFull) return fail(BM_ERR_INVALID_ARG, "batch must be in [1, 2^32 - 1]");
    const MlpLayout L = mlp_layout(n_members, batch, false);
    rc = check_ws(L, d_ws, ws_bytes);
    if (rc) return rc;
    int dev;
    rc = check_device(&dev);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    const hipError_t e = launch_infer(n_members, d_x, batch, (const bf16_t *)d_wbf, d_params, d_y, s);
    return e == hipSuccess ? ok() : hip_fail(e, "bm_mlp_forward");
}

extern "C" int bm_mlp_backward(uint32_t n_members, const float *d_params, const uint16_t *d_wbf, const float *d_x,
                               const float *d_t, const uint32_t *d_idx, uint64_t batch, float *d_grad,
                               float *d_loss, void *d_ws, size_t ws_bytes, void *stream)
{
    int rc = check_members(n_members);
    if (rc) return rc;
    if (!d_params || !d_wbf || !d_x || !d_t || !d_grad) return fail(BM_ERR_INVALID_ARG, "NULL pointer");
    if (batch < 64 || batch % 64 != 0 || batch > 65536)
        return fail(BM_ERR_INVALID_ARG, "training batch must be a multiple of 64 and <= 65536");
    const MlpLayout L = mlp_layout(n_members, batch, true);
    rc = check_ws(L, d_ws, ws_bytes);
    if (rc) return rc;
    int dev;
    rc = check_device(&dev);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    char *ws = (char *)d_ws;
    TrainArgs a{};
    a.x = d_x;
    a.t = d_t;
    a.idx = d_idx;
    a.wbf = (const bf16_t *)d_wbf;
    a.params = d_params;
    a.B = (int)batch;
    a.a1T = (bf16_t *)(ws + L.a1);
    a.a2T = (bf16_t *)(ws + L.a2);
    a.dz1T = (bf16_t *)(ws + L.dz1);
    a.dz2T = (bf16_t *)(ws + L.dz2);
    a.dz3T = (bf16_t *)(ws + L.dz3);
    a.u = (float *)(ws + L.u);
    a.hpart = (float *)(ws + L.hpart);
    a.members = (int)n_members;
    a.groups = train_groups(n_members, batch);
    a.grad = d_grad;
    a.loss = d_loss;
    hipLaunchKernelGGL(k_train_rows, dim3((uint32_t)a.groups, n_members), dim3(TBT), 0, s, a);
    auto wgrad = [&](auto kernel, int wgm) {
        hipLaunchKernelGGL(kernel, dim3(wg_blocks(wgm) * n_members), dim3(TBT), 0, s, a);
    };
    switch (wgrad_split((int)batch)) {
    case 1: wgrad(&k_train_wgrad<1, 32>, 32); break;
    case 2:
        if (n_members >= WGRAD_TALL) wgrad(&k_train_wgrad<2, 64>, 64);
        else wgrad(&k_train_wgrad<2, 32>, 32);
        break;
    case 4: wgrad(&k_train_wgrad<4, 32>, 32); break;
    default: wgrad(&k_train_wgrad<8, 32>, 32); break;
    }
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? ok() : hip_fail(e, "bm_mlp_backward");
}

extern "C" int bm_mlp_adam_step(uint32_t n_members, float *d_params, const float *d_grad, float *d_m, float *d_v,
                           uint16_t *d_wbf, uint32_t step, float lr, float beta1, float beta2, float eps,
                           void *stream)
{
    int rc = check_members(n_members);
    if (rc) return rc;
    if (!d_params || !d_grad || !d_m || !d_v || !d_wbf) return fail(BM_ERR_INVALID_ARG, "NULL pointer");
    if (step < 1) return fail(BM_ERR_INVALID_ARG, "step counts from 1");
    if (!(lr > 0) || !(beta1 >= 0 && beta1 < 1) || !(beta2 >= 0 && beta2 < 1) || !(eps > 0))
        return fail(BM_ERR_INVALID_ARG, "need lr > 0, 0 <= beta < 1, eps > 0");
    int dev;
    rc = check_device(&dev);
    if (rc) return rc;
    const uint64_t total = (uint64_t)n_members * NPARAM;
    const float c1 = (float)(1.0 / (1.0 - std::pow((double)beta1, (double)step)));
    const float c2 = (float)(1.0 / (1.0 - std::pow((double)beta2, (double)step)));
    hipLaunchKernelGGL(k_adam, dim3((uint32_t)((total + 255) / 256)), dim3(256), 0, (hipStream_t)stream, d_params,
                       d_grad, d_m, d_v, (bf16_t *)d_wbf, total, lr, beta1, beta2, eps, c1, c2);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? ok() : hip_fail(e, "bm_mlp_adam_step");
}

// Most work-groups of 256 rows whose counts every compacting group adds up for itself:
// the sums are nblk / 512 loads per thread and group, side by side, where the scan is one
// group's serial work and a launch, but their work grows with the square.  Sums against scan
// and compaction: 4.4 and 8.9 us at 1000 groups, 6.4 and 13.7 at 4000, 12.4 and 23.4 at 8192,
// 29 and 39 at 16384, 81 and 76 at 32768; 8192 keeps clear of where the lead turns.
static constexpr uint64_t COMPACT_SUMS = 8192;

// The kernels of a query: fused inference of every member into y, then mean, std,
// routing flags and per-256-row counts (blk), and the ordered compaction of the routed
// rows.  Every element of y and blk a call reads is first
// written by that call, so neither buffer needs clearing.
static hipError_t enqueue_query(uint32_t n_members, const float *d_params, const uint16_t *d_wbf, const float *d_x,
                                uint64_t batch, float threshold, float *d_mean, float *d_std,
                                uint32_t *d_fallback_idx, uint32_t *d_fallback_count, float *y, uint32_t *blk,
                                hipStream_t s)
{
    hipError_t e = launch_infer(n_members, d_x, batch, (const bf16_t *)d_wbf, d_params, y, s);
    if (e != hipSuccess) return e;
    const uint64_t nblk = (batch + 255) / 256;
    if (batch <= ROUTE_ROWS) {
        hipLaunchKernelGGL(k_route_small, dim3(1), dim3((uint32_t)(batch + 63) / 64 * 64), 0, s, (const float *)y,
                           (int)n_members, (uint32_t)batch, threshold, d_mean, d_std, d_fallback_idx, d_fallback_count);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_stats, dim3((uint32_t)nblk), dim3(256), 0, s, (const float *)y, (int)n_members, batch,
                       threshold, d_mean, d_std, blk);
    if (nblk <= COMPACT_SUMS) {
        hipLaunchKernelGGL(k_compact<false>, dim3((uint32_t)nblk), dim3(256), 0, s, (const float *)d_std, batch,
                           threshold, (const uint32_t *)blk, d_fallback_idx, d_fallback_count);
    } else {
        hipLaunchKernelGGL(k_scan_counts, dim3(1), dim3(256), 0, s, blk, nblk, d_fallback_count);
        hipLaunchKernelGGL(k_compact<true>, dim3((uint32_t)nblk), dim3(256), 0, s, (const float *)d_std, batch,
                           threshold, (const uint32_t *)blk, d_fallback_idx, d_fallback_count);
    }
    e = hipGetLastError();
    return e;
}

static int check_query(uint32_t n_members, const float *d_params, const uint16_t *d_wbf, const float *d_x,
                       uint64_t batch, float threshold, float *d_mean, float *d_std, uint32_t *d_fallback_idx,
                       uint32_t *d_fallback_count)
{
    int rc = check_members(n_members);
    if (rc) return rc;
    if (!d_params || !d_wbf || !d_x || !d_mean || !d_std || !d_fallback_idx || !d_fallback_count)
        return fail(BM_ERR_INVALID_ARG, "NULL pointer");
    if (batch < 1 || batch > 0xFFFFFFFFull) return fail(BM_ERR_INVALID_ARG, "batch must be in [1, 2^32 - 1]");
    if (!(threshold >= 0)) return fail(BM_ERR_INVALID_ARG, "threshold must be >= 0");
    return BM_OK;
}

extern "C" int bm_surrogate_query(uint32_t n_members, const float *d_params, const uint16_t *d_wbf,
                                  const float *d_x, uint64_t batch, float threshold, float *d_mean, float *d_std,
                                  uint32_t *d_fallback_idx, uint32_t *d_fallback_count, void *d_ws,
                                  size_t ws_bytes, void *stream)
{
    int rc = check_query(n_members, d_params, d_wbf, d_x, batch, threshold, d_mean, d_std, d_fallback_idx,
                         d_fallback_count);
    if (rc) return rc;
    const MlpLayout L = mlp_layout(n_members, batch, false);
    rc = check_ws(L, d_ws, ws_bytes);
    if (rc) return rc;
    int dev;
    rc = check_device(&dev);
    if (rc) return rc;
    char *ws = (char *)d_ws;
    const hipError_t e = enqueue_query(n_members, d_params, d_wbf, d_x, batch, threshold, d_mean, d_std,
                                       d_fallback_idx, d_fallback_count, (float *)(ws + L.y),
                                       (uint32_t *)(ws + L.blk), (hipStream_t)stream);
    return e == hipSuccess ? ok() : hip_fail(e, "bm_surrogate_query");
}


// ---------------------------------------------------------------------------
// Ensemble query without a caller workspace and without any allocation: the
// members' predictions and the per-256-row counts live in `scratch`, a file-scope
// device array (one copy per GPU, held until the process ends).  In host code the
// array's name stands for a host-side shadow, so its device address is looked up
// once per device with hipGetSymbolAddress and only that address is ever passed to
// a kernel.  Every element a query reads is first written by the same query, so
// the array needs no clearing between calls.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[BM_QUERY_SCRATCH_BYTES];

namespace {
constexpr int SCRATCH_MAX_DEVICES = 64;
std::mutex scratch_mu;
void *scratch_dev[SCRATCH_MAX_DEVICES];     // device address of `scratch` on each device

// Device address of `scratch` on device `dev` (the current device), looked up on the
// first call for that device.
int scratch_address(int dev, char **out)
{
    if (dev < 0 || dev >= SCRATCH_MAX_DEVICES)
        return fail(BM_ERR_DEVICE, "device index %d beyond the %d the scratch table holds", dev,
                    SCRATCH_MAX_DEVICES);
    std::lock_guard<std::mutex> lock(scratch_mu);
    if (!scratch_dev[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return hip_fail(e, "hipGetSymbolAddress(scratch)");
        if (!p) return fail(BM_ERR_DEVICE, "hipGetSymbolAddress(scratch) returned NULL");
        scratch_dev[dev] = p;
    }
    *out = (char *)scratch_dev[dev];
    return BM_OK;
}
} // namespace

extern "C" int bm_surrogate_query_noalloc(uint32_t n_members, const float *d_params, const uint16_t *d_wbf,
                                          const float *d_x, uint64_t batch, float threshold, float *d_mean,
                                          float *d_std, uint32_t *d_fallback_idx, uint32_t *d_fallback_count,
                                          void *stream)
{
    int rc = check_query(n_members, d_params, d_wbf, d_x, batch, threshold, d_mean, d_std, d_fallback_idx,
                         d_fallback_count);
    if (rc) return rc;
    const MlpLayout L = mlp_layout(n_members, batch, false);
    if (L.total > BM_QUERY_SCRATCH_BYTES)
        return fail(BM_ERR_WORKSPACE,
                    "query of %u members x %llu rows needs %zu B of scratch; the built-in scratch holds %zu B "
                    "(use bm_surrogate_query with a workspace)",
                    n_members, (unsigned long long)batch, L.total, (size_t)BM_QUERY_SCRATCH_BYTES);
    int dev;
    rc = check_device(&dev);
    if (rc) return rc;
    char *ws = nullptr;
    rc = scratch_address(dev, &ws);
    if (rc) return rc;
    const hipError_t e = enqueue_query(n_members, d_params, d_wbf, d_x, batch, threshold, d_mean, d_std,
                                       d_fallback_idx, d_fallback_count, (float *)(ws + L.y),
                                       (uint32_t *)(ws + L.blk), (hipStream_t)stream);
    return e == hipSuccess ? ok() : hip_fail(e, "bm_surrogate_query_noalloc");
}
