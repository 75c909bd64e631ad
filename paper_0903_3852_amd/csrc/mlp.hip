// mlp.hip -- ensemble MLP surrogate of the mean velocity <v> of the
// Josephson junction: training (forward, back-propagation, MSE, Adam) and
// inference with hand-written FP32 kernels, and the scan that falls back to
// the integrator where the ensemble disagrees.
//
// Training works on minibatches of B samples for all members at once, three
// launches a step, all products on the FP32 matrix cores
// (v_mfma_f32_16x16x4_f32): the rows of the batch forward and back through
// every layer, the weight gradients, the update.  A whole epoch of steps is
// recorded once as a HIP graph; the Adam step count is a device counter, so
// the same graph replays every epoch.
//
// Inference is one fused kernel for all members, the hidden weights packed
// once per call into its operand layout.  Wide networks (mlp_split_infer_kernel):
// the FP32 products from BF16 ones of operands in three exact parts,
// activations in registers from layer to layer, weights streamed through LDS.  Narrow ones
// and those with one hidden layer (mlp_infer_mfma_kernel): a workgroup takes
// 64 queries whose activations stay in LDS in the operand layout of the next
// layer, each of its 4 waves computes 16 queries x all outputs of a layer on
// v_mfma_f32_16x16x4_f32 with the weights streamed from L2.  In both, bias
// and GELU write the next operand, and the output layer, the members' mean
// and their sample standard deviation follow.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <new>
#include <numeric>
#include <random>

#include "device_common.h"
#include "sde_internal.h"

struct sde_surrogate {
    sde_ctx* ctx = nullptr;
    std::vector<uint32_t> widths;
    std::vector<uint64_t> w_off, b_off;  // offsets of W_l, b_l in a member's packed parameters
    uint32_t members = 0;
    uint64_t P = 0;                      // parameters per member
    float* params = nullptr;             // device [members][P]
    float* grads = nullptr;              // device [members][P]
    float* adam_m = nullptr;             // device [members][P]
    float* adam_v = nullptr;
    uint64_t* adam_t = nullptr;          // device [members] Adam step counts
    sde_surrogate_scaling sc{};
    // training workspace
    float* work = nullptr;
    size_t work_bytes = 0;
    uint32_t* perm = nullptr;            // device [members][n] sample order of the epoch
    size_t perm_cap = 0;
    // inference: hidden-layer weights in the FP32 MFMA operand layout, and the
    // members' outputs of a call that gives each a workgroup
    float* packed = nullptr;
    size_t packed_bytes = 0;
    hipEvent_t raw_done = nullptr;       // the last such call has read them,
    int raw_last = 0;                    // 0 none yet, 1 on the null stream (not recorded), 2 on another
};

namespace sde {

constexpr uint32_t kTagMlpInit = 5;
constexpr int kMaxLayers = 8;

__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad(float z)
{
    return 0.5f * (1.f + erff(z * 0.70710678118654752f)) + z * 0.39894228040143268f * expf(-0.5f * z * z);
}

// ------------------------------------------------------------ parameters --
struct InitArgs {
    float* params;
    uint64_t P;
    uint32_t members;
    uint32_t n_layers;
    uint64_t layer_end[kMaxLayers];  // packed offset where layer l's (W, b) ends
    float bound[kMaxLayers];         // 1 / sqrt(fan_in)
    uint32_t key0, key1;
};

__global__ void mlp_init_kernel(InitArgs A)
{
    const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= A.P * A.members) return;
    const uint32_t m = (uint32_t)(g / A.P);
    const uint64_t k = g % A.P;
    uint32_t l = 0;
    while (l + 1 < A.n_layers && k >= A.layer_end[l]) ++l;
    const U4 x = philox4x32_10(U4{(uint32_t)(k >> 2), m, 0u, kTagMlpInit}, A.key0, A.key1);
    const uint32_t w = (k & 3) == 0 ? x.x : (k & 3) == 1 ? x.y : (k & 3) == 2 ? x.z : x.w;
    const float u = (float)(w >> 8) * 0x1p-24f;
    A.params[g] = A.bound[l] * (2.f * u - 1.f);
}

// ------------------------------------------------------------- features --
struct NormArgs {
    const float* X;          // [n][w0] raw features
    const float* y;          // [n] targets or null
    float* Xn;               // [n][w0]
    float* yn;               // [n] or null
    uint64_t n;
    uint32_t w0;
    sde_surrogate_scaling sc;
};

__global__ void mlp_normalize_kernel(NormArgs A)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= A.n) return;
    for (uint32_t j = 0; j < A.w0; ++j)
        A.Xn[i * A.w0 + j] = (A.X[i * A.w0 + j] - A.sc.in_center[j]) / A.sc.in_scale[j];
    if (A.y) {
        float t = A.y[i];
        if (A.sc.target_over_omega) t /= A.X[i * A.w0 + 1];
        A.yn[i] = (t - A.sc.out_mean) / A.sc.out_std;
    }
}

// ------------------------------------------------------------- training ---
// A step is three launches.
//  1. mlp_rows_kernel: forward and the chain of input gradients.  Both are
//     local to a sample, so a workgroup takes 16 or 32 of them through every
//     layer and back, activations and gradients in LDS in the operand layout
//     of the next product, the weights streamed from L2 in the layout the
//     matrix cores read (kept up to date by launch 3).  What the weight
//     gradients need (activations, dZ) goes to memory once.
//  2. mlp_grads_kernel: every layer's weight gradient dW = dZ^T A in k slices,
//     the bias gradients in slices of rows, the loss.
//  3. mlp_update_kernel: the slices added in order, Adam, the packed weights.
// The sums keep a fixed order that does not depend on this split (every
// product adds its k in ascending order on v_mfma_f32_16x16x4_f32, which
// rounds each multiply-add of its four k in turn as an FMA chain does), so a
// seed gives the same weights bit for bit as one launch per product did.
// What bounded that: 31 launches a step, and 64 x 64 tiles staged through LDS
// in 16-k slices with nothing in flight over a slice (15 TFLOP/s).  Five
// members of 5-256-256-256-1, 1024 samples: 413 us a step then, 100 now (rows
// 61, of which the products' MFMAs are 34; gradients 24; update 10).
typedef float f32x4_t __attribute__((ext_vector_type(4)));

// Operands of a 16 x 16 block (16 rows or output columns by 16 k) of the FP32
// products are one 1 KB run: lane l = i % 16 + 16 * (k % 4) holds the float4 of
// k = k % 4 + {0, 4, 8, 12}, the operands of four consecutive MFMAs.
__device__ __forceinline__ uint32_t frag32_index(uint32_t i, uint32_t k, uint32_t kb16)
{
    return (((i >> 4) * kb16 + (k >> 4)) * 64 + ((i & 15u) + 16u * (k & 3u))) * 4 + ((k & 15u) >> 2);
}

constexpr int kGK = 16;   // granularity of the k slices
constexpr int kGT = 64;   // tile of the weight gradients
constexpr uint32_t kColSlice = 64;  // rows per bias-gradient slice

// Shapes and buffers of one step; layer l < hidden is hidden, layer `hidden`
// is the output.  Sample rows have a pitch of Hp = H rounded up to 16, the
// columns past H are zero.
struct TrainArgs {
    const float* Xn;          // [n][w0] normalized inputs
    const float* yn;          // [n] normalized targets
    const uint32_t* rows;     // sample order of each member, or null
    uint64_t rows_mstride;
    uint32_t rows_offset;     // first row of this minibatch
    uint32_t B, w0, H, Hp, hidden, members;
    float* params;            // [members][P]
    uint64_t P;
    uint64_t w_off[kMaxLayers], b_off[kMaxLayers];
    float* wf;                // [members][hidden - 1][Hp * Hp] operands of the forward products
    float* wb;                // the same of the input gradients
    float* act;               // [hidden][members][B][Hp] activations
    float* slope;             // GELU' at the pre-activations
    float* dz;                // gradients of the pre-activations
    float* y;                 // [members][B] outputs
    float* dy;                // their gradients
    float* part_h;            // [hidden - 1][members][ks_h][Hp * Hp] dW slices
    float* part_in;           // [members][ks_in][H * w0] of the first layer
    float* part_out;          // [members][ks_out][H] of the output layer
    float* part_b;            // [hidden][members][col_slices][Hp] dB slices
    float* part_bo;           // [members][col_slices] of the output bias
    uint32_t ks_h, ks_in, ks_out, col_slices;
    float* loss;              // [members][loss_stride]
    uint32_t loss_slot, loss_stride;
    // update
    float* grads;             // [members][P], or null (Adam steps do not keep them)
    float* m;
    float* v;                 // Adam state, null: gradients only
    uint64_t* t;              // [members] Adam step counts
    float* bc;                // [members][2] the step's bias corrections
    float lr, b1, b2, eps;

    __host__ __device__ uint64_t layer_stride() const { return (uint64_t)members * B * Hp; }
};

__device__ __forceinline__ uint64_t train_row(const TrainArgs& A, uint32_t mem, uint32_t b)
{
    return A.rows ? A.rows[mem * A.rows_mstride + A.rows_offset + b] : b;
}

constexpr int kRowsThreads = 512;
constexpr int kRowsWaves = kRowsThreads / 64;  // wave w has columns 32 w .. 32 w + 31

// The products of a workgroup's rows with packed weights: start() sends for
// the first two k blocks of a wave's 32 columns, run() multiplies (in: LDS,
// operand layout), always two blocks of weights ahead.
template <int RB>
struct RowsProduct {
    uint32_t KB, wave, lane;
    const float* wp[2];
    f32x4_t w0[2], w1[2];

    __device__ __forceinline__ void load(uint32_t kb, f32x4_t (&w)[2])
    {
        const uint32_t k = min(kb, KB - 1);
#pragma unroll
        for (int n = 0; n < 2; ++n) w[n] = *reinterpret_cast<const f32x4_t*>(wp[n] + k * 256);
    }
    __device__ __forceinline__ void start(const float* W)
    {
#pragma unroll
        for (int n = 0; n < 2; ++n)  // a wave past the last column block repeats it (and drops the result)
            wp[n] = W + (min(2 * wave + n, KB - 1) * KB * 64 + lane) * 4;
        load(0, w0);
        load(1, w1);
    }
    __device__ __forceinline__ void block(const float* in, uint32_t kb, const f32x4_t (&w)[2], f32x4_t (&acc)[RB][2])
    {
        f32x4_t a[RB];
#pragma unroll
        for (int m = 0; m < RB; ++m) a[m] = *reinterpret_cast<const f32x4_t*>(in + ((m * KB + kb) * 64 + lane) * 4);
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int m = 0; m < RB; ++m)
#pragma unroll
                for (int n = 0; n < 2; ++n)
                    acc[m][n] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[m][j], w[n][j], acc[m][n], 0, 0, 0);
    }
    __device__ __forceinline__ void run(const float* in, f32x4_t (&acc)[RB][2])
    {
#pragma unroll
        for (int m = 0; m < RB; ++m)
#pragma unroll
            for (int n = 0; n < 2; ++n) acc[m][n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        for (uint32_t kb = 0; kb + 1 < KB; kb += 2) {  // no branch: loads in flight are counted, not drained
            const f32x4_t c[2] = {w0[0], w0[1]};
            load(kb + 2, w0);
            __builtin_amdgcn_sched_barrier(0);  // the loads go out first, two blocks ahead of their use
            block(in, kb, c, acc);
            __builtin_amdgcn_sched_barrier(0);
            const f32x4_t d[2] = {w1[0], w1[1]};
            load(kb + 3, w1);
            __builtin_amdgcn_sched_barrier(0);
            block(in, kb + 1, d, acc);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (KB & 1u) block(in, KB - 1, w0, acc);
    }
};

// Forward and input gradients of samples blockIdx.x * 16 RB .. of member
// blockIdx.y.
template <int RB>
__global__ __launch_bounds__(kRowsThreads) void mlp_rows_kernel(TrainArgs A)
{
    constexpr uint32_t kRows = 16 * RB;
    __shared__ __attribute__((aligned(16))) float buf[2][kRows * 256];
    __shared__ float xs[kRows][8], ts[kRows], dys[kRows];
    const uint32_t mem = blockIdx.y, r0 = blockIdx.x * kRows;
    const uint32_t wave = uniform_u32(threadIdx.x >> 6), lane = threadIdx.x & 63u;
    const uint32_t H = A.H, Hp = A.Hp, KB = Hp / 16, hidden = A.hidden, B = A.B;
    const float* prm = A.params + mem * A.P;
    const uint64_t ls = A.layer_stride();
    for (uint32_t e = threadIdx.x; e < kRows * 8; e += kRowsThreads) {
        const uint32_t row = e / 8, j = e % 8;
        const bool ok = r0 + row < B;
        const uint64_t sample = ok ? train_row(A, mem, r0 + row) : 0u;
        xs[row][j] = ok && j < A.w0 ? A.Xn[sample * A.w0 + j] : 0.f;
        if (j == 7) ts[row] = ok ? A.yn[sample] : 0.f;
    }
    // Lane l of a 16 x 16 block holds rows 4 (l / 16) + q, column l % 16: this
    // lane's first element in a [row][Hp] array and in the operand layout.
    const uint32_t lrow = 4 * (lane >> 4), lcol = wave * 32 + (lane & 15u);
    const uint64_t at = ((uint64_t)mem * B + r0 + lrow) * Hp + lcol;
    const uint32_t frag = frag32_index(lrow, lcol, KB);
    auto each = [&](auto f) {
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            const uint32_t col = lcol + 16 * n;
            if (wave * 32 + 16 * n >= Hp) continue;
#pragma unroll
            for (int m = 0; m < RB; ++m)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    f(m, n, q, (uint32_t)(m * 16 + q) + lrow, col, (m * 16 + q) * Hp + 16 * n,
                      frag + (m * KB + n) * 256 + 4 * q);
        }
    };
    const bool whole = r0 + kRows <= B;  // every row is a sample
    RowsProduct<RB> prod{KB, wave, lane};
    const uint64_t hh = (uint64_t)Hp * Hp;
    const float* wf = A.wf + (uint64_t)mem * (hidden - 1) * hh;  // forward operands of layer 1
    const float* wb = A.wb + (uint64_t)mem * (hidden - 1) * hh;
    if (hidden > 1) prod.start(wf);
    __syncthreads();
    // pre-activation z of layer l -> its activation and slope
    auto activate = [&](float* act, float* slope, uint32_t row, uint32_t col, uint32_t off, float z, float* out) {
        float a = 0.f, d = 0.f;
        if (col < H) {
            a = gelu(z);
            d = gelu_grad(z);
        }
        *out = a;
        if (whole || r0 + row < B) {
            act[off] = a;
            slope[off] = d;
        }
    };
    uint32_t cur = 0;
    f32x4_t acc[RB][2];
    if (hidden) {
        const float* W = prm + A.w_off[0];
        const float* b = prm + A.b_off[0];
        float wx[2][8], bias[2];
#pragma unroll
        for (int n = 0; n < 2; ++n) {
            const uint32_t col = min(lcol + 16 * n, H - 1);
            bias[n] = b[col];
#pragma unroll
            for (int j = 0; j < 8; ++j) wx[n][j] = (uint32_t)j < A.w0 ? W[col * A.w0 + j] : 0.f;
        }
        each([&](int, int n, int, uint32_t row, uint32_t col, uint32_t off, uint32_t fi) {
            float z = 0.f;
#pragma unroll
            for (int j = 0; j < 8; ++j) z = fmaf(xs[row][j], wx[n][j], z);  // zeros past the inputs
            activate(A.act + at, A.slope + at, row, col, off, z + bias[n], buf[0] + fi);
        });
    }
    __syncthreads();
    for (uint32_t l = 1; l < hidden; ++l) {
        const float* b = prm + A.b_off[l];
        const float bias[2] = {b[min(lcol, H - 1)], b[min(lcol + 16, H - 1)]};
        prod.run(buf[cur], acc);
        prod.start(l + 1 < hidden ? wf + l * hh : wb + (hidden - 2) * hh);  // the next product's first weights
        each([&](int m, int n, int q, uint32_t row, uint32_t col, uint32_t off, uint32_t fi) {
            activate(A.act + l * ls + at, A.slope + l * ls + at, row, col, off, acc[m][n][q] + bias[n],
                     buf[cur ^ 1] + fi);
        });
        cur ^= 1;
        __syncthreads();
    }
    // output layer, the loss' gradient
    if (threadIdx.x < kRows) {
        const uint32_t row = threadIdx.x;
        const float* W = prm + A.w_off[hidden];
        float z = 0.f;
        if (hidden) {
            // k in ascending order; a float4 of the operand layout holds every fourth
            const float* a = buf[cur] + frag32_index(row, 0, KB);
            for (uint32_t kb = 0; kb < KB; ++kb) {
                f32x4_t x[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) x[r] = *reinterpret_cast<const f32x4_t*>(a + kb * 256 + r * 64);
#pragma unroll
                for (int k = 0; k < 16; ++k) z = fmaf(x[k & 3][k >> 2], W[min(kb * 16 + k, H - 1)], z);  // zeros past H
            }
        } else {
            for (uint32_t j = 0; j < A.w0; ++j) z = fmaf(xs[row][j], W[j], z);
        }
        z += prm[A.b_off[hidden]];
        float g = 0.f;
        if (r0 + row < B) {
            g = 2.f * (z - ts[row]) / (float)B;
            A.y[(uint64_t)mem * B + r0 + row] = z;
            A.dy[(uint64_t)mem * B + r0 + row] = g;
        }
        dys[row] = g;
    }
    if (!hidden) return;
    // dZ of layer l from the gradient of its activation; slopes were sent for
    // before the product
    float slope[RB][2][4];
    auto load_slopes = [&](uint32_t l) {
        const float* p = A.slope + l * ls + at;
        each([&](int m, int n, int q, uint32_t row, uint32_t, uint32_t off, uint32_t) {
            slope[m][n][q] = whole || r0 + row < B ? p[off] : 0.f;
        });
    };
    auto store_dz = [&](float* dz, uint32_t row, uint32_t off, float g, float* out) {
        *out = g;
        if (whole || r0 + row < B) dz[off] = g;
    };
    load_slopes(hidden - 1);
    {
        const float* W = prm + A.w_off[hidden];
        const float w[2] = {W[min(lcol, H - 1)], W[min(lcol + 16, H - 1)]};
        __syncthreads();
        each([&](int m, int n, int q, uint32_t row, uint32_t, uint32_t off, uint32_t fi) {
            store_dz(A.dz + (hidden - 1) * ls + at, row, off, dys[row] * w[n] * slope[m][n][q], buf[cur ^ 1] + fi);
        });
        cur ^= 1;
        __syncthreads();
    }
    for (uint32_t l = hidden - 1; l > 0; --l) {
        load_slopes(l - 1);
        prod.run(buf[cur], acc);
        if (l > 1) prod.start(wb + (l - 2) * hh);
        each([&](int m, int n, int q, uint32_t row, uint32_t, uint32_t off, uint32_t fi) {
            store_dz(A.dz + (l - 1) * ls + at, row, off, acc[m][n][q] * slope[m][n][q], buf[cur ^ 1] + fi);
        });
        cur ^= 1;
        __syncthreads();
    }
}

// The k range of slice ks of kslices, in whole k steps.
__device__ __forceinline__ void k_range(uint32_t K, uint32_t kslices, uint32_t ks, uint32_t& k_begin, uint32_t& k_end)
{
    const uint32_t per = ((K + kslices - 1) / kslices + kGK - 1) / kGK * kGK;
    k_begin = min(K, ks * per);
    k_end = min(K, k_begin + per);
}

// The work of mlp_grads_kernel's workgroups, in this order: 64-row bands of
// the hidden layers' dW (a wave per 64 columns), the first layer's dW, the
// output layer's dW, bias slices of 64 rows per hidden layer, bias slices of
// the output with them, the loss.
struct GradsGrid {
    uint32_t hidden, in, out, bias, loss;
    __host__ __device__ explicit GradsGrid(const TrainArgs& A)
    {
        hidden = A.hidden > 1 ? (A.hidden - 1) * A.members * A.ks_h * ((A.Hp + kGT - 1) / kGT) : 0u;
        in = A.hidden ? A.members * A.ks_in : 0u;
        out = A.members * A.ks_out;
        bias = A.members * A.col_slices * (A.hidden + 1);
        loss = A.members;
    }
    __host__ __device__ uint32_t total() const { return hidden + in + out + bias + loss; }
};

// One wave's 64 x 64 tile of dW = dZ^T A over k (samples) in [kb, ke).  Both
// operands lie with k in rows, so a lane's float4 of 4 neighbouring columns
// (16 lanes and 4 rows: 4 runs of 256 B) is its operand of 4 MFMAs: operand j
// of row or column i is row or column 4 i + j of the tile.  Four k steps of 4
// are in flight ahead of the 64 MFMAs of the current ones.
__device__ __forceinline__ void grads_tile(const float* dz, const float* act, uint32_t Hp, uint32_t m0, uint32_t n0,
                                           uint32_t kb, uint32_t ke, uint32_t lane, float* part)
{
    const uint32_t i = 4 * (lane & 15u), kq = lane >> 4;
    const bool n_ok = n0 + i < Hp;
    // a lane past the last row or column takes the first one's values; what
    // they give is not stored
    const float* pa = dz + (uint64_t)kq * Hp + m0 + (m0 + i < Hp ? i : 0u);
    const float* pb = act + (uint64_t)kq * Hp + n0 + (n_ok ? i : 0u);
    f32x4_t acc[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto products = [&](const f32x4_t& x, const f32x4_t& y) {
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 4; ++b) acc[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[a], y[b], acc[a][b], 0, 0, 0);
    };
    // whole blocks of 16 k; the loads have no condition on them (the last
    // block sends for itself again), so none is waited for early
    const uint32_t full = kb + (ke - kb) / 16 * 16;
    f32x4_t fa[4], fb[4];
    auto load = [&](uint32_t k0) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            fa[u] = *reinterpret_cast<const f32x4_t*>(pa + (uint64_t)(k0 + 4 * u) * Hp);
            fb[u] = *reinterpret_cast<const f32x4_t*>(pb + (uint64_t)(k0 + 4 * u) * Hp);
        }
    };
    if (full > kb) {
        load(kb);
        for (uint32_t k0 = kb; k0 < full; k0 += 16) {
            f32x4_t ca[4], cb[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                ca[u] = fa[u];
                cb[u] = fb[u];
            }
            load(min(k0 + 16, full - 16));
            __builtin_amdgcn_sched_barrier(0);  // the loads go out before the products
#pragma unroll
            for (int u = 0; u < 4; ++u) products(ca[u], cb[u]);
        }
    }
    for (uint32_t k0 = full; k0 < ke; k0 += 4) {  // the batch's last k, zeros past its end
        f32x4_t x = {0.f, 0.f, 0.f, 0.f}, y = x;
        if (k0 + kq < ke) {
            x = *reinterpret_cast<const f32x4_t*>(pa + (uint64_t)k0 * Hp);
            y = *reinterpret_cast<const f32x4_t*>(pb + (uint64_t)k0 * Hp);
        }
        products(x, y);
    }
    if (!n_ok) return;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t m = m0 + 4 * (4 * kq + q) + a;
            if (m >= Hp) continue;
            *reinterpret_cast<f32x4_t*>(part + (uint64_t)m * Hp + n0 + i) =
                f32x4_t{acc[a][0][q], acc[a][1][q], acc[a][2][q], acc[a][3][q]};
        }
}

__global__ __launch_bounds__(256) void mlp_grads_kernel(TrainArgs A)
{
    const GradsGrid G(A);
    const uint32_t tid = threadIdx.x, H = A.H, Hp = A.Hp, B = A.B;
    const uint64_t ls = A.layer_stride();
    uint32_t w = blockIdx.x, kb, ke;
    if (w < G.hidden) {
        const uint32_t bands = (Hp + kGT - 1) / kGT, band = w % bands, ks = w / bands % A.ks_h;
        const uint32_t mem = w / bands / A.ks_h % A.members, l = 1 + w / bands / A.ks_h / A.members;
        const uint32_t n0 = (tid >> 6) * kGT;
        if (n0 >= Hp) return;
        k_range(B, A.ks_h, ks, kb, ke);
        const uint64_t o = (uint64_t)mem * B * Hp;
        grads_tile(A.dz + l * ls + o, A.act + (l - 1) * ls + o, Hp, band * kGT, n0, kb, ke, tid & 63u,
                   A.part_h + (((uint64_t)(l - 1) * A.members + mem) * A.ks_h + ks) * Hp * Hp);
        return;
    }
    w -= G.hidden;
    if (w < G.in) {  // dW of the first layer: thread per output, the samples' inputs through LDS
        const uint32_t ks = w % A.ks_in, mem = w / A.ks_in;
        __shared__ __attribute__((aligned(16))) float xs[64][8];
        k_range(B, A.ks_in, ks, kb, ke);
        float acc[8] = {};
        const float* dz = A.dz + (uint64_t)mem * B * Hp + min(tid, H - 1);
        for (uint32_t k0 = kb; k0 < ke; k0 += 64) {
            __syncthreads();
            for (uint32_t e = tid; e < 64 * 8; e += 256) {
                const uint32_t k = k0 + e / 8, j = e % 8;
                xs[e / 8][j] = k < ke && j < A.w0 ? A.Xn[train_row(A, mem, k) * A.w0 + j] : 0.f;
            }
            __syncthreads();
            const uint32_t n = min(64u, ke - k0);
#pragma unroll 16
            for (uint32_t k = 0; k < n; ++k) {
                const float d = dz[(uint64_t)(k0 + k) * Hp];
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] = fmaf(d, xs[k][j], acc[j]);
            }
        }
        if (tid >= H) return;
        float* out = A.part_in + ((uint64_t)mem * A.ks_in + ks) * H * A.w0 + (uint64_t)tid * A.w0;
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if ((uint32_t)j < A.w0) out[j] = acc[j];
        return;
    }
    w -= G.in;
    if (w < G.out) {  // dW of the output layer: thread per input
        const uint32_t ks = w % A.ks_out, mem = w / A.ks_out, in = A.hidden ? H : A.w0;
        if (tid >= in) return;
        k_range(B, A.ks_out, ks, kb, ke);
        const float* dy = A.dy + (uint64_t)mem * B;
        const float* act = A.act + (A.hidden ? (A.hidden - 1) * ls : 0u) + (uint64_t)mem * B * Hp + tid;
        float acc = 0.f;
#pragma unroll 16
        for (uint32_t k = kb; k < ke; ++k)
            acc = fmaf(dy[k], A.hidden ? act[(uint64_t)k * Hp] : A.Xn[train_row(A, mem, k) * A.w0 + tid], acc);
        A.part_out[((uint64_t)mem * A.ks_out + ks) * in + tid] = acc;
        return;
    }
    w -= G.out;
    if (w < G.bias) {  // db[n] = sum_b dZ[b][n], one slice of rows
        const uint32_t sl = w % A.col_slices, mem = w / A.col_slices % A.members, l = w / A.col_slices / A.members;
        const uint32_t b0 = sl * kColSlice, b1 = min(B, b0 + kColSlice);
        const bool last = l == A.hidden;
        if (tid >= (last ? 1u : H)) return;
        const float* p = last ? A.dy + (uint64_t)mem * B : A.dz + l * ls + (uint64_t)mem * B * Hp + tid;
        const uint64_t pitch = last ? 1u : Hp;
        float s = 0.f;
#pragma unroll 16
        for (uint32_t b = b0; b < b1; ++b) s += p[b * pitch];
        if (last)
            A.part_bo[(uint64_t)mem * A.col_slices + sl] = s;
        else
            A.part_b[(((uint64_t)l * A.members + mem) * A.col_slices + sl) * Hp + tid] = s;
        return;
    }
    // loss = mean (y - t)^2 (FP64 block sum), and the step count
    const uint32_t mem = w - G.bias;
    __shared__ double lds[4];
    double s = 0.0;
    for (uint32_t b = tid; b < B; b += 256) {
        const float r = A.y[(uint64_t)mem * B + b] - A.yn[train_row(A, mem, b)];
        s += (double)r * (double)r;
    }
    s = wave_sum(s);
    if ((tid & 63u) == 0) lds[tid >> 6] = s;
    __syncthreads();
    if (tid == 0) {
        A.loss[(uint64_t)mem * A.loss_stride + A.loss_slot] = (float)((lds[0] + lds[1] + lds[2] + lds[3]) / B);
        if (A.t) {
            const uint64_t t = A.t[mem] + 1;
            A.t[mem] = t;
            A.bc[2 * mem] = (float)(1.0 - pow((double)A.b1, (double)t));
            A.bc[2 * mem + 1] = (float)(1.0 - pow((double)A.b2, (double)t));
        }
    }
}

// A hidden weight W_l[o][k] (l >= 1) into both operand layouts.
__device__ __forceinline__ void pack_weight(const TrainArgs& A, uint32_t mem, uint32_t l, uint32_t o, uint32_t k, float x)
{
    const uint64_t base = ((uint64_t)mem * (A.hidden - 1) + l - 1) * A.Hp * A.Hp;
    A.wf[base + frag32_index(o, k, A.Hp / 16)] = x;
    A.wb[base + frag32_index(k, o, A.Hp / 16)] = x;
}

// The update's workgroups: per layer the blocks of 256 weights, then one
// block for the biases (at most 256).
__host__ __device__ inline uint32_t layer_in(const TrainArgs& A, uint32_t l) { return l ? A.H : A.w0; }
__host__ __device__ inline uint32_t layer_out(const TrainArgs& A, uint32_t l) { return l == A.hidden ? 1u : A.H; }
__host__ __device__ inline uint32_t update_blocks(const TrainArgs& A, uint32_t l)
{
    return (layer_in(A, l) * layer_out(A, l) + 255) / 256 + 1;
}

// Gradients from their slices, one Adam step (bias-corrected), the packed
// weights.  Thread per parameter of member blockIdx.y; the step count and the
// corrections that go with it were written by the launch before.
__global__ __launch_bounds__(256) void mlp_update_kernel(TrainArgs A)
{
    const uint32_t mem = blockIdx.y;
    uint32_t l = 0, blk = blockIdx.x;
    for (; blk >= update_blocks(A, l); ++l) blk -= update_blocks(A, l);
    const bool bias = blk + 1 == update_blocks(A, l);
    const uint32_t e = (bias ? 0u : blk * 256) + threadIdx.x;
    if (e >= (bias ? layer_out(A, l) : layer_in(A, l) * layer_out(A, l))) return;
    // slices: part[k * pitch], k < n
    const float* part;
    uint64_t pitch;
    uint32_t n, o = 0, k = 0;
    if (bias) {
        n = A.col_slices;
        part = l == A.hidden ? A.part_bo + (uint64_t)mem * n : A.part_b + ((uint64_t)l * A.members + mem) * n * A.Hp + e;
        pitch = l == A.hidden ? 1u : A.Hp;
    } else if (l == A.hidden) {
        n = A.ks_out;
        pitch = layer_in(A, l);
        part = A.part_out + (uint64_t)mem * n * pitch + e;
    } else if (l == 0) {
        n = A.ks_in;
        pitch = (uint64_t)A.H * A.w0;
        part = A.part_in + (uint64_t)mem * n * pitch + e;
    } else {
        n = A.ks_h;
        pitch = (uint64_t)A.Hp * A.Hp;
        o = e / A.H;
        k = e % A.H;
        part = A.part_h + ((uint64_t)(l - 1) * A.members + mem) * n * pitch + (uint64_t)o * A.Hp + k;
    }
    float g = 0.f;
#pragma unroll 4
    for (uint32_t s = 0; s < n; ++s) g += part[s * pitch];
    const uint64_t j = mem * A.P + (bias ? A.b_off[l] : A.w_off[l]) + e;
    if (A.grads) A.grads[j] = g;
    if (!A.m) return;
    // the roundings spelled out, so that no compilation moves them
    const float m = fmaf(1.f - A.b1, g, A.b1 * A.m[j]);
    const float v = fmaf(g, (1.f - A.b2) * g, A.b2 * A.v[j]);
    A.m[j] = m;
    A.v[j] = v;
    const float p = A.params[j] - A.lr * (m / A.bc[2 * mem]) / (sqrtf(v / A.bc[2 * mem + 1]) + A.eps);
    A.params[j] = p;
    if (!bias && l > 0 && l < A.hidden) pack_weight(A, mem, l, o, k, p);
}

// Both operand layouts of every hidden weight, zero past H.
__global__ __launch_bounds__(256) void mlp_pack_train_kernel(TrainArgs A)
{
    const uint64_t per = (uint64_t)A.Hp * A.Hp;
    const uint64_t g = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (g >= per * (A.hidden - 1) * A.members) return;
    const uint32_t mem = (uint32_t)(g / (per * (A.hidden - 1))), l = 1 + (uint32_t)(g / per % (A.hidden - 1));
    const uint32_t o = (uint32_t)(g % per / A.Hp), k = (uint32_t)(g % A.Hp);
    pack_weight(A, mem, l, o, k,
                o < A.H && k < A.H ? A.params[mem * A.P + A.w_off[l] + (uint64_t)o * A.H + k] : 0.f);
}

// ------------------------------------------------------------ inference ---
// Fused ensemble forward for widths w0 -> H -> ... -> H -> 1 with H <= 256.
constexpr int kInfH = 256;

struct InferArgs {
    const float* X;          // [n][w0] raw features
    const float* params;     // [members][P]
    float* mean;             // [n]
    float* spread;           // [n]
    uint64_t n, P;
    uint32_t members, n_layers, w0, H;
    uint64_t w_off[kMaxLayers], b_off[kMaxLayers];
    sde_surrogate_scaling sc;
};

// Members' mean and sample standard deviation at `query`, in units of <v>.
template <typename Out>
__device__ __forceinline__ void store_prediction(const InferArgs& A, uint64_t query, Out out)
{
    const float omega = A.sc.target_over_omega ? A.X[query * A.w0 + 1] : 1.f;
    float v[8], s = 0.f;
#pragma unroll
    for (uint32_t m = 0; m < 8; ++m)
        if (m < A.members) {
            v[m] = (A.sc.out_mean + A.sc.out_std * out(m)) * omega;
            s += v[m];
        }
    const float mu = s / (float)A.members;
    float ss = 0.f;
#pragma unroll
    for (uint32_t m = 0; m < 8; ++m)
        if (m < A.members) ss += (v[m] - mu) * (v[m] - mu);
    A.mean[query] = mu;
    A.spread[query] = A.members > 1 ? sqrtf(ss / (float)(A.members - 1)) : 0.f;
}

// The same from the members' outputs of queries first .., raw[members][n - first].
__global__ __launch_bounds__(256) void mlp_combine_kernel(InferArgs A, uint64_t first, const float* raw)
{
    const uint64_t q = (uint64_t)blockIdx.x * 256 + threadIdx.x, n = A.n - first;
    if (q < n) store_prediction(A, first + q, [&](uint32_t m) { return raw[m * n + q]; });
}

// FP32 MFMA forward (v_mfma_f32_16x16x4_f32) in the operand layout of
// frag32_index.  The hidden weights are packed that way once per call
// (B(k, c) = W[c][k]); the activations stay in LDS in the same layout, as the
// A operand of the next layer.
struct PackArgs {
    const float* params;
    uint64_t P;
    uint32_t members, hidden, H, Hp;
    uint64_t w_off[kMaxLayers];  // of hidden layer 1 + l at index l
    float* packed;               // [members][hidden][Hp * Hp]
};

// packed[m][l] (Hp x Hp, zero padded) from the hidden weights W_{l+1} of member m
__global__ void mlp_pack_hidden_kernel(PackArgs A)
{
    const uint64_t per = (uint64_t)A.Hp * A.Hp;
    const uint64_t g = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (g >= (uint64_t)A.members * A.hidden * per) return;
    const uint32_t m = (uint32_t)(g / (A.hidden * per));
    const uint32_t l = (uint32_t)((g / per) % A.hidden);
    const uint32_t e = (uint32_t)(g % per), c = e / A.Hp, k = e % A.Hp;
    const float* W = A.params + (uint64_t)m * A.P + A.w_off[l];
    A.packed[((uint64_t)m * A.hidden + l) * per + frag32_index(c, k, A.Hp / 16)] =
        (c < A.H && k < A.H) ? W[(uint64_t)c * A.H + k] : 0.f;
}

// Networks of width 65 and more with two hidden layers or more go to
// mlp_split_infer_kernel, so a product here has 4 column blocks at the most.
constexpr uint32_t kSplitMinH = 65;
constexpr uint32_t kInfBlocks = (kSplitMinH - 1) / 16;
// Queries per workgroup: one 16-row block per wave.  LDS is sized by the
// width, so that several workgroups (20 KB each at 64) share a CU and one's
// GELU epilogue overlaps the other's products: 200000 queries of five
// 5-64-64-64-1 networks 801 us with room for 256 columns, 420 us so.
constexpr uint32_t kInfMRows = 64;

__global__ __launch_bounds__(256, 2) void mlp_infer_mfma_kernel(InferArgs A, const float* packed, uint32_t Hp,
                                                               float* raw)
{
    extern __shared__ float smem[];
    float* act = smem;                      // [kInfMRows x Hp] in the operand layout
    float* xn = act + kInfMRows * Hp;       // [kInfMRows][8] normalized features
    float* outs = xn + kInfMRows * 8;       // [kInfMRows][8] member outputs
    const uint64_t r0 = (uint64_t)blockIdx.x * kInfMRows;
    const uint32_t H = A.H, KB = Hp / 16, NB = KB;
    const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
    for (uint32_t e = threadIdx.x; e < kInfMRows * A.w0; e += 256) {
        const uint32_t row = e / A.w0, j = e % A.w0;
        const uint64_t gi = r0 + row;
        xn[row * 8 + j] = gi < A.n ? (A.X[gi * A.w0 + j] - A.sc.in_center[j]) / A.sc.in_scale[j] : 0.f;
    }
    __syncthreads();
    const uint32_t hidden = A.n_layers - 2;
    const uint32_t mem0 = raw ? blockIdx.y : 0, mem1 = raw ? mem0 + 1 : A.members;
    for (uint32_t mem = mem0; mem < mem1; ++mem) {
        const float* prm = A.params + (uint64_t)mem * A.P;
        {   // layer 1 from the normalized features
            const float* W = prm + A.w_off[0];
            const float* b = prm + A.b_off[0];
            for (uint32_t e = threadIdx.x; e < kInfMRows * Hp; e += 256) {
                const uint32_t row = e / Hp, col = e % Hp;
                float z = 0.f;
                if (col < H) {
                    z = b[col];
                    for (uint32_t j = 0; j < A.w0; ++j) z = fmaf(W[col * A.w0 + j], xn[row * 8 + j], z);
                    z = gelu(z);
                }
                act[frag32_index(row, col, KB)] = z;
            }
            __syncthreads();
        }
        // hidden layers: wave w computes rows 16 w .. 16 w + 15, all columns
        for (uint32_t l = 0; l < hidden; ++l) {
            const float* Bp = packed + ((uint64_t)mem * hidden + l) * Hp * Hp;
            const float* b = prm + A.b_off[l + 1];
            f32x4_t acc[kInfBlocks];
#pragma unroll
            for (int n = 0; n < (int)kInfBlocks; ++n) acc[n] = f32x4_t{0.f, 0.f, 0.f, 0.f};
            for (uint32_t kb = 0; kb < KB; ++kb) {
                const f32x4_t a = *reinterpret_cast<const f32x4_t*>(act + ((wave * KB + kb) * 64 + lane) * 4);
                f32x4_t w[kInfBlocks];
#pragma unroll
                for (int n = 0; n < (int)kInfBlocks; ++n)
                    if ((uint32_t)n < NB)
                        w[n] = *reinterpret_cast<const f32x4_t*>(Bp + (((uint64_t)n * KB + kb) * 64 + lane) * 4);
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int n = 0; n < (int)kInfBlocks; ++n)
                        if ((uint32_t)n < NB) acc[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], w[n][j], acc[n], 0, 0, 0);
            }
            __syncthreads();  // every wave has read this layer's input
#pragma unroll
            for (int n = 0; n < (int)kInfBlocks; ++n) {
                if ((uint32_t)n >= NB) continue;
                const uint32_t col = n * 16 + (lane & 15u);
                const float bias = col < H ? b[col] : 0.f;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const uint32_t row = wave * 16 + 4 * (lane >> 4) + q;
                    act[frag32_index(row, col, KB)] = col < H ? gelu(acc[n][q] + bias) : 0.f;
                }
            }
            __syncthreads();
        }
        // output layer H -> 1: four lanes per row, each a quarter of the columns
        {
            const float* W = prm + A.w_off[A.n_layers - 1];
            const float bo = prm[A.b_off[A.n_layers - 1]];
            const uint32_t row = threadIdx.x >> 2, quarter = threadIdx.x & 3u;
            float part = 0.f;
            for (uint32_t col = quarter; col < H; col += 4) part = fmaf(act[frag32_index(row, col, KB)], W[col], part);
            part += __shfl_xor(part, 1, 4);
            part += __shfl_xor(part, 2, 4);
            if (quarter == 0) outs[row * 8 + mem] = part + bo;
            __syncthreads();
        }
    }
    const uint64_t gi = r0 + threadIdx.x;
    if (threadIdx.x >= kInfMRows || gi >= A.n) return;
    const float* out = outs + threadIdx.x * 8;
    if (raw)
        raw[mem0 * A.n + gi] = out[mem0];
    else
        store_prediction(A, gi, [&](uint32_t m) { return out[m]; });
}

// Wide networks (H > 64, two hidden layers or more): FP32 products on the BF16
// matrix cores.  An FP32 operand is the sum of three BF16 parts exactly (24
// bits in three times eight, and FP32's exponents, so nothing is scaled), and
// of the nine products of parts the six above 2^-24 of the whole are formed:
// what is left out is below the rounding of an FP32 product, and a sum of 256
// has 16 roundings of FP32 accumulators where the FP32 chain has 256.
//
// A wave owns 16 queries; every wave of the workgroup goes through all output
// features, 16 at a time, with the weights (A operand, rows = features)
// streamed through LDS in chunks of 32 features that the eight waves share.
// The k order of a product is free as long as both operands agree, and it is
// chosen so that the C values a lane ends with (4 neighbouring features of
// its query) are the 8 k values its B operand of the next layer needs: the
// activations never leave the lane.  They are kept in FP32 (64 registers at
// 256 columns) and split as the first 16 features of a layer are multiplied
// (96 for the parts), when no GELU is due.  The weights go to LDS past the
// registers (global_load_lds), which have no room for a chunk in flight.
//
// Bound by the vector unit's GELU and splitting next to the products and the
// LDS reads of the weights (200000 queries, five 5-256-256-256-1 networks: 620
// us each at their peaks), so the three have to overlap: a step's products are
// issued between the parts of the step before's GELU, and the weights two
// blocks ahead.  Eight waves of 16 queries fill the registers (256 each); four
// waves of 32 would halve the LDS reads, but a wave alone on its SIMD issues
// too slowly.  That call: 4482 us with FP32 products, 1420 so (185 TFLOP/s of
// the network's own products); 5-128-128-128-1 1750 -> 500.  Two FP16 parts and
// three products took 1090 us, but lost the operands' last bit and the products
// of the lower parts: 1.3e-7 to 2.2e-7 of the norm off in networks of one to
// four weights a row, where FP32 is 0.8e-7 to 1.5e-7 and this 0.7e-7 to 1.2e-7
// (dense rows: 2.0e-7, 4.3e-7, 1.7e-7).
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
constexpr uint32_t kSplitQueries = 16;  // per wave
constexpr uint32_t kSplitWaves = 8;
constexpr uint32_t kSplitThreads = kSplitWaves * kWave;
constexpr uint32_t kSplitParts = 3;

// Two values to their three parts, pairs in a register.
__device__ __forceinline__ void split_pair(float a0, float a1, uint32_t (&part)[kSplitParts])
{
    f32x2_t r = {a0, a1};
#pragma unroll
    for (uint32_t i = 0; i < kSplitParts; ++i) {
        part[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, bf16x2_t));
        r[0] -= __uint_as_float(part[i] << 16);  // exact
        r[1] -= __uint_as_float(part[i] & 0xffff0000u);
    }
}

// GELU(z), in four parts so that a caller can put matrix instructions between
// them.  |z| < 1: z / 2 + z^2 P(z^2), P = (Phi(z) - 1/2) / z.  From 1 on:
// max(z, 0) - t q(t) with t = |z|, q(t) = erfc(t / sqrt 2) / 2 =
// exp(-t^2 / 2) R(t), R a polynomial in u = 1 / (1 + 0.3 t); no cancellation
// for negative z.  Minimax fits, P to 2.6e-10, t q to 4.4e-9 of its size.
// Rounded to FP32 the error against 64 bits is below that of z (1 + erff) / 2
// over every range of z (0.5 <= z < 1: 1.8e-8 rms against 2.3e-8, 1 to 2:
// 3.4e-8 against 4.8e-8, 3 to 6: 1.1e-7 against 1.4e-7).
struct Gelu {
    float z, h, u, e, r, p;
    __device__ __forceinline__ void begin(float x)
    {
        z = x;
        h = z * z;
        u = __builtin_amdgcn_rcpf(fmaf(fabsf(z), 0.3f, 1.f));
        e = __builtin_amdgcn_exp2f(h * -0.72134752044448170f);
    }
    __device__ __forceinline__ void first()
    {
        r = fmaf(-0x1.757d7ep-4f, u, 0x1.0b8df4p-2f);
        r = fmaf(r, u, -0x1.31abb8p-4f);
        r = fmaf(r, u, 0x1.735f5cp-3f);
        r = fmaf(r, u, 0x1.9dfa2p-4f);
        r = fmaf(r, u, 0x1.f4b1c4p-4f);
    }
    __device__ __forceinline__ void second()
    {
        r = fmaf(r, u, -0x1.2f7cfp-13f);
        p = fmaf(-0x1.012f18p-17f, h, 0x1.dc1b46p-14f);
        p = fmaf(p, h, -0x1.36fecep-10f);
        p = fmaf(p, h, 0x1.46ce5ep-7f);
        p = fmaf(p, h, -0x1.105832p-4f);
        p = fmaf(p, h, 0x1.988454p-2f);
    }
    __device__ __forceinline__ float end() const
    {
        const float tail = fmaf(-fabsf(z), e * r, __builtin_elementwise_maximum(z, 0.f));  // fmaxf would drop a NaN
        return fabsf(z) < 1.f ? fmaf(h, p, 0.5f * z) : tail;
    }
};

// A member's table, rows of Hq: the biases of each layer l < hidden, the
// output layer's weights, the first layer's weights [Hq][wpad]; then the
// output layer's bias.
__host__ __device__ constexpr uint32_t split_table(uint32_t hidden, uint32_t Hq, uint32_t wpad)
{
    return (hidden + 1 + wpad) * Hq + 4;
}

struct SplitArgs {
    InferArgs in;
    uint32_t Hq;      // H rounded up to 128 or 256
    uint32_t hidden;
    __bf16* packed;   // [members][hidden - 1][Hq / 16 features][Hq / 32 k][3 parts][64 lanes][8]
    uint32_t wpad;    // inputs the kernel is built for, 5 or 8
    float* info;      // [members][split_table]
    uint64_t first;   // of the launch's queries
    float* raw;       // null, or [members][n - first] outputs where a workgroup takes one member (blockIdx.y)
};

// One workgroup per 16 features of a layer (z = member * hidden + layer): the
// table's entries, then (l >= 1) the rows' parts in the operand layout: per
// 32 k three runs of 1 KB, lane i + 16 g holding feature i,
// k = 32 kb + 16 (s / 4) + 4 g + s % 4 for its s = 0 .. 7.
__global__ __launch_bounds__(256) void mlp_split_pack_kernel(SplitArgs A)
{
    const uint32_t mem = blockIdx.y / A.hidden, l = blockIdx.y % A.hidden, ob = blockIdx.x;
    const uint32_t H = A.in.H, K = l ? H : A.in.w0;
    const float* prm = A.in.params + mem * A.in.P;
    const float* W = prm + A.in.w_off[l];
    float* table = A.info + (uint64_t)mem * split_table(A.hidden, A.Hq, A.wpad);
    if (threadIdx.x < 16) {
        const uint32_t o = ob * 16 + threadIdx.x;
        table[l * A.Hq + o] = o < H ? prm[A.in.b_off[l] + o] : 0.f;
        if (l == 0) table[A.hidden * A.Hq + o] = o < H ? prm[A.in.w_off[A.hidden] + o] : 0.f;
    }
    if (l == 0) {
        float* w_in = table + (A.hidden + 1) * A.Hq;
        for (uint32_t e = threadIdx.x; e < 16 * A.wpad; e += 256) {
            const uint32_t o = ob * 16 + e / A.wpad, j = e % A.wpad;
            w_in[ob * 16 * A.wpad + e] = o < H && j < K ? W[(uint64_t)o * K + j] : 0.f;
        }
        if (ob == 0 && threadIdx.x == 0) w_in[A.Hq * A.wpad] = prm[A.in.b_off[A.hidden]];
        return;
    }
    const uint32_t KB = A.Hq / 32;
    u32x4_t* out = reinterpret_cast<u32x4_t*>(A.packed) +
                   ((uint64_t)(mem * (A.hidden - 1) + l - 1) * (A.Hq / 16) + ob) * KB * kSplitParts * 64;
    for (uint32_t e = threadIdx.x; e < KB * 64; e += 256) {
        const uint32_t kb = e >> 6, lane = e & 63u, g = lane >> 4, o = ob * 16 + (lane & 15u);
        u32x4_t x[kSplitParts];
#pragma unroll
        for (int sl = 0; sl < 8; sl += 2) {
            const uint32_t k = kb * 32 + 16 * (sl >> 2) + 4 * g + (sl & 3);
            uint32_t part[kSplitParts];
            split_pair(o < H && k < H ? W[(uint64_t)o * H + k] : 0.f, o < H && k + 1 < H ? W[(uint64_t)o * H + k + 1] : 0.f,
                       part);
#pragma unroll
            for (uint32_t i = 0; i < kSplitParts; ++i) x[i][sl >> 1] = part[i];
        }
#pragma unroll
        for (uint32_t i = 0; i < kSplitParts; ++i) out[(kb * kSplitParts + i) * 64 + lane] = x[i];
    }
}

template <int KB, int W0>
__global__ __launch_bounds__(kSplitThreads) void mlp_split_infer_kernel(SplitArgs S)
{
    constexpr uint32_t HQ = 32 * KB;
    constexpr uint32_t kChunk = 2 * KB * kSplitParts * 64;  // 16-byte operands per chunk of 32 features
    constexpr uint32_t kPer = kChunk / kSplitThreads;       // of them per thread
    // two arrays, so that the reads of one do not wait for the loads into the other
    __shared__ u32x4_t ring0[kChunk], ring1[kChunk];
    __shared__ float outs[8][kSplitWaves * kSplitQueries];        // the members' outputs
    extern __shared__ __attribute__((aligned(16))) float info[];  // the member's table
    const InferArgs& A = S.in;
    const uint32_t tid = threadIdx.x, wave = uniform_u32(tid >> 6), lane = tid & 63u, g = lane >> 4;
    const uint32_t hidden = S.hidden;
    const uint64_t query = S.first + ((uint64_t)blockIdx.x * kSplitWaves + wave) * kSplitQueries + (lane & 15u);
    float x[W0];
#pragma unroll
    for (int j = 0; j < W0; ++j) {
        const bool ok = query < A.n && (uint32_t)j < A.w0;
        x[j] = ok ? (A.X[query * A.w0 + j] - A.sc.in_center[j]) / A.sc.in_scale[j] : 0.f;
    }
    const uint32_t mem0 = S.raw ? blockIdx.y : 0, mem1 = S.raw ? mem0 + 1 : A.members;
    // the chunk stream: every layer of every member in turn
    const u32x4_t* src = reinterpret_cast<const u32x4_t*>(S.packed) + (uint64_t)mem0 * (hidden - 1) * KB * kChunk;
    const u32x4_t* last = src + ((uint64_t)(mem1 - mem0) * (hidden - 1) * KB - 1) * kChunk;
    auto fetch = [&](u32x4_t* ring) {  // the next chunk, past the end the last one again
#pragma unroll
        for (uint32_t i = 0; i < kPer; ++i)
            __builtin_amdgcn_global_load_lds(static_cast<const void*>(src + i * kSplitThreads + tid),
                                             (void __attribute__((address_space(3)))*)(ring + i * kSplitThreads + wave * 64),
                                             16, 0, 0);
        src = src < last ? src + kChunk : last;
    };
    const uint32_t table = split_table(hidden, HQ, W0);
    const float* w_out = info + hidden * HQ;
    const float* w_in = w_out + HQ;
    constexpr uint32_t kCopies = (split_table(kMaxLayers - 1, HQ, W0) / 4 + kSplitThreads - 1) / kSplitThreads;
    fetch(ring0);
    for (uint32_t mem = mem0; mem < mem1; ++mem) {
        {   // sent for at once, and past the table's end its last entry again
            const f32x4_t* from = reinterpret_cast<const f32x4_t*>(S.info + (uint64_t)mem * table);
            f32x4_t t[kCopies];
#pragma unroll
            for (uint32_t i = 0; i < kCopies; ++i) t[i] = from[min(i * kSplitThreads + tid, table / 4 - 1)];
            __syncthreads();
#pragma unroll
            for (uint32_t i = 0; i < kCopies; ++i)
                if (i * kSplitThreads + tid < table / 4) reinterpret_cast<f32x4_t*>(info)[i * kSplitThreads + tid] = t[i];
        }
        __builtin_amdgcn_s_waitcnt(0);  // the first chunk has landed
        __syncthreads();
        float c[2 * KB][4];             // activations: features 16 s + 4 g + q of the query
#pragma unroll
        for (int s = 0; s < 2 * KB; ++s) {
            const uint32_t f0 = s * 16 + 4 * g;
            const f32x4_t bias = *reinterpret_cast<const f32x4_t*>(info + f0);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float z = bias[q];
#pragma unroll
                for (int j = 0; j < W0; ++j) z = fmaf(w_in[(f0 + q) * W0 + j], x[j], z);
                Gelu a;
                a.begin(z);
                a.first();
                a.second();
                c[s][q] = a.end();
            }
            // without these the compiler sends for several blocks' operands at
            // once and spills the activations
            __builtin_amdgcn_sched_barrier(0);
        }
        for (uint32_t l = 1; l < hidden; ++l) {
            const float* bias_l = info + l * HQ;
            u32x4_t b[KB][kSplitParts];  // the activations' parts, in pairs
            auto split = [&](int k) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    uint32_t part[kSplitParts];
                    split_pair(c[2 * k + (i >> 1)][2 * (i & 1)], c[2 * k + (i >> 1)][2 * (i & 1) + 1], part);
#pragma unroll
                    for (uint32_t j = 0; j < kSplitParts; ++j) b[k][j][i] = part[j];
                }
                // operands in four neighbouring registers, here and now
                asm("" : "+v"(b[k][0]), "+v"(b[k][1]), "+v"(b[k][2]));
            };
            auto operand = [](const u32x4_t& v) { return __builtin_bit_cast(bf16x8_t, v); };
            // 16 features a step, 32 k a block of 6 products; between the
            // products of a step, a part at a time, the vector unit makes
            // activations of the results of the step before, or in the first
            // step splits the next block's operands
            f32x4_t prev[2], bias;
            Gelu z[2];
            auto tables = [&](int s) { bias = *reinterpret_cast<const f32x4_t*>(bias_l + s * 16 + 4 * g); };
            auto part = [&](int s, int n) {  // of eight
                const int i = n >> 2;        // which two of the four values
#pragma unroll
                for (int j = 0; j < 2; ++j) {
                    const int q = 2 * i + j;
                    if ((n & 3) == 0)
                        z[j].begin(prev[0][q] + prev[1][q] + bias[q]);
                    else if ((n & 3) == 1)
                        z[j].first();
                    else if ((n & 3) == 2)
                        z[j].second();
                    else
                        c[s][q] = z[j].end();
                }
            };
            split(0);
#pragma unroll
            for (int p = 0; p < KB; ++p) {
                fetch(p & 1 ? ring0 : ring1);  // at a member's end the next member's first
                const u32x4_t* w = (p & 1 ? ring1 : ring0) + lane;
                u32x4_t a[2][kSplitParts];     // the next two blocks of weights
                auto weights = [&](int blk) {
#pragma unroll
                    for (uint32_t i = 0; i < kSplitParts; ++i) a[blk & 1][i] = w[(blk * kSplitParts + i) * 64];
                };
                weights(0);
                weights(1);
                f32x4_t acc[2];  // of the largest products, and of the others
#pragma unroll
                for (int blk = 0; blk < 2 * KB; ++blk) {
                    const int k = blk % KB, s = 2 * p + blk / KB;
                    if (k == 0) {
                        acc[0] = acc[1] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                        if (s > 0) tables(s - 1);
                    }
                    auto product = [&](int to, int i, int j) {
                        acc[to] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(operand(a[blk & 1][i]), operand(b[k][j]), acc[to],
                                                                          0, 0, 0);
                    };
                    product(1, 1, 1);
                    product(0, 0, 0);
                    product(1, 2, 0);
                    product(1, 0, 2);
                    product(1, 1, 0);
                    product(1, 0, 1);
                    if (blk + 2 < 2 * KB) weights(blk + 2);
                    if (s > 0) {
#pragma unroll
                        for (int n = 0; n < 8 / KB; ++n) part(s - 1, k * (8 / KB) + n);
                    } else if (k + 1 < KB)
                        split(k + 1);
                    __builtin_amdgcn_sched_barrier(0);
                    if (k == KB - 1) {
                        prev[0] = acc[0];
                        prev[1] = acc[1];
                    }
                }
                __builtin_amdgcn_s_waitcnt(0);  // the next chunk has landed
                __syncthreads();
            }
            tables(2 * KB - 1);
#pragma unroll
            for (int n = 0; n < 8; ++n) part(2 * KB - 1, n);
        }
        float y = 0.f;
#pragma unroll
        for (int s = 0; s < 2 * KB; ++s) {
            const f32x4_t wo = *reinterpret_cast<const f32x4_t*>(w_out + s * 16 + 4 * g);
#pragma unroll
            for (int q = 0; q < 4; ++q) y = fmaf(c[s][q], wo[q], y);
        }
        y += __shfl_xor(y, 16, 64);
        y += __shfl_xor(y, 32, 64);
        if (g == 0) outs[mem][wave * kSplitQueries + lane] = y + info[table - 4];
    }
    if (g || query >= A.n) return;
    if (S.raw)
        S.raw[mem0 * (A.n - S.first) + query - S.first] = outs[mem0][wave * kSplitQueries + lane];
    else
        store_prediction(A, query, [&](uint32_t m) { return outs[m][wave * kSplitQueries + lane]; });
}

// ------------------------------------------------------------ scan glue ---
__global__ void scan_flag_kernel(const float* spread, float spread_max, uint64_t n, uint8_t* flag)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) flag[i] = spread[i] > spread_max ? 1 : 0;
}

__global__ void scan_merge_kernel(const float* mean, const uint8_t* flag, const uint64_t* fb_index,
                                  const double* fb_sums, const uint32_t* fb_paths, uint64_t n_fb, uint64_t n,
                                  double* v_out, uint8_t* used)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        if (!flag[i]) v_out[i] = (double)mean[i];  // flagged entries are written below
        if (used) used[i] = flag[i];
    }
    if (i < n_fb) v_out[fb_index[i]] = fb_sums[2 * i] / (double)fb_paths[i];
}

}  // namespace sde

using namespace sde;

// ------------------------------------------------------------------ host --
namespace {

int check_s(sde_surrogate* s) { return s && s->ctx ? SDE_OK : SDE_ERR_INVALID; }

void layout(sde_surrogate* s)
{
    s->w_off.clear();
    s->b_off.clear();
    uint64_t k = 0;
    for (size_t l = 0; l + 1 < s->widths.size(); ++l) {
        s->w_off.push_back(k);
        k += (uint64_t)s->widths[l + 1] * s->widths[l];
        s->b_off.push_back(k);
        k += s->widths[l + 1];
    }
    s->P = k;
}

int alloc_surrogate(sde_ctx* ctx, const uint32_t* widths, uint32_t n_widths, uint32_t members, sde_surrogate** out)
{
    if (!ctx || !widths || !out || n_widths < 2 || n_widths > (uint32_t)kMaxLayers + 1 || members == 0 || members > 8)
        return fail(ctx, SDE_ERR_INVALID, "surrogate: need 2..%d widths and 1..8 members", kMaxLayers + 1);
    if (widths[n_widths - 1] != 1) return fail(ctx, SDE_ERR_INVALID, "surrogate: the output width must be 1");
    if (widths[0] == 0 || widths[0] > 8) return fail(ctx, SDE_ERR_INVALID, "surrogate: 1..8 input features");
    for (uint32_t l = 1; l + 1 < n_widths; ++l)
        if (widths[l] == 0 || widths[l] > (uint32_t)kInfH || (l > 1 && widths[l] != widths[1]))
            return fail(ctx, SDE_ERR_INVALID, "surrogate: hidden layers must share one width <= %d", kInfH);
    sde_surrogate* s = new (std::nothrow) sde_surrogate();
    if (!s) return SDE_ERR_NOMEM;
    s->ctx = ctx;
    s->widths.assign(widths, widths + n_widths);
    s->members = members;
    layout(s);
    const size_t bytes = (size_t)members * s->P * sizeof(float);
    if (hipMalloc(&s->params, bytes) != hipSuccess || hipMalloc(&s->grads, bytes) != hipSuccess ||
        hipMalloc(&s->adam_m, bytes) != hipSuccess || hipMalloc(&s->adam_v, bytes) != hipSuccess ||
        hipMalloc(&s->adam_t, 8 * sizeof(uint64_t)) != hipSuccess) {
        (void)hipGetLastError();
        sde_surrogate_destroy(s);
        return fail(ctx, SDE_ERR_NOMEM, "surrogate: cannot allocate parameters");
    }
    if (hipMemset(s->adam_m, 0, bytes) != hipSuccess || hipMemset(s->adam_v, 0, bytes) != hipSuccess ||
        hipMemset(s->adam_t, 0, 8 * sizeof(uint64_t)) != hipSuccess) {
        sde_surrogate_destroy(s);
        return fail(ctx, SDE_ERR_DEVICE, "surrogate: hipMemset failed");
    }
    for (int i = 0; i < 8; ++i) {
        s->sc.in_center[i] = 0.f;
        s->sc.in_scale[i] = 1.f;
    }
    s->sc.out_mean = 0.f;
    s->sc.out_std = 1.f;
    *out = s;
    return SDE_OK;
}

int ensure_work(sde_surrogate* s, size_t bytes)
{
    if (s->work_bytes >= bytes) return SDE_OK;
    if (s->work) {
        SDE_HIP(s->ctx, hipDeviceSynchronize());
        SDE_HIP(s->ctx, hipFree(s->work));
        s->work = nullptr;
        s->work_bytes = 0;
        ++s->ctx->ws_generation;
    }
    if (hipMalloc(&s->work, bytes) != hipSuccess) {
        (void)hipGetLastError();
        return fail(s->ctx, SDE_ERR_NOMEM, "surrogate: cannot allocate %zu bytes of workspace", bytes);
    }
    s->work_bytes = bytes;
    ++s->ctx->ws_generation;
    return SDE_OK;
}

// Slices of the batch sum of a weight-gradient product: enough workgroups to
// cover the CUs (the M x N tiles alone give few), at least 64 rows each.
constexpr uint32_t kMaxKSlices = 16;
static uint32_t dw_kslices(uint32_t M, uint32_t N, uint32_t K, uint32_t members)
{
    const uint32_t tiles = ((N + kGT - 1) / kGT) * ((M + kGT - 1) / kGT) * members;
    uint32_t k = (320 + tiles - 1) / tiles;
    k = std::min(k, std::max(1u, K / 64));
    return std::max(1u, std::min(k, kMaxKSlices));
}

// Shapes of a step on minibatches of B, and its buffers in the workspace
// (16-float aligned sections); returns the floats they take.
size_t carve(sde_surrogate* s, uint64_t n, uint32_t B, uint32_t steps, TrainArgs& A)
{
    A = TrainArgs{};
    A.B = B;
    A.w0 = s->widths[0];
    A.hidden = (uint32_t)s->widths.size() - 2;
    A.H = A.hidden ? s->widths[1] : 0u;
    A.Hp = (A.H + 15u) & ~15u;
    A.members = s->members;
    A.params = s->params;
    A.P = s->P;
    for (size_t l = 0; l < s->w_off.size(); ++l) {
        A.w_off[l] = s->w_off[l];
        A.b_off[l] = s->b_off[l];
    }
    A.ks_h = A.hidden > 1 ? dw_kslices(A.H, A.H, B, A.members) : 0u;
    A.ks_in = A.hidden ? dw_kslices(A.H, A.w0, B, A.members) : 0u;
    A.ks_out = dw_kslices(1, A.hidden ? A.H : A.w0, B, A.members);
    A.col_slices = (B + kColSlice - 1) / kColSlice;
    A.loss_stride = steps;
    size_t at = 0;
    auto take = [&](size_t floats) {
        float* p = s->work + at;
        at += (floats + 15) & ~(size_t)15;
        return p;
    };
    const size_t M = A.members, hh = (size_t)A.Hp * A.Hp, pairs = A.hidden > 1 ? A.hidden - 1 : 0;
    const size_t layers = A.hidden * A.layer_stride();
    A.Xn = take(n * A.w0);
    A.yn = take(n);
    A.act = take(layers);
    A.slope = take(layers);
    A.dz = take(layers);
    A.y = take(M * B);
    A.dy = take(M * B);
    A.wf = take(M * pairs * hh);
    A.wb = take(M * pairs * hh);
    A.part_h = take(pairs * M * A.ks_h * hh);
    A.part_in = take(M * A.ks_in * A.H * A.w0);
    A.part_out = take(M * A.ks_out * (A.hidden ? A.H : A.w0));
    A.part_b = take((size_t)A.hidden * M * A.col_slices * A.Hp);
    A.part_bo = take(M * A.col_slices);
    A.loss = take(M * steps);
    A.bc = take(2 * M);
    return at;
}

// Sizes the workspace for it first.
int prepare_steps(sde_surrogate* s, uint64_t n, uint32_t B, uint32_t steps, TrainArgs& A)
{
    const size_t floats = carve(s, n, B, steps, A);
    if (const int e = ensure_work(s, floats * sizeof(float))) return e;
    carve(s, n, B, steps, A);
    return SDE_OK;
}

int pack_weights(sde_surrogate* s, const TrainArgs& A, hipStream_t st)
{
    if (A.hidden < 2) return SDE_OK;
    const uint64_t total = (uint64_t)A.members * (A.hidden - 1) * A.Hp * A.Hp;
    hipLaunchKernelGGL(mlp_pack_train_kernel, dim3((uint32_t)((total + 255) / 256)), dim3(256), 0, st, A);
    SDE_HIP(s->ctx, hipGetLastError());
    return SDE_OK;
}

// One step (forward, loss, backward, and Adam where A holds its state).
int record_step(sde_ctx* ctx, const TrainArgs& A, hipStream_t st)
{
    // 16 samples a workgroup up to three workgroups a CU, then 32, which halve
    // the traffic of the weights.  An epoch of 16384 samples, 16 against 32:
    // five members, batch 1024 (320 workgroups) 1679 against 1737 us, 2048
    // (640) 1277 against 1421; eight members, 1536 (768) 1789 against 1935,
    // but 2048 (1024) 1852 against 1778 and 4096 1796 against 1736.
    if ((uint64_t)((A.B + 15) / 16) * A.members <= 3 * (uint64_t)ctx->n_cu)
        hipLaunchKernelGGL(mlp_rows_kernel<1>, dim3((A.B + 15) / 16, A.members), dim3(kRowsThreads), 0, st, A);
    else
        hipLaunchKernelGGL(mlp_rows_kernel<2>, dim3((A.B + 31) / 32, A.members), dim3(kRowsThreads), 0, st, A);
    hipLaunchKernelGGL(mlp_grads_kernel, dim3(GradsGrid(A).total()), dim3(256), 0, st, A);
    uint32_t blocks = 0;
    for (uint32_t l = 0; l <= A.hidden; ++l) blocks += update_blocks(A, l);
    hipLaunchKernelGGL(mlp_update_kernel, dim3(blocks, A.members), dim3(256), 0, st, A);
    SDE_HIP(ctx, hipGetLastError());
    return SDE_OK;
}

int normalize(sde_surrogate* s, const float* X, const float* y, uint64_t n, const TrainArgs& t, hipStream_t st)
{
    NormArgs a;
    a.X = X;
    a.y = y;
    a.Xn = const_cast<float*>(t.Xn);
    a.yn = const_cast<float*>(t.yn);
    a.n = n;
    a.w0 = s->widths[0];
    a.sc = s->sc;
    hipLaunchKernelGGL(mlp_normalize_kernel, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, st, a);
    SDE_HIP(s->ctx, hipGetLastError());
    return SDE_OK;
}

}  // namespace

extern "C" {

int sde_surrogate_create(sde_ctx* ctx, const uint32_t* widths, uint32_t n_widths, uint32_t n_members, uint64_t seed,
                         sde_surrogate** out)
{
    if (!ctx) return SDE_ERR_INVALID;
    ctx->last_error.clear();
    sde_surrogate* s = nullptr;
    int st = alloc_surrogate(ctx, widths, n_widths, n_members, &s);
    if (st) return st;
    InitArgs a{};
    a.params = s->params;
    a.P = s->P;
    a.members = s->members;
    a.n_layers = (uint32_t)s->widths.size() - 1;
    for (uint32_t l = 0; l < a.n_layers; ++l) {
        a.layer_end[l] = s->b_off[l] + s->widths[l + 1];
        a.bound[l] = (float)(1.0 / std::sqrt((double)s->widths[l]));
    }
    a.key0 = (uint32_t)seed;
    a.key1 = (uint32_t)(seed >> 32);
    const uint64_t total = s->P * s->members;
    hipLaunchKernelGGL(mlp_init_kernel, dim3((uint32_t)((total + 255) / 256)), dim3(256), 0, 0, a);
    if (hipGetLastError() != hipSuccess || hipDeviceSynchronize() != hipSuccess) {
        sde_surrogate_destroy(s);
        return fail(ctx, SDE_ERR_DEVICE, "surrogate: initialization kernel failed");
    }
    *out = s;
    return SDE_OK;
}

void sde_surrogate_destroy(sde_surrogate* s)
{
    if (!s) return;
    (void)hipDeviceSynchronize();
    for (void* p : {(void*)s->params, (void*)s->grads, (void*)s->adam_m, (void*)s->adam_v, (void*)s->adam_t,
                    (void*)s->work, (void*)s->perm, (void*)s->packed})
        if (p) (void)hipFree(p);
    if (s->raw_done) (void)hipEventDestroy(s->raw_done);
    delete s;
}

uint64_t sde_surrogate_param_count(const sde_surrogate* s) { return s ? s->P : 0; }

int sde_surrogate_set_params(sde_surrogate* s, uint32_t member, const float* host, uint64_t n)
{
    if (check_s(s)) return SDE_ERR_INVALID;
    if (!host || member >= s->members || n != s->P) return fail(s->ctx, SDE_ERR_INVALID, "set_params: bad member/size");
    const size_t b = s->P * sizeof(float);
    SDE_HIP(s->ctx, hipDeviceSynchronize());
    SDE_HIP(s->ctx, hipMemcpy(s->params + member * s->P, host, b, hipMemcpyHostToDevice));
    SDE_HIP(s->ctx, hipMemset(s->adam_m + member * s->P, 0, b));
    SDE_HIP(s->ctx, hipMemset(s->adam_v + member * s->P, 0, b));
    uint64_t zero = 0;
    SDE_HIP(s->ctx, hipMemcpy(s->adam_t + member, &zero, sizeof zero, hipMemcpyHostToDevice));
    return SDE_OK;
}

int sde_surrogate_get_params(sde_surrogate* s, uint32_t member, float* host, uint64_t n)
{
    if (check_s(s)) return SDE_ERR_INVALID;
    if (!host || member >= s->members || n != s->P) return fail(s->ctx, SDE_ERR_INVALID, "get_params: bad member/size");
    SDE_HIP(s->ctx, hipDeviceSynchronize());
    SDE_HIP(s->ctx, hipMemcpy(host, s->params + member * s->P, s->P * sizeof(float), hipMemcpyDeviceToHost));
    return SDE_OK;
}

int sde_surrogate_set_scaling(sde_surrogate* s, const sde_surrogate_scaling* sc)
{
    if (check_s(s) || !sc) return SDE_ERR_INVALID;
    for (uint32_t j = 0; j < s->widths[0]; ++j)
        if (!std::isfinite(sc->in_center[j]) || !std::isfinite(sc->in_scale[j]) || sc->in_scale[j] == 0.f)
            return fail(s->ctx, SDE_ERR_INVALID, "scaling: feature %u needs a finite center and nonzero scale", j);
    if (!std::isfinite(sc->out_mean) || !std::isfinite(sc->out_std) || sc->out_std == 0.f || sc->reserved != 0)
        return fail(s->ctx, SDE_ERR_INVALID, "scaling: bad output scaling");
    if (sc->target_over_omega && s->widths[0] < 2)
        return fail(s->ctx, SDE_ERR_INVALID, "scaling: <v>/omega needs omega as feature 1");
    s->sc = *sc;
    return SDE_OK;
}

int sde_surrogate_get_scaling(const sde_surrogate* s, sde_surrogate_scaling* sc)
{
    if (!s || !sc) return SDE_ERR_INVALID;
    *sc = s->sc;
    return SDE_OK;
}

int sde_surrogate_loss_grad(sde_surrogate* s, uint32_t member, const float* X, const float* y, uint64_t n,
                            float* host_grad, double* host_loss, void* hip_stream)
{
    if (check_s(s)) return SDE_ERR_INVALID;
    sde_ctx* ctx = s->ctx;
    ctx->last_error.clear();
    if (!X || !y || n == 0 || n > (1u << 20) || member >= s->members)
        return fail(ctx, SDE_ERR_INVALID, "loss_grad: bad arguments");
    hipStream_t st = static_cast<hipStream_t>(hip_stream);
    const uint32_t B = (uint32_t)n;
    int e;
    TrainArgs t;
    if ((e = prepare_steps(s, n, B, 1, t))) return e;
    t.grads = s->grads;
    if ((e = normalize(s, X, y, n, t, st)) || (e = pack_weights(s, t, st)) || (e = record_step(ctx, t, st))) return e;
    SDE_HIP(ctx, hipStreamSynchronize(st));
    if (host_grad)
        SDE_HIP(ctx, hipMemcpy(host_grad, s->grads + member * s->P, s->P * sizeof(float), hipMemcpyDeviceToHost));
    if (host_loss) {
        float l = 0.f;
        SDE_HIP(ctx, hipMemcpy(&l, t.loss + member, sizeof(float), hipMemcpyDeviceToHost));
        *host_loss = l;
    }
    return SDE_OK;
}

int sde_surrogate_train(sde_surrogate* s, const float* X, const float* y, uint64_t n, const sde_train_opts* o,
                        float* loss_curve, void* hip_stream)
{
    if (check_s(s)) return SDE_ERR_INVALID;
    const TraceRange range("sde_surrogate_train");
    sde_ctx* ctx = s->ctx;
    ctx->last_error.clear();
    if (!X || !y || !o || n == 0 || o->epochs == 0 || o->batch == 0 || o->batch > n || n > 0xffffffffull)
        return fail(ctx, SDE_ERR_INVALID, "train: need X, y, options, 0 < batch <= n");
    if (!(o->lr > 0) || !(o->beta1 >= 0 && o->beta1 < 1) || !(o->beta2 >= 0 && o->beta2 < 1) || !(o->eps > 0))
        return fail(ctx, SDE_ERR_INVALID, "train: bad Adam hyper-parameters");
    try {
        hipStream_t st = static_cast<hipStream_t>(hip_stream);
        const uint32_t B = o->batch;
        const uint32_t steps = (uint32_t)(n / B);
        int e;
        TrainArgs t;
        if ((e = prepare_steps(s, n, B, steps, t))) return e;
        if ((e = normalize(s, X, y, n, t, st)) || (e = pack_weights(s, t, st))) return e;
        const size_t perm_elems = (size_t)s->members * n;
        if (s->perm_cap < perm_elems) {
            SDE_HIP(ctx, hipDeviceSynchronize());
            if (s->perm) SDE_HIP(ctx, hipFree(s->perm));
            s->perm = nullptr;
            s->perm_cap = 0;
            SDE_HIP(ctx, hipMalloc(&s->perm, perm_elems * sizeof(uint32_t)));
            s->perm_cap = perm_elems;
            ++ctx->ws_generation;
        }
        t.rows = s->perm;
        t.rows_mstride = n;
        t.m = s->adam_m;
        t.v = s->adam_v;
        t.t = s->adam_t;
        t.lr = o->lr;
        t.b1 = o->beta1;
        t.b2 = o->beta2;
        t.eps = o->eps;
        std::vector<uint32_t> perm(perm_elems);
        std::vector<float> losses(steps);
        uint32_t* hperm = nullptr;
        SDE_HIP(ctx, hipHostMalloc(&hperm, perm_elems * sizeof(uint32_t), hipHostMallocDefault));
        char key[256];
        snprintf(key, sizeof key, "mlp-epoch|%p|%p|%p|%llu|%u|%u|%a|%a|%a|%a", (void*)s, (void*)s->work, (void*)s->perm,
                 (unsigned long long)n, B, steps, o->lr, o->beta1, o->beta2, o->eps);
        for (uint32_t ep = 0; ep < o->epochs; ++ep) {
            // the sample order of this epoch, one permutation per member
            for (uint32_t m = 0; m < s->members; ++m) {
                std::mt19937_64 rng(o->shuffle_seed * 1000003ull + (uint64_t)ep * 131ull + m);
                uint32_t* p = perm.data() + (size_t)m * n;
                std::iota(p, p + n, 0u);
                std::shuffle(p, p + n, rng);
            }
            SDE_HIP(ctx, hipStreamSynchronize(st));  // the previous epoch no longer reads hperm
            std::memcpy(hperm, perm.data(), perm_elems * sizeof(uint32_t));
            SDE_HIP(ctx, hipMemcpyAsync(s->perm, hperm, perm_elems * sizeof(uint32_t), hipMemcpyHostToDevice, st));
            e = run_recorded(ctx, key, st, [&](hipStream_t cs) -> int {
                for (uint32_t k = 0; k < steps; ++k) {
                    t.rows_offset = k * B;
                    t.loss_slot = k;
                    if (const int r = record_step(ctx, t, cs)) return r;
                }
                return SDE_OK;
            });
            if (e) {
                (void)hipHostFree(hperm);
                return e;
            }
            if (loss_curve) {
                SDE_HIP(ctx, hipMemcpyAsync(losses.data(), t.loss, steps * sizeof(float), hipMemcpyDeviceToHost, st));
                SDE_HIP(ctx, hipStreamSynchronize(st));
                double sum = 0.0;
                for (float l : losses) sum += l;
                loss_curve[ep] = (float)(sum / steps);
            }
        }
        SDE_HIP(ctx, hipStreamSynchronize(st));
        SDE_HIP(ctx, hipHostFree(hperm));
        return SDE_OK;
    } catch (...) {
        return fail(ctx, SDE_ERR_NOMEM, "host allocation failed");
    }
}

static int ensure_packed(sde_surrogate* s, size_t need)
{
    sde_ctx* ctx = s->ctx;
    if (s->packed_bytes >= need) return SDE_OK;
    if (s->packed) SDE_HIP(ctx, hipFree(s->packed));
    s->packed = nullptr;
    s->packed_bytes = 0;
    SDE_HIP(ctx, hipMalloc(&s->packed, need));
    s->packed_bytes = need;
    return SDE_OK;
}

// The members' outputs that mlp_combine_kernel reads are the handle's, one
// region for every stream: a call waits on its stream for the call before to
// have read them.  Two calls in turn on the null stream are ordered by it, and
// need no event (one query of five 5-64-64-64-1 networks 25 us, 29 with one).
// A call that is being captured gives no workgroup to one member, since its
// replays could be ordered with nothing.
static bool members_apart(hipStream_t st)
{
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(st, &status) == hipSuccess) return status == hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return false;
}

static int raw_begin(sde_surrogate* s, hipStream_t st)
{
    if (s->raw_last == 0 || (!st && s->raw_last == 1)) return SDE_OK;
    if (s->raw_last == 1) {
        if (!s->raw_done) SDE_HIP(s->ctx, hipEventCreateWithFlags(&s->raw_done, hipEventDisableTiming));
        SDE_HIP(s->ctx, hipEventRecord(s->raw_done, nullptr));
    }
    SDE_HIP(s->ctx, hipStreamWaitEvent(st, s->raw_done, 0));
    return SDE_OK;
}

static int raw_end(sde_surrogate* s, hipStream_t st)
{
    SDE_HIP(s->ctx, hipGetLastError());
    if (st) {
        if (!s->raw_done) SDE_HIP(s->ctx, hipEventCreateWithFlags(&s->raw_done, hipEventDisableTiming));
        SDE_HIP(s->ctx, hipEventRecord(s->raw_done, st));
    }
    s->raw_last = st ? 2 : 1;
    return SDE_OK;
}

// Widths past 64 with products between hidden layers.  Below the line the
// operands would be padded to 128 columns: 200000 queries of five networks with
// three hidden layers take 420 us at H = 64 on the FP32 products, 483 at H = 65
// here; at H = 100 (two hidden layers) 310 us here, 1060 there.
static int predict_split(sde_surrogate* s, const InferArgs& a, hipStream_t st)
{
    sde_ctx* ctx = s->ctx;
    SplitArgs S{};
    S.in = a;
    S.hidden = a.n_layers - 1;
    S.Hq = a.H <= 128 ? 128 : 256;
    S.wpad = a.w0 <= 5 ? 5 : 8;
    const size_t parts = (size_t)a.members * (S.hidden - 1) * S.Hq * S.Hq * kSplitParts;
    const uint32_t table = split_table(S.hidden, S.Hq, S.wpad);
    // Workgroups past the last full round over the CUs: a workgroup per member
    // where that takes at most half a round's time (a call of one query 204
    // -> 53 us, of 200000, 6.1 rounds, 1565 -> 1422).
    const uint32_t per = kSplitQueries * kSplitWaves;
    const uint64_t blocks = (a.n + per - 1) / per, n_cu = (uint64_t)ctx->n_cu, tail = blocks % n_cu;
    const bool by_member = tail && 2 * ((tail * a.members + n_cu - 1) / n_cu) <= a.members && members_apart(st);
    const size_t floats = (size_t)a.members * table, raw = (size_t)a.members * n_cu * per;
    if (const int e = ensure_packed(s, parts * sizeof(__bf16) + (floats + raw) * sizeof(float))) return e;
    S.packed = reinterpret_cast<__bf16*>(s->packed);
    S.info = reinterpret_cast<float*>(S.packed + parts);
    hipLaunchKernelGGL(mlp_split_pack_kernel, dim3(S.Hq / 16, a.members * S.hidden), dim3(256), 0, st, S);
    SDE_HIP(ctx, hipGetLastError());
    void (*kern)(SplitArgs) = S.Hq == 128 ? (S.wpad == 5 ? mlp_split_infer_kernel<4, 5> : mlp_split_infer_kernel<4, 8>)
                                          : (S.wpad == 5 ? mlp_split_infer_kernel<8, 5> : mlp_split_infer_kernel<8, 8>);
    const size_t lds = table * sizeof(float);
    const uint64_t full = by_member ? blocks - tail : blocks;
    if (full) {
        SplitArgs F = S;
        F.in.n = std::min<uint64_t>(a.n, full * per);
        hipLaunchKernelGGL(kern, dim3((uint32_t)full), dim3(kSplitThreads), lds, st, F);
        SDE_HIP(ctx, hipGetLastError());
    }
    if (by_member) {
        S.first = full * per;
        S.raw = S.info + floats;
        if (const int e = raw_begin(s, st)) return e;
        hipLaunchKernelGGL(kern, dim3((uint32_t)tail, a.members), dim3(kSplitThreads), lds, st, S);
        SDE_HIP(ctx, hipGetLastError());
        hipLaunchKernelGGL(mlp_combine_kernel, dim3((uint32_t)((a.n - S.first + 255) / 256)), dim3(256), 0, st, a,
                           S.first, static_cast<const float*>(S.raw));
        if (const int e = raw_end(s, st)) return e;
    }
    return SDE_OK;
}

static int predict_impl(sde_surrogate* s, const float* X, uint64_t n, float* mean, float* spread, hipStream_t st)
{
    sde_ctx* ctx = s->ctx;
    if (s->widths.size() - 1 < 2) return fail(ctx, SDE_ERR_UNSUPPORTED, "predict: needs at least one hidden layer");
    InferArgs a{};
    a.X = X;
    a.params = s->params;
    a.mean = mean;
    a.spread = spread;
    a.n = n;
    a.P = s->P;
    a.members = s->members;
    a.n_layers = (uint32_t)s->widths.size() - 1;
    a.w0 = s->widths[0];
    a.H = s->widths[1];
    for (uint32_t l = 0; l < a.n_layers; ++l) {
        a.w_off[l] = s->w_off[l];
        a.b_off[l] = s->b_off[l];
    }
    a.sc = s->sc;
    if (a.n_layers >= 3 && a.H >= kSplitMinH) return predict_split(s, a, st);
    // hidden weights into the MFMA operand layout (Hp = H rounded up to 16)
    const uint32_t H = a.H, Hp = (H + 15u) & ~15u, hidden = a.n_layers - 2;
    // Up to one workgroup a CU: a workgroup per member, several of which share
    // a CU (five 5-64-64-64-1 networks, one query 94 -> 25 us, 16384 96 -> 45).
    const uint64_t blocks = (n + kInfMRows - 1) / kInfMRows;
    const bool by_member = a.members > 1 && blocks <= (uint64_t)ctx->n_cu && members_apart(st);
    const size_t weights = (size_t)s->members * hidden * Hp * Hp, raw = (size_t)s->members * ctx->n_cu * kInfMRows;
    if (const int e = ensure_packed(s, (weights + raw) * sizeof(float))) return e;
    if (hidden > 0) {
        PackArgs pk{};
        pk.params = s->params;
        pk.P = s->P;
        pk.members = s->members;
        pk.hidden = hidden;
        pk.H = H;
        pk.Hp = Hp;
        for (uint32_t l = 0; l < hidden; ++l) pk.w_off[l] = s->w_off[l + 1];
        pk.packed = s->packed;
        const uint64_t total = (uint64_t)s->members * hidden * Hp * Hp;
        hipLaunchKernelGGL(mlp_pack_hidden_kernel, dim3((uint32_t)((total + 255) / 256)), dim3(256), 0, st, pk);
        SDE_HIP(ctx, hipGetLastError());
    }
    const size_t lds = (size_t)kInfMRows * (Hp + 16) * sizeof(float);
    static bool attr_set = false;
    if (!attr_set) {
        SDE_HIP(ctx, hipFuncSetAttribute(reinterpret_cast<const void*>(mlp_infer_mfma_kernel),
                                         hipFuncAttributeMaxDynamicSharedMemorySize,
                                         (int)(kInfMRows * (kInfH + 16) * sizeof(float))));
        attr_set = true;
    }
    float* members_out = by_member ? s->packed + weights : nullptr;
    if (by_member)
        if (const int e = raw_begin(s, st)) return e;
    hipLaunchKernelGGL(mlp_infer_mfma_kernel, dim3((uint32_t)blocks, by_member ? a.members : 1), dim3(256), lds, st, a,
                       static_cast<const float*>(s->packed), Hp, members_out);
    SDE_HIP(ctx, hipGetLastError());
    if (by_member) {
        hipLaunchKernelGGL(mlp_combine_kernel, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, st, a, (uint64_t)0,
                           static_cast<const float*>(members_out));
        if (const int e = raw_end(s, st)) return e;
    }
    return SDE_OK;
}

int sde_surrogate_predict(sde_surrogate* s, const float* X, uint64_t n, float* mean, float* spread, void* hip_stream)
{
    if (check_s(s)) return SDE_ERR_INVALID;
    const TraceRange range("sde_surrogate_predict");
    s->ctx->last_error.clear();
    if (!X || !mean || !spread || n == 0 || (n + kInfMRows - 1) / kInfMRows > 0x7fffffffull)
        return fail(s->ctx, SDE_ERR_INVALID, "predict: bad arguments");
    if (!aligned(X, 4) || !aligned(mean, 4) || !aligned(spread, 4))
        return fail(s->ctx, SDE_ERR_INVALID, "predict: misaligned pointer");
    return predict_impl(s, X, n, mean, spread, static_cast<hipStream_t>(hip_stream));
}

int sde_surrogate_scan(sde_surrogate* s, const sde_jj_point* q, uint64_t n, float spread_max, const sde_run* fb,
                       double* v_out, uint8_t* used, sde_scan_stats* stats, void* hip_stream)
{
    if (check_s(s)) return SDE_ERR_INVALID;
    const TraceRange range("sde_surrogate_scan");
    sde_ctx* ctx = s->ctx;
    ctx->last_error.clear();
    if (!q || n == 0 || !fb || !v_out || !(spread_max >= 0) || s->widths[0] != 5)
        return fail(ctx, SDE_ERR_INVALID, "scan: bad arguments (the surrogate must take 5 features)");
    if (!aligned(v_out, 8)) return fail(ctx, SDE_ERR_INVALID, "scan: misaligned v_out");
    try {
        const auto t0 = std::chrono::steady_clock::now();
        hipStream_t st = static_cast<hipStream_t>(hip_stream);
        std::vector<float> feat(n * 5);
        for (uint64_t i = 0; i < n; ++i) {
            if (!(q[i].D > 0) || q[i].m != 1.0)
                return fail(ctx, SDE_ERR_INVALID, "scan: query %llu needs D > 0 and m = 1", (unsigned long long)i);
            feat[5 * i] = (float)q[i].a;
            feat[5 * i + 1] = (float)q[i].omega;
            feat[5 * i + 2] = (float)q[i].f;
            feat[5 * i + 3] = (float)std::log10(q[i].D);
            feat[5 * i + 4] = (float)q[i].gamma;
        }
        // workspace: features | mean | spread | flags
        int e = upload(ctx, kSlotMisc, 3, feat.data(), feat.size() * sizeof(float), st);
        if (e) return e;
        void* w = nullptr;
        if ((e = ensure_ws(ctx, kSlotObs, n * (2 * sizeof(float) + 1) + 256, &w))) return e;
        float* X = static_cast<float*>(ctx->ws[kSlotMisc].ptr);
        float* mean = static_cast<float*>(w);
        float* spread = mean + n;
        uint8_t* flag = reinterpret_cast<uint8_t*>(spread + n);
        hipEvent_t e0, e1, e2, e3;
        SDE_HIP(ctx, hipEventCreate(&e0));
        SDE_HIP(ctx, hipEventCreate(&e1));
        SDE_HIP(ctx, hipEventCreate(&e2));
        SDE_HIP(ctx, hipEventCreate(&e3));
        SDE_HIP(ctx, hipEventRecord(e0, st));
        if ((e = predict_impl(s, X, n, mean, spread, st))) return e;
        hipLaunchKernelGGL(scan_flag_kernel, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, st, spread, spread_max,
                           n, flag);
        SDE_HIP(ctx, hipEventRecord(e1, st));
        std::vector<uint8_t> hflag(n);
        SDE_HIP(ctx, hipMemcpyAsync(hflag.data(), flag, n, hipMemcpyDeviceToHost, st));
        SDE_HIP(ctx, hipStreamSynchronize(st));
        std::vector<sde_jj_point> fpts;
        std::vector<uint64_t> fidx;
        std::vector<uint32_t> fpaths;
        for (uint64_t i = 0; i < n; ++i)
            if (hflag[i]) {
                fpts.push_back(q[i]);
                fidx.push_back(i);
                fpaths.push_back(q[i].n_paths);
            }
        const uint64_t nf = fpts.size();
        // fallback simulation: one persistent launch over the uncertain points
        void* fbw = nullptr;
        if ((e = ensure_ws(ctx, kSlotTune, std::max<uint64_t>(nf, 1) * (2 * sizeof(double) + sizeof(uint64_t) + 4) + 64,
                           &fbw)))
            return e;
        double* fsums = static_cast<double*>(fbw);
        uint64_t* didx = reinterpret_cast<uint64_t*>(fsums + 2 * std::max<uint64_t>(nf, 1));
        uint32_t* dpaths = reinterpret_cast<uint32_t*>(didx + std::max<uint64_t>(nf, 1));
        SDE_HIP(ctx, hipEventRecord(e2, st));
        if (nf) {
            sde_run r = *fb;
            r.init = SDE_INIT_PHILOX;
            r.step0 = 0;
            r.sync = 0;
            if ((e = jj_integrate_impl(ctx, fpts.data(), (uint32_t)nf, &r, nullptr, nullptr, nullptr, nullptr, fsums,
                                       st)))
                return e;
            SDE_HIP(ctx, hipMemcpyAsync(didx, fidx.data(), nf * sizeof(uint64_t), hipMemcpyHostToDevice, st));
            SDE_HIP(ctx, hipMemcpyAsync(dpaths, fpaths.data(), nf * sizeof(uint32_t), hipMemcpyHostToDevice, st));
        }
        hipLaunchKernelGGL(scan_merge_kernel, dim3((uint32_t)((n + 255) / 256)), dim3(256), 0, st, mean, flag, didx,
                           fsums, dpaths, nf, n, v_out, used);
        SDE_HIP(ctx, hipEventRecord(e3, st));
        SDE_HIP(ctx, hipStreamSynchronize(st));
        if (stats) {
            float a = 0.f, b = 0.f;
            SDE_HIP(ctx, hipEventElapsedTime(&a, e0, e1));
            SDE_HIP(ctx, hipEventElapsedTime(&b, e2, e3));
            stats->n_queries = n;
            stats->n_fallback = nf;
            stats->predict_ms = a;
            stats->fallback_ms = b;
            stats->total_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
        }
        for (hipEvent_t ev : {e0, e1, e2, e3}) (void)hipEventDestroy(ev);
        return sync_and_check(ctx, st);
    } catch (...) {
        return fail(ctx, SDE_ERR_NOMEM, "host allocation failed");
    }
}

int sde_surrogate_save(const sde_surrogate* s, const char* path)
{
    if (!s || !path) return SDE_ERR_INVALID;
    std::vector<float> p(s->P * s->members);
    if (hipDeviceSynchronize() != hipSuccess ||
        hipMemcpy(p.data(), s->params, p.size() * sizeof(float), hipMemcpyDeviceToHost) != hipSuccess)
        return fail(s->ctx, SDE_ERR_DEVICE, "save: cannot read parameters");
    FILE* f = std::fopen(path, "wb");
    if (!f) return fail(s->ctx, SDE_ERR_INVALID, "save: cannot open %s", path);
    const uint32_t hdr[4] = {0x53444553u /* "SDES" */, 1u, (uint32_t)s->widths.size(), s->members};
    bool ok = std::fwrite(hdr, sizeof hdr, 1, f) == 1 &&
              std::fwrite(s->widths.data(), sizeof(uint32_t), s->widths.size(), f) == s->widths.size() &&
              std::fwrite(&s->sc, sizeof s->sc, 1, f) == 1 && std::fwrite(p.data(), sizeof(float), p.size(), f) == p.size();
    ok = (std::fclose(f) == 0) && ok;
    return ok ? SDE_OK : fail(s->ctx, SDE_ERR_DEVICE, "save: write failed");
}

int sde_surrogate_load(sde_ctx* ctx, const char* path, sde_surrogate** out)
{
    if (!ctx || !path || !out) return SDE_ERR_INVALID;
    ctx->last_error.clear();
    FILE* f = std::fopen(path, "rb");
    if (!f) return fail(ctx, SDE_ERR_INVALID, "load: cannot open %s", path);
    uint32_t hdr[4];
    std::vector<uint32_t> widths;
    sde_surrogate_scaling sc;
    int st = SDE_ERR_INVALID;
    sde_surrogate* s = nullptr;
    if (std::fread(hdr, sizeof hdr, 1, f) == 1 && hdr[0] == 0x53444553u && hdr[1] == 1u && hdr[2] >= 2 && hdr[2] <= 9) {
        widths.resize(hdr[2]);
        if (std::fread(widths.data(), sizeof(uint32_t), hdr[2], f) == hdr[2] && std::fread(&sc, sizeof sc, 1, f) == 1 &&
            (st = alloc_surrogate(ctx, widths.data(), hdr[2], hdr[3], &s)) == SDE_OK) {
            std::vector<float> p(s->P * s->members);
            if (std::fread(p.data(), sizeof(float), p.size(), f) == p.size() &&
                hipMemcpy(s->params, p.data(), p.size() * sizeof(float), hipMemcpyHostToDevice) == hipSuccess) {
                s->sc = sc;
                st = SDE_OK;
            } else {
                st = SDE_ERR_INVALID;
            }
        }
    }
    std::fclose(f);
    if (st != SDE_OK) {
        sde_surrogate_destroy(s);
        return st == SDE_ERR_INVALID ? fail(ctx, st, "load: %s is not a surrogate file", path) : st;
    }
    *out = s;
    return SDE_OK;
}

}  // extern "C"
