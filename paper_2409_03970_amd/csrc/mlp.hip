// The learned key-CDF model: an fp32 perceptron 1 -> 32 -> 32 -> 1 with ReLU
// that maps a key to (an estimate of) its rank fraction.  It predicts the
// partition points of the parallel merge (Sec. 2.1); an exact bounded search
// corrects every prediction, so sort results never depend on it.
//
// Kernels:
//   forward      one thread per sample, parameters staged in LDS;
//   gradient     forward and backward of 32 samples at a time on the fp32
//                matrix cores (see cdf_grad_kernel), every workgroup leaving
//                its sums over a fixed set of samples in a row of partials;
//   reduce       one entry's partials added in a fixed order, in training
//                followed at once by the entry's Adam step (Kingma and Ba
//                2015, Algorithm 1).  Every sum has a fixed order, so reruns
//                are bitwise identical;
//   minibatch    sample positions from SplitMix64 (Steele, Lea, Flood 2014)
//                on a counter, key -> x, position/m -> target, drawn by the
//                gradient kernel itself.
#include "hvms.h"
#include "hvms_internal.h"
#include "mlp_common.h"

namespace hvms {

namespace {

constexpr int H = 32;
constexpr int NP = HVMS_CDF_PARAMS;  // 1153
constexpr int CHUNK = 128;           // samples a workgroup takes at a time (4 waves x 32)
constexpr int GRAD_WGS = 256;        // rows of partials at most: one workgroup per CU

__global__ __launch_bounds__(256) void cdf_forward_kernel(const float *__restrict__ p,
                                                          const float *__restrict__ x,
                                                          float *__restrict__ y, int64_t b)
{
    __shared__ float P[NP];
    for (int i = threadIdx.x; i < NP; i += blockDim.x)
        P[i] = p[i];
    __syncthreads();
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < b;
         i += (int64_t)gridDim.x * blockDim.x)
        y[i] = cdf_eval(P, x[i]);
}

// The model sampled on the unit interval: table[i] = F(i / 2^16), i <= 2^16.
// The co-rank predictor reads it instead of evaluating the model per merge
// pair and pass (see cdf_lookup).
__global__ __launch_bounds__(256) void cdf_table_kernel(const float *__restrict__ p,
                                                        float *__restrict__ table)
{
    __shared__ float P[NP];
    for (int i = threadIdx.x; i < NP; i += blockDim.x)
        P[i] = p[i];
    __syncthreads();
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i <= kCdfTableSteps)
        table[i] = cdf_eval(P, (float)i * (1.0f / kCdfTableSteps));
}

typedef float f32x16 __attribute__((ext_vector_type(16)));

// The 32x32 matrix product's operands in a wave (v_mfma_f32_32x32x2_f32):
// A[i][k] and B[k][j] sit in lane 32 k + i and 32 k + j, D[i][j] in register
// r of lane 32 g + j with i = unit(r, g).  The sixteen k steps of a product
// may take the units in any order, so step r takes units unit(r, 0) and
// unit(r, 1): a product's result registers are then the next one's B operand
// as they stand.
__device__ __forceinline__ constexpr int unit(int r, int g) { return 8 * (r >> 2) + 4 * g + (r & 3); }

// Sum over the 32 lanes of each half of the wave, in its last lane.
__device__ __forceinline__ float half_sum(float v)
{
    const auto add = [](float x, int y) { return x + __builtin_bit_cast(float, y); };
    const auto bits = [](float x) { return __builtin_bit_cast(int, x); };
    v = add(v, __builtin_amdgcn_update_dpp(0, bits(v), 0x111, 0xF, 0xF, true));  // row_shr:1
    v = add(v, __builtin_amdgcn_update_dpp(0, bits(v), 0x112, 0xF, 0xF, true));  // row_shr:2
    v = add(v, __builtin_amdgcn_update_dpp(0, bits(v), 0x114, 0xF, 0xF, true));  // row_shr:4
    v = add(v, __builtin_amdgcn_update_dpp(0, bits(v), 0x118, 0xF, 0xF, true));  // row_shr:8
    v = add(v, __builtin_amdgcn_update_dpp(0, bits(v), 0x142, 0xA, 0xF, false)); // row_bcast:15
    return v;
}

// Loss and gradient sums of a fixed share of the samples, one row of NP + 1
// partials per workgroup.
//
// A wave takes 32 samples (lane 32 g + s: sample s): h1 in registers, then
// z2 = W2 h1, dh1 = W2^T dz2 and dW2 += dz2 h1^T as 16 matrix steps each, in
// fp32; only the last needs its operands turned (samples along k), through
// LDS.  The other sums stay in the lanes until the end.  48 matrix steps of
// 64 cycles bound a block of samples: 65,536 samples are two blocks per SIMD,
// 2.6 us.  Before, the per-sample factors of every gradient entry went
// through memory (34 MB for 65,536 samples), one workgroup per 128 samples
// multiplied them on the VALU, and five workgroups added 512 rows of partials
// one after the other: 478 us a training step, now 14 us (11.5 here, 3.9 in the
// reduction; drawing the second block's samples during the first was no faster).
// Apart from the matrix steps a launch's fixed part shows (1,024 samples: 10.5
// us a step): the last sums over the lanes go through LDS, since DPP adds, a
// dependent chain for each of 64 registers, cost 1 us more.  Eight waves of
// half the blocks (the layers' vectors read again for each) take as long at
// 65,536 samples, 12% less at 2^18 and a fifth more at 32,768 and below.
//
// TRAIN: the samples are a minibatch drawn here, position
// i_k = SplitMix64(seed, step * 2^32 + k) mod m of the sorted sample, x its
// key on the unit interval, target i_k / m.
template <bool TRAIN>
__global__ __launch_bounds__(256, 1) void cdf_grad_kernel(
    const float *__restrict__ p, const float *__restrict__ x, const float *__restrict__ tgt,
    const int32_t *__restrict__ sorted, int64_t m, uint64_t seed, uint64_t step, int64_t b,
    float *__restrict__ partial)
{
    constexpr int LD = H + 1;
    __shared__ float turn[4][2][H * LD];  // dz2 and h1, [sample][unit]
    __shared__ float sums[4][NP + 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int s = lane & 31, g = lane >> 5;
    const float *W1 = p, *b1 = p + H, *W2 = p + 2 * H, *b2 = p + 2 * H + H * H;
    const float *W3 = p + 3 * H + H * H;
    const float b3 = p[4 * H + H * H];
    float w1[16], c1[16], c2[16], w3[16], w2a[16], w2t[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int u = unit(r, g);
        w1[r] = W1[u];
        c1[r] = b1[u];
        c2[r] = b2[u];
        w3[r] = W3[u];
        w2a[r] = W2[s * H + u];
        w2t[r] = W2[u * H + s];
    }
    float gw1[16], gb1[16], gb2[16], gw3[16], gb3 = 0.0f, loss = 0.0f;
    f32x16 gw2;
#pragma unroll
    for (int r = 0; r < 16; ++r)
        gw1[r] = gb1[r] = gb2[r] = gw3[r] = gw2[r] = 0.0f;

    for (int64_t i0 = (int64_t)blockIdx.x * CHUNK; i0 < b; i0 += (int64_t)gridDim.x * CHUNK) {
        // lanes past the last sample repeat it with dy = 0: their products with
        // its activations are finite wherever its own gradient is
        const bool in = i0 + wave * 32 + s < b;
        const int64_t i = in ? i0 + wave * 32 + s : b - 1;
        float xi, ti;
        if constexpr (TRAIN) {
            const int64_t k =
                (int64_t)(splitmix64(seed, (step << 32) + (uint64_t)i) % (uint64_t)m);
            xi = key_to_unit(sorted[k]);
            ti = (float)((double)k / (double)m);
        } else {
            xi = x[i];
            ti = tgt[i];
        }
        float h1[16];
        f32x16 z2;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            h1[r] = fmaxf(fmaf(w1[r], xi, c1[r]), 0.0f);
            z2[r] = c2[r];
        }
#pragma unroll
        for (int r = 0; r < 16; ++r)
            z2 = __builtin_amdgcn_mfma_f32_32x32x2f32(w2a[r], h1[r], z2, 0, 0, 0);
        float y = 0.0f;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            y = fmaf(w3[r], fmaxf(z2[r], 0.0f), y);
        y += __shfl_xor(y, 32) + b3;
        const float diff = in ? y - ti : 0.0f;
        const float dy = in ? 2.0f * diff / (float)b : 0.0f;
        gb3 += dy;
        loss = fmaf(diff, diff, loss);
        float dz2[16];
        f32x16 dh;
        float *tz = turn[wave][0], *th = turn[wave][1];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            dz2[r] = in && z2[r] > 0.0f ? dy * w3[r] : 0.0f;
            gw3[r] = fmaf(dy, fmaxf(z2[r], 0.0f), gw3[r]);
            gb2[r] += dz2[r];
            dh[r] = 0.0f;
            tz[s * LD + unit(r, g)] = dz2[r];
            th[s * LD + unit(r, g)] = in ? h1[r] : 0.0f;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r)
            dh = __builtin_amdgcn_mfma_f32_32x32x2f32(w2t[r], dz2[r], dh, 0, 0, 0);
        // one wave's LDS operations complete in order; keep the compiler to it
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int r = 0; r < 16; ++r)
            gw2 = __builtin_amdgcn_mfma_f32_32x32x2f32(tz[(2 * r + g) * LD + s],
                                                      th[(2 * r + g) * LD + s], gw2, 0, 0, 0);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const float dz1 = h1[r] > 0.0f ? dh[r] : 0.0f;
            gw1[r] = fmaf(dz1, xi, gw1[r]);
            gb1[r] += dz1;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }

    // The lanes' sums of the four vectors, turned like the operands above:
    // then half g of the wave adds up vector g, a unit to a lane.
    const auto column_sums = [&](const float(&v0)[16], const float(&v1)[16], int at) {
        float *t = turn[wave][0];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            t[s * LD + unit(r, g)] = v0[r];
            t[H * LD + s * LD + unit(r, g)] = v1[r];
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        float q[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int i = 0; i < H; ++i)
            q[i & 3] += t[(g * H + i) * LD + s];
        sums[wave][at + lane] = (q[0] + q[1]) + (q[2] + q[3]);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    column_sums(gw1, gb1, 0);
    column_sums(gb2, gw3, 2 * H + H * H);
#pragma unroll
    for (int r = 0; r < 16; ++r)
        sums[wave][2 * H + unit(r, g) * H + s] = gw2[r];
    gb3 = half_sum(gb3);
    loss = half_sum(loss);
    if (lane == 31) {
        sums[wave][NP - 1] = gb3;
        sums[wave][NP] = loss;
    }
    __syncthreads();
    for (int j = threadIdx.x; j <= NP; j += 256)
        partial[(int64_t)blockIdx.x * (NP + 1) + j] =
            (sums[0][j] + sums[1][j]) + (sums[2][j] + sums[3][j]);
}

struct AdamArgs {
    float *p, *m, *v;
    float lr, beta1, beta2, eps, bc1, bc2;
};

__device__ __forceinline__ void adam_entry(const AdamArgs &a, int j, float gj)
{
    const float mj = a.beta1 * a.m[j] + (1.0f - a.beta1) * gj;
    const float vj = a.beta2 * a.v[j] + (1.0f - a.beta2) * gj * gj;
    a.m[j] = mj;
    a.v[j] = vj;
    a.p[j] -= a.lr * (mj / a.bc1) / (sqrtf(vj / a.bc2) + a.eps);
}

// Entry j's partials: 16 threads add every sixteenth row, then the sixteen
// sums are added in order.  A workgroup takes 64 entries, so that the rows
// are read in 256-byte pieces and all at once.  ADAM: the entry's Adam step
// follows, and grad and loss are not stored.
template <bool ADAM>
__global__ __launch_bounds__(1024) void cdf_reduce_kernel(const float *__restrict__ partial,
                                                          int rows, int64_t b,
                                                          float *__restrict__ grad,
                                                          float *__restrict__ loss, AdamArgs a)
{
    __shared__ float part[16][64];
    const int e = threadIdx.x & 63, q = threadIdx.x >> 6;
    const int j = blockIdx.x * 64 + e;
    float s = 0.0f;
    if (j <= NP) {
#pragma unroll 16
        for (int c = q; c < rows; c += 16)
            s += partial[(int64_t)c * (NP + 1) + j];
    }
    part[q][e] = s;
    __syncthreads();
    if (q != 0 || j > NP)
        return;
    s = 0.0f;
#pragma unroll
    for (int c = 0; c < 16; ++c)
        s += part[c][e];
    if constexpr (ADAM) {
        if (j < NP)
            adam_entry(a, j, s);
    } else {
        if (j < NP)
            grad[j] = s;
        else
            loss[0] = s / (float)b;
    }
}

__global__ __launch_bounds__(256) void cdf_adam_kernel(const float *__restrict__ g, AdamArgs a)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < NP)
        adam_entry(a, j, g[j]);
}

__global__ void cdf_zero_kernel(float *__restrict__ a, float *__restrict__ b)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j < NP) {
        a[j] = 0.0f;
        b[j] = 0.0f;
    }
}

// out[k] = keys[SplitMix64(seed, k) mod n]: a uniform sample with replacement.
__global__ __launch_bounds__(256) void cdf_sample_kernel(const int32_t *__restrict__ keys, int64_t n,
                                                         int64_t m, uint64_t seed,
                                                         int32_t *__restrict__ out)
{
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < m;
         k += (int64_t)gridDim.x * blockDim.x)
        out[k] = keys[splitmix64(seed, (uint64_t)k) % (uint64_t)n];
}

// Rows of partials of a batch, which are all that its workspace holds.
int grad_rows(int64_t b)
{
    const int64_t chunks = b / CHUNK + (b % CHUNK != 0);
    return (int)(chunks < GRAD_WGS ? chunks : GRAD_WGS);
}

int64_t partial_bytes(int64_t b)
{
    return ((int64_t)grad_rows(b) * (NP + 1) * 4 + 255) & ~(int64_t)255;
}

// What hvms_cdf_backward has always asked for: 132 floats a sample and a row
// of partials for each CHUNK of them.
int64_t backward_bytes(int64_t b)
{
    const int64_t chunks = (b + CHUNK - 1) / CHUNK;
    return ((132 * b * 4 + 255) & ~(int64_t)255) +
           ((chunks * (NP + 1) * 4 + 255) & ~(int64_t)255);
}

AdamArgs adam_args(float *p, float *m, float *v, int step, float lr, float beta1, float beta2,
                   float eps)
{
    return {p, m, v, lr, beta1, beta2, eps, (float)(1.0 - pow((double)beta1, (double)step)),
            (float)(1.0 - pow((double)beta2, (double)step))};
}

int status(hipError_t e)
{
    if (e == hipSuccess)
        return HVMS_OK;
    set_last_hip_error((int)e);
    return HVMS_ERR_HIP;
}

int check(void *ws, size_t bytes, int64_t need)
{
    if (!ws || (int64_t)bytes < need || ((uintptr_t)ws & 255))
        return HVMS_ERR_WORKSPACE;
    return HVMS_OK;
}

}  // namespace

hipError_t launch_cdf_table(const float *params, float *table, hipStream_t s)
{
    hipLaunchKernelGGL(cdf_table_kernel, dim3((kCdfTableSteps + 256) / 256), dim3(256), 0, s,
                       params, table);
    return hipGetLastError();
}

}  // namespace hvms

using namespace hvms;

extern "C" {

int64_t hvms_cdf_param_count(void) { return HVMS_CDF_PARAMS; }

int hvms_cdf_forward(const float *d_params, const float *d_x, float *d_y, int64_t b, void *stream)
{
    if (b < 0 || (b > 0 && (!d_params || !d_x || !d_y)))
        return HVMS_ERR_INVALID_ARG;
    if (b == 0)
        return HVMS_OK;
    int64_t blocks = (b + 255) / 256;
    if (blocks > 8192)
        blocks = 8192;
    hipLaunchKernelGGL(cdf_forward_kernel, dim3((unsigned)blocks), dim3(256), 0,
                       (hipStream_t)stream, d_params, d_x, d_y, b);
    return status(hipGetLastError());
}

int64_t hvms_cdf_workspace_bytes(int64_t b)
{
    if (b < 0)
        return HVMS_ERR_INVALID_ARG;
    return backward_bytes(b);
}

int hvms_cdf_backward(const float *d_params, const float *d_x, const float *d_t, float *d_grad,
                      float *d_loss, int64_t b, void *d_ws, size_t ws_bytes, void *stream)
{
    if (b <= 0 || !d_params || !d_x || !d_t || !d_grad || !d_loss)
        return HVMS_ERR_INVALID_ARG;
    const int st = check(d_ws, ws_bytes, backward_bytes(b));
    if (st)
        return st;
    float *partial = (float *)d_ws;
    const int rows = grad_rows(b);
    hipLaunchKernelGGL(cdf_grad_kernel<false>, dim3(rows), dim3(256), 0, (hipStream_t)stream,
                       d_params, d_x, d_t, nullptr, (int64_t)0, (uint64_t)0, (uint64_t)0, b,
                       partial);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return status(e);
    hipLaunchKernelGGL(cdf_reduce_kernel<false>, dim3((NP + 64) / 64), dim3(1024), 0,
                       (hipStream_t)stream, partial, rows, b, d_grad, d_loss, AdamArgs{});
    return status(hipGetLastError());
}

int hvms_cdf_adam_step(float *d_params, float *d_m, float *d_v, const float *d_grad, int32_t step,
                       float lr, float beta1, float beta2, float eps, void *stream)
{
    if (!d_params || !d_m || !d_v || !d_grad || step < 1 || !(beta1 >= 0.0f && beta1 < 1.0f) ||
        !(beta2 >= 0.0f && beta2 < 1.0f))
        return HVMS_ERR_INVALID_ARG;
    hipLaunchKernelGGL(cdf_adam_kernel, dim3((NP + 255) / 256), dim3(256), 0,
                       (hipStream_t)stream, d_grad,
                       adam_args(d_params, d_m, d_v, step, lr, beta1, beta2, eps));
    return status(hipGetLastError());
}

int64_t hvms_cdf_train_workspace_bytes(int64_t batch)
{
    if (batch <= 0)
        return HVMS_ERR_INVALID_ARG;
    return partial_bytes(batch);
}

int hvms_cdf_train(float *d_params, float *d_m, float *d_v, const int32_t *d_sorted, int64_t m,
                   int64_t batch, int32_t steps, float lr, uint64_t seed, void *d_ws,
                   size_t ws_bytes, void *stream)
{
    if (!d_params || !d_m || !d_v || !d_sorted || m <= 0 || batch <= 0 || steps < 0)
        return HVMS_ERR_INVALID_ARG;
    int st = check(d_ws, ws_bytes, partial_bytes(batch));
    if (st)
        return st;
    hipStream_t s = (hipStream_t)stream;
    float *partial = (float *)d_ws;
    const int rows = grad_rows(batch);
    hipLaunchKernelGGL(cdf_zero_kernel, dim3((NP + 255) / 256), dim3(256), 0, s, d_m, d_v);
    st = status(hipGetLastError());
    for (int step = 1; step <= steps && !st; ++step) {
        hipLaunchKernelGGL(cdf_grad_kernel<true>, dim3(rows), dim3(256), 0, s, d_params, nullptr,
                           nullptr, d_sorted, m, seed, (uint64_t)(step - 1), batch, partial);
        // no Adam step on partials that were not written
        st = status(hipGetLastError());
        if (st)
            return st;
        hipLaunchKernelGGL(cdf_reduce_kernel<true>, dim3((NP + 64) / 64), dim3(1024), 0, s,
                           partial, rows, batch, nullptr, nullptr,
                           adam_args(d_params, d_m, d_v, step, lr, 0.9f, 0.999f, 1e-8f));
        st = status(hipGetLastError());
    }
    return st;
}

int hvms_cdf_sample_i32(const int32_t *d_keys, int64_t n, int64_t m, uint64_t seed,
                        int32_t *d_out, void *stream)
{
    if (n < 0 || m < 0 || (m > 0 && (n == 0 || !d_keys || !d_out)))
        return HVMS_ERR_INVALID_ARG;
    if (m == 0)
        return HVMS_OK;
    int64_t blocks = (m + 255) / 256;
    if (blocks > 16384)
        blocks = 16384;
    hipLaunchKernelGGL(cdf_sample_kernel, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream,
                       d_keys, n, m, seed, d_out);
    return status(hipGetLastError());
}

}  // extern "C"
