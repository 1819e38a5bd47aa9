// gf_mlp.hip -- the launch-config predictor: a 3-layer FP32 MLP
// (8 -> 64 -> ReLU -> 64 -> ReLU -> 32) with hand-written forward, backward,
// masked-MSE loss and Adam kernels, plus a host forward pass for inference
// at launch time. FP32 VALU arithmetic: the network is tiny and latency-bound,
// nothing here is worth a matrix core.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>

#include "gf_internal.h"

namespace gf {

constexpr int kIn = GF_MLP_IN;
constexpr int kH = GF_MLP_HIDDEN;
constexpr int kOut = GF_MLP_OUT;
// parameter layout: W1[kH][kIn] b1[kH] W2[kH][kH] b2[kH] W3[kOut][kH] b3[kOut]
constexpr int kOffW1 = 0;
constexpr int kOffB1 = kOffW1 + kH * kIn;
constexpr int kOffW2 = kOffB1 + kH;
constexpr int kOffB2 = kOffW2 + kH * kH;
constexpr int kOffW3 = kOffB2 + kH;
constexpr int kOffB3 = kOffW3 + kOut * kH;
constexpr int kNParams = kOffB3 + kOut;
static_assert(kNParams == GF_MLP_NPARAMS, "parameter count");

constexpr int kMlpThreads = 512;      // eight wavefronts, two samples each
constexpr int kSamplesPerBlock = 16;
constexpr int kWaveSamples = kSamplesPerBlock / (kMlpThreads / kWave);
constexpr int kPitch = kH + 4;        // LDS row of W2 and W3: lanes read their rows 16 bytes at a time without conflicts
constexpr int kSumThreads = 64;       // k_mlp_update: one wavefront per workgroup
constexpr int kSumLoads = 48;         // partial rows a thread has in flight
constexpr int kLossParts = 32;        // partial sums of the loss, over 256 elements each per turn
constexpr int kLossSpan = 256;
constexpr int kLossLoads = 48;        // loads in flight per thread

// A kernel argument may be aligned to 4 bytes only.
typedef float gf_f4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float gf_f4 __attribute__((ext_vector_type(4)));

// What a wavefront's lanes wrote to LDS can be read by its other lanes.
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// *loss = inv_norm * the partial sums in order.
__device__ __forceinline__ void loss_final(const float *__restrict__ part, float inv_norm, float *__restrict__ loss)
{
    float p[kLossParts];
#pragma unroll
    for (int i = 0; i < kLossParts; ++i)
        p[i] = part[i];
    float acc = 0.0f;
#pragma unroll
    for (int i = 0; i < kLossParts; ++i)
        acc += p[i];
    *loss = acc * inv_norm;
}

// Partial sum `b` of sum m (y - t)^2, by T threads (one wavefront, or four): 256
// strands of elements b * 256 + strand + i * 32 * 256, each thread 256 / T of
// them, halved pairwise. The sum does not depend on T.
template <int T>
__device__ __forceinline__ void loss_part(const float *__restrict__ y, const float *__restrict__ tgt,
                                          const float *__restrict__ mask, int64_t count, int b,
                                          float *__restrict__ part)
{
    constexpr int Q = kLossSpan / T;             // strands of a thread
    constexpr int R = kLossLoads / (3 * Q);      // turns in flight
    const int tid = threadIdx.x;
    float acc[Q] = {};
    for (int64_t base = (int64_t)b * kLossSpan; base < count; base += R * kLossParts * kLossSpan) {
        float yv[R][Q], tv[R][Q], mv[R][Q];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int64_t i = base + r * kLossParts * kLossSpan + q * T + tid;
                const int64_t at = i < count ? i : count - 1;
                yv[r][q] = y[at];
                tv[r][q] = tgt[at];
                mv[r][q] = mask[at];
            }
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const int64_t i = base + r * kLossParts * kLossSpan + q * T + tid;
                const float d = yv[r][q] - tv[r][q];
                const float t = mv[r][q] * d * d;
                acc[q] = i < count ? acc[q] + t : acc[q];
            }
    }
    float s;
    if constexpr (T == kWave) {
        s = (acc[0] + acc[2]) + (acc[1] + acc[3]);
    } else {
        __shared__ float s_acc[kLossSpan];
        s_acc[tid] = acc[0];
        __syncthreads();
        const int l = tid & (kWave - 1);
        s = (s_acc[l] + s_acc[l + 2 * kWave]) + (s_acc[l + kWave] + s_acc[l + 3 * kWave]);
    }
#pragma unroll
    for (int w = kWave / 2; w > 0; w >>= 1)
        s += __shfl_down(s, w, kWave);
    if (tid == 0)
        part[b] = s;
}

// Forward and (or) backward pass. Workgroup b takes the 16 samples from
// 16 b, a wavefront two of them at once: lane j computes hidden unit j of
// both, W2 and W3 coming from LDS, the other units' values broadcast
// from there. The backward pass of the masked MSE
// L = sum m (y - t)^2 * inv_norm keeps the 16 samples' activations and
// deltas in LDS; then every thread adds its parameters' gradients over the
// samples, in order, into the workgroup's row part[b][kNParams], and
// k_mlp_update adds the rows in order: gradients are deterministic.
// FWD computes z1, z2 (stored where given) and y; without it the backward
// pass reads them. Both together leave z1 and z2 in the registers.
// Every sum has the order of the serial loop over its index. Bound by
// latency and issue: a workgroup per 16 samples leaves one on a CU at 4,096
// samples. With one wavefront per 16 samples, one sample at a time, forward
// took 28.8 us and backward 36.6 at 4,000 samples; the two together now take
// 11 (14 with four wavefronts of four samples: the LDS reads of one wavefront
// per SIMD are not hidden).
// A workgroup past the samples' closes the previous epoch's loss.
template <bool FWD, bool BWD>
__global__ void __launch_bounds__(kMlpThreads) k_mlp_pass(
    const float *__restrict__ P, const float *__restrict__ feats, float *__restrict__ z1_, float *__restrict__ z2_,
    float *__restrict__ y_, const float *__restrict__ tgt, const float *__restrict__ mask, int32_t batch,
    float inv_norm, float *__restrict__ part, const float *__restrict__ lpart, float *__restrict__ loss)
{
    __shared__ __align__(16) float s_w2[kH * kPitch], s_w3[kOut * kPitch];
    __shared__ __align__(16) float s_f[kSamplesPerBlock][kIn];
    __shared__ __align__(16) float s_a1[kSamplesPerBlock][kH], s_a2[kSamplesPerBlock][kH];
    __shared__ __align__(16) float s_dz1[kSamplesPerBlock][kH], s_dz2[kSamplesPerBlock][kH];
    __shared__ __align__(16) float s_dy[kSamplesPerBlock][kOut];
    const int tid = threadIdx.x, j = tid & (kWave - 1);
    const int s0 = blockIdx.x * kSamplesPerBlock;
    if (s0 >= batch) {
        if (tid == 0)
            loss_final(lpart, inv_norm, loss);
        return;
    }
    const int ns = batch - s0 < kSamplesPerBlock ? batch - s0 : kSamplesPerBlock;
#pragma unroll
    for (int q = 0; q < kH * kH / 4 / kMlpThreads; ++q) {
        const int e = 4 * (q * kMlpThreads + tid);
        *(gf_f4 *)(s_w2 + e / kH * kPitch + e % kH) = *(const gf_f4u *)(P + kOffW2 + e);
    }
#pragma unroll
    for (int q = 0; q < kOut * kH / 4 / kMlpThreads; ++q) {
        const int e = 4 * (q * kMlpThreads + tid);
        *(gf_f4 *)(s_w3 + e / kH * kPitch + e % kH) = *(const gf_f4u *)(P + kOffW3 + e);
    }
    if (tid < kSamplesPerBlock * kIn) {
        const int s = tid / kIn < ns ? tid / kIn : ns - 1;
        s_f[tid / kIn][tid % kIn] = feats[(int64_t)(s0 + s) * kIn + tid % kIn];
    }
    // the wavefront's samples: m0, m0 + 1 of the workgroup, those past the
    // last one computed on its values and not used
    const int m0 = __builtin_amdgcn_readfirstlane(tid / kWave) * kWaveSamples;
    int64_t g[kWaveSamples];
#pragma unroll
    for (int i = 0; i < kWaveSamples; ++i)
        g[i] = s0 + (m0 + i < ns ? m0 + i : ns - 1);
    float z1[kWaveSamples], z2[kWaveSamples];
    if constexpr (FWD) {
        gf_f4u w1[kIn / 4];
#pragma unroll
        for (int k = 0; k < kIn / 4; ++k)
            w1[k] = *(const gf_f4u *)(P + kOffW1 + j * kIn + 4 * k);
        const float b1 = P[kOffB1 + j], b2 = P[kOffB2 + j], b3 = P[kOffB3 + j % kOut];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kWaveSamples; ++i) {
            z1[i] = b1;
#pragma unroll
            for (int k = 0; k < kIn; ++k)
                z1[i] += w1[k / 4][k % 4] * s_f[m0 + i][k];
            if (z1_ && m0 + i < ns)
                z1_[g[i] * kH + j] = z1[i];
            s_a1[m0 + i][j] = z1[i] > 0.0f ? z1[i] : 0.0f;
            z2[i] = b2;
        }
        wave_sync();
#pragma unroll 4
        for (int k = 0; k < kH; k += 4) {
            const gf_f4 w = *(const gf_f4 *)(s_w2 + j * kPitch + k);
#pragma unroll
            for (int i = 0; i < kWaveSamples; ++i) {
                const gf_f4 a = *(const gf_f4 *)&s_a1[m0 + i][k];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    z2[i] += w[q] * a[q];
            }
        }
#pragma unroll
        for (int i = 0; i < kWaveSamples; ++i) {
            if (z2_ && m0 + i < ns)
                z2_[g[i] * kH + j] = z2[i];
            s_a2[m0 + i][j] = z2[i] > 0.0f ? z2[i] : 0.0f;
        }
        wave_sync();
        // outputs: half the lanes per sample
        const int c = j % kOut, h = j / kOut;
        float o[kWaveSamples / 2];
#pragma unroll
        for (int i = 0; i < kWaveSamples / 2; ++i)
            o[i] = b3;
#pragma unroll 4
        for (int k = 0; k < kH; k += 4) {
            const gf_f4 w = *(const gf_f4 *)(s_w3 + c * kPitch + k);
#pragma unroll
            for (int i = 0; i < kWaveSamples / 2; ++i) {
                const gf_f4 a = *(const gf_f4 *)&s_a2[m0 + 2 * i + h][k];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    o[i] += w[q] * a[q];
            }
        }
#pragma unroll
        for (int i = 0; i < kWaveSamples / 2; ++i) {
            const int m = m0 + 2 * i + h;
            if (m < ns)
                y_[(int64_t)(s0 + m) * kOut + c] = o[i];
            if constexpr (BWD) {
                const int64_t at = (int64_t)(s0 + (m < ns ? m : ns - 1)) * kOut + c;
                s_dy[m][c] = 2.0f * mask[at] * (o[i] - tgt[at]) * inv_norm;
            }
        }
    } else {
        const int c = j % kOut, h = j / kOut;
#pragma unroll
        for (int i = 0; i < kWaveSamples; ++i) {
            z1[i] = z1_[g[i] * kH + j];
            z2[i] = z2_[g[i] * kH + j];
            s_a1[m0 + i][j] = z1[i] > 0.0f ? z1[i] : 0.0f;
            s_a2[m0 + i][j] = z2[i] > 0.0f ? z2[i] : 0.0f;
        }
#pragma unroll
        for (int i = 0; i < kWaveSamples / 2; ++i) {
            const int m = m0 + 2 * i + h;
            const int64_t at = (int64_t)(s0 + (m < ns ? m : ns - 1)) * kOut + c;
            s_dy[m][c] = 2.0f * mask[at] * (y_[at] - tgt[at]) * inv_norm;
        }
        __syncthreads();
    }
    if constexpr (BWD) {
        wave_sync();
        // dz2_j = relu'(z2_j) * sum_c W3[c][j] dy_c, then dz1 likewise from W2 and dz2
        float da[kWaveSamples] = {};
#pragma unroll 4
        for (int c = 0; c < kOut; c += 4) {
            float w[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                w[q] = s_w3[(c + q) * kPitch + j];
#pragma unroll
            for (int i = 0; i < kWaveSamples; ++i) {
                const gf_f4 d = *(const gf_f4 *)&s_dy[m0 + i][c];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    da[i] += w[q] * d[q];
            }
        }
#pragma unroll
        for (int i = 0; i < kWaveSamples; ++i) {
            s_dz2[m0 + i][j] = z2[i] > 0.0f ? da[i] : 0.0f;
            da[i] = 0.0f;
        }
        wave_sync();
#pragma unroll 4
        for (int u = 0; u < kH; u += 4) {
            float w[4];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                w[q] = s_w2[(u + q) * kPitch + j];
#pragma unroll
            for (int i = 0; i < kWaveSamples; ++i) {
                const gf_f4 d = *(const gf_f4 *)&s_dz2[m0 + i][u];
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    da[i] += w[q] * d[q];
            }
        }
#pragma unroll
        for (int i = 0; i < kWaveSamples; ++i)
            s_dz1[m0 + i][j] = z1[i] > 0.0f ? da[i] : 0.0f;
        __syncthreads();
        // gradients: a thread holds 2 x 4 of W2, four of W3, one of W1 and
        // (the first 160) a bias
        const int r3 = tid / 16, r2 = 2 * r3, k4 = tid % 16 * 4, r1 = tid / kIn, k1 = tid % kIn;
        const float *bias = tid < kH ? &s_dz1[0][tid] : tid < 2 * kH ? &s_dz2[0][tid - kH] : &s_dy[0][tid % kOut];
        const int bstep = tid < 2 * kH ? kH : kOut;
        gf_f4 gw2[2] = {}, gw3 = {};
        float gw1 = 0.0f, gb = 0.0f;
#pragma unroll 4
        for (int s = 0; s < ns; ++s) {
            const gf_f4 a1 = *(const gf_f4 *)&s_a1[s][k4], a2 = *(const gf_f4 *)&s_a2[s][k4];
            const float d20 = s_dz2[s][r2], d21 = s_dz2[s][r2 + 1], d3 = s_dy[s][r3];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                gw2[0][q] += d20 * a1[q];
                gw2[1][q] += d21 * a1[q];
                gw3[q] += d3 * a2[q];
            }
            gw1 += s_dz1[s][r1] * s_f[s][k1];
            gb += bias[s * bstep];
        }
        float *row = part + (int64_t)blockIdx.x * kNParams;
        *(gf_f4 *)(row + kOffW2 + r2 * kH + k4) = gw2[0];
        *(gf_f4 *)(row + kOffW2 + (r2 + 1) * kH + k4) = gw2[1];
        *(gf_f4 *)(row + kOffW3 + r3 * kH + k4) = gw3;
        row[kOffW1 + r1 * kIn + k1] = gw1;
        if (tid < 2 * kH + kOut)
            row[tid < kH ? kOffB1 + tid : tid < 2 * kH ? kOffB2 + tid - kH : kOffB3 + tid - 2 * kH] = gb;
    }
}
static_assert(kMlpThreads == 8 * kH && kIn == 8 && kOut == kH / 2, "the gradient tiles of k_mlp_pass");
static_assert(kNParams % 4 == 0 && kOffW2 % 4 == 0 && kOffW3 % 4 == 0, "16-byte stores of the partial rows");

// Adam (Kingma & Ba): m = b1 m + (1-b1) g; v = b2 v + (1-b2) g^2;
// p -= lr * (m / (1 - b1^t)) / (sqrt(v / (1 - b2^t)) + eps).
struct AdamStep {
    float lr, b1, b2, eps, c1, c2;
};

__device__ __forceinline__ void adam_update(const AdamStep &a, float gi, float *p, float *m, float *v, int i)
{
    const float mi = a.b1 * m[i] + (1.0f - a.b1) * gi;
    const float vi = a.b2 * v[i] + (1.0f - a.b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    p[i] -= a.lr * (mi / a.c1) / (sqrtf(vi / a.c2) + a.eps);
}

__global__ void k_adam(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m,
                       float *__restrict__ v, int32_t n, AdamStep a)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n)
        adam_update(a, g[i], p, m, v, i);
}

// Gradient of one parameter per thread: the workgroups' partial rows added in
// order, stored (g) or, in training, given to Adam at once. Bound by the
// latency of the rows, which the pass before left in other XCDs' part of the
// memory: 48 of them are in flight per thread, and one wavefront per
// workgroup spreads the parameters over 107 CUs. One row at a time took 57.5
// us at 4,000 samples (250 rows); with Adam and the loss's partial sums
// (workgroups past the parameters') this takes 7.
template <bool ADAM>
__global__ void __launch_bounds__(kSumThreads) k_mlp_update(const float *__restrict__ part, int32_t nblocks,
                                                            float *__restrict__ g, float *__restrict__ p,
                                                            float *__restrict__ m, float *__restrict__ v, AdamStep a,
                                                            const float *__restrict__ y,
                                                            const float *__restrict__ tgt,
                                                            const float *__restrict__ mask, int64_t count,
                                                            float *__restrict__ lpart)
{
    constexpr int kSumBlocks = (kNParams + kSumThreads - 1) / kSumThreads;
    if (ADAM && blockIdx.x >= kSumBlocks) {
        loss_part<kWave>(y, tgt, mask, count, blockIdx.x - kSumBlocks, lpart);
        return;
    }
    const int i = blockIdx.x * kSumThreads + threadIdx.x;
    if (i >= kNParams)
        return;
    float acc = 0.0f;
    for (int b = 0; b < nblocks; b += kSumLoads) {
        float t[kSumLoads];
#pragma unroll
        for (int q = 0; q < kSumLoads; ++q)
            t[q] = part[(int64_t)(b + q < nblocks ? b + q : nblocks - 1) * kNParams + i];
#pragma unroll
        for (int q = 0; q < kSumLoads; ++q)
            if (b + q < nblocks)
                acc += t[q];
    }
    if constexpr (ADAM)
        adam_update(a, acc, p, m, v, i);
    else
        g[i] = acc;
}

// Masked MSE: partial sums of m (y - t)^2, summed in order by one thread of the
// last launch. Alone on the chip a part takes four wavefronts: with one,
// 50,000 samples took 47 us, 18 with four.
__global__ void __launch_bounds__(kLossSpan) k_mlp_loss_part(const float *__restrict__ y, const float *__restrict__ tgt,
                                                         const float *__restrict__ mask, int64_t count,
                                                         float *__restrict__ part)
{
    loss_part<kLossSpan>(y, tgt, mask, count, blockIdx.x, part);
}

__global__ void k_mlp_loss_final(const float *__restrict__ part, float inv_norm, float *__restrict__ loss)
{
    if (threadIdx.x == 0 && blockIdx.x == 0)
        loss_final(part, inv_norm, loss);
}

int mlp_blocks(int32_t batch) { return (batch + kSamplesPerBlock - 1) / kSamplesPerBlock; }

namespace {

constexpr int kUpdateBlocks = (kNParams + kSumThreads - 1) / kSumThreads;

AdamStep adam_step(float lr, float b1, float b2, float eps, int32_t t)
{
    return {lr, b1, b2, eps, 1.0f - std::pow(b1, (float)t), 1.0f - std::pow(b2, (float)t)};
}

}  // namespace

hipError_t launch_mlp_forward(const float *P, const float *feats, int32_t batch, float *y, float *z1, float *z2,
                              hipStream_t s)
{
    if (batch <= 0)
        return hipSuccess;
    hipLaunchKernelGGL((k_mlp_pass<true, false>), dim3(mlp_blocks(batch)), dim3(kMlpThreads), 0, s, P, feats, z1, z2,
                       y, nullptr, nullptr, batch, 0.0f, nullptr, nullptr, nullptr);
    return hipGetLastError();
}

hipError_t launch_mlp_backward(const float *P, const float *feats, const float *z1, const float *z2, const float *y,
                               const float *tgt, const float *mask, int32_t batch, float inv_norm, float *part,
                               float *grads, hipStream_t s)
{
    const int nb = mlp_blocks(batch);
    hipLaunchKernelGGL((k_mlp_pass<false, true>), dim3(nb), dim3(kMlpThreads), 0, s, P, feats, (float *)z1,
                       (float *)z2, (float *)y, tgt, mask, batch, inv_norm, part, nullptr, nullptr);
    hipLaunchKernelGGL((k_mlp_update<false>), dim3(kUpdateBlocks), dim3(kSumThreads), 0, s, part, nb, grads, nullptr,
                       nullptr, nullptr, AdamStep{}, nullptr, nullptr, nullptr, (int64_t)0, nullptr);
    return hipGetLastError();
}

hipError_t launch_mlp_loss(const float *y, const float *tgt, const float *mask, int64_t count, float inv_norm,
                           float *part, float *loss, hipStream_t s)
{
    hipLaunchKernelGGL(k_mlp_loss_part, dim3(kLossParts), dim3(kLossSpan), 0, s, y, tgt, mask, count, part);
    hipLaunchKernelGGL(k_mlp_loss_final, dim3(1), dim3(kWave), 0, s, part, inv_norm, loss);
    return hipGetLastError();
}

// Two launches per epoch: the forward and backward pass, then gradients, Adam
// and the loss's partial sums. The next epoch's first launch (the last one's
// k_mlp_loss_final) closes the loss. Seven launches took 134 us an epoch at
// 4,000 samples.
hipError_t launch_mlp_train(float *P, float *m, float *v, const float *feats, const float *tgt, const float *mask,
                            int32_t batch, float inv_norm, int32_t epochs, float lr, float *part, float *y,
                            float *lpart, float *loss_hist, hipStream_t s)
{
    const int nb = mlp_blocks(batch);
    for (int32_t e = 0; e < epochs; ++e) {
        const bool close = loss_hist && e > 0;
        hipLaunchKernelGGL((k_mlp_pass<true, true>), dim3(nb + (close ? 1 : 0)), dim3(kMlpThreads), 0, s, P, feats,
                           nullptr, nullptr, y, tgt, mask, batch, inv_norm, part, lpart,
                           close ? loss_hist + e - 1 : nullptr);
        hipLaunchKernelGGL((k_mlp_update<true>), dim3(kUpdateBlocks + (loss_hist ? kLossParts : 0)),
                           dim3(kSumThreads), 0, s, part, nb, nullptr, P, m, v,
                           adam_step(lr, 0.9f, 0.999f, 1e-8f, e + 1), y, tgt, mask, (int64_t)batch * kOut, lpart);
        const hipError_t r = hipGetLastError();
        if (r != hipSuccess)
            return r;
    }
    if (loss_hist && epochs > 0)
        hipLaunchKernelGGL(k_mlp_loss_final, dim3(1), dim3(kWave), 0, s, lpart, inv_norm, loss_hist + epochs - 1);
    return hipGetLastError();
}

hipError_t launch_adam(float *p, const float *g, float *m, float *v, int32_t n, float lr, float b1, float b2, float eps,
                       int32_t t, hipStream_t s)
{
    hipLaunchKernelGGL(k_adam, dim3((n + 255) / 256), dim3(256), 0, s, p, g, m, v, n, adam_step(lr, b1, b2, eps, t));
    return hipGetLastError();
}

// Host forward pass (FP32, same layer order as the kernel) for single
// launch-time predictions without a device round trip.
void mlp_forward_host(const float *P, const float *f, float *out)
{
    float a1[kH], a2[kH];
    for (int j = 0; j < kH; ++j) {
        float z = P[kOffB1 + j];
        for (int k = 0; k < kIn; ++k)
            z += P[kOffW1 + j * kIn + k] * f[k];
        a1[j] = z > 0.0f ? z : 0.0f;
    }
    for (int j = 0; j < kH; ++j) {
        float z = P[kOffB2 + j];
        for (int k = 0; k < kH; ++k)
            z += P[kOffW2 + j * kH + k] * a1[k];
        a2[j] = z > 0.0f ? z : 0.0f;
    }
    for (int c = 0; c < kOut; ++c) {
        float o = P[kOffB3 + c];
        for (int k = 0; k < kH; ++k)
            o += P[kOffW3 + c * kH + k] * a2[k];
        out[c] = o;
    }
}

}  // namespace gf
