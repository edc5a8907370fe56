// surrogate.hip -- training, evaluation and certification of the learned
// K(x, y) surrogate (not part of the paper's method; the series of §2.4
// stays its fallback and the measure of its error).
//
//  * labels: the plain method's K in binary64 (series for x^2+y^2 < 100,
//    3-node rule beyond, §2.4), turned into the target
//    z = asinh(ln(K/G3)/tau);
//  * training step: one workgroup per 64 samples runs the forward pass, the
//    mean-squared-error gradient and the backward pass (the 64x64 products
//    dW = dZ^T A and dA = dZ W on the matrix cores) and writes its partial
//    gradient; the update kernel sums the partials in a fixed order and
//    applies Adam (Kingma & Ba 2015), then rewrites the bfloat16 copies.
//    No atomics: the result does not depend on scheduling;
//  * certification: one workgroup per cell of (x, log10 y) compares the
//    surrogate at a 16x16 lattice of the cell's points (edges included) with
//    the binary64 series and returns the cell's largest relative error.
#include <cmath>

#include "surrogate_dev.h"

namespace hk {
namespace {

using namespace surr;

// The plain method's K(x, y) in binary64 (x >= 0, y > 0): series of the
// Faddeeva function with step 1/2 (A&S 7.1.29) for x^2+y^2 < 100, one exp
// per term; the 3-node rule up to 1e6; the 1-node rule beyond.
__device__ __forceinline__ double plain_K(double x, double y)
{
    const double r = x * x + y * y;
    const double kPiD = 3.14159265358979323846;
    if (r >= 100.0) {
        if (r >= 1.0e6) return (y / kPiD) * (1.7724538509055160 / r);
        const double t1 = 1.2247448713915890, w0 = 1.1816359006036774, w1 = 0.29540897515091934;
        return (y / kPiD) * (w0 / r + w1 / ((x - t1) * (x - t1) + y * y) + w1 / ((x + t1) * (x + t1) + y * y));
    }
    const int N = 2 * (int)ceil(x) + 14;
    double s1 = 0.0, s2 = 0.0, s3 = 0.0;
    for (int n = 1; n <= N; ++n) {
        const double hn = 0.5 * n;
        const double den = hn * hn + y * y;
        s1 += exp(-(hn * hn + x * x)) / den;
        s2 += exp(-(hn + x) * (hn + x)) / den;
        s3 += exp(-(hn - x) * (hn - x)) / den;
    }
    const double ex2 = exp(-x * x);
    const double c2 = cos(2.0 * x * y);
    const double s = sin(x * y);
    return ex2 * erfcx(y) * c2 + (ex2 * s * s / y) / kPiD + (-y * c2 * s1 + 0.5 * y * (s2 + s3)) / kPiD;
}

__device__ double gh3_K(double x, double y)
{
    const double kPiD = 3.14159265358979323846;
    const double t1 = 1.2247448713915890, w0 = 1.1816359006036774, w1 = 0.29540897515091934;
    return (y / kPiD) * (w0 / (x * x + y * y) + w1 / ((x - t1) * (x - t1) + y * y) +
                         w1 / ((x + t1) * (x + t1) + y * y));
}

__global__ __launch_bounds__(256) void label_kernel(const float* __restrict__ x, const float* __restrict__ y,
                                                   int64_t n, float* __restrict__ z)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const double xd = fabs((double)x[i]), yd = (double)y[i];
    const double t = log(plain_K(xd, yd) / gh3_K(xd, yd));
    z[i] = (float)asinh(t / 1e-5);
}

// Parameters (binary32) -> the bfloat16 compute copy; thread per parameter.
__device__ void write_copy(const float* __restrict__ theta, int p, MlpBf16* __restrict__ P)
{
    const float v = theta[p];
    if (p < kOffB1) {
        P->W1[p] = f2bf(v);
    } else if (p < kOffW2) {
        P->b[0][p - kOffB1] = v;
    } else if (p < kOffW5) {
        const int q = p - kOffW2, k = q / (kHid * kHid + kHid), e = q % (kHid * kHid + kHid);
        if (e < kHid * kHid) {
            const int o = e / kHid, i = e % kHid;
            P->W[k][o * kHid + i] = f2bf(v);
            P->WT[k][i * kHid + o] = f2bf(v);
        } else {
            P->b[k + 1][e - kHid * kHid] = v;
        }
    } else if (p < kOffB5) {
        P->w5[p - kOffW5] = f2bf(v);
    } else {
        P->b5 = v;
    }
}

__global__ __launch_bounds__(256) void pack_kernel(const float* __restrict__ theta, MlpBf16* __restrict__ P)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < kNParams) write_copy(theta, p, P);
}

// LDS of the training step (one workgroup per 64 samples)
struct alignas(16) TrainLds {
    float Z[4][kHid][kHid + 1];     // pre-activations of layers 1-4, [s][o] (padded: layer 1 writes a column per lane)
    uint16_t inT[4][kHid][kLd];   // bfloat16 inputs of layers 2-5, [i][s]
    uint16_t act[2][kHid][kLd];   // forward activations [s][i], two in turn
    uint16_t dz[kHid][kLd];       // bfloat16 dZ of the current layer, [s][o]
    uint16_t dzT[kHid][kLd];      // the same, [o][s]
    float f1[kHid], f2[kHid], dout[kHid];
};
constexpr int kTrainWaves = 4;

// Forward, loss and backward of 64 samples; samples j = (base + 64 w + l)
// mod n for 64 w + l < batch (other lanes are padding with zero gradient).
// Loss: mean of w(z) (z_hat - z)^2 with w(z) = 1 / (1 + (z/wscale)^2), or
// w = 1 when wscale = 0.  part_grad[w][p]; part_loss[w] = the weighted sum.
//
// Four wavefronts share the 64 samples, each taking 16 of the 64 outputs of
// every layer (and inputs, on the way back): a step's batch of 4096 is only
// 64 groups of samples, so one wavefront a group left a quarter of the CUs
// with one wavefront each and the rest idle, bound by that wavefront's serial
// chain.  Every value is the same sequence of operations as with one
// wavefront, bit for bit.  (Batch 4096: 36 -> 15 us, of which 8 pass before the
// first layer, in launch and the weights' way from the update of the step
// before.  Sixteen wavefronts, a tile each: 17 us.)
__global__ __launch_bounds__(64 * kTrainWaves) void train_kernel(
    const MlpBf16* __restrict__ P, const float* __restrict__ xs, const float* __restrict__ ys,
    const float* __restrict__ zs, int64_t n, int64_t base, int32_t batch, float wscale,
    float* __restrict__ part_grad, float* __restrict__ part_loss)
{
    __shared__ __align__(16) TrainLds L;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int row = lane & 15, kq = 8 * (lane >> 4);
    const int o = 16 * wave + row;  // this lane's output of the products
    // every weight this lane needs, asked for before anything waits: the update
    // of the step before has just written them elsewhere, and each of the
    // seven layers' passes would wait for its own
    bf16x8 w0[3], w1[3], t0[3], t1[3];
    float bias[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        w0[k] = ld8(P->W[k] + o * kHid + kq);
        w1[k] = ld8(P->W[k] + o * kHid + 32 + kq);
        t0[k] = ld8(P->WT[k] + o * kHid + kq);
        t1[k] = ld8(P->WT[k] + o * kHid + 32 + kq);
        bias[k] = P->b[k + 1][o];
    }
    const float w5 = bf2f(P->w5[o]), b5 = P->b5;
    const int64_t b = (int64_t)blockIdx.x * kHid + lane;
    const bool active = b < batch;
    int64_t j = base + b;
    if (j >= n) j -= n;
    if (j >= n) j %= n;  // (rarely: a batch, or a start, beyond 2 n)
    const float x = active ? fabsf(xs[j]) : 0.0f, y = active ? ys[j] : 1.0f;
    const float zt = active ? zs[j] : 0.0f;
    uint4 w5v[kHid / 8];  // the output layer's weights (wavefront 0)
#pragma unroll
    for (int q = 0; q < kHid / 8; ++q) w5v[q] = reinterpret_cast<const uint4*>(P->w5)[q];
    const float f1 = feature_x(x), f2 = feature_y(y);
    if (wave == 0) {
        L.f1[lane] = f1;
        L.f2[lane] = f2;
    }
    // layer 1 (2 -> 64), a sample per lane, 16 outputs per wavefront
#pragma unroll
    for (int q = 16 * wave; q < 16 * wave + 16; q += 8) {
        uint16_t hv[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const float z = fmaf(bf2f(P->W1[2 * (q + e)]), f1, fmaf(bf2f(P->W1[2 * (q + e) + 1]), f2, P->b[0][q + e]));
            hv[e] = f2bf(silu(z));
            L.Z[0][lane][q + e] = z;
            L.inT[0][q + e][lane] = hv[e];
        }
        uint4 pk;
        pk.x = hv[0] | ((uint32_t)hv[1] << 16);
        pk.y = hv[2] | ((uint32_t)hv[3] << 16);
        pk.z = hv[4] | ((uint32_t)hv[5] << 16);
        pk.w = hv[6] | ((uint32_t)hv[7] << 16);
        *reinterpret_cast<uint4*>(&L.act[0][lane][q]) = pk;
    }
    __syncthreads();
    // layers 2-4 on the matrix cores: every sample, this wavefront's outputs
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const uint16_t* act = &L.act[k & 1][0][0];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const bf16x8 a0 = ld8(act + (16 * m + row) * kLd + kq);
            const bf16x8 a1 = ld8(act + (16 * m + row) * kLd + 32 + kq);
            floatx4 c = {0.0f, 0.0f, 0.0f, 0.0f};
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, w0[k], c, 0, 0, 0);
            c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, w1[k], c, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int s = 16 * m + 4 * (lane >> 4) + r;
                const float z = c[r] + bias[k];
                const uint16_t h = f2bf(silu(z));
                L.act[(k + 1) & 1][s][o] = h;
                L.Z[k + 1][s][o] = z;
                L.inT[k + 1][o][s] = h;
            }
        }
        __syncthreads();
    }
    float* G = part_grad + (int64_t)blockIdx.x * kNParams;
    // output (64 -> 1) and loss, a sample per lane
    if (wave == 0) {
        const uint16_t* act = &L.act[1][0][0];
        float out = b5;
#pragma unroll
        for (int q = 0; q < kHid; q += 8) {
            const uint4 v = *reinterpret_cast<const uint4*>(act + lane * kLd + q);
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
            const uint32_t u[4] = {w5v[q / 8].x, w5v[q / 8].y, w5v[q / 8].z, w5v[q / 8].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                out = fmaf(__uint_as_float(u[e] << 16), __uint_as_float(w[e] << 16), out);
                out = fmaf(__uint_as_float(u[e] & 0xFFFF0000u), __uint_as_float(w[e] & 0xFFFF0000u), out);
            }
        }
        const float res = active ? out - zt : 0.0f;
        const float q = wscale > 0.0f ? zt / wscale : 0.0f;
        const float wgt = 1.0f / fmaf(q, q, 1.0f);
        const float dout = 2.0f * wgt * res / (float)batch;
        L.dout[lane] = dout;
        float sq = wgt * res * res;
        for (int sh = 32; sh > 0; sh >>= 1) sq += __shfl_xor(sq, sh, 64);
        if (lane == 0) part_loss[blockIdx.x] = sq;
        float db5 = dout;
        for (int sh = 32; sh > 0; sh >>= 1) db5 += __shfl_xor(db5, sh, 64);
        if (lane == 0) G[kOffB5] = db5;
    }
    __syncthreads();
    // output layer: dw5[o] = sum_s dout[s] in5[s][o], a lane per output
    if (wave == 3) {
        float g = 0.0f;
#pragma unroll 16
        for (int s = 0; s < kHid; ++s) g = fmaf(L.dout[s], bf2f(L.inT[3][lane][s]), g);
        G[kOffW5 + lane] = g;
    }
    // dH4 in the product layout: dH[s][o] = dout[s] w5[o]
    floatx4 dh[4];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) dh[m][r] = L.dout[16 * m + 4 * (lane >> 4) + r] * w5;
#pragma unroll
    for (int k = 3; k >= 1; --k) {  // layers 4, 3, 2 (weights P->W[k-1])
        // dZ = dH * SiLU'(Z); bias gradient; bfloat16 dZ in both layouts
        float bsum = 0.0f;
#pragma unroll
        for (int m = 0; m < 4; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int s = 16 * m + 4 * (lane >> 4) + r;
                const float dz = dh[m][r] * dsilu(L.Z[k][s][o]);
                bsum += dz;
                const uint16_t h = f2bf(dz);
                L.dz[s][o] = h;
                L.dzT[o][s] = h;
            }
        bsum += __shfl_xor(bsum, 16, 64);
        bsum += __shfl_xor(bsum, 32, 64);
        if (lane < 16) G[kOffB2 + (k - 1) * (kHid * kHid + kHid) + 16 * wave + lane] = bsum;
        __syncthreads();
        // dW[o][i] = sum_s dZ[s][o] in[s][i]:  A = dZ^T (rows o), B = in^T rows i
        {
            const uint16_t* inT = &L.inT[k - 1][0][0];
            const bf16x8 a0 = ld8(&L.dzT[o][kq]);
            const bf16x8 a1 = ld8(&L.dzT[o][32 + kq]);
            float* GW = G + kOffW2 + (k - 1) * (kHid * kHid + kHid);
#pragma unroll
            for (int nn = 0; nn < 4; ++nn) {
                const bf16x8 b0 = ld8(inT + (16 * nn + row) * kLd + kq);
                const bf16x8 b1 = ld8(inT + (16 * nn + row) * kLd + 32 + kq);
                floatx4 c = {0.0f, 0.0f, 0.0f, 0.0f};
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, b0, c, 0, 0, 0);
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, b1, c, 0, 0, 0);
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    GW[(16 * wave + 4 * (lane >> 4) + r) * kHid + 16 * nn + row] = c[r];
            }
        }
        // dH_prev[s][i] = sum_o dZ[s][o] W[o][i]:  A = dZ (rows s), B = W^T rows i
        {
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const bf16x8 a0 = ld8(&L.dz[16 * m + row][kq]);
                const bf16x8 a1 = ld8(&L.dz[16 * m + row][32 + kq]);
                floatx4 c = {0.0f, 0.0f, 0.0f, 0.0f};
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, t0[k - 1], c, 0, 0, 0);
                dh[m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, t1[k - 1], c, 0, 0, 0);
            }
        }
        __syncthreads();  // dz / dzT are rewritten by the next layer
    }
    // layer 1: dZ1 = dH1 SiLU'(Z1), kept in place of Z1
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int s = 16 * m + 4 * (lane >> 4) + r;
            L.Z[0][s][o] = dh[m][r] * dsilu(L.Z[0][s][o]);
        }
    __syncthreads();
    if (wave == 0) {
        float g = 0.0f;
#pragma unroll 16
        for (int s = 0; s < kHid; ++s) g = fmaf(L.Z[0][s][lane], L.f1[s], g);
        G[kOffW1 + 2 * lane] = g;
    } else if (wave == 1) {
        float g = 0.0f;
#pragma unroll 16
        for (int s = 0; s < kHid; ++s) g = fmaf(L.Z[0][s][lane], L.f2[s], g);
        G[kOffW1 + 2 * lane + 1] = g;
    } else if (wave == 2) {
        float g = 0.0f;
#pragma unroll 16
        for (int s = 0; s < kHid; ++s) g += L.Z[0][s][lane];
        G[kOffB1 + lane] = g;
    }
}

// Sum of the per-workgroup partials in workgroup order; thread per parameter.
// (Sixteen loads are in flight before the first is added: one at a time, the
// 64 partials of a batch of 4096 took a memory latency each.)
__device__ inline float sum_partials(const float* __restrict__ part, int32_t n_wg, int p)
{
    float g = 0.0f;
    int w = 0;
    for (; w + 16 <= n_wg; w += 16) {
        float v[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) v[e] = part[(int64_t)(w + e) * kNParams + p];
#pragma unroll
        for (int e = 0; e < 16; ++e) g += v[e];
    }
    for (; w < n_wg; ++w) g += part[(int64_t)w * kNParams + p];
    return g;
}
// The losses of the workgroups, summed in workgroup order by one lane (the
// other lanes of its wavefront load them).
__device__ inline float sum_losses(const float* __restrict__ part_loss, int32_t n_wg)
{
    const int lane = threadIdx.x & 63;
    float s = 0.0f;
    for (int w0 = 0; w0 < n_wg; w0 += 64) {
        const float v = w0 + lane < n_wg ? part_loss[w0 + lane] : 0.0f;
        for (int e = 0; e < min(64, n_wg - w0); ++e)
            s += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), e));
    }
    return s;
}
constexpr int kUpdateThreads = 64;  // a wavefront per workgroup: 200 of them, spread over the CUs

__global__ __launch_bounds__(kUpdateThreads) void adam_kernel(float* __restrict__ theta, float* __restrict__ m,
                                                   float* __restrict__ v, const float* __restrict__ part,
                                                   int32_t n_wg, float lr, float beta1, float beta2, float eps,
                                                   float c1, float c2, MlpBf16* __restrict__ P,
                                                   const float* __restrict__ part_loss, int32_t batch,
                                                   float* __restrict__ loss_out)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (blockIdx.x == 0 && loss_out) {
        const float s = sum_losses(part_loss, n_wg);
        if (p == 0) *loss_out = s / (float)batch;
    }
    if (p >= kNParams) return;
    const float g = sum_partials(part, n_wg, p);
    const float mm = beta1 * m[p] + (1.0f - beta1) * g;
    const float vv = beta2 * v[p] + (1.0f - beta2) * g * g;
    m[p] = mm;
    v[p] = vv;
    theta[p] -= lr * (mm * c1) / (sqrtf(vv * c2) + eps);
    write_copy(theta, p, P);
}

__global__ __launch_bounds__(kUpdateThreads) void reduce_kernel(const float* __restrict__ part, int32_t n_wg,
                                                     float* __restrict__ grad, const float* __restrict__ part_loss,
                                                     int32_t batch, float* __restrict__ loss_out)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (blockIdx.x == 0 && loss_out) {
        const float s = sum_losses(part_loss, n_wg);
        if (p == 0) *loss_out = s / (float)batch;
    }
    if (p < kNParams) grad[p] = sum_partials(part, n_wg, p);
}

// Network output and K_hat at given points; four wavefronts of 64 samples.
__global__ __launch_bounds__(256) void eval_kernel(const MlpBf16* __restrict__ P, const float* __restrict__ xs,
                                                   const float* __restrict__ ys, int64_t n,
                                                   float* __restrict__ z_out, float* __restrict__ K_out)
{
    __shared__ __align__(16) uint16_t act[4][kHid * kLd];
    const int wave = threadIdx.x >> 6;
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    const float x = i < n ? fabsf(xs[i]) : 0.0f, y = i < n ? ys[i] : 1.0f;
    const float z = mlp_forward(P, act[wave], feature_x(x), feature_y(y));
    if (i < n) {
        z_out[i] = z;
        if (K_out) K_out[i] = surrogate_K(x, y, z);
    }
}

// One workgroup per cell c = iy * kCellsX + ix, sampling its 16x16 lattice
// (edges included): thread t takes (i, j) = (t % 16, t / 16),
// x = (ix + i/15) w, log10 y = -4 + (iy + j/15) h; err[c] = the largest
// relative error of K_hat against the binary64 series.  A dense-sampling
// check, not a bound: the network and the method are smooth on the cell's
// scale, and the deployed error is checked on whole bins against the oracle.
constexpr int kCertSide = 16;
__global__ __launch_bounds__(256) void certify_kernel(const MlpBf16* __restrict__ P, double* __restrict__ err)
{
    __shared__ __align__(16) uint16_t act[4][kHid * kLd];
    __shared__ double wmax[4];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int c = blockIdx.x;
    const int ix = c % kCellsX, iy = c / kCellsX;
    const int i = threadIdx.x % kCertSide, j = threadIdx.x / kCertSide;
    const float x = ((float)ix + (float)i / (float)(kCertSide - 1)) * kCellW;
    const float ly = -4.0f + ((float)iy + (float)j / (float)(kCertSide - 1)) * kCellH;
    const float y = exp10f(ly);
    const float z = mlp_forward(P, act[wave], feature_x(x), feature_y(y));
    const double K = (double)surrogate_K(x, y, z);
    const double ref = plain_K((double)x, (double)y);
    double e = fabs(K / ref - 1.0);
    if (!(e == e)) e = 1e300;
    for (int o = 32; o > 0; o >>= 1) e = fmax(e, __shfl_xor(e, o, 64));
    if (lane == 0) wmax[wave] = e;
    __syncthreads();
    if (threadIdx.x == 0) err[c] = fmax(fmax(wmax[0], wmax[1]), fmax(wmax[2], wmax[3]));
}
static_assert(kCertSide * kCertSide == 256, "one lattice point per thread");

}  // namespace

size_t surrogate_params_bytes() { return sizeof(MlpBf16); }
int32_t surrogate_n_params() { return kNParams; }
int32_t surrogate_cells() { return kCellsX * kCellsY; }

hipError_t launch_surrogate_labels(const float* x, const float* y, int64_t n, float* z, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    label_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s>>>(x, y, n, z);
    return hipGetLastError();
}

hipError_t launch_surrogate_pack(const float* theta, void* P, hipStream_t s)
{
    pack_kernel<<<dim3((kNParams + 255) / 256), dim3(256), 0, s>>>(theta, static_cast<MlpBf16*>(P));
    return hipGetLastError();
}

hipError_t launch_surrogate_train_step(const void* P, const float* x, const float* y, const float* z, int64_t n,
                                       int64_t base, int32_t batch, float wscale, float* part_grad,
                                       float* part_loss, hipStream_t s)
{
    const int n_wg = (batch + kHid - 1) / kHid;
    train_kernel<<<dim3(n_wg), dim3(64 * kTrainWaves), 0, s>>>(static_cast<const MlpBf16*>(P), x, y, z, n, base, batch, wscale,
                                                 part_grad, part_loss);
    return hipGetLastError();
}

hipError_t launch_surrogate_adam(float* theta, float* m, float* v, const float* part_grad, int32_t batch,
                                 float lr, float beta1, float beta2, float eps, float c1, float c2, void* P,
                                 const float* part_loss, float* loss_out, hipStream_t s)
{
    const int n_wg = (batch + kHid - 1) / kHid;
    adam_kernel<<<dim3((kNParams + kUpdateThreads - 1) / kUpdateThreads), dim3(kUpdateThreads), 0, s>>>(theta, m, v, part_grad, n_wg, lr, beta1, beta2,
                                                                   eps, c1, c2, static_cast<MlpBf16*>(P),
                                                                   part_loss, batch, loss_out);
    return hipGetLastError();
}

hipError_t launch_surrogate_reduce(const float* part_grad, int32_t batch, float* grad, const float* part_loss,
                                   float* loss_out, hipStream_t s)
{
    const int n_wg = (batch + kHid - 1) / kHid;
    reduce_kernel<<<dim3((kNParams + kUpdateThreads - 1) / kUpdateThreads), dim3(kUpdateThreads), 0, s>>>(part_grad, n_wg, grad, part_loss, batch,
                                                                     loss_out);
    return hipGetLastError();
}

hipError_t launch_surrogate_eval(const void* P, const float* x, const float* y, int64_t n, float* z, float* K,
                                 hipStream_t s)
{
    if (n == 0) return hipSuccess;
    eval_kernel<<<dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s>>>(static_cast<const MlpBf16*>(P), x, y, n, z,
                                                                        K);
    return hipGetLastError();
}

hipError_t launch_surrogate_certify(const void* P, double* err, hipStream_t s)
{
    certify_kernel<<<dim3(kCellsX * kCellsY), dim3(256), 0, s>>>(static_cast<const MlpBf16*>(P), err);
    return hipGetLastError();
}

}  // namespace hk
