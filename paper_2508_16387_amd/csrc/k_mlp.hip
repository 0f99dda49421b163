// k_mlp.hip -- BF16 matrix-core inference and training of the learned
// star-pressure guess, and the guess kernel of the FIVER work queue.
//
// One wavefront evaluates 16 samples at a time with the 16x16x16 BF16 MFMA
// (FP32 accumulation), in the transposed orientation Z^T = W X^T so that the
// output tile of one layer is already the B operand of the next:
//   MFMA lane layout (checked on gfx950): A[i][k] in lane i + 16(k/4),
//   element k%4; B[k][j] in lane j + 16(k/4), element k%4; D[i][j] in lane
//   j + 16(i/4), element i%4.
// Layer 1: Z1^T (64x16) = W1 (64x8, K padded to 16) X^T   -> 4 MFMA
// Layer 2: Z2^T (64x16) = W2 (64x64) H1^T                 -> 16 MFMA
// Layer 3: y (16) = w3 . H2^T + b3                         -> lane sums + shuffles
// Backward (training): dW2 = dZ2^T H1 and dW1 = dZ1^T X accumulate over the
// block's samples in MFMA accumulators (the transposes go through LDS),
// dH1^T = W2^T dZ2^T reuses dZ2^T in place as the B operand.
#include "m2c_device.h"
#include "m2c_internal.h"
#include "m2c_kernels.h"
#include "m2c_mlp.h"
#include "m2c_mlp_infer.h"

namespace m2c {

// Sum over the 16 lanes of this lane's group (lanes with equal lane/16).
__device__ __forceinline__ float group16_sum(float v)
{
    v += __shfl_xor(v, 1);
    v += __shfl_xor(v, 2);
    v += __shfl_xor(v, 4);
    v += __shfl_xor(v, 8);
    return v;
}

// Forward pass of 16 samples held by one wave, the weights in registers.
// xb: this lane's B operand of layer 1 (features 4g..4g+3 of sample l%16,
// zero for g >= 2).  Produces the hidden activations in D layout (h1[c][e] =
// H1^T[16c+4g+e][l%16], same for h2) and y of sample l%16 in every lane of
// that sample.
struct Fwd {
    float h1[4][4], h2[4][4];
    float y;
};

__device__ __forceinline__ void mlp_fwd16(const MlpRegs& w, bf16x4 xb, Fwd& f)
{
    // layer 1
    bf16x4 hb[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const f32x4 z = mfma(w.a1[t], xb, f32x4{0.f, 0.f, 0.f, 0.f});
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float h = tanhf(z[e] + w.b1[t][e]);
            f.h1[t][e] = h;
            hb[t][e] = to_bf16(h);
        }
    }
    // layer 2
    float part = 0.f;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < 4; ++c) z = mfma(w.a2[u][c], hb[c], z);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float v = tanhf(z[e] + w.b2[u][e]);
            f.h2[u][e] = v;
            part += w.w3[u][e] * v;
        }
    }
    // layer 3: sum the four lane groups of each sample
    part += __shfl_xor(part, 16);
    part += __shfl_xor(part, 32);
    f.y = part + w.b3;
}

// This lane's features 4g..4g+3 of sample i (zeros for g >= 2 and beyond
// the samples), and the layer-1 B operand they make.
__device__ __forceinline__ void load_features(const float* __restrict__ X, long long n, long long i, bool live,
                                              float x[4])
{
    const int g = (threadIdx.x & 63) >> 4;
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = live && g < 2 ? X[(4 * g + e) * n + i] : 0.f;
}

__device__ __forceinline__ bf16x4 xb_of(const float x[4])
{
    bf16x4 b;
#pragma unroll
    for (int e = 0; e < 4; ++e) b[e] = to_bf16(x[e]);
    return b;
}

// ---------------------------------------------------------------------------
// Features of n Riemann problems (SoA in [6][n], eos [4][n]) -> X [8][n],
// and, when p* is given, the targets ln((p* - p_lo)/P).
__global__ __launch_bounds__(256) void k_mlp_features(long long n, const double* __restrict__ in,
                                                      const double* __restrict__ eos, const double* __restrict__ ps,
                                                      float* __restrict__ X, float* __restrict__ tg)
{
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x) {
        float x[8];
        double plo, P;
        mlp_features(in[i], in[n + i], in[2 * n + i], eos[i], eos[n + i], in[3 * n + i], in[4 * n + i],
                     in[5 * n + i], eos[2 * n + i], eos[3 * n + i], x, plo, P);
#pragma unroll
        for (int k = 0; k < 8; ++k) X[k * n + i] = x[k];
        if (ps && tg) tg[i] = (float)log((ps[i] - plo) / P);
    }
}

hipError_t launch_mlp_features(long long n, const double* in, const double* eos, const double* ps, float* X,
                               float* tg, hipStream_t s)
{
    long long nb = (n + 255) / 256;
    if (nb > 65536) nb = 65536;
    if (nb < 1) nb = 1;
    hipLaunchKernelGGL(k_mlp_features, dim3((unsigned)nb), dim3(256), 0, s, n, in, eos, ps, X, tg);
    return hipGetLastError();
}

// Inference on n feature vectors X [8][n] -> y [n].  One wave per 16-sample
// chunk (grid-stride); samples past n are computed on zeros and dropped.
__global__ __launch_bounds__(256) void k_mlp_forward(long long n, const float* __restrict__ X,
                                                     const float* __restrict__ P, const uint16_t* __restrict__ wbf,
                                                     float* __restrict__ y)
{
    const int l = threadIdx.x & 63, r = l & 15;
    const long long wave = (blockIdx.x * (long long)blockDim.x + threadIdx.x) >> 6;
    const long long nw = ((long long)gridDim.x * blockDim.x) >> 6;
    if (wave * 16 >= n) return;                                   // wave-uniform
    MlpRegs w;
    mlp_load_regs(P, wbf, w);
    for (long long c = wave; c * 16 < n; c += nw) {
        const long long i = c * 16 + r;
        float x[4];
        load_features(X, n, i, i < n, x);
        Fwd f;
        mlp_fwd16(w, xb_of(x), f);
        if (l < 16 && i < n) y[i] = f.y;
    }
}

hipError_t launch_mlp_forward(long long n, const float* X, const MlpDev& m, float* y, hipStream_t s)
{
    long long nb = (n + 63) / 64;               // 4 waves x 16 samples per block
    if (nb > 1536) nb = 1536;                  // two rounds of the resident blocks, so that the weights are loaded rarely
    if (nb < 1) nb = 1;
    hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned)nb), dim3(256), 0, s, n, X, m.master, m.wbf, y);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Gradient of the mean squared error over samples [i0, i0 + cnt) of a
// minibatch of size B.  A block of four waves takes 64 samples at a time,
// wave w the 16-sample chunk w of the forward pass and of dH1^T = W2^T dZ2^T;
// the operands of the two weight gradients then go through LDS, and wave w
// forms rows 16w..16w+15 of dW2 and dW1 over all 64 samples, so that no sum
// over waves is left for them.  Each block writes its partial gradient (and
// sum of squared errors) to part[block][GRAD_STRIDE]; k_adam / k_grad_sum
// add the blocks up in a fixed order.
//
// What bounds it: a minibatch is a few thousand samples, so the kernel is one
// chain of latencies (weights, two layers of tanh, transposes) on a fraction
// of the chip.  Before, one wave per 64 samples walked four such chains,
// loaded its weights two bytes at a time and added 4801 values per wave
// atomically: 46 us for 4096 samples; now 14 us, of which the 32 tanh of a lane are a third.
constexpr int GRAD_SAMPLES = 64;                   // per block and pass
constexpr int GRAD_PITCH = GRAD_SAMPLES + 4;       // LDS row pitch: 16 rows, 8-byte reads, no bank twice
static_assert(GRAD_SSE == MLP_NPARAM && GRAD_STRIDE >= GRAD_SSE + 1, "gradient partial layout");

__global__ __launch_bounds__(256) void k_mlp_grad(long long i0, long long cnt, long long ntot, float invB,
                                                  const float* __restrict__ X, const float* __restrict__ T,
                                                  const float* __restrict__ P, const uint16_t* __restrict__ wbf,
                                                  float* __restrict__ part)
{
    __shared__ __align__(8) short sA[64 * GRAD_PITCH];      // dZ2^T, then dZ1^T, as [hidden][sample]
    __shared__ __align__(8) short sB[64 * GRAD_PITCH];      // H1^T as [hidden][sample]
    __shared__ __align__(8) short sWT[64 * GRAD_PITCH];     // W2^T as [hidden 1][hidden 2]
    __shared__ __align__(8) short sX[MLP_IN * GRAD_PITCH];  // X as [feature][sample]
    __shared__ float sSum[4][3 * 64 + 2];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63, g = l >> 4, r = l & 15;
    MlpRegs net;
    mlp_load_regs(P, wbf, net);
    {
        // thread t: row t/4 of W2, 16 columns from 16 (t%4)
        const int row = threadIdx.x >> 2, c0 = 16 * (threadIdx.x & 3);
#pragma unroll
        for (int c = 0; c < 16; c += 4) {
            const bf16x4 v = ld_bf16x4(wbf + 512 + row * MLP_H + c0 + c);
#pragma unroll
            for (int e = 0; e < 4; ++e) sWT[(c0 + c + e) * GRAD_PITCH + row] = v[e];
        }
    }
    f32x4 dW2[4], dW1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int v = 0; v < 4; ++v) dW2[v] = f32x4{0.f, 0.f, 0.f, 0.f};
    float gw3[4][4] = {}, gb2[4][4] = {}, gb1[4][4] = {};
    float gb3 = 0.f, err2 = 0.f;
    const short* const row16 = sA + (16 * w + r) * GRAD_PITCH + 4 * g;
    for (long long s0 = (long long)blockIdx.x * GRAD_SAMPLES; s0 < cnt; s0 += (long long)gridDim.x * GRAD_SAMPLES) {
        const long long i = i0 + s0 + 16 * w + r;
        const bool live = i < i0 + cnt;
        float x[4];
        load_features(X, ntot, i, live, x);
        const float ti = live ? T[i] : 0.f;
        const bf16x4 xb = xb_of(x);
        Fwd f;
        mlp_fwd16(net, xb, f);
        const float err = live ? f.y - ti : 0.f, dy = 2.f * err * invB;
        if (l < 16) {
            err2 += err * err;
            gb3 += dy;
        }
        // dZ2^T (D layout), the per-hidden-unit sums, and the LDS operands
        bf16x4 dz2b[4];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float h2 = f.h2[u][e];
                gw3[u][e] += dy * h2;
                const float d = net.w3[u][e] * dy * (1.f - h2 * h2);
                gb2[u][e] += d;
                dz2b[u][e] = to_bf16(d);
            }
        __syncthreads();                           // the pass before has read its operands (and sWT is whole)
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int o = (16 * u + 4 * g + e) * GRAD_PITCH + 16 * w + r;
                sA[o] = dz2b[u][e];
                sB[o] = to_bf16(f.h1[u][e]);
            }
        if (g < 2) {
#pragma unroll
            for (int e = 0; e < 4; ++e) sX[(4 * g + e) * GRAD_PITCH + 16 * w + r] = xb[e];
        }
        // dH1^T = W2^T dZ2^T: A[i][k] = W2^T[16v+i][16c+k], B = dZ2^T tile c
        float dz1[4][4];
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            f32x4 z = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int c = 0; c < 4; ++c)
                z = mfma(*reinterpret_cast<const bf16x4*>(sWT + (16 * v + r) * GRAD_PITCH + 16 * c + 4 * g), dz2b[c], z);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float h1 = f.h1[v][e];
                const float d = z[e] * (1.f - h1 * h1);
                dz1[v][e] = d;
                gb1[v][e] += d;
            }
        }
        __syncthreads();
        // dW2[a][b] += sum_j dZ2^T[a][j] H1^T[b][j], rows a of this wave:
        // A[i][k=j] = sA[16w+i][j], B[k=j][n] = sB[16v+n][j]
#pragma unroll
        for (int q = 0; q < GRAD_SAMPLES / 16; ++q) {
            const bf16x4 a = *reinterpret_cast<const bf16x4*>(row16 + 16 * q);
#pragma unroll
            for (int v = 0; v < 4; ++v)
                dW2[v] = mfma(a, *reinterpret_cast<const bf16x4*>(sB + (16 * v + r) * GRAD_PITCH + 16 * q + 4 * g), dW2[v]);
        }
        __syncthreads();
#pragma unroll
        for (int v = 0; v < 4; ++v)
#pragma unroll
            for (int e = 0; e < 4; ++e) sA[(16 * v + 4 * g + e) * GRAD_PITCH + 16 * w + r] = to_bf16(dz1[v][e]);
        __syncthreads();
        // dW1[a][k] += sum_j dZ1^T[a][j] X[j][k] (columns 8..15 of the tile unused)
#pragma unroll
        for (int q = 0; q < GRAD_SAMPLES / 16; ++q) {
            const bf16x4 a = *reinterpret_cast<const bf16x4*>(row16 + 16 * q);
            dW1 = mfma(a, *reinterpret_cast<const bf16x4*>(sX + (r & 7) * GRAD_PITCH + 16 * q + 4 * g), dW1);
        }
    }
    // per-hidden-unit sums: over the 16 samples of the wave, then its waves
#pragma unroll
    for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int h = 16 * u + 4 * g + e;
            const float s3 = group16_sum(gw3[u][e]), s2 = group16_sum(gb2[u][e]), s1 = group16_sum(gb1[u][e]);
            if (r == 0) {
                sSum[w][h] = s3;
                sSum[w][64 + h] = s2;
                sSum[w][128 + h] = s1;
            }
        }
    gb3 = group16_sum(gb3);
    err2 = group16_sum(err2);
    if (l == 0) {
        sSum[w][192] = gb3;
        sSum[w][193] = err2;
    }
    // D layout: dW2 tile (w,v) element e of lane l = dW2[16w + 4g + e][16v + r]
    float* const out = part + (long long)blockIdx.x * GRAD_STRIDE;
#pragma unroll
    for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int e = 0; e < 4; ++e) out[MLP_OFF_W2 + (16 * w + 4 * g + e) * MLP_H + 16 * v + r] = dW2[v][e];
    if (r < MLP_IN) {
#pragma unroll
        for (int e = 0; e < 4; ++e) out[MLP_OFF_W1 + (16 * w + 4 * g + e) * MLP_IN + r] = dW1[e];
    }
    __syncthreads();
    if (threadIdx.x < 194) {
        const int q = threadIdx.x;
        const float s = (sSum[0][q] + sSum[1][q]) + (sSum[2][q] + sSum[3][q]);
        const int o = q < 64 ? MLP_OFF_W3 + q : (q < 128 ? MLP_OFF_B2 + q - 64 : (q < 192 ? MLP_OFF_B1 + q - 128
                                                                                 : (q == 192 ? MLP_OFF_B3 : GRAD_SSE)));
        out[o] = s;
    }
}

// Sum over the blocks' partial gradients of the parameter this thread's lane
// owns (64 parameters per block; the four waves share the partials), valid
// in wave 0.
__device__ __forceinline__ float grad_total(const float* __restrict__ part, int nblk, int p, float (*sPart)[64])
{
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    float s = 0.f;
    if (p <= GRAD_SSE) {
#pragma unroll 8
        for (int b = w; b < nblk; b += 4) s += part[(long long)b * GRAD_STRIDE + p];
    }
    sPart[w][l] = s;
    __syncthreads();
    return (sPart[0][l] + sPart[1][l]) + (sPart[2][l] + sPart[3][l]);
}

__global__ void k_fill_f32(float* p, long long n, float v)
{
    for (long long i = blockIdx.x * (long long)blockDim.x + threadIdx.x; i < n;
         i += (long long)gridDim.x * blockDim.x)
        p[i] = v;
}

// At most GRAD_MAX_BLOCKS blocks (one per CU; the partials are read back by
// the sum).
int mlp_grad_blocks(long long cnt)
{
    const long long nb = (cnt + GRAD_SAMPLES - 1) / GRAD_SAMPLES;
    return (int)(nb < GRAD_MAX_BLOCKS ? nb : GRAD_MAX_BLOCKS);
}

hipError_t launch_mlp_grad(long long i0, long long cnt, long long ntot, float invB, const float* X, const float* T,
                           const MlpDev& m, float* part, hipStream_t s)
{
    const int nb = mlp_grad_blocks(cnt);
    if (nb < 1) return hipSuccess;
    hipLaunchKernelGGL(k_mlp_grad, dim3(nb), dim3(256), 0, s, i0, cnt, ntot, invB, X, T, m.master, m.wbf, part);
    return hipGetLastError();
}

// grad[0 .. MLP_NPARAM] = the summed gradient, then the sum of squared errors.
__global__ __launch_bounds__(256) void k_grad_sum(const float* __restrict__ part, int nblk, float* __restrict__ grad)
{
    __shared__ float sPart[4][64];
    const int p = blockIdx.x * 64 + (threadIdx.x & 63);
    const float g = grad_total(part, nblk, p, sPart);
    if (threadIdx.x < 64 && p <= GRAD_SSE) grad[p] = g;
}

hipError_t launch_grad_sum(const float* part, int nblk, float* grad, hipStream_t s)
{
    hipLaunchKernelGGL(k_grad_sum, dim3((GRAD_SSE + 64) / 64), dim3(256), 0, s, part, nblk, grad);
    return hipGetLastError();
}

hipError_t launch_fill_f32(float* p, long long n, float v, hipStream_t s)
{
    long long nb = (n + 255) / 256;
    if (nb > 4096) nb = 4096;
    if (nb < 1) nb = 1;
    hipLaunchKernelGGL(k_fill_f32, dim3((unsigned)nb), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

// Adam (Kingma and Ba) on the FP32 master parameters from the blocks' partial
// gradients, then refresh the BF16 copies; the sum of squared errors is added
// to *sse.
__global__ __launch_bounds__(256) void k_adam(float* __restrict__ P, uint16_t* __restrict__ wbf,
                                              float* __restrict__ m, float* __restrict__ v,
                                              const float* __restrict__ part, int nblk, float* __restrict__ sse,
                                              float lr, float b1, float b2, float eps, float c1, float c2)
{
    __shared__ float sPart[4][64];
    const int i = blockIdx.x * 64 + (threadIdx.x & 63);
    const float gi = grad_total(part, nblk, i, sPart);
    if (threadIdx.x >= 64 || i > GRAD_SSE) return;
    if (i == GRAD_SSE) {
        *sse += gi;
        return;
    }
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float p = P[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    P[i] = p;
    if (i < MLP_OFF_B1) wbf[i] = (uint16_t)to_bf16(p);
    else if (i >= MLP_OFF_W2 && i < MLP_OFF_B2) wbf[512 + (i - MLP_OFF_W2)] = (uint16_t)to_bf16(p);
}

hipError_t launch_adam(const MlpDev& md, float* m, float* v, const float* part, int nblk, float* sse, float lr,
                       float b1, float b2, float eps, int step, hipStream_t s)
{
    const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3((GRAD_SSE + 64) / 64), dim3(256), 0, s, md.master, md.wbf, m, v, part, nblk, sse,
                       lr, b1, b2, eps, c1, c2);
    return hipGetLastError();
}

// BF16 copies of the weight matrices from the master parameters.
__global__ void k_mlp_sync_bf16(const float* __restrict__ P, uint16_t* __restrict__ wbf)
{
    for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < MLP_NBF; i += gridDim.x * blockDim.x) {
        const float p = i < 512 ? P[MLP_OFF_W1 + i] : P[MLP_OFF_W2 + i - 512];
        wbf[i] = (uint16_t)to_bf16(p);
    }
}

hipError_t launch_mlp_sync(const MlpDev& m, hipStream_t s)
{
    hipLaunchKernelGGL(k_mlp_sync_bf16, dim3(18), dim3(256), 0, s, m.master, m.wbf);
    return hipGetLastError();
}

// Learned guesses of independent problems (in [6][n], eos [4][n]) for the
// kernel-level solver.
__global__ __launch_bounds__(256) void k_points_guess(long long n, const double* __restrict__ in,
                                                      const double* __restrict__ eos, const MlpDev m,
                                                      double* __restrict__ guess)
{
    const int l = threadIdx.x & 63;
    const long long wave = (blockIdx.x * (long long)blockDim.x + threadIdx.x) >> 6;
    const long long nw = ((long long)gridDim.x * blockDim.x) >> 6;
    if (wave * 64 >= n) return;                                   // wave-uniform
    MlpRegs w;
    mlp_load_regs(m.master, m.wbf, w);
    for (long long c = wave; c * 64 < n; c += nw) {
        const long long i = c * 64 + l;
        float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        double plo = 0.0, P = 1.0;
        bool skip = true;
        if (i < n) {
            const double rL = in[i], uL = in[n + i], pL = in[2 * n + i], rR = in[3 * n + i], uR = in[4 * n + i],
                         pR = in[5 * n + i];
            const double gL = eos[i], pcL = eos[n + i], gR = eos[2 * n + i], pcR = eos[3 * n + i];
            skip = acoustic_suffices(rL, uL, pL, gL, pcL, rR, uR, pR, gR, pcR);
            if (!skip) mlp_features(rL, uL, pL, gL, pcL, rR, uR, pR, gR, pcR, x, plo, P);
        }
        const double gs = guess64(w, x, plo, P, skip);
        if (i < n) guess[i] = gs;
    }
}

hipError_t launch_points_guess(long long n, const double* in, const double* eos, const MlpDev& m, double* guess,
                               hipStream_t s)
{
    long long nb = (n + 255) / 256;
    if (nb > 4096) nb = 4096;
    if (nb < 1) nb = 1;
    hipLaunchKernelGGL(k_points_guess, dim3((unsigned)nb), dim3(256), 0, s, n, in, eos, m, guess);
    return hipGetLastError();
}

}  // namespace m2c
