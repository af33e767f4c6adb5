// Learned troubled-cell / AMR indicator for gfx950: a 16 -> 64 -> 64 -> 1 ReLU
// network with BF16 weights, MSE loss and Adam on FP32 master weights.
// Inference multiplies BF16 operands (weights, inputs, first hidden layer) on
// the matrix cores with FP32 accumulation; training runs in FP32 arithmetic on
// the BF16 weights.
//
// Parameter vector (5313 floats): W1[64][16], b1[64], W2[64][64], b2[64],
// W3[64], b3 (W[j][k]: output unit j, input k).  The device keeps the FP32
// masters, Adam's moments and a BF16 copy (round to nearest even) that the
// forward and backward passes read; the gradient is taken at the BF16 weights
// and applied to the masters.
//
//  k_mlp_forward   inference on the matrix cores (BF16 products, FP32
//                  accumulation), 32 samples per wave
//  k_mlp_grad      64 samples per pass and four waves, every product of the
//                  forward and backward pass on the matrix cores in FP32; the
//                  weight gradients stay in their accumulators over the
//                  block's passes; one partial row per block
//  k_mlp_update    16 threads per parameter: sums the block partials in a fixed
//                  order (deterministic), Adam step, new BF16 copy
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <string>

#include "dgidp_internal.h"
#include "dgidp_mlp_dev.h"

namespace dgidp {

namespace {

using namespace mlp;

constexpr int kRow = kNP + 1;   // partial row: gradient, then the loss sum
constexpr int kGS = 64;         // samples per pass of the gradient kernel
constexpr int kMaxGradBlocks = 256;  // one per compute unit (107 of its 160 KB of LDS each)

__global__ __launch_bounds__(256) void k_mlp_round(const float* __restrict__ master,
                                                   uint16_t* __restrict__ wb)
{
    const int p = blockIdx.x * blockDim.x + threadIdx.x;
    if (p < kNP) wb[p] = bf16_rne(master[p]);
}

// inference: 32 samples per wave (the matrix-core pass of forward32), four
// waves per block sharing one LDS copy of the weights; each wave loops over
// its tiles
__global__ __launch_bounds__(256) void k_mlp_forward(const float* __restrict__ x, int B,
                                                     const uint16_t* __restrict__ wb,
                                                     float* __restrict__ y)
{
    __shared__ __align__(16) LdsWeights sW;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int c = lane & 31, hf = lane >> 5;
    stage_weights(sW, wb, threadIdx.x, 256);
    __syncthreads();
    const int ntiles = (B + 31) / 32;
#pragma unroll 1
    for (int tile = blockIdx.x * 4 + wv; tile < ntiles; tile += gridDim.x * 4) {
        const int s = tile * 32 + c;
        float v[8];
        if (s < B) {
            const float4 p0 = *(const float4*)(x + (size_t)s * kNin + hf * 8);
            const float4 p1 = *(const float4*)(x + (size_t)s * kNin + hf * 8 + 4);
            v[0] = p0.x; v[1] = p0.y; v[2] = p0.z; v[3] = p0.w;
            v[4] = p1.x; v[5] = p1.y; v[6] = p1.z; v[7] = p1.w;
        } else {
#pragma unroll
            for (int t = 0; t < 8; ++t) v[t] = 0.0f;
        }
        // an opaque zero offset keeps the weight reads inside the loop (hoisted,
        // they would hold some 140 registers)
        int z = 0;
        asm volatile("" : "+v"(z));
        const LdsWeights& L = *reinterpret_cast<const LdsWeights*>(reinterpret_cast<const char*>(&sW) + z);
        const float o = forward32(L, pack_bf16x8(v), lane);
        if (hf == 0 && s < B) y[s] = o;
    }
}

// Gradient of loss = (1/B) sum (y - t)^2 at the BF16 weights; block b handles
// the passes b, b + gridDim.x, ... of kGS samples and writes one partial row.
//
// Every layer is a 64 x 64 (units x samples) product of 32 x 32 tiles, one per
// wave: v_mfma_f32_32x32x2_f32, lane l = (i, h) = (l % 32, l / 32) holding row
// (column) i and K entry h of A (B), the result's column i and rows
// 8 (r / 4) + 4 h + r % 4, r = 0..15.  The K entries may come in any order common to
// both operands, so a lane takes four consecutive ones, 8 g + 4 h + 0..3, with one
// 16-byte LDS read for four products; the hidden vectors are kept by sample and
// by unit for that (rows of kLd floats).  FP32 throughout, as a product by
// vector instructions would be.
// Bound: the waves' serial chain of 104 products of 64 cycles and eight barriers,
// some 4 us; a batch of 8,192 fills 128 blocks.  With vector products whose
// operands came from LDS one value at a time it took 43 us, now 10.5 us (14.4 before the
// weights came 16 bytes at a time and the samples a pass ahead).
constexpr int kLd = kNh + 4;    // row stride of the 64-wide arrays, floats
constexpr int kLx = kNin + 4;   // of the 16-wide ones

__device__ __forceinline__ float4 ld4(const float* p) { return *reinterpret_cast<const float4*>(p); }
__device__ __forceinline__ void mfma4(f32x16& d, float4 a, float4 b)
{
    d = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, b.x, d, 0, 0, 0);
    d = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, b.y, d, 0, 0, 0);
    d = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, b.z, d, 0, 0, 0);
    d = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, b.w, d, 0, 0, 0);
}
typedef float f32x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void k_mlp_grad(const float* __restrict__ x,
                                                  const float* __restrict__ t, int B,
                                                  const uint16_t* __restrict__ wb,
                                                  float* __restrict__ partial)
{
    __shared__ __align__(16) float sW1[kNh * kLx];
    __shared__ __align__(16) float sW2[kNh * kLd];
    __shared__ float sB1[kNh], sB2[kNh], sW3[kNh];
    __shared__ __align__(16) float sX[kGS * kLx], sXT[kNin * kLd];
    // H1 by sample, later dy H2 by unit; H1 by unit; D2 by sample, later D1 by unit; D2 by unit
    __shared__ __align__(16) float sA[kGS * kLd], sB[kGS * kLd], sC[kGS * kLd], sD[kGS * kLd];
    __shared__ float sY[2][kGS], sDY[kGS], sRed[4][4][kNh];
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int i = lane & 31, h = lane >> 5, rt = wv >> 1, ct = wv & 1;
    const int npass = (B + kGS - 1) / kGS;
    // the samples of the first pass (later ones are loaded a pass ahead), then the
    // weights, 16 bytes a thread and turn (whole rows or halves of them)
    float xv[4];
    auto fetch = [&](int pass) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int e = tid + 256 * c, sm = e >> 4;
            xv[c] = pass * kGS + sm < B ? x[(size_t)pass * kGS * kNin + e] : 0.0f;
        }
    };
    fetch(blockIdx.x);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        const int ch = tid + 256 * c, p = 8 * ch;
        if (p >= kOffB3) continue;
        const uint4 v = reinterpret_cast<const uint4*>(wb)[ch];
        const uint32_t word[4] = {v.x, v.y, v.z, v.w};
        float* to = p < kOffB1 ? &sW1[(p / kNin) * kLx + p % kNin]
                    : p < kOffW2 ? &sB1[p - kOffB1]
                    : p < kOffB2 ? &sW2[((p - kOffW2) / kNh) * kLd + (p - kOffW2) % kNh]
                    : p < kOffW3 ? &sB2[p - kOffB2] : &sW3[p - kOffW3];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            to[2 * j] = __uint_as_float(word[j] << 16);
            to[2 * j + 1] = __uint_as_float(word[j] & 0xFFFF0000u);
        }
    }
    const float b3 = bf16_f(wb[kOffB3]);
    const float invB = 1.0f / (float)B;
    const int row = (32 * rt + i), col = (32 * ct + i);  // this lane's A row and B column
    const int su = tid & 63, sq = tid >> 6;              // unit and quarter of the samples of the sums
    f32x16 gw2 = {};
    f32x4 gw1 = {};
    float gb1 = 0.0f, gb2 = 0.0f, gw3 = 0.0f, gb3 = 0.0f, loss = 0.0f;
    for (int pass = blockIdx.x; pass < npass; pass += gridDim.x) {
        __syncthreads();  // the previous pass is done with the arrays; weights staged
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int e = tid + 256 * c, sm = e >> 4, k = e & 15;
            sX[sm * kLx + k] = xv[c];
            sXT[k * kLd + sm] = xv[c];
        }
        const float tv = tid < kGS && pass * kGS + tid < B ? t[pass * kGS + tid] : 0.0f;
        fetch(pass + gridDim.x);
        __syncthreads();
        // hidden layer 1
        float h1[16], h2[16];
        {
            f32x16 z = {};
#pragma unroll
            for (int g = 0; g < kNin / 8; ++g)
                mfma4(z, ld4(&sW1[row * kLx + 8 * g + 4 * h]), ld4(&sX[col * kLx + 8 * g + 4 * h]));
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int u = 32 * rt + 8 * q + 4 * h;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    h1[4 * q + r] = fmaxf(z[4 * q + r] + sB1[u + r], 0.0f);
                    sB[(u + r) * kLd + col] = h1[4 * q + r];
                }
                *reinterpret_cast<float4*>(&sA[col * kLd + u]) =
                    make_float4(h1[4 * q], h1[4 * q + 1], h1[4 * q + 2], h1[4 * q + 3]);
            }
        }
        __syncthreads();
        // hidden layer 2 and the output
        {
            f32x16 z = {};
#pragma unroll
            for (int g = 0; g < kNh / 8; ++g)
                mfma4(z, ld4(&sW2[row * kLd + 8 * g + 4 * h]), ld4(&sA[col * kLd + 8 * g + 4 * h]));
            float y = 0.0f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int j = 32 * rt + 8 * (r >> 2) + 4 * h + (r & 3);
                h2[r] = fmaxf(z[r] + sB2[j], 0.0f);
                y = fmaf(sW3[j], h2[r], y);
            }
            y += __shfl_xor(y, 32, 64);
            if (h == 0) sY[rt][col] = y;
        }
        __syncthreads();
        if (tid < kGS) {
            const int gs = pass * kGS + tid;
            const float r = gs < B ? sY[0][tid] + sY[1][tid] + b3 - tv : 0.0f;
            const float dy = 2.0f * r * invB;
            sDY[tid] = dy;
            gb3 += dy;
            loss = fmaf(r, r, loss);
        }
        __syncthreads();
        // output gradients of layer 2, by sample and by unit, and dy H2 by unit
        {
            const float dy = sDY[col];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int u = 32 * rt + 8 * q + 4 * h;
                float d[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    d[r] = h2[4 * q + r] > 0.0f ? dy * sW3[u + r] : 0.0f;
                    sD[(u + r) * kLd + col] = d[r];
                    sA[(u + r) * kLd + col] = dy * h2[4 * q + r];
                }
                *reinterpret_cast<float4*>(&sC[col * kLd + u]) = make_float4(d[0], d[1], d[2], d[3]);
            }
        }
        __syncthreads();
        // layer 1: D1 = W2^T D2 where H1 > 0; dW2 += D2 H1^T
        f32x16 d1 = {};
#pragma unroll
        for (int g = 0; g < kNh / 8; ++g) {
            const float* w = &sW2[(8 * g + 4 * h) * kLd + row];
            mfma4(d1, make_float4(w[0], w[kLd], w[2 * kLd], w[3 * kLd]), ld4(&sC[col * kLd + 8 * g + 4 * h]));
            mfma4(gw2, ld4(&sD[row * kLd + 8 * g + 4 * h]), ld4(&sB[col * kLd + 8 * g + 4 * h]));
        }
        __syncthreads();
#pragma unroll
        for (int r = 0; r < 16; ++r)
            sC[(32 * rt + 8 * (r >> 2) + 4 * h + (r & 3)) * kLd + col] = h1[r] > 0.0f ? d1[r] : 0.0f;
        __syncthreads();
        // dW1 += D1 X^T in 16 x 16 tiles (v_mfma_f32_16x16x4_f32: lane l holds row or
        // column l % 16 and K entry l / 16, the result's column l % 16 and rows
        // 4 (l / 16) + 0..3), one per wave; the sums over the samples
#pragma unroll
        for (int g = 0; g < kGS / 16; ++g) {
            const int o = 16 * g + 4 * (lane >> 4);
            const float4 a = ld4(&sC[(16 * wv + (lane & 15)) * kLd + o]), b = ld4(&sXT[(lane & 15) * kLd + o]);
            gw1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.x, b.x, gw1, 0, 0, 0);
            gw1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.y, b.y, gw1, 0, 0, 0);
            gw1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.z, b.z, gw1, 0, 0, 0);
            gw1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a.w, b.w, gw1, 0, 0, 0);
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int o = su * kLd + 16 * sq + 4 * c;
            const float4 v1 = ld4(&sC[o]), v2 = ld4(&sD[o]), v3 = ld4(&sA[o]);
            gb1 += (v1.x + v1.y) + (v1.z + v1.w);
            gb2 += (v2.x + v2.y) + (v2.z + v2.w);
            gw3 += (v3.x + v3.y) + (v3.z + v3.w);
        }
    }
    __syncthreads();
    sRed[0][sq][su] = gb1;
    sRed[1][sq][su] = gb2;
    sRed[2][sq][su] = gw3;
    if (tid < kGS) {
        sRed[3][0][tid] = gb3;
        sRed[3][1][tid] = loss;
    }
    float* out = partial + (size_t)blockIdx.x * kRow;
#pragma unroll
    for (int r = 0; r < 16; ++r)
        out[kOffW2 + (32 * rt + 8 * (r >> 2) + 4 * h + (r & 3)) * kNh + col] = gw2[r];
#pragma unroll
    for (int r = 0; r < 4; ++r) out[(16 * wv + 4 * (lane >> 4) + r) * kNin + (lane & 15)] = gw1[r];
    __syncthreads();
    if (tid < 3 * kNh) {
        const int a = tid / kNh, u = tid % kNh;
        const int at = a == 0 ? kOffB1 : a == 1 ? kOffB2 : kOffW3;
        out[at + u] = (sRed[a][0][u] + sRed[a][1][u]) + (sRed[a][2][u] + sRed[a][3][u]);
    } else {
        // the last wave: the two sums over the samples' threads
        float v = sRed[3][0][lane], w = sRed[3][1][lane];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            v += __shfl_xor(v, o, 64);
            w += __shfl_xor(w, o, 64);
        }
        if (lane == 0) {
            out[kOffB3] = v;
            out[kNP] = w;
        }
    }
}

// Sum of the block partials; Adam when lr > 0.  Thread (c, p) of a block of 16 x 64
// adds rows c, c + 16, ... of parameter p, the 16 sums are added in order: fixed
// for a given number of blocks.  Bound: latency, a serial chain of nblk / 16 + 16
// additions; one thread per parameter took 31 us for 128 rows, this 3.4 us.
constexpr int kUpP = 64, kUpC = 16;
__global__ __launch_bounds__(kUpP* kUpC) void k_mlp_update(const float* __restrict__ partial, int nblk,
                                                           float* master, float* m, float* v,
                                                           uint16_t* wb, float lr, float bc1, float bc2,
                                                           float* grad_out, float* loss_out, int B)
{
    __shared__ float sS[kUpC][kUpP];
    const int c = threadIdx.x / kUpP, pl = threadIdx.x % kUpP, p = blockIdx.x * kUpP + pl;
    float g = 0.0f;
    if (p <= kNP) {
#pragma unroll 4
        for (int b = c; b < nblk; b += kUpC) g += partial[(size_t)b * kRow + p];
    }
    sS[c][pl] = g;
    __syncthreads();
    if (c != 0 || p > kNP) return;
#pragma unroll
    for (int k = 1; k < kUpC; ++k) g += sS[k][pl];
    if (p == kNP) {
        if (loss_out) *loss_out = g / (float)B;
        return;
    }
    if (grad_out) grad_out[p] = g;
    if (lr > 0.0f) {
        const float b1 = 0.9f, b2 = 0.999f, eps = 1e-8f;
        const float mn = b1 * m[p] + (1.0f - b1) * g;
        const float vn = b2 * v[p] + (1.0f - b2) * g * g;
        m[p] = mn;
        v[p] = vn;
        const float w = master[p] - lr * (mn / bc1) / (sqrtf(vn / bc2) + eps);
        master[p] = w;
        wb[p] = bf16_rne(w);
    }
}

}  // namespace

struct MlpState {
    float* master = nullptr;
    float* m = nullptr;
    float* v = nullptr;
    uint16_t* wb = nullptr;
    float* partial = nullptr;
    float* loss = nullptr;
    float* scratch[4] = {nullptr, nullptr, nullptr, nullptr};
    size_t scratch_cap[4] = {0, 0, 0, 0};
    int t = 0;
    bool has_weights = false;
};

int mlp_num_params() { return kNP; }

MlpState* mlp_create()
{
    MlpState* s = new MlpState();
    if (hipMalloc((void**)&s->master, kNP * sizeof(float)) != hipSuccess ||
        hipMalloc((void**)&s->m, kNP * sizeof(float)) != hipSuccess ||
        hipMalloc((void**)&s->v, kNP * sizeof(float)) != hipSuccess ||
        hipMalloc((void**)&s->wb, kNPpad * sizeof(uint16_t)) != hipSuccess ||
        hipMalloc((void**)&s->partial, (size_t)kMaxGradBlocks * kRow * sizeof(float)) != hipSuccess ||
        hipMalloc((void**)&s->loss, sizeof(float)) != hipSuccess ||
        hipMemset(s->wb, 0, kNPpad * sizeof(uint16_t)) != hipSuccess) {
        mlp_destroy(s);
        return nullptr;
    }
    return s;
}

void mlp_destroy(MlpState* s)
{
    if (!s) return;
    for (void* p : {(void*)s->master, (void*)s->m, (void*)s->v, (void*)s->wb, (void*)s->partial,
                    (void*)s->loss})
        if (p) (void)hipFree(p);
    for (int i = 0; i < 4; ++i)
        if (s->scratch[i]) (void)hipFree(s->scratch[i]);
    delete s;
}

bool mlp_has_weights(const MlpState* s) { return s && s->has_weights; }

float* mlp_scratch(MlpState* s, int which, size_t floats)
{
    if (which < 0 || which >= 4) return nullptr;
    if (s->scratch_cap[which] < floats) {
        if (s->scratch[which]) (void)hipFree(s->scratch[which]);
        s->scratch[which] = nullptr;
        s->scratch_cap[which] = 0;
        if (hipMalloc((void**)&s->scratch[which], std::max<size_t>(floats, 1) * sizeof(float)) != hipSuccess)
            return nullptr;
        s->scratch_cap[which] = floats;
    }
    return s->scratch[which];
}

int mlp_set_weights(MlpState* s, const float* host_w, hipStream_t st)
{
    if (hipMemcpyAsync(s->master, host_w, kNP * sizeof(float), hipMemcpyHostToDevice, st) != hipSuccess ||
        hipMemsetAsync(s->m, 0, kNP * sizeof(float), st) != hipSuccess ||
        hipMemsetAsync(s->v, 0, kNP * sizeof(float), st) != hipSuccess)
        return -1;
    hipLaunchKernelGGL(k_mlp_round, dim3((kNP + 255) / 256), dim3(256), 0, st, s->master, s->wb);
    if (hipGetLastError() != hipSuccess || hipStreamSynchronize(st) != hipSuccess) return -1;
    s->t = 0;
    s->has_weights = true;
    return 0;
}

int mlp_get_weights(MlpState* s, float* host_w, hipStream_t st)
{
    if (hipMemcpyAsync(host_w, s->master, kNP * sizeof(float), hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess)
        return -1;
    return 0;
}

const uint16_t* mlp_weights_bf16(const MlpState* s) { return s->wb; }  // kNPpad values, 16-B aligned

int mlp_forward(MlpState* s, const float* x, int64_t B, float* y, hipStream_t st)
{
    if (B <= 0) return 0;
    // four waves (128 samples) per block and round; at most 1,024 blocks
    const int64_t tiles = (B + 31) / 32;
    const unsigned grid = (unsigned)std::min<int64_t>((tiles + 3) / 4, 1024);
    hipLaunchKernelGGL(k_mlp_forward, dim3(grid), dim3(256), 0, st, x, (int)B, s->wb, y);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int mlp_grad_step(MlpState* s, const float* x, const float* t, int64_t B, float lr, float* grad,
                  float* loss_host, hipStream_t st)
{
    const int npass = (int)((B + kGS - 1) / kGS);
    const int nblk = std::min(npass, kMaxGradBlocks);
    hipLaunchKernelGGL(k_mlp_grad, dim3(nblk), dim3(256), 0, st, x, t, (int)B, s->wb, s->partial);
    if (hipGetLastError() != hipSuccess) return -1;
    float bc1 = 1.0f, bc2 = 1.0f;
    if (lr > 0.0f) {
        s->t += 1;
        bc1 = (float)(1.0 - std::pow(0.9, (double)s->t));
        bc2 = (float)(1.0 - std::pow(0.999, (double)s->t));
    }
    hipLaunchKernelGGL(k_mlp_update, dim3((kNP + kUpP) / kUpP), dim3(kUpP * kUpC), 0, st, s->partial, nblk,
                       s->master, s->m, s->v, s->wb, lr, bc1, bc2, grad, s->loss, (int)B);
    if (hipGetLastError() != hipSuccess) return -1;
    if (loss_host) {
        if (hipMemcpyAsync(loss_host, s->loss, sizeof(float), hipMemcpyDeviceToHost, st) != hipSuccess ||
            hipStreamSynchronize(st) != hipSuccess)
            return -1;
    }
    return 0;
}

}  // namespace dgidp
