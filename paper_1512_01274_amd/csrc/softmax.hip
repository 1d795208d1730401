// Softmax output layer: p[n][k] = exp(z[n][k] - max_j z[n][j]) / sum_j exp(...), and the gradient of the
// cross-entropy against integer labels, (p - onehot(label)) * scale.  One workgroup per row; fp32
// arithmetic whatever the storage type; row maximum and sum reduced through LDS in a fixed order.
#include "mxc_internal.h"

namespace mxc {
namespace {

constexpr int SM_THREADS = 256;

__device__ __forceinline__ float block_reduce(float v, float *red, bool is_max)
{
    red[threadIdx.x] = v;
    __syncthreads();
    for (int half = SM_THREADS / 2; half > 0; half >>= 1) {
        if ((int)threadIdx.x < half) red[threadIdx.x] = is_max ? fmaxf(red[threadIdx.x], red[threadIdx.x + half])
                                                               : red[threadIdx.x] + red[threadIdx.x + half];
        __syncthreads();
    }
    const float r = red[0];
    __syncthreads();
    return r;
}

template <typename T>
__global__ __launch_bounds__(SM_THREADS) void softmax_fwd_kernel(const T *__restrict__ z, T *__restrict__ p, int K)
{
    __shared__ float red[SM_THREADS];
    const T *zr = z + (size_t)blockIdx.x * K;
    T *pr = p + (size_t)blockIdx.x * K;
    float mx = -3.0e38f;
    for (int k = threadIdx.x; k < K; k += SM_THREADS) mx = fmaxf(mx, load_f32(zr + k));
    mx = block_reduce(mx, red, true);
    float sum = 0.f;
    for (int k = threadIdx.x; k < K; k += SM_THREADS) sum += expf(load_f32(zr + k) - mx);
    sum = block_reduce(sum, red, false);
    const float inv = 1.f / sum;
    for (int k = threadIdx.x; k < K; k += SM_THREADS) store_f32(pr + k, expf(load_f32(zr + k) - mx) * inv);
}

// Rows of whole 16-byte pieces that a wave, or four, holds in registers: read once, without a barrier where one wave does it (the general
// form reads a row three times and meets at twenty barriers: 128 rows of 1000 bf16 4.3 -> 2.8 us, 188 of 3272 7.5 -> 3.3).  Lane l of the row's 64*W has pieces
// l, l + 64*W, ...; fixed order.
template <typename T, int W, int PIECES>
__global__ __launch_bounds__(64 * W) void softmax_fwd_vec_kernel(const uint4 *z, uint4 *p, int pieces)      // (may be the same rows)
{
    constexpr int V = 16 / (int)sizeof(T);
    __shared__ float red[2][W];
    const size_t row = (size_t)blockIdx.x * pieces;
    float v[PIECES][V];
    float mx = -3.0e38f;
#pragma unroll
    for (int q = 0; q < PIECES; ++q) {
        const int at = q * 64 * W + (int)threadIdx.x;
        uint4 u = make_uint4(0, 0, 0, 0);
        if (at < pieces) u = z[row + at];
        const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
        for (int e = 0; e < V; ++e) {
            if constexpr (V == 8) v[q][e] = __uint_as_float(e & 1 ? w[e / 2] & 0xFFFF0000u : w[e / 2] << 16);
            else v[q][e] = __uint_as_float(w[e]);
            if (at < pieces) mx = fmaxf(mx, v[q][e]);
        }
    }
    auto meet = [&](float x, int slot, bool is_max) {
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) {
            const float o = __shfl_xor(x, d);
            x = is_max ? fmaxf(x, o) : x + o;
        }
        if constexpr (W > 1) {
            if ((threadIdx.x & 63) == 0) red[slot][threadIdx.x >> 6] = x;
            __syncthreads();
            x = red[slot][0];
#pragma unroll
            for (int w = 1; w < W; ++w) x = is_max ? fmaxf(x, red[slot][w]) : x + red[slot][w];
        }
        return x;
    };
    mx = meet(mx, 0, true);
    float sum = 0.f;
#pragma unroll
    for (int q = 0; q < PIECES; ++q)
#pragma unroll
        for (int e = 0; e < V; ++e) {
            v[q][e] = expf(v[q][e] - mx);
            if (q * 64 * W + (int)threadIdx.x < pieces) sum += v[q][e];
        }
    const float inv = 1.f / meet(sum, 1, false);
#pragma unroll
    for (int q = 0; q < PIECES; ++q) {
        const int at = q * 64 * W + (int)threadIdx.x;
        if (at >= pieces) continue;
        alignas(16) T out[V];
#pragma unroll
        for (int e = 0; e < V; ++e) store_f32(out + e, v[q][e] * inv);
        p[row + at] = *reinterpret_cast<uint4 *>(out);
    }
}

template <typename T>
bool softmax_fwd_vec(int N, int K, const T *z, T *p, hipStream_t st)
{
    constexpr int V = 16 / (int)sizeof(T);
    const int pieces = K / V;
    if (K % V != 0 || pieces > 1024) return false;       // (z and p begin on 16 bytes: mxc_softmax_fwd)
    const uint4 *zv = (const uint4 *)z;
    uint4 *pv = (uint4 *)p;
    if (pieces <= 64) hipLaunchKernelGGL((softmax_fwd_vec_kernel<T, 1, 1>), dim3((unsigned)N), dim3(64), 0, st, zv, pv, pieces);
    else if (pieces <= 128) hipLaunchKernelGGL((softmax_fwd_vec_kernel<T, 1, 2>), dim3((unsigned)N), dim3(64), 0, st, zv, pv, pieces);
    else if (pieces <= 256) hipLaunchKernelGGL((softmax_fwd_vec_kernel<T, 4, 1>), dim3((unsigned)N), dim3(256), 0, st, zv, pv, pieces);
    else if (pieces <= 512) hipLaunchKernelGGL((softmax_fwd_vec_kernel<T, 4, 2>), dim3((unsigned)N), dim3(256), 0, st, zv, pv, pieces);
    else hipLaunchKernelGGL((softmax_fwd_vec_kernel<T, 4, 4>), dim3((unsigned)N), dim3(256), 0, st, zv, pv, pieces);
    return true;
}

template <typename T>
__global__ __launch_bounds__(SM_THREADS) void softmax_xent_bwd_kernel(const T *__restrict__ p, const int *__restrict__ labels,
                                                                      T *__restrict__ dz, int K, float scale)
{
    const T *pr = p + (size_t)blockIdx.x * K;
    T *dr = dz + (size_t)blockIdx.x * K;
    const int label = labels[blockIdx.x];
    for (int k = threadIdx.x; k < K; k += SM_THREADS) store_f32(dr + k, (load_f32(pr + k) - (k == label ? 1.f : 0.f)) * scale);
}

}  // namespace

int softmax_fwd(int N, int K, int dtype, const void *z, void *p, hipStream_t st)
{
    if (dtype == MXC_BF16 ? softmax_fwd_vec(N, K, (const bf16_t *)z, (bf16_t *)p, st) : softmax_fwd_vec(N, K, (const float *)z, (float *)p, st))
        return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
    if (dtype == MXC_BF16) hipLaunchKernelGGL(softmax_fwd_kernel<bf16_t>, dim3((unsigned)N), dim3(SM_THREADS), 0, st, (const bf16_t *)z, (bf16_t *)p, K);
    else hipLaunchKernelGGL(softmax_fwd_kernel<float>, dim3((unsigned)N), dim3(SM_THREADS), 0, st, (const float *)z, (float *)p, K);
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
}

int softmax_xent_bwd(int N, int K, int dtype, const void *p, const int *labels, void *dz, float scale, hipStream_t st)
{
    if (dtype == MXC_BF16)
        hipLaunchKernelGGL(softmax_xent_bwd_kernel<bf16_t>, dim3((unsigned)N), dim3(SM_THREADS), 0, st, (const bf16_t *)p, labels,
                           (bf16_t *)dz, K, scale);
    else
        hipLaunchKernelGGL(softmax_xent_bwd_kernel<float>, dim3((unsigned)N), dim3(SM_THREADS), 0, st, (const float *)p, labels,
                           (float *)dz, K, scale);
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
}

}  // namespace mxc
