// Direct (one thread per output element) convolution kernels.
//
// These cover every shape and both element types, and are the path for shapes the
// matrix-core kernels do not take (stride > 4, tensors of 2 GiB and more, more than
// 127 taps) and for the smallest NHWC gradients of ragged K.  Working layout:
// activations NHWC, filters KRSC, fp32 accumulation in a fixed order (deterministic).
#include "resum.h"

namespace mxc {

namespace {

// y[n,p,q,k] = sum_{r,s,c} x[n,p*st-pad+r,q*st-pad+s,c] * w[k,r,s,c]
template <typename T>
__global__ __launch_bounds__(256) void direct_fwd_kernel(ConvShape s, const T *__restrict__ x, const T *__restrict__ w,
                                                         T *__restrict__ y, size_t total, const float *__restrict__ bias, int relu)
{
    const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= total) return;
    size_t t = gid;
    const int k = (int)(t % s.K); t /= s.K;
    const int q = (int)(t % s.Q); t /= s.Q;
    const int p = (int)(t % s.P); t /= s.P;
    const int n = (int)t;
    float acc = 0.f;
    for (int r = 0; r < s.R; ++r) {
        const int h = p * s.stride - s.pad + r;
        if (h < 0 || h >= s.H) continue;
        for (int ss = 0; ss < s.S; ++ss) {
            const int v = q * s.stride - s.pad + ss;
            if (v < 0 || v >= s.W) continue;
            const T *xp = x + (((size_t)n * s.H + h) * s.W + v) * s.C;
            const T *wp = w + (((size_t)k * s.R + r) * s.S + ss) * s.C;
            for (int c = 0; c < s.C; ++c) acc = fmaf(load_f32(xp + c), load_f32(wp + c), acc);
        }
    }
    if (bias != nullptr) acc += bias[k];
    if (relu) acc = fmaxf(acc, 0.f);
    store_f32(y + gid, acc);
}

template <typename T>
__global__ __launch_bounds__(256) void direct_bwd_data_kernel(ConvShape s, const T *__restrict__ dy,
                                                              const T *__restrict__ w, T *__restrict__ dx, size_t total,
                                                              const T *__restrict__ mask)
{
    const size_t gid = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= total) return;
    size_t t = gid;
    const int c = (int)(t % s.C); t /= s.C;
    const int v = (int)(t % s.W); t /= s.W;
    const int h = (int)(t % s.H); t /= s.H;
    const int n = (int)t;
    float acc = sum_dx<T, false>(s, dy, w, n, h, v, c);
    if (mask != nullptr && !mask_keeps(mask + gid)) acc = 0.f;
    store_f32(dx + gid, acc);
}

// partial[split][k,r,s,c] = sum over the split's pixel range of dy[n,p,q,k] * x[n,h,v,c]
template <typename T>
__global__ __launch_bounds__(256) void direct_bwd_weight_kernel(ConvShape s, const T *__restrict__ x,
                                                                const T *__restrict__ dy, float *__restrict__ partial,
                                                                int pix_per_split)
{
    const int wtotal = s.K * s.R * s.S * s.C;
    const int gid = blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= wtotal) return;
    int t = gid;
    const int c = t % s.C; t /= s.C;
    const int ss = t % s.S; t /= s.S;
    const int r = t % s.R; t /= s.R;
    const int k = t;
    const long long npq = (long long)s.N * s.P * s.Q;
    const long long m0 = (long long)blockIdx.y * pix_per_split;
    long long m1 = m0 + pix_per_split;
    if (m1 > npq) m1 = npq;
    float acc = 0.f;
    for (long long m = m0; m < m1; ++m) {
        const int q = (int)(m % s.Q);
        const int p = (int)((m / s.Q) % s.P);
        const int n = (int)(m / ((long long)s.P * s.Q));
        const int h = p * s.stride - s.pad + r, v = q * s.stride - s.pad + ss;
        if (h < 0 || h >= s.H || v < 0 || v >= s.W) continue;
        acc = fmaf(load_f32(dy + (size_t)m * s.K + k), load_f32(x + (((size_t)n * s.H + h) * s.W + v) * s.C + c), acc);
    }
    partial[(size_t)blockIdx.y * wtotal + gid] = acc;
}

// ---- results of the matrix-core kernels that padding made NaN (see resum.h) --------------------------------------
// The two kernels below read the results and sum those that are NaN once more.  What bounds them is the launch: they read what
// was just written (a 64x30x45x37 dx 2.5 us, a 50x30x3x3 dw 2.2).  Where a kernel passes over the results anyway - the last
// conversion to NCHW, the mapped split reduction - it does so itself: the NCHW training step of that layer is 71.1 us without,
// 75.9 with the two kernels, 72.1 that way.
// dx, eight elements per thread
template <bool NCHW>
__global__ __launch_bounds__(256) void resum_dx_kernel(ConvShape s, const bf16_t *__restrict__ dy, const bf16_t *__restrict__ w, bf16_t *dx,
                                                       size_t total)
{
    const size_t at = ((size_t)blockIdx.x * 256 + threadIdx.x) * 8;
    if (at >= total) return;
    const int n_el = total - at < 8 ? (int)(total - at) : 8;
    unsigned bad = 0;
    if (n_el == 8) bad = nan_bits(*reinterpret_cast<const uint4 *>(dx + at));
    else
        for (int e = 0; e < n_el; ++e) bad |= (is_nan(dx[at + e]) ? 1u : 0u) << e;
    for (; bad != 0; bad &= bad - 1) {
        const size_t i = at + (__ffs(bad) - 1);
        size_t t = i;
        int c = 0;
        if (!NCHW) { c = (int)(t % s.C); t /= s.C; }
        const int v = (int)(t % s.W); t /= s.W;
        const int h = (int)(t % s.H); t /= s.H;
        if (NCHW) { c = (int)(t % s.C); t /= s.C; }
        store_f32(dx + i, sum_dx<bf16_t, NCHW>(s, dy, w, (int)t, h, v, c));     // a masked element is not NaN
    }
}

// dw, `per` elements per workgroup: its threads share the pixels of each sum, and their shares meet in a tree
template <typename OUT, bool NCHW>
__global__ __launch_bounds__(256) void resum_dw_kernel(ConvShape s, const bf16_t *__restrict__ x, const bf16_t *__restrict__ dy, OUT *dw, int total,
                                                       int per)
{
    __shared__ float red[256];
    __shared__ int bad[256];
    const int tid = threadIdx.x, RS = s.R * s.S, gid = blockIdx.x * per + tid;
    const bool mine = tid < per && gid < total && is_nan(dw[gid]);
    bad[tid] = mine;
    if (!__syncthreads_or(mine)) return;
    for (int i = 0; i < per; ++i) {
        if (!bad[i]) continue;                       // the same for every thread
        const int at = blockIdx.x * per + i;
        const int c = NCHW ? at / RS % s.C : at % s.C, rs = NCHW ? at % RS : at / s.C % RS, k = at / (RS * s.C);
        red[tid] = sum_dw<NCHW>(s, x, dy, k, c, rs / s.S, rs % s.S, tid, 256);
        __syncthreads();
        for (int half = 128; half > 0; half >>= 1) {
            if (tid < half) red[tid] += red[tid + half];
            __syncthreads();
        }
        if (tid == 0) store_f32(dw + at, red[0]);
        __syncthreads();
    }
}

inline int ok() { return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH; }

}  // namespace

int direct_fwd(const ConvShape &s, int dtype, const void *x, const void *w, void *y, hipStream_t st, const PostOp &post)
{
    const size_t total = (size_t)s.N * s.P * s.Q * s.K;
    const size_t blocks = (total + 255) / 256;
    if (blocks > 0x7FFFFFFFull) return MXC_ERR_SHAPE;
    if (dtype == MXC_BF16)
        hipLaunchKernelGGL(direct_fwd_kernel<bf16_t>, dim3((unsigned)blocks), dim3(256), 0, st, s, (const bf16_t *)x,
                           (const bf16_t *)w, (bf16_t *)y, total, post.bias, post.relu);
    else
        hipLaunchKernelGGL(direct_fwd_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, st, s, (const float *)x,
                           (const float *)w, (float *)y, total, post.bias, post.relu);
    return ok();
}

int direct_bwd_data(const ConvShape &s, int dtype, const void *dy, const void *w, void *dx, hipStream_t st, const PostOp &post)
{
    const size_t total = (size_t)s.N * s.H * s.W * s.C;
    const size_t blocks = (total + 255) / 256;
    if (blocks > 0x7FFFFFFFull) return MXC_ERR_SHAPE;
    if (dtype == MXC_BF16)
        hipLaunchKernelGGL(direct_bwd_data_kernel<bf16_t>, dim3((unsigned)blocks), dim3(256), 0, st, s,
                           (const bf16_t *)dy, (const bf16_t *)w, (bf16_t *)dx, total, (const bf16_t *)post.mask);
    else
        hipLaunchKernelGGL(direct_bwd_data_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, st, s,
                           (const float *)dy, (const float *)w, (float *)dx, total, (const float *)post.mask);
    return ok();
}

int resum_dx(const Resum &q, void *dx, hipStream_t st)
{
    const ConvShape &s = q.s;
    const size_t total = (size_t)s.N * s.H * s.W * s.C, blocks = (total + 2047) / 2048;
    if (blocks > 0x7FFFFFFFull) return MXC_ERR_SHAPE;
    if (q.nchw) hipLaunchKernelGGL(resum_dx_kernel<true>, dim3((unsigned)blocks), dim3(256), 0, st, s, q.a, q.b, (bf16_t *)dx, total);
    else hipLaunchKernelGGL(resum_dx_kernel<false>, dim3((unsigned)blocks), dim3(256), 0, st, s, q.a, q.b, (bf16_t *)dx, total);
    return ok();
}

template <typename OUT>
static int resum_dw_to(const Resum &q, OUT *dw, hipStream_t st)
{
    const ConvShape &s = q.s;
    const int total = s.K * s.R * s.S * s.C;        // below 2^31: checked with the shape
    // few elements per workgroup where there are few: should they all be NaN, the chip shares the work
    int per = (total + 1023) / 1024;
    per = per < 4 ? 4 : per > 256 ? 256 : per;
    const dim3 grid((unsigned)((total + (long long)per - 1) / per)), block(256);
    if (q.nchw) hipLaunchKernelGGL((resum_dw_kernel<OUT, true>), grid, block, 0, st, s, q.a, q.b, dw, total, per);
    else hipLaunchKernelGGL((resum_dw_kernel<OUT, false>), grid, block, 0, st, s, q.a, q.b, dw, total, per);
    return ok();
}

int resum_dw(const Resum &q, void *dw, bool dw_bf16, hipStream_t st)
{
    return dw_bf16 ? resum_dw_to(q, (bf16_t *)dw, st) : resum_dw_to(q, (float *)dw, st);
}

int direct_bwd_weight_splits(const ConvShape &s)
{
    // Enough splits to occupy the chip when the filter is small, never more than the pixel count.
    const long long wtotal = (long long)s.K * s.R * s.S * s.C;
    const long long npq = (long long)s.N * s.P * s.Q;
    long long blocks = (wtotal + 255) / 256;
    long long splits = (2048 + blocks - 1) / blocks;
    if (splits > 256) splits = 256;
    if (splits > npq) splits = npq;
    if (splits < 1) splits = 1;
    return (int)splits;
}

int direct_bwd_weight(const ConvShape &s, int dtype, const void *x, const void *dy, void *dw, bool dw_bf16, float *partial,
                      int splits, hipStream_t st)
{
    const long long wtotal_ll = (long long)s.K * s.R * s.S * s.C;
    if (wtotal_ll > 0x7FFFFFFFll) return MXC_ERR_SHAPE;
    const int wtotal = (int)wtotal_ll;
    const long long npq = (long long)s.N * s.P * s.Q;
    const long long pps = (npq + splits - 1) / splits;
    if (pps > 0x7FFFFFFFll) return MXC_ERR_SHAPE;
    dim3 grid((unsigned)((wtotal + 255) / 256), (unsigned)splits), block(256);
    if (dtype == MXC_BF16)
        hipLaunchKernelGGL(direct_bwd_weight_kernel<bf16_t>, grid, block, 0, st, s, (const bf16_t *)x,
                           (const bf16_t *)dy, partial, (int)pps);
    else
        hipLaunchKernelGGL(direct_bwd_weight_kernel<float>, grid, block, 0, st, s, (const float *)x, (const float *)dy,
                           partial, (int)pps);
    if (ok() != MXC_OK) return MXC_ERR_LAUNCH;
    return sum_splits(partial, dw, dw_bf16, wtotal, splits, st);
}

}  // namespace mxc
