// One result of a convolution gradient as the definition has it: the taps inside, and nothing else.  For the one-thread
// kernels, and for results of the matrix-core kernels on zero-padded channels (bf16 layers of ragged K) that padding made NaN:
// there a tap outside the image, and a place that a first layer's packing leaves empty, is a product with zero, which is NaN
// where the other operand is infinite or NaN, although the sum does not have that term.  Such a result is NaN itself.
#pragma once
#include "mxc_internal.h"

namespace mxc {

__device__ __forceinline__ bool is_nan(float v) { return v != v; }
__device__ __forceinline__ bool is_nan(bf16_t v) { return (v & 0x7FFFu) > 0x7F80u; }
// which of eight bf16 are NaN, as bits; the usual answer is none
__device__ __forceinline__ unsigned nan_bits(uint4 v)
{
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    const auto mag = [](uint32_t u) { return __builtin_bit_cast(u16x2, u & 0x7FFF7FFFu); };
    const u16x2 most = __builtin_elementwise_max(__builtin_elementwise_max(mag(v.x), mag(v.y)), __builtin_elementwise_max(mag(v.z), mag(v.w)));
    if (most.x <= 0x7F80u && most.y <= 0x7F80u) return 0;
    const uint32_t u[4] = {v.x, v.y, v.z, v.w};
    unsigned bad = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) bad |= (is_nan((bf16_t)(u[e >> 1] >> ((e & 1) * 16))) ? 1u : 0u) << e;
    return bad;
}

// dx[n,h,v,c] = sum over taps (r,s) with (h+pad-r)%st==0, (v+pad-s)%st==0, p,q in range, and k.
template <typename T, bool NCHW>
__device__ __forceinline__ float sum_dx(const ConvShape &s, const T *__restrict__ dy, const T *__restrict__ w, int n, int h, int v, int c)
{
    const size_t plane = (size_t)s.P * s.Q, wk = (size_t)s.R * s.S * s.C;
    float acc = 0.f;
    for (int r = 0; r < s.R; ++r) {
        const int hp = h + s.pad - r;
        if (hp < 0 || hp % s.stride != 0) continue;
        const int p = hp / s.stride;
        if (p >= s.P) continue;
        for (int ss = 0; ss < s.S; ++ss) {
            const int vq = v + s.pad - ss;
            if (vq < 0 || vq % s.stride != 0) continue;
            const int q = vq / s.stride;
            if (q >= s.Q) continue;
            const size_t pq = (size_t)p * s.Q + q, rs = (size_t)r * s.S + ss;
            const T *dyp = dy + (NCHW ? (size_t)n * s.K * plane + pq : ((size_t)n * plane + pq) * s.K);
            const T *wp = w + (NCHW ? (size_t)c * (s.R * s.S) + rs : rs * s.C + c);
            const size_t dk = NCHW ? plane : 1;
            for (int k = 0; k < s.K; ++k) acc = fmaf(load_f32(dyp + (size_t)k * dk), load_f32(wp + (size_t)k * wk), acc);
        }
    }
    return acc;
}

// the share of dw[k,c,r,s] of pixels first, first + step, ...; a sum that has turned NaN ends
template <bool NCHW>
__device__ __forceinline__ float sum_dw(const ConvShape &s, const bf16_t *__restrict__ x, const bf16_t *__restrict__ dy, int k, int c, int r, int ss,
                                        int first, int step)
{
    const long long npq = (long long)s.N * s.P * s.Q;
    const size_t plane = (size_t)s.P * s.Q, xplane = (size_t)s.H * s.W;
    float acc = 0.f;
    for (long long m = first; m < npq && !is_nan(acc); m += step) {
        const int q = (int)(m % s.Q), p = (int)(m / s.Q % s.P), n = (int)(m / (long long)plane);
        const int h = p * s.stride - s.pad + r, v = q * s.stride - s.pad + ss;
        if (h < 0 || h >= s.H || v < 0 || v >= s.W) continue;
        acc = fmaf(load_f32(dy + (NCHW ? ((size_t)n * s.K + k) * plane + (size_t)p * s.Q + q : (size_t)m * s.K + k)),
                   load_f32(x + (NCHW ? ((size_t)n * s.C + c) * xplane + (size_t)h * s.W + v : ((size_t)n * xplane + (size_t)h * s.W + v) * s.C + c)), acc);
    }
    return acc;
}

}  // namespace mxc
