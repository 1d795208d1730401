// Internal declarations shared by the library's translation units (not installed).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/mxc.h"

namespace mxc {

typedef uint16_t bf16_t;  // raw bf16 bit pattern

// One convolution problem in the library's working layout: activations NHWC,
// filters KRSC.  P and Q are derived by the ABI layer.
// Kr, Cr: where the tensors carry more channels than the problem has (padded to a multiple of 8 with zeros), the
// problem's own counts; 0 = the same.  The filter always has the problem's own K rows.
struct ConvShape {
    int N, C, H, W, K, R, S, stride, pad, P, Q;
    int Kr = 0, Cr = 0;
};
inline int real_k(const ConvShape &s) { return s.Kr ? s.Kr : s.K; }
inline int real_c(const ConvShape &s) { return s.Cr ? s.Cr : s.C; }

// The caller's operands of a gradient whose results may have to be summed again (see resum.h), with the problem's own
// channel counts: dx: a = dy, b = w; dw: a = x, b = dy
struct Resum {
    ConvShape s;
    bool nchw;
    const bf16_t *a, *b;
};

__device__ __forceinline__ float bf16_to_f32(bf16_t v) { return __uint_as_float(((uint32_t)v) << 16); }

// Round-to-nearest-even; inputs are finite in this library's use.
__device__ __forceinline__ bf16_t f32_to_bf16(float f)
{
    uint32_t u = __float_as_uint(f);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (bf16_t)(u >> 16);
}

// two values at once (v_cvt_pk_bf16_f32): `lo` in bits 0..15; the same rounding as f32_to_bf16 for finite inputs
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    typedef float f32x2_t __attribute__((ext_vector_type(2)));
    const f32x2_t f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2_t));
}

__device__ __forceinline__ float load_f32(const float *p) { return *p; }
__device__ __forceinline__ float load_f32(const bf16_t *p) { return bf16_to_f32(*p); }
__device__ __forceinline__ void store_f32(float *p, float v) { *p = v; }
__device__ __forceinline__ void store_f32(bf16_t *p, float v) { *p = f32_to_bf16(v); }

// Order of a launch's tiles.  Each XCD, whose L2 is its own, gets `share` tiles that follow each other: what they read between
// them is least when the tiles that share the larger operand's rows are neighbours.  bm, bn: what a tile reads of either operand.  True:
// the row tiles of a column follow each other, which has to save a quarter (5850 pixels, 112 columns, 5x5 on 176 channels, near the
// tie: 16.6 us with the column tiles together, 17.9 with the row tiles).
inline bool rows_inner(long long share, long long m_tiles, double bm, long long n_tiles, double bn)
{
    const auto read = [&](long long inner, double inner_rows, double outer_rows) {
        return share >= inner ? inner * inner_rows + (share + inner - 1) / inner * outer_rows : share * inner_rows + outer_rows;
    };
    return read(m_tiles, bm, bn) < 0.75 * read(n_tiles, bn, bm);
}

// What the kernel that produces a result applies to it before the store (the grouped forms of the
// convolution: see mxc_conv2d_fwd_bias_act / mxc_conv2d_bwd_data_relu).  Default: nothing.
struct PostOp {
    const float *bias = nullptr;   // forward: + bias[k], one fp32 value per output channel
    int relu = 0;                  // forward: max(0, .) after the bias
    const void *mask = nullptr;    // backward-data: result is 0 where mask <= 0; same shape, type and layout as dx
    struct PlaneOut *planes = nullptr;
    bool copied = false;           // the result is a copy that a re-layout reads next
};
// An NCHW problem on NHWC copies: a kernel that can stores the result straight to its planes and says so.
struct PlaneOut {
    void *out;                     // [N][cols][plane]
    const void *mask;              // PostOp::mask in that layout
    int cols;                      // the problem's own columns
    bool stored;
};

// keeps the halves of v (two bf16) whose mask half is > 0
__device__ __forceinline__ uint32_t mask_bf16x2(uint32_t v, uint32_t m)
{
    // per half: min(m, 1) as signed integers is 1 where m > 0 and at most 0 elsewhere; 0 - max(that, 0) is all ones or zero
    typedef short s2 __attribute__((ext_vector_type(2)));
    const s2 one = __builtin_elementwise_max(__builtin_elementwise_min(__builtin_bit_cast(s2, m), s2{1, 1}), s2{0, 0});
    return v & __builtin_bit_cast(uint32_t, s2{0, 0} - one);
}
__device__ __forceinline__ bool mask_keeps(const float *m) { return *m > 0.f; }
__device__ __forceinline__ bool mask_keeps(const bf16_t *m) { return (int16_t)*m > 0; }

// ---- asynchronous global -> LDS transfers (the MFMA kernels' operand path) ---------------------------
// A wave-wide 16-byte-per-lane buffer load whose data goes straight to LDS: lane l's 16 bytes land at
// lds_base + 16*l, where lds_base is wave-uniform.  Lanes whose byte offset lies outside the buffer deposit
// zeros (how padding, ragged edges and reduction tails are filled).
//
// Written as inline assembly on purpose.  Issued through the compiler's builtin, the transfer is known to the
// compiler as a write to LDS, and it then guards LDS reads that it cannot prove disjoint (every read made
// with a transposing-read builtin, every read after a control-flow join, everything once more than eight LDS
// objects are in play) with a wait for ALL outstanding transfers, which empties a ring of stages at every
// stage.  This way the compiler sees no LDS write at all; the kernels order the transfers against their LDS
// reads themselves (s_waitcnt vmcnt(N) + barrier before a stage is read).  M0 holds the LDS base for the
// instruction; nothing else in these kernels uses M0.
typedef int buf_rsrc_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ buf_rsrc_t make_buf_rsrc(const void *base, unsigned bytes)
{
    const uint64_t a = (uint64_t)base;
    buf_rsrc_t r;
    r.x = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    r.y = __builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xFFFFu));   // stride 0: raw buffer
    r.z = __builtin_amdgcn_readfirstlane((int)bytes);                              // out-of-range above this
    r.w = 0x00020000;
    return r;
}
__device__ __forceinline__ void lds_dma16(buf_rsrc_t rsrc, unsigned byte_off, const void *lds_base_uniform)
{
    typedef __attribute__((address_space(3))) const void *lds_cvptr;
    const unsigned lds_addr = (unsigned)(uintptr_t)(lds_cvptr)lds_base_uniform;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :
                 : "s"(lds_addr), "v"(byte_off), "s"(rsrc)
                 : "memory");
}

// the same with 4 bytes per lane: lane l's dword lands at lds_base + 4*l
__device__ __forceinline__ void lds_dma4(buf_rsrc_t rsrc, unsigned byte_off, const void *lds_base_uniform)
{
    typedef __attribute__((address_space(3))) const void *lds_cvptr;
    const unsigned lds_addr = (unsigned)(uintptr_t)(lds_cvptr)lds_base_uniform;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds"
                 :
                 : "s"(lds_addr), "v"(byte_off), "s"(rsrc)
                 : "memory");
}

// lds_dma16 marked non-temporal: a streaming read that the caches need not keep
__device__ __forceinline__ void lds_dma16_nt(buf_rsrc_t rsrc, unsigned byte_off, const void *lds_base_uniform)
{
    typedef __attribute__((address_space(3))) const void *lds_cvptr;
    const unsigned lds_addr = (unsigned)(uintptr_t)(lds_cvptr)lds_base_uniform;
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen nt lds"
                 :
                 : "s"(lds_addr), "v"(byte_off), "s"(rsrc)
                 : "memory");
}
// 16-byte store through a buffer resource: a lane whose byte_off lies beyond the resource's size writes nothing,
// which takes the place of a bounds branch.  These are compiler builtins, not inline assembly, so that the compiler
// itself keeps the wait states between a store wider than 8 bytes and the next write of its data registers.
typedef __amdgpu_buffer_rsrc_t out_rsrc_t;
__device__ __forceinline__ out_rsrc_t make_out_rsrc(void *base, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(base, 0, (int)bytes, 0x00020000);     // stride 0: raw buffer
}
__device__ __forceinline__ void buffer_store16(out_rsrc_t rsrc, unsigned byte_off, uint4 v)
{
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{v.x, v.y, v.z, v.w}, rsrc, (int)byte_off, 0, 0);
}
__device__ __forceinline__ void buffer_store16_nt(out_rsrc_t rsrc, unsigned byte_off, uint4 v)
{
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    __builtin_amdgcn_raw_buffer_store_b128(u32x4{v.x, v.y, v.z, v.w}, rsrc, (int)byte_off, 0, 2);   // 2: non-temporal
}

// 16-byte load through a buffer resource: a lane whose byte_off lies beyond the resource's size gets zeros
__device__ __forceinline__ uint4 buffer_load16(out_rsrc_t rsrc, unsigned byte_off)
{
    typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)byte_off, 0, 0);
    return make_uint4(v.x, v.y, v.z, v.w);
}
// Results that leave un-packed from space-to-depth order (streaming and window kernels): row (n, h2, w2), column
// (dh*s + dw)*Cq + c goes to dx[n][h2*s + dh - pad][w2*s + dw - pad][c] of an N x H x W x C tensor; s = 0: off.
struct S2DStore {
    int s, pad, C, Cq, H, W;
};

__host__ __device__ inline bool s2d_pairs(const S2DStore &q)
{
    return q.Cq == q.C && (q.s * q.C) % 2 == 0 && (q.pad * q.C) % 2 == 0 && (q.W * q.C) % 2 == 0;
}
// store instructions for the 32 rows of a wave (s is even)
__host__ __device__ inline int s2d_stores(const S2DStore &q) { return q.s * (q.s * q.C / (s2d_pairs(q) ? 2 : 1)) / 2; }

// Stores the 32 rows of a wave from its staging area.  A unit is two neighbouring elements of an image row where the two
// always share a dword, else one.  Units are numbered (dh, row, place in the row's run of s*C elements): for one dh the
// units of consecutive rows are consecutive in the image, so a store instruction writes 128 or 256 bytes in a piece.
struct S2DWave {
    bool pair;
    int run_u, u0, r0, du, dr;      // units per run; this lane's first unit, and the step to the one 64 further on
    __device__ __forceinline__ S2DWave(const S2DStore &q, int lane)
    {
        pair = s2d_pairs(q);
        run_u = q.s * q.C / (pair ? 2 : 1);
        r0 = lane / run_u; u0 = lane - r0 * run_u;
        dr = 64 / run_u; du = 64 - dr * run_u;
    }
    __device__ __forceinline__ int stores(const S2DStore &q) const { return q.s * run_u / 2; }
    __device__ __forceinline__ void next(int &u, int &r, int &dh) const
    {
        u += du;
        const int carry = u >= run_u ? 1 : 0;
        u -= carry ? run_u : 0;
        r += dr + carry;
        dh += r >> 5;
        r &= 31;
    }
    // the GEMM's column of element e of the run at dh
    __device__ __forceinline__ int column(const S2DStore &q, int dh, int e) const
    {
        if (q.Cq == q.C) return dh * q.s * q.C + e;
        const int dw = q.C == 3 ? (e * 86) >> 8 : q.C == 2 ? e >> 1 : e;        // e / C: C <= 3 and e < 16 here
        return (dh * q.s + dw) * q.Cq + e - dw * q.C;
    }
    // lane l (and l + 32) brings row l's position: image n, block (h2, w2), or ok = false; staged(r, col) points at a result
    template <class F>
    __device__ __forceinline__ void store(const S2DStore &q, out_rsrc_t rs_out, int n, int h2, int w2, bool row_ok, F &&staged) const
    {
        const int h0 = h2 * q.s - q.pad, w0 = w2 * q.s - q.pad;
        const int base = ((n * q.H + h0) * q.W + w0) * q.C;
        const int hw = row_ok ? (h0 & 0xFFFF) | (w0 << 16) : (-16384) & 0xFFFF;
        const int row_e = q.W * q.C, iters = stores(q);
        int u = u0, r = r0 & 31, dh = r0 >> 5;
        for (int k = 0; k < iters; ++k) {
            const int rb = __shfl(base, r), rhw = __shfl(hw, r);
            const int e = pair ? 2 * u : u;
            const uint16_t *src = staged(r, column(q, dh, e));
            const int h = (int)(short)rhw + dh, we = (rhw >> 16) * q.C + e;
            const bool ok = (unsigned)h < (unsigned)q.H && (unsigned)we < (unsigned)row_e;
            const unsigned off = ok ? (unsigned)(rb + dh * row_e + e) * 2u : 0x80000000u;      // rejected by the resource
            if (pair) __builtin_amdgcn_raw_buffer_store_b32(*reinterpret_cast<const uint32_t *>(src), rs_out, (int)off, 0, 0);
            else __builtin_amdgcn_raw_buffer_store_b16(*src, rs_out, (int)off, 0, 0);
            next(u, r, dh);
        }
    }
};

__device__ __forceinline__ uint4 mask_bf16x8(uint4 v, uint4 m)
{
    return make_uint4(mask_bf16x2(v.x, m.x), mask_bf16x2(v.y, m.y), mask_bf16x2(v.z, m.z), mask_bf16x2(v.w, m.w));
}

// n / d for 0 <= n < 2^31 as a multiplication, by the method of Granlund and Montgomery (Division by Invariant Integers using
// Multiplication, PLDI 1994): m = floor(2^32 * (2^l - d) / d) + 1 with 2^(l-1) < d <= 2^l, and n / d = (mulhi(m, n) + n) >> l.
// The compiler's division by a variable is some thirty instructions, and a tile's setup has dozens of them (they were two thirds
// of a small layer's kernel time).
struct FastDiv {
    unsigned mul = 0, shift = 0;
    int d = 1;
    FastDiv() = default;
    explicit FastDiv(int divisor) : d(divisor > 0 ? divisor : 1)
    {
        while (shift < 31 && (1u << shift) < (unsigned)d) ++shift;
        mul = (unsigned)(((1ull << 32) * ((1ull << shift) - (unsigned)d)) / (unsigned)d + 1);
    }
    __device__ __forceinline__ int div(int n) const { return (int)((__umulhi(mul, (unsigned)n) + (unsigned)n) >> shift); }
    __device__ __forceinline__ int mod(int n) const { return n - div(n) * d; }
};

// floor(t / d) for 0 <= t <= 127, 1 <= d <= 127
__device__ __forceinline__ int small_div(int t, int magic) { return (t * magic) >> 16; }
inline int small_magic(int d) { return (65536 + d - 1) / d; }

static inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
static inline size_t elem_size(int dtype) { return dtype == MXC_BF16 ? 2 : 4; }

// ---- layout.hip ------------------------------------------------------------
// Batched 2-D transpose: src[b][rows][cols] -> dst[b][cols][rows], element size 2 or 4 bytes.
int launch_transpose(const void *src, void *dst, int batch, int rows, int cols, int elem_bytes,
                     hipStream_t stream);
// whether launch_transpose can run this problem (its grid holds batch x ceil(rows/64) x ceil(cols/64) workgroups)
bool transpose_launchable(long long batch, long long rows, long long cols);
int launch_copy(const void *src, void *dst, size_t bytes, hipStream_t stream);

// Re-layouts of 2-byte elements, up to MAX_RELAY_JOBS in one launch (see relayout_kernel).
enum { RELAY_TRANSPOSE = 0, RELAY_PAD = 1, RELAY_FILTER_KRSC = 2, RELAY_FILTER_KCRS = 3 };
constexpr int MAX_RELAY_JOBS = 3;
struct RelayJob {
    const void *src;
    void *dst;
    long long batch, src_batch, dst_batch;
    int kind, rows, cols, src_pitch, run, dst_pitch, run_tiles;     // run: length of a destination run (>= rows: zeros beyond)
    int C, class_C, R, S, stride;
    unsigned blocks;
};
// one or two plain transposes of 4-byte elements in one launch
int relayout4(const RelayJob *jobs, int n, hipStream_t st);
RelayJob relay_to_nhwc(const void *src, void *dst, int n, int c, int hw, int c_pitch);      // [n][c][hw] -> [n][hw][c_pitch]
RelayJob relay_to_nchw(const void *src, void *dst, int n, int c, int hw, int c_pitch);      // [n][hw][c_pitch] -> [n][c][hw]
RelayJob relay_pad(const void *src, void *dst, long long rows, int c, int c_pitch);         // [rows][c] -> [rows][c_pitch]
// the filter matrices of backward-data, one per stride residue class: wt[class][c][(j*TS + i)*K + k] (see igemm_bwd_data)
RelayJob relay_bwd_filter(const ConvShape &s, const void *w, void *wt, bool kcrs);
// resum: the one job brings dx to its place
int relayout(const RelayJob *jobs, int n, hipStream_t st, const Resum *resum = nullptr);

// ---- probe.hip: matrix-pipe ceiling measurement -------------------------------------
// launches the register-resident MFMA loop; *flops = floating-point operations the launch performs
int probe_mfma(int workgroups, int iters, float *out, double *flops, hipStream_t st);

// ---- update.hip: SGD with momentum and weight decay on fp32 master weights -------------
int sgd_update(size_t n, float *w, const float *g, float *v, void *w_copy, float lr, float momentum, float wd, hipStream_t st);

// ---- softmax.hip: softmax output layer --------------------------------------------------
int softmax_fwd(int N, int K, int dtype, const void *z, void *p, hipStream_t st);
int softmax_xent_bwd(int N, int K, int dtype, const void *p, const int *labels, void *dz, float scale, hipStream_t st);

// ---- bias.hip: bias gradient ------------------------------------------------------------
size_t bias_grad_scratch(long long N, int K, long long PQ, int dtype, int layout);      // bytes of partial vectors
int bias_grad(long long N, int K, long long PQ, int dtype, int layout, const void *dy, float *db, float *partial, hipStream_t st);

// ---- direct.hip: one-thread-per-output kernels, any shape, NHWC/KRSC --------
int direct_fwd(const ConvShape &s, int dtype, const void *x, const void *w, void *y, hipStream_t st, const PostOp &post = PostOp());
int direct_bwd_data(const ConvShape &s, int dtype, const void *dy, const void *w, void *dx, hipStream_t st,
                    const PostOp &post = PostOp());
// partial: fp32 scratch of direct_bwd_weight_splits(s) * K*R*S*C floats
int direct_bwd_weight_splits(const ConvShape &s);
// dw: fp32, or bf16 (the fp32 sum rounded once) when dw_bf16
int direct_bwd_weight(const ConvShape &s, int dtype, const void *x, const void *dy, void *dw, bool dw_bf16,
                      float *partial, int splits, hipStream_t st);

// After the matrix-core kernels on zero-padded channels (see resum.h): results that padding made NaN, summed again without it
int resum_dx(const Resum &q, void *dx, hipStream_t st);
int resum_dw(const Resum &q, void *dw, bool dw_bf16, hipStream_t st);

// ---- taps_dx.hip: backward-data of first layers at stride 1 in one launch ----------------------------------
const char *taps_dx_name();
bool taps_dx_supported(const ConvShape &s);
bool taps_dx_faster(const ConvShape &s);      // of a supported layer
int taps_dx(const ConvShape &s, const void *dy, const void *w, bool packed, int packed_cols, void *dx, hipStream_t st, const PostOp &post);

// ---- fp32.hip: fp32 matrix-core convolution, NHWC/KRSC or NCHW/KCRS operands read in place -----------------
bool f32_supported(const ConvShape &s);
// `copies`: with NCHW, what f32_copies answered (at least 0: the operands are NHWC / KRSC copies, the result goes to its planes)
int f32_copies(const ConvShape &s, bool bwd, bool masked);
int f32_fwd(const ConvShape &s, bool nchw, int copies, const void *x, const void *w, void *y, hipStream_t st, const char **variant,
            const PostOp &post);
int f32_bwd_data(const ConvShape &s, bool nchw, int copies, const void *dy, const void *w, void *dx, hipStream_t st, const char **variant,
                 const PostOp &post);
size_t f32_wgrad_workspace(const ConvShape &s);       // bytes of fp32 partial tensors
int f32_wgrad(const ConvShape &s, bool nchw, const void *x, const void *dy, void *dw, float *partial, hipStream_t st, const char **variant);
const char *f32_tile_name(int index);
const char *f32_wave_name(int index);

// ---- igemm.hip: bf16 MFMA implicit GEMM (NHWC/KRSC) ---------------------------
bool igemm_fwd_supported(const ConvShape &s);
// split_ws: scratch of igemm_fwd_split_bytes(s) bytes for a split reduction (may be null: never split)
size_t igemm_fwd_split_bytes(const ConvShape &s);
int igemm_fwd(const ConvShape &s, const void *x, const void *w, void *y, hipStream_t st, const char **variant,
              const PostOp &post = PostOp(), void *split_ws = nullptr);
bool igemm_bwd_data_supported(const ConvShape &s);
size_t igemm_bwd_data_workspace(const ConvShape &s);   // bytes for the re-packed filter
size_t igemm_bwd_data_split_bytes(const ConvShape &s);   // scratch for a split reduction (0: never split)
// Filter preparation (re-pack per stride residue class / transpose of a 1x1 filter) into wt; a filter that the
// kernel reads in place is copied to wt only when copy_in_place_filter is set.
// (kcrs: w lies in KCRS order)
int igemm_bwd_data_prepare(const ConvShape &s, const void *w, void *wt, hipStream_t st, bool copy_in_place_filter, bool kcrs = false);
// whether igemm_bwd_data reads this layer's filter as it is; otherwise relay_bwd_filter makes the form it reads
bool bwd_data_reads_filter_in_place(const ConvShape &s);
// ... or reads the KRSC filter it is handed in place although its prepared form is the re-packed one; strided dx likewise
bool bwd_data_small_in_place(const ConvShape &s, bool masked);
bool bwd_data_classes_in_place(const ConvShape &s, bool masked);
// whether dx of an NCHW problem, its filter re-packed, goes straight to its planes (see PlaneOut)
bool igemm_bwd_data_planes(const ConvShape &s, bool masked);
int igemm_bwd_data(const ConvShape &s, const void *dy, const void *w_in_place, void *dx, const void *wt, hipStream_t st,
                   const char **variant, const PostOp &post = PostOp(), void *split_ws = nullptr);
// stride-1 backward-data whose result is stored un-packed from space-to-depth order: the kernel that can and should, or none
enum ImageStore { IMAGE_NONE = 0, IMAGE_STREAM, IMAGE_WINDOW };
ImageStore igemm_bwd_data_image_store(const ConvShape &s2, const S2DStore &q);
// w2: the KRSC filter where the streaming kernel is to read it, or null: wt, as igemm_bwd_data_prepare left it
int igemm_bwd_data_image(ImageStore kind, const ConvShape &s2, const S2DStore &q, const void *dy, const void *w2, const void *wt, void *dx, hipStream_t st,
                         const char **variant);

// backward-data for C <= 4: G output columns form one GEMM row (see igemm.hip)
bool igemm_bwd_data_smallc_supported(const ConvShape &s);
void igemm_bwd_data_smallc_workspace(const ConvShape &s, size_t *w2_bytes, size_t *dx4_bytes);
int igemm_bwd_data_smallc_columns(const ConvShape &s);       // dy columns per row of the packed filter
int igemm_bwd_data_smallc_prepare(const ConvShape &s, const void *w, void *w2, hipStream_t st);
int igemm_bwd_data_smallc(const ConvShape &s, const void *dy, const void *w2, void *dx, void *dx4, hipStream_t st,
                          const char **variant, const PostOp &post = PostOp());

// names of the tile shapes the two MFMA kernel families are built in (nullptr past the last)
const char *igemm_tile_name(int index);
const char *igemm_stream_name(int index);   // names of the whole-launch kernels' plans (streaming kernel, window kernel)
// key (rows, output columns, reduction length) of the calling thread's last implicit-GEMM plan lookup
void igemm_last_plan_key(long long *M, int *Co, int *Kd);
const char *wgrad_tile_name(int index);
// dw[i] = sum over z of partial[z][i] in a fixed order (see the reduce kernels of wgrad.hip); dw fp32, or bf16 rounded once
int sum_splits(const float *partial, void *dw, bool dw_bf16, long long total, int splits, hipStream_t st);

// ---- the implicit GEMM as its kernels see it (igemm.hip, stream.hip) ----------------------------------
constexpr int MAX_TAPS = 127;   // tap table capacity (11x11 = 121 fits)

struct RowStep { int n, a, b; };
inline RowStep row_step(int rows, int Mh, int Mw) { return RowStep{rows / (Mh * Mw), rows % (Mh * Mw) / Mw, rows % Mw}; }

// Out[m][co] = sum_{t,ci} In[pixel(m) + tap(t)][ci] * Wm[co][t*Ci + ci]; m runs over (image, row, column) of the
// launch's output grid, t over a TR x TS grid of filter taps, ci over the channels of a tap's contiguous run.
struct IgemmParams {
    const bf16_t *in;    // activations [N][Hi][Wi][Ci]
    const bf16_t *wm;    // filter matrix [Co][T*Ci]
    bf16_t *out;         // output tensor [N][Ho][Wo][Co]
    int N, Hi, Wi;
    int Ci;              // reduction elements per tap: a contiguous run starting at the tap's pixel
    int pix;             // elements per pixel in memory (== Ci for plain NHWC; smaller when a run spans pixels)
    int Co;
    int Cw;              // rows of the filter matrix and bias values that exist (columns beyond are zero); 0: Co
    int TR, TS, tstep_h, tstep_w;   // tap grid and the direction (+1 or -1) taps advance in, per axis
    int Mh, Mw;          // output grid of this launch (per image)
    int in_mul_h, in_mul_w, in_off_h, in_off_w;     // input coordinate of tap 0: a*in_mul + in_off
    int Ho, Wo, out_mul_h, out_mul_w, out_off_h, out_off_w;  // output coordinate: a*out_mul + out_off
    // A step of so many GEMM rows as images + grid rows + grid columns, set by the launcher: of a load's rows to the next
    // load's, and of a store's rows to the next store's (walked by additions: a division costs a wave some hundred clocks)
    RowStep in_step, out_step;
    int linear_out;      // output pixel index == m (forward, and stride-1 backward-data)
    int M;               // N*Mh*Mw (< 2^31, checked by the launcher)
    int m_begin, m_end;  // GEMM rows [m_begin, m_end) belong to this launch (a problem may be cut in two launches of
                         // different tile shapes: see Plan); tile 0 starts at m_begin
    int m_tiles, n_tiles;
    unsigned in_bytes, wm_bytes;   // sizes of the two operand buffers (< 2^31)
    // BT kernels (stride-1 backward-data straight from the filter, no re-packed copy): wm = w[K][T][Co]; reduction element
    // (tap, k) is filter row k*T + tap, whose Co output columns are contiguous.
    unsigned bt_w_bytes; // size of the filter
    int wm_by_k;         // streaming kernel: wm is that filter too, transposed on its way into LDS
    // split reduction (few tiles, long reduction): workgroup (tile, z) runs stages [z*split_stages, (z+1)*split_stages)
    // and stores its fp32 accumulators to partial[z][m][co]; a second kernel adds the splits in ascending z and
    // applies bias / ReLU / mask.  splits <= 1: off.
    float *partial;
    int splits, split_stages;
    int tap_row_inner;   // tap t = (column step)*TR + (row step) instead of (row step)*TS + (column step)
    S2DStore s2d;        // `out` is the image and not the GEMM's [m][co]
    int f32_out;         // store the fp32 accumulators to `partial` ([m][co], one split) instead of a rounded result to `out`
    int zero_rest;       // dx of a 1x1 filter at stride 2: the three pixels of a 2x2 block that no tap reaches are written too, as zeros
    int nt_out;          // the 16-byte result stores are non-temporal
    unsigned out_bytes;  // size of the output tensor when below 2 GiB (buffer stores with range-checked offsets), else 0
    int tap_inner;       // reduction order (see tap_inner_order): 1 = all taps of a channel block before the next block
    // applied to the accumulators before the store (all optional)
    const float *bias;   // + bias[co]
    int relu;            // max(0, .)
    int copied;          // see PostOp (here, where the fields before it leave a gap: the kernels' arguments stay where they are)
    const bf16_t *mask;  // indexed like `out`: the stored value is 0 where mask <= 0
};

// out[m][n] = sum_k a[m][k] * b[n][k] in fp32 from bf16 operands (k contiguous in both), on the tiled kernel
bool igemm_gemm_f32_supported(long long M, int Kd, int Nn);
int igemm_gemm_f32(long long M, int Kd, int Nn, const void *a, const void *b, float *out, hipStream_t st, const char **variant);

// ---- winograd.hip: 3x3 stride-1 forward in the transform domain, F(2x2, 3x3) ----------------------------
bool winograd_supported(const ConvShape &s);
// bytes of the three workspace parts: transformed filter U [16][K][C] bf16, transformed input V [16][tiles][C] bf16,
// products M [16][tiles][K] fp32
void winograd_workspace(const ConvShape &s, size_t *u_bytes, size_t *v_bytes, size_t *m_bytes);
int winograd_fwd(const ConvShape &s, const void *x, const void *w, void *y, void *u, void *v, void *m, hipStream_t st,
                 const char **variant, const PostOp &post);

// stream.hip: the same GEMM for short reductions and few output columns (see there); whether it can run p,
// and the launch over all rows (both take p as a launch site fills it: the fields the launcher derives -
// M, row range, tile counts, byte sizes, linear_out, tap_inner - are ignored and recomputed).
bool stream_applicable(const IgemmParams &p);
bool stream_pays(const IgemmParams &p, bool masked, double other);      // 1x1 filters at stride 1: rather than a kernel modelled at `other` us
int stream_launch(const IgemmParams &p, hipStream_t st);
// window.hip: the same GEMM for multi-tap stride-1 layers of at most 64 input channels, from an LDS-resident input
// window and filter (see there); same conventions as the streaming kernel.
bool window_applicable(const IgemmParams &p);
// two patches or more for every CU, at most a third of their rows past the image
bool window_fills_chip(const IgemmParams &p);
int window_launch(const IgemmParams &p, hipStream_t st);
// runs.hip: the same GEMM for stride-1 filters of 3 or 5 columns whose output rows are as wide as the input's (see there)
const char *run_name(int shape);
int run_forced(const char *name, const IgemmParams &p);
bool run_applicable(const IgemmParams &p);
int run_best(long long M, int Co, int Ci, int TR, int TS, bool masked, double *us);      // the shape of least modelled time and that time
int run_launch(int shape, IgemmParams p, hipStream_t st, bool bt = false);      // bt: wm is the KRSC filter

// wave.hip: the same GEMM for problems that fill a fraction of the chip and for short reductions (see there).  Shapes are
// numbered from 0; bwd: backward-data, whose shapes can all read the filter in place; bt: wm is the KRSC filter itself (see
// IgemmParams).  wave_best: the shape of least modelled time and that time, or -1.
const char *wave_name(int shape);
int wave_forced(const char *name, bool bwd);
int wave_best(long long M, int Co, int Kd, bool bwd, bool masked, double *us);
int wave_launch(int shape, const IgemmParams &p, hipStream_t st, bool bt, PlaneOut *planes = nullptr);
// dx of a layer of stride 2: bt: p.wm is the KRSC filter itself, else as igemm_bwd_data_prepare left it
bool wave_has_classes(int shape);
int wave_best_classes(const ConvShape &s, bool masked, double *us, double *other);
int wave_launch_classes(int shape, const ConvShape &s, const IgemmParams &p, hipStream_t st, bool bt);

// ---- prep.hip: re-packing for channel counts that are not a multiple of 8 ---------
// Small-C (C <= 4) image packing: `pix` channels per pixel, explicit zero border, padded size Hp x Wp;
// one filter row's taps form a contiguous run of `run` elements.
struct SmallCGeom { int pix, Hp, Wp, run; };
SmallCGeom smallc_geom(const ConvShape &s);
int smallc_pack_x(const ConvShape &s, const void *x, void *xp, hipStream_t st);   // xp: N*Hp*Wp*pix elements
int smallc_pack_w(const ConvShape &s, const void *w, void *wp, hipStream_t st);   // wp: K*R*run elements
// Space-to-depth (C <= 4, stride 2 or 4): s x s pixel blocks become channels of a stride-1 problem.
struct S2DGeom { int s, Cq, C2, R2, S2, H2, W2; };
S2DGeom s2d_geom(const ConvShape &s);
bool s2d_applicable(const ConvShape &s);
ConvShape s2d_shape(const ConvShape &s);      // the equivalent stride-1 problem: x2[N][H2][W2][C2], w2[K][R2][S2][C2]
int s2d_pack_x(const ConvShape &s, const void *x, void *x2, hipStream_t st);
int s2d_pack_w(const ConvShape &s, const void *w, void *w2, hipStream_t st);
int s2d_pack_wt(const ConvShape &s, const void *w, void *wt, hipStream_t st);       // ... as igemm_bwd_data_prepare makes of it
int s2d_unpack_dx(const ConvShape &s, const void *dx2, void *dx, hipStream_t st, const void *mask = nullptr);   // mask: see PostOp
bool igemm_fwd_smallc_supported(const ConvShape &s);
int igemm_fwd_smallc(const ConvShape &s, const void *xp, const void *wp, void *y, hipStream_t st, const char **variant,
                     const PostOp &post = PostOp());

// ---- wgrad.hip: bf16 MFMA backward-weight with split reduction ------------------
// The problem as the kernel sees it: x[N][H][W][pix], dy[N][P][Q][K]; filter columns are TR*TS taps of
// `run` contiguous elements each; dw[k][r][s][c] (dense R,S,C) is read back from column
// r*col_r + s*col_s + c.
// With s2d > 1 the columns come from a space-to-depth problem: filter tap (r,s) sits in block
// (r/s2d, s/s2d) at channel ((r%s2d)*s2d + s%s2d)*Cq + c.
struct WgradGeom {
    int N, H, W, pix, K, P, Q, stride, pad, TR, TS, run, R, S, C, col_r, col_s, s2d, Cq;
    int Kout;                    // rows of dw (K counts dy's channels, padded to a multiple of 8)
    int oH, oW, ostride, opad;   // the caller's problem (with N, C, K, R, S: the key of the measured-plan table)
};
WgradGeom wgrad_geom_s2d(const ConvShape &s);       // x already packed by s2d_pack_x
WgradGeom wgrad_geom_plain(const ConvShape &s);     // C % 8 == 0
WgradGeom wgrad_geom_chanpad(const ConvShape &s);   // x already padded to C8 channels
WgradGeom wgrad_geom_smallc(const ConvShape &s);    // x already packed by smallc_pack_x
// Where an element of the summed [K][ncols] tensor belongs: dw has the same order, or it is dw[k][r][s][c] (or
// dw[k][c][r][s]) of column (r/d)*col_r + (s/d)*col_s + ((r%d)*d + s%d)*Cq + c, and padded rows and columns are dropped.
enum { DW_SAME = 0, DW_KRSC = 1, DW_KCRS = 2 };
struct DwMap {
    int order, ncols, Kout, R, S, C, col_r, col_s, d, Cq;
};
// element (k, col)'s place in dw and its filter tap (r, s) and channel, or -1
__device__ __forceinline__ long long dw_place(const DwMap &m, int k, int col, int &r, int &s, int &c)
{
    const int rb = col / m.col_r, in_r = col - rb * m.col_r, sb = in_r / m.col_s, in_s = in_r - sb * m.col_s;
    const int blk = m.d > 1 ? in_s / m.Cq : 0;
    c = in_s - blk * m.Cq;
    r = rb * m.d + blk / m.d; s = sb * m.d + blk % m.d;
    if (k >= m.Kout || r >= m.R || s >= m.S || c >= m.C) return -1;
    return m.order == DW_KRSC ? (((long long)k * m.R + r) * m.S + s) * m.C + c : (((long long)k * m.C + c) * m.R + r) * m.S + s;
}

// wave_dw.hip: backward-weight of small problems (see there).  Shapes are numbered from 0.  out: `ranges` partial tensors
// [K][ncols] of `span` pixels each (a multiple of 32), or with one range dw itself, mapped or (map null) as it lies.
// wave_dw_best: the shape and ranges (at most max_ranges) of least modelled time and that time, or -1.
const char *wave_dw_name(int shape);
int wave_dw_ranges(long long M, int ranges, int *span);        // the number of ranges there are, none empty, and their length
int wave_dw_best(const WgradGeom &g, bool copies, int max_ranges, int *ranges, double *us);
int wave_dw_launch(int shape, const WgradGeom &g, int ranges, int span, const void *x, const void *dy, void *out, const DwMap *map, bool dw_bf16, int rows,
                   hipStream_t st);

// runs_dw.hip: backward-weight of stride-1 filters of 3 or 5 columns whose output rows are as wide as the input's (see there).  out: partial
// tensors as above, or with one range dw itself where its columns are in KRSC order
const char *run_dw_name(int shape);
bool run_dw_applicable(const WgradGeom &g);
bool run_dw_has(int shape, int columns);       // whether the shape is built for filters of so many columns
int run_dw_ranges(int shape, long long M, int ranges, int *span);
int run_dw_best(const WgradGeom &g, int most_ranges, bool copies, int *ranges, int *span, double *us);      // the shape of least modelled time, as wave_dw_best
double dw_places_us(int ranges, double mb);      // what a dw of so many MB costs besides on copies (see there)
int run_dw_launch(int shape, const WgradGeom &g, int ranges, int span, const void *x, const void *dy, float *out, int rows, hipStream_t st);

bool wgrad_supported(const WgradGeom &g);
size_t wgrad_workspace(const WgradGeom &g);            // bytes of fp32 partial tiles
// dw: fp32, or bf16 (the fp32 sum rounded once, by the reduce kernel) when dw_bf16; KRSC, or KCRS when kcrs
int wgrad(const WgradGeom &g, const void *x, const void *dy, void *dw, bool dw_bf16, bool kcrs, float *partial, hipStream_t st,
          const char **variant, const Resum *resum = nullptr);

}  // namespace mxc
