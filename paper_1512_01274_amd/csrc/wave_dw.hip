// bf16 backward-weight of small problems: the waves of a workgroup share a tile's pixels.
//
//     dw[k][col] = sum_m dy[m][k] * xcol[m][col],   col = tap*run + e  (see wgrad.hip)
//
// The counterpart of wave.hip.  A wave reduces every KG-th step of 32 pixels of its workgroup's range through a ring of its
// own, no barrier before the KG partial tiles meet in LDS; a problem whose pixels one workgroup per tile can take is one
// launch, in the order and type of dw, and with several ranges there are KG times fewer partial tensors to write and add.
//
// Both operands lie pixel by pixel, [32 pixels][16*B columns] per step and operand, brought by direct global->LDS loads of
// contiguous 64 or 128 bytes per pixel and fetched with the transposing read ds_read_b64_tr_b16; the 16-byte chunks of a row
// are exchanged by bits of its number so that the rows a read touches fall on different banks.  v_mfma_f32_16x16x32_bf16 with x
// first: lane 16*g + i holds columns 4*g .. 4*g + 3 of filter k = i of a block, 16 bytes of dw.
//
// What bounds it: the loads, 4-8 KB per wave and step, while the chip is part-filled their latency.  Measured (us with the
// summing launch where there is one, planned tile -> this kernel): 440 pixels, 256 filters x 112 columns 8.4 -> 3.4; 1944,
// 144 x 800 13.6 -> 5.7; 28120, 32 x 288 13.0 -> 8.4; 21318, 208 x 96 15.0 -> 10.0.  Which problems it gets: make_plan in wgrad.hip.
#include <stdlib.h>
#include <string.h>

#include "mxc_internal.h"

namespace mxc {

namespace {

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16x4 __attribute__((address_space(3))) * lds_bf16x4_ptr;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x2 __attribute__((ext_vector_type(2)));

constexpr unsigned OOB = 0x80000000u;   // a buffer offset no operand reaches: the load returns zeros

struct DwParams {
    const bf16_t *x, *dy;
    void *out;                  // dw, or the partial tensors
    unsigned x_bytes, dy_bytes;
    int units, tiles, M, span;  // span: pixels per range, a multiple of 32
    int K, ncols, rows;         // rows: of the result that are stored
    int hw_lim, px2, row2, img2, stride, pad;
    int P, Q;
    int adv_q, adv_p, adv_n;    // KG*32 pixels further
    int rows_inner;                  // (see rows_inner)
    FastDiv by_tiles, by_inner, by_q, by_p, by_run, by_ts;
    int mapped, dw_bf16;        // the result is dw: `map` says where an element belongs
    DwMap map;
};

template <int N> __device__ __forceinline__ void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ void wait_lgkmcnt0() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// chunk exchange of row r in a tile of 2*B chunks per row
template <int B> __device__ __forceinline__ int row_swz(int r) { return B == 2 ? ((r >> 3) & 1) << 1 : ((r >> 1) & 1) << 1 | ((r >> 3) & 1) << 2; }

// MB blocks of 16 filters x NB blocks of 16 columns per tile, KG waves, a ring of NS sets of U steps.  LINEAR: a 1x1 filter at
// stride 1 without padding, whose x rows are the pixels themselves.
template <int MB, int NB, int KG, int U, int NS, bool LINEAR>
__global__ __launch_bounds__(64 * KG) void wave_dw_kernel(const DwParams p)
{
    constexpr int BLK = 512, SET = U * (MB + NB) * BLK, RING = NS * SET, L = U * (MB + NB);
    static_assert((MB == 2 || MB == 4) && (NB == 2 || NB == 4), "rows of 64 or 128 bytes");
    static_assert(L * (NS - 1) < 64 && MB * NB * 512 <= RING, "vmcnt range; a wave's partial tile must fit its ring");
    __shared__ __attribute__((aligned(1024))) bf16_t ring[KG * RING];

    const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    bf16_t *mine = ring + wave * RING;
    // consecutive workgroups go round-robin to the 8 XCDs: a contiguous range each, tiles of one pixel range side by side
    const int per_xcd = (p.units + 7) / 8;
    const int unit = ((int)blockIdx.x & 7) * per_xcd + ((int)blockIdx.x >> 3);
    if (unit >= p.units) return;
    const int z = p.by_tiles.div(unit), tile = unit - z * p.tiles, outer = p.by_inner.div(tile), inner = tile - outer * p.by_inner.d;
    const int k0 = (p.rows_inner ? inner : outer) * 16 * MB, n0 = (p.rows_inner ? outer : inner) * 16 * NB;
    const int m_lo = z * p.span, m_end = min(m_lo + p.span, p.M);
    const int turns = (m_end - m_lo + 32 * KG * U - 1) / (32 * KG * U);

    const buf_rsrc_t rs_x = make_buf_rsrc(p.x, p.x_bytes), rs_dy = make_buf_rsrc(p.dy, p.dy_bytes);

    // ---- what this lane loads: of load j, chunk (lane % CH) of pixel row ROWS*j + lane/CH of the step ------------------
    constexpr int ACH = 2 * MB, AROWS = 64 / ACH, BCH = 2 * NB, BROWS = 64 / BCH;
    const int m_first = m_lo + wave * 32;
    int a_m = m_first + lane / ACH;                 // dy row of load 0; AROWS further for each next
    unsigned a_off[MB];
#pragma unroll
    for (int j = 0; j < MB; ++j) {
        const int r = AROWS * j + lane / ACH, k = k0 + ((lane % ACH) ^ row_swz<MB>(r)) * 8;
        a_off[j] = k < p.K ? ((unsigned)(m_first + r) * (unsigned)p.K + (unsigned)k) * 2u : OOB;
    }
    int b_m = m_first + lane / BCH;
    int b_off[NB], b_q[NB], b_p[NB], b_tap[NB];     // byte offset of the pixel's element, its position, the tap's packed offset
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int r = BROWS * j + lane / BCH, col = n0 + ((lane % BCH) ^ row_swz<NB>(r)) * 8;
        const int m = m_first + r;
        if constexpr (LINEAR) {
            b_off[j] = col < p.ncols ? m * p.px2 + col * 2 : (int)OOB;
        } else {
            const int tap = p.by_run.div(col), fr = p.by_ts.div(tap), fs = tap - fr * p.by_ts.d;
            const int t = p.by_q.div(m), n = p.by_p.div(t);
            b_q[j] = m - t * p.Q; b_p[j] = t - n * p.P;
            b_off[j] = n * p.img2 + (b_p[j] * p.stride + fr - p.pad) * p.row2 + (b_q[j] * p.stride + fs - p.pad) * p.px2 + (col - tap * p.by_run.d) * 2;
            b_tap[j] = col < p.ncols ? ((fr - p.pad) & 0xFFFF) | ((fs - p.pad) << 16) : (-16384) & 0xFFFF;
        }
    }
    const unsigned a_adv = (unsigned)(KG * 32) * (unsigned)(p.K * 2);
    auto issue = [&](bf16_t *dst) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            bf16_t *to = dst + u * (MB + NB) * BLK;
#pragma unroll
            for (int j = 0; j < MB; ++j) {
                lds_dma16(rs_dy, a_m + AROWS * j < m_end && a_off[j] < OOB ? a_off[j] : OOB, to + j * BLK);
                a_off[j] += a_off[j] < OOB ? a_adv : 0u;
            }
            a_m += KG * 32;
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                const bool in = b_m + BROWS * j < m_end;
                if constexpr (LINEAR) {
                    lds_dma16(rs_x, in ? (unsigned)b_off[j] : OOB, to + (MB + j) * BLK);
                    b_off[j] += (unsigned)b_off[j] < OOB ? KG * 32 * p.px2 : 0;
                } else {
                    const int h0 = b_p[j] * p.stride, w0 = b_q[j] * p.stride;
                    const s16x2 hw = __builtin_bit_cast(s16x2, (h0 & 0xFFFF) | (w0 << 16)) + __builtin_bit_cast(s16x2, b_tap[j]);
                    const s16x2 d = __builtin_bit_cast(s16x2, p.hw_lim) - hw;
                    const int bad = (__builtin_bit_cast(int, hw) | __builtin_bit_cast(int, d)) & (int)0x80008000;
                    lds_dma16(rs_x, bad == 0 && in ? (unsigned)b_off[j] : OOB, to + (MB + j) * BLK);
                    const int sp = p.stride * p.px2, sr = p.stride * p.row2;
                    int off = b_off[j] + p.adv_n * p.img2 + p.adv_p * sr + p.adv_q * sp;
                    int q = b_q[j] + p.adv_q;
                    const bool cq = q >= p.Q;
                    q -= cq ? p.Q : 0;
                    off += cq ? sr - p.Q * sp : 0;
                    int pr = b_p[j] + p.adv_p + (cq ? 1 : 0);
                    const bool cp = pr >= p.P;
                    pr -= cp ? p.P : 0;
                    off += cp ? p.img2 - p.P * sr : 0;
                    b_q[j] = q; b_p[j] = pr; b_off[j] = off;
                }
            }
            b_m += KG * 32;
        }
    };
    f32x4 acc[MB][NB];
#pragma unroll
    for (int b = 0; b < MB; ++b)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[b][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // fragments: eight pixels 8*g .. of column i of a block, four rows per read; the second read's rows are 4 further on,
    // which changes none of the swizzled bits
    const int fr = 8 * g + (i >> 2);
    int ta[MB], tb[NB];
#pragma unroll
    for (int b = 0; b < MB; ++b) ta[b] = fr * (16 * MB) + ((2 * b + ((i & 3) >> 1)) ^ row_swz<MB>(fr)) * 8 + (i & 1) * 4;
#pragma unroll
    for (int j = 0; j < NB; ++j) tb[j] = fr * (16 * NB) + ((2 * j + ((i & 3) >> 1)) ^ row_swz<NB>(fr)) * 8 + (i & 1) * 4;
    auto fetch = [&](const bf16_t *at, int pitch) __attribute__((always_inline)) {
        const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)at);
        const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(at + 4 * pitch));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    auto step = [&](bf16_t *src, bool refill) __attribute__((always_inline)) {
        bf16x8 fa[U][MB], fb[U][NB];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bf16_t *from = src + u * (MB + NB) * BLK;
#pragma unroll
            for (int b = 0; b < MB; ++b) fa[u][b] = fetch(from + ta[b], 16 * MB);
#pragma unroll
            for (int j = 0; j < NB; ++j) fb[u][j] = fetch(from + MB * BLK + tb[j], 16 * NB);
        }
        wait_lgkmcnt0();                          // the slot's operands are in registers: it may be refilled
        __builtin_amdgcn_sched_barrier(0);
        if (refill) issue(src);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int b = 0; b < MB; ++b)
#pragma unroll
                for (int j = 0; j < NB; ++j) acc[b][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fb[u][j], fa[u][b], acc[b][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    // the ring: see wave.hip
    const int ahead = min(turns, NS);
#pragma unroll
    for (int q = 0; q < NS; ++q)
        if (q < ahead) issue(mine + q * SET);
    int slot = 0;
    for (int t = turns; t > NS; --t) {
        wait_vmcnt<L * (NS - 1)>();
        step(mine + slot * SET, true);
        slot = slot + 1 == NS ? 0 : slot + 1;
    }
#pragma unroll
    for (int q = NS; q > 0; --q)
        if (q <= ahead) {
            if (q == 4) wait_vmcnt<L * 3>();
            else if (q == 3) wait_vmcnt<L * 2>();
            else if (q == 2) wait_vmcnt<L>();
            else wait_vmcnt<0>();
            step(mine + slot * SET, false);
            slot = slot + 1 == NS ? 0 : slot + 1;
        }

    // ---- the KG partial tiles, block by block, in ascending order -----------------------------------------------------
    f32x4 *part = reinterpret_cast<f32x4 *>(ring);
    constexpr int PITCH = RING / 8;
#pragma unroll
    for (int b = 0; b < MB; ++b)
#pragma unroll
        for (int j = 0; j < NB; ++j) part[wave * PITCH + (b * NB + j) * 64 + lane] = acc[b][j];
    __syncthreads();
    for (int blk = wave; blk < MB * NB; blk += KG) {
        f32x4 v = part[blk * 64 + lane];
#pragma unroll
        for (int w = 1; w < KG; ++w) v += part[w * PITCH + blk * 64 + lane];
        const int k = k0 + blk / NB * 16 + i, col = n0 + blk % NB * 16 + 4 * g;
        if (k >= p.rows || col >= p.ncols) continue;
        if (!p.mapped) {
            *reinterpret_cast<f32x4 *>((float *)p.out + ((size_t)z * p.K + k) * p.ncols + col) = v;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                int r, sc, c;
                const long long at = dw_place(p.map, k, col + e, r, sc, c);
                if (at < 0) continue;
                if (p.dw_bf16) ((bf16_t *)p.out)[at] = f32_to_bf16(v[e]);
                else ((float *)p.out)[at] = v[e];
            }
        }
    }
}

// The shapes and, for each, the time model that picks one (us, fitted to 543 gradients of 50 to 740 thousand pixels on the device,
// 9-10% off): fixed + round * (rounds of workgroups that fit a CU) + turn * (rounds times steps per wave) + mb * (MB that all
// workgroups load) + area * (ten blocks of the CU with most tiles) + dw * (MB of dw) + with several ranges 2.45 and part * (MB of
// partial tensors).
struct DwShape { int mb, nb, kg, u, ns; const char *name; float fixed, round, turn, load, area, dw, part; };
#define SHAPES(X) \
    X(0, 2, 2, 8, 1, 4, "wgrad_wave_32x32_w8", 2.53f, 0.919f, 0.197f, 0.033f, 0.f, 0.020f, 0.304f) \
    X(1, 2, 4, 8, 1, 3, "wgrad_wave_32x64_w8", 2.28f, 1.184f, 0.370f, 0.026f, 0.f, 0.186f, 0.405f) \
    X(2, 4, 2, 8, 1, 3, "wgrad_wave_64x32_w8", 2.31f, 1.079f, 0.354f, 0.021f, 0.f, 0.195f, 0.535f) \
    X(3, 4, 4, 8, 1, 2, "wgrad_wave_64x64_w8", 2.57f, 0.f, 0.571f, 0.016f, 0.737f, 0.259f, 0.481f)
#define X(I, MB, NB, KG, U, NS, NAME, ...) {MB, NB, KG, U, NS, NAME, __VA_ARGS__},
const DwShape kShapes[] = {SHAPES(X)};
#undef X
constexpr int N_SHAPES = sizeof(kShapes) / sizeof(kShapes[0]);

template <int MB, int NB, int KG, int U, int NS>
int launch(DwParams &p, bool linear, hipStream_t st)
{
    const dim3 grid((unsigned)((p.units + 7) / 8 * 8)), block(64 * KG);
    if (linear) hipLaunchKernelGGL((wave_dw_kernel<MB, NB, KG, U, NS, true>), grid, block, 0, st, p);
    else hipLaunchKernelGGL((wave_dw_kernel<MB, NB, KG, U, NS, false>), grid, block, 0, st, p);
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
}

}  // namespace

const char *wave_dw_name(int shape) { return shape >= 0 && shape < N_SHAPES ? kShapes[shape].name : nullptr; }

int wave_dw_ranges(long long M, int ranges, int *span)
{
    *span = (int)(((M + ranges - 1) / ranges + 31) / 32 * 32);
    return (int)((M + *span - 1) / *span);
}

// copies: x and dy have just been written by the launch before, so a CU's loads find them in no cache of its own XCD.  32x32, one
// range, 112 x 80 filters: 0.25 us per step of the waves where they lie in the L2, 0.8 as copies (48 images of 11x16: 12.0 and 32.0 us;
// 16 to 64 channels 3x3 13.6 and 21.3), and a third launch in a row costs its 2.6 us in full.  The model's
// term is 0.3 a step for every shape: over 220 gradients of copies its choices take as long as with 0.55 (within 0.1% in the mean), and
// 4.5% less than without a term.
int wave_dw_best(const WgradGeom &g, bool copies, int max_ranges, int *ranges, double *us)
{
    const long long M = (long long)g.N * g.P * g.Q;
    const int ncols = g.TR * g.TS * g.run;
    const double mb = 4e-6 * g.K * ncols;
    int best = -1;
    if (M > 1 << 30) return -1;
    for (int i = 0; i < N_SHAPES; ++i) {
        const DwShape &s = kShapes[i];
        const long long tiles = (long long)((g.K + 16 * s.mb - 1) / (16 * s.mb)) * ((ncols + 16 * s.nb - 1) / (16 * s.nb));
        const int slots = 160 / (s.kg * s.ns * s.u * (s.mb + s.nb));
        for (int fill = 64; fill <= 512; fill *= 2) {       // one range, then as many as give 128, 256 and 512 workgroups
            long long z = fill == 64 ? 1 : fill / tiles;
            if (z > max_ranges) z = max_ranges;
            if (z < 1) z = 1;
            int span;
            z = wave_dw_ranges(M, (int)z, &span);
            const long long per_cu = (tiles * z + 255) / 256;
            const double rounds = (double)((per_cu + slots - 1) / slots), turns = (double)((span + 32 * s.kg * s.u - 1) / (32 * s.kg * s.u));
            double t = s.fixed + s.round * rounds + (s.turn + (copies ? 0.3f : 0.f)) * rounds * turns + s.load * 1e-3 * tiles * z * turns * s.kg * s.u * (s.mb + s.nb) +
                       s.area * 0.1 * per_cu * s.mb * s.nb + s.dw * mb;
            if (z > 1) t += (copies ? 3.0 : 2.45) + s.part * z * mb;
            else if (g.K != g.Kout && g.opad > 0) t += 2.4;       // sums that padding made NaN: a launch of its own looks
            if (best < 0 || t < *us) { best = i; *us = t; *ranges = (int)z; }
        }
    }
    return best;
}

int wave_dw_launch(int shape, const WgradGeom &g, int ranges, int span, const void *x, const void *dy, void *out, const DwMap *map, bool dw_bf16, int rows,
                   hipStream_t st)
{
    const DwShape &s = kShapes[shape];
    DwParams p{};
    p.x = (const bf16_t *)x; p.dy = (const bf16_t *)dy; p.out = out;
    p.M = g.N * g.P * g.Q;
    p.K = g.K; p.ncols = g.TR * g.TS * g.run; p.rows = rows;
    p.span = span;
    const int n_tiles = (p.ncols + 16 * s.nb - 1) / (16 * s.nb);
    const int k_tiles = (g.K + 16 * s.mb - 1) / (16 * s.mb);
    const long long tiles = (long long)k_tiles * n_tiles;
    if (tiles * ranges > 0x3FFFFFFFll) return MXC_ERR_SHAPE;
    p.tiles = (int)tiles; p.units = (int)(tiles * ranges);
    p.x_bytes = (unsigned)((long long)g.N * g.H * g.W * g.pix * 2);
    p.dy_bytes = (unsigned)((long long)p.M * g.K * 2);
    p.hw_lim = ((g.H - 1) & 0xFFFF) | ((g.W - 1) << 16);
    p.px2 = g.pix * 2; p.row2 = g.W * p.px2; p.img2 = g.H * p.row2;
    p.stride = g.stride; p.pad = g.pad; p.P = g.P; p.Q = g.Q;
    const int adv = 32 * s.kg, rows_adv = adv / g.Q;
    p.adv_q = adv % g.Q; p.adv_p = rows_adv % g.P; p.adv_n = rows_adv / g.P;
    // (several ranges: an XCD has all tiles of one, and either order reads the same)
    const int taps = g.TR * g.TS;
    p.rows_inner = ranges == 1 && rows_inner((p.units + 7) / 8, k_tiles, 16.0 * s.mb, n_tiles, 16.0 * s.nb * (taps > 1 ? 2.0 / taps : 1.0));      // the taps share x
    p.by_tiles = FastDiv(p.tiles); p.by_inner = FastDiv(p.rows_inner ? k_tiles : n_tiles); p.by_q = FastDiv(g.Q); p.by_p = FastDiv(g.P);
    p.by_run = FastDiv(g.run); p.by_ts = FastDiv(g.TS);
    p.mapped = map != nullptr; p.dw_bf16 = dw_bf16;
    if (map) p.map = *map;
    const bool linear = g.TR * g.TS == 1 && g.stride == 1 && g.pad == 0 && g.H == g.P && g.W == g.Q && g.run == g.pix;
    switch (shape) {
#define X(I, MB, NB, KG, U, NS, ...) case I: return launch<MB, NB, KG, U, NS>(p, linear, st);
    SHAPES(X)
#undef X
    default: return MXC_ERR_UNSUPPORTED;
    }
}

}  // namespace mxc
