// The implicit GEMM of igemm.hip for small problems: the waves of a workgroup share a tile's reduction, each with a ring of
// its own.
//
//     Out[m][co] = sum_{t,ci} In[pixel(m) + tap(t)][ci] * Wm[co][t*Ci + ci]
//
// What bounds a GEMM that fills a fraction of the chip is the chain of latencies between its launch and its last store, and
// not bytes or MFMAs.  Here a wave computes its whole tile over every KG-th step of 32 reduction elements, and nothing waits
// at a barrier before the KG partial tiles meet in LDS, where they are added in ascending order (same bits from run to run).
//
// Instruction: v_mfma_f32_16x16x32_bf16, the product formed transposed (filter first): lane 16*g + i holds columns
// 4*g .. 4*g + 3 of a block for pixel i.  Operands pass through LDS although no wave reads another's: the instruction wants
// neighbouring lanes on different rows, and loads in that order run at one lane a clock (37 KB/us per CU, measured; four
// lanes on 64 contiguous bytes: 110).  A block of 16 rows x 32 elements is one direct global->LDS load: lane l brings chunk
// (l%4) ^ (l/16) of row l/4, which makes the ds_read_b128 fetches conflict-free.  A filter that lies transposed (backward-data
// reading the KRSC filter in place: BT) lands as 32 rows of 16*NB columns and is fetched with ds_read_b64_tr_b16.
//
// Measured (us, pixels x columns x reduction, igemm.hip's tile -> this kernel): 392 x 56 x 448 6.4 -> 3.4; 392 x 56 x 576 in 3x3
// taps 6.7 -> 3.7; 2704 x 160 x 1000 10.8 -> 6.0; 46464 x 288 x 24 15.1 -> 10.9.
#include <math.h>
#include <stdlib.h>
#include <string.h>

#include <type_traits>

#include "mxc_internal.h"

namespace mxc {

namespace {

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef bf16x4 __attribute__((address_space(3))) * lds_bf16x4_ptr;
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr unsigned OOB = 0x80000000u;   // a buffer offset no operand reaches: the load returns zeros
constexpr int FAR = (-16384) & 0xFFFF;  // a packed position that is outside whatever is added to it

// The output pixels of a launch, or of one residue class of strided backward-data: an Mh x Mw grid per image and its taps.
struct WaveGrid {
    FastDiv by_mw, by_mh;
    int M, Kd, turns, TS, ts_magic;   // rows, reduction, a wave's sets of steps; taps: divisor of the tap index
    int off_h, off_w;                 // input position of tap 0: grid position * mul + off
    int out_off_h, out_off_w;
    int tile0, tap0, tap_row, tap_col;        // classes: first row tile; class tap (j, q) is the filter's tap0 + j*tap_row + q*tap_col
    unsigned wm_off;                  // bytes before the class's matrix in a re-packed filter
};
struct WaveParams {
    const bf16_t *in, *wm;
    bf16_t *out;
    const float *bias;
    const bf16_t *mask;
    unsigned in_bytes, wm_bytes;
    WaveGrid grid;
    int units, Co, Cw, Ci, T;         // T: taps of the filter
    int hw_lim;                       // last row and column of the image, packed
    int px2, row2, img2;              // bytes from pixel to pixel, row to row, image to image
    int mul_h, mul_w;
    int tap_h, tap_w, th2, tv2;       // a tap's steps in pixels and in bytes
    int row_inner;                    // tap t = (column step)*TR + (row step)
    FastDiv by_inner, by_ci;
    int rows_inner;                   // the tiles of a column follow each other, not those of a row
    int kq, kr;                       // a wave's step of KG*32 reduction elements as taps + channels
    int linear_out, Ho, Wo, out_mul_h, out_mul_w;
    int relu;
    int cols;                         // PLANES: the result's planes per image
};
constexpr int MAX_CLASSES = 4;
struct WaveClassParams : WaveParams { WaveGrid cls[MAX_CLASSES]; int n_cls; };

// How a step's 32 reduction elements lie: anyhow; in one tap, the same for all lanes (Ci % 32 == 0: the tap arithmetic is
// scalar); or there is one tap and every pixel is inside the image (a 1x1 filter without padding, Ci % 32 == 0 too).
enum { STEP_ANY = 0, STEP_TAP = 1, STEP_1X1 = 2 };

template <int N> __device__ __forceinline__ void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ void wait_lgkmcnt0() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// MB x NB blocks of 16 pixels x 16 columns per wave, a ring of NS sets of U steps; KG waves share a tile's reduction, MG of
// them stand side by side along the pixels.
// PLANES: the operands are NHWC copies of an NCHW problem and the result goes straight to its planes: the product is formed the other
// way round, lane 16*g + i holds pixels 4*g .. 4*g + 3 of column i.  One launch and one pass over the result less (us, forward
// and dx): 32 to 32 channels 3x3 on 4 20x20 images 8.2 -> 6.0, 9.4 -> 7.3; 96 to 128 1x1 on 64 14x14 13.3 -> 9.1, 14.3 -> 10.9.
template <int MB, int NB, int KG, int MG, int U, int NS, bool BT, int STEP, bool PLANES, bool CLASSES>
__global__ __launch_bounds__(64 * KG * MG) void wave_kernel(const std::conditional_t<CLASSES, WaveClassParams, WaveParams> p)
{
    constexpr int BM = 16 * MB * MG, BN = 16 * NB, NW = KG * MG;
    constexpr int BLK = 512;                                        // elements of a block: 16 rows x 32
    constexpr int SET = U * (MB + NB) * BLK, RING = NS * SET;       // elements of a set, and of a wave's ring
    constexpr int L = U * (MB + NB);                                // loads per set
    static_assert(L * (NS - 1) < 64, "vmcnt range");
    static_assert(KG == 1 || MB * NB * 256 * 2 <= RING, "a wave's partial tile must fit its ring");
    static_assert(NB == 1 || NB % 2 == 0, "results leave in pairs of blocks");
    static_assert(!BT || NB == 2 || NB == 4, "rows of a transposed filter tile");
    __shared__ __attribute__((aligned(1024))) bf16_t ring[NW * RING];

    const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int kg = wave % KG, mg = wave / KG;
    bf16_t *mine = ring + wave * RING;
    // consecutive workgroups go round-robin to the 8 XCDs; each XCD gets a contiguous range of tiles
    const int per_xcd = (p.units + 7) / 8;
    const int unit = ((int)blockIdx.x & 7) * per_xcd + ((int)blockIdx.x >> 3);
    if (unit >= p.units) return;
    const int outer = p.by_inner.div(unit), inner = unit - outer * p.by_inner.d;
    const int n0 = (p.rows_inner ? outer : inner) * BN;
    int m_tile = p.rows_inner ? inner : outer;
    const WaveGrid *grid = &p.grid;
    if constexpr (CLASSES) {
        int c = 0;
        while (c + 1 < p.n_cls && m_tile >= p.cls[c + 1].tile0) ++c;
        grid = &p.cls[c];
        m_tile -= grid->tile0;
    }
    const WaveGrid &gr = *grid;
    const int m0 = m_tile * BM + mg * 16 * MB;

    const buf_rsrc_t rs_in = make_buf_rsrc(p.in, p.in_bytes);
    const buf_rsrc_t rs_wm = make_buf_rsrc(p.wm, p.wm_bytes);

    // ---- what this lane loads: row l/4 of every block, chunk (l%4) ^ (l/16) of its step ------------------------------
    const int ld_row = lane >> 2, chunk = ((lane & 3) ^ (lane >> 4)) * 8;
    int a_off[MB], a_hw[MB];       // byte offset and position of tap 0
#pragma unroll
    for (int b = 0; b < MB; ++b) {
        const int m = m0 + 16 * b + ld_row;
        const int t = gr.by_mw.div(m), col = m - t * gr.by_mw.d, n = gr.by_mh.div(t), row = t - n * gr.by_mh.d;
        const int h = row * p.mul_h + gr.off_h, w = col * p.mul_w + gr.off_w;
        a_off[b] = n * p.img2 + h * p.row2 + w * p.px2;
        a_hw[b] = m < gr.M ? (h & 0xFFFF) | (w << 16) : FAR;
    }
    if constexpr (STEP == STEP_1X1) {
#pragma unroll
        for (int b = 0; b < MB; ++b) a_off[b] = a_hw[b] == FAR ? (int)OOB : a_off[b] + chunk * 2;
    }
    // position in the reduction: kd = tap*Ci + ci, of the lane's own chunk (STEP_ANY) or of the step
    const int in_kd = STEP == STEP_ANY ? chunk : 0, in_off = chunk - in_kd;
    int kd = kg * 32 + in_kd;
    int tap = STEP == STEP_1X1 ? 0 : p.by_ci.div(kd), ci = kd - tap * p.Ci;
    // filter rows; of a transposed one the columns of 16-byte chunk bt_c, whose row within a load is bt_r
    constexpr int BCH = BT ? 2 * NB : 4, BROWS = 64 / BCH;          // BT: chunks per row, rows per load
    const int bt_r = lane / BCH;
    unsigned f_off[NB];
    if constexpr (BT) {
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int r = BROWS * j + bt_r, c = (lane % BCH) ^ (NB == 2 ? ((r >> 3) & 1) << 1 : ((r >> 1) & 1) << 1 | ((r >> 3) & 1) << 2);
            f_off[j] = n0 + c * 8 < p.Co ? (unsigned)(n0 + c * 8) * 2u : OOB;
        }
    } else {
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int co = n0 + 16 * j + ld_row;
            f_off[j] = co < p.Cw ? ((unsigned)co * (unsigned)gr.Kd + (unsigned)in_off) * 2u + (CLASSES ? gr.wm_off : 0u) : OOB;
        }
    }
    // BT: (tap, k) of the lane's filter rows: row k0 + BROWS*j + bt_r of the step.  With whole steps per tap the tap is the step's.
    [[maybe_unused]] int bt_kd = kg * 32;

    auto issue = [&](bf16_t *dst) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bool k_ok = kd < gr.Kd;
            bf16_t *to = dst + u * (MB + NB) * BLK;
            if constexpr (STEP == STEP_1X1) {
                // (an offset beyond the resource stays there: kd*2 < 2^31)
#pragma unroll
                for (int b = 0; b < MB; ++b) lds_dma16(rs_in, k_ok ? (unsigned)a_off[b] + (unsigned)kd * 2u : OOB, to + b * BLK);
            } else {
                const int q = small_div(tap, gr.ts_magic), rem = tap - q * gr.TS;
                const int th = p.row_inner ? rem : q, tv = p.row_inner ? q : rem;
                const int t_hw = k_ok ? (th * p.tap_h & 0xFFFF) | (tv * p.tap_w) << 16 : FAR;
                const int base = th * p.th2 + tv * p.tv2 + ci * 2 + in_off * 2;
#pragma unroll
                for (int b = 0; b < MB; ++b) {
                    const s16x2 hw = __builtin_bit_cast(s16x2, a_hw[b]) + __builtin_bit_cast(s16x2, t_hw);
                    const s16x2 d = __builtin_bit_cast(s16x2, p.hw_lim) - hw;
                    const int bad = (__builtin_bit_cast(int, hw) | __builtin_bit_cast(int, d)) & (int)0x80008000;
                    lds_dma16(rs_in, bad == 0 ? (unsigned)(a_off[b] + base) : OOB, to + b * BLK);
                }
            }
            if constexpr (BT) {
                // filter row (k, tap) lies at (k*T + tap)*Co
                auto filter_tap = [&](int t) __attribute__((always_inline)) {
                    if constexpr (!CLASSES) return t;
                    const int q = small_div(t, gr.ts_magic);
                    return gr.tap0 + q * gr.tap_row + (t - q * gr.TS) * gr.tap_col;
                };
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    const int at = bt_kd + BROWS * j + bt_r;                   // reduction element of this lane's row
                    int t = 0, k = at;
                    if constexpr (STEP == STEP_TAP) { t = tap; k = ci + BROWS * j + bt_r; }
                    if constexpr (STEP == STEP_ANY) { t = p.by_ci.div(at); k = at - t * p.Ci; }
                    lds_dma16(rs_wm, at < gr.Kd && f_off[j] != OOB ? f_off[j] + (unsigned)(k * p.T + filter_tap(t)) * (unsigned)(p.Co * 2) : OOB,
                              to + (MB + j) * BLK);
                }
            } else {
#pragma unroll
                for (int j = 0; j < NB; ++j)
                    lds_dma16(rs_wm, k_ok && f_off[j] != OOB ? f_off[j] + (unsigned)kd * 2u : OOB, to + (MB + j) * BLK);
            }
            kd += KG * 32;
            bt_kd += KG * 32;
            if constexpr (STEP != STEP_1X1) {
                ci += p.kr;
                const int carry = ci >= p.Ci ? 1 : 0;
                ci -= carry ? p.Ci : 0;
                tap += p.kq + carry;
            }
        }
    };
    f32x4 acc[MB][NB];
#pragma unroll
    for (int b = 0; b < MB; ++b)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[b][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // ---- fragments: lane 16*g + i fetches chunk g of row i; BT: eight rows 8*g .. of column i, four at a time ----------
    const int frag = i * 32 + ((g ^ (i >> 2)) & 3) * 8;
    int tr[BT ? NB : 1];
    if constexpr (BT) {
        const int r = 8 * g + (i >> 2);           // the second read's rows are 4 further on, which changes none of the swizzled bits
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int c = 2 * j + ((i & 3) >> 1);
            const int swz = c ^ (NB == 2 ? ((r >> 3) & 1) << 1 : ((r >> 1) & 1) << 1 | ((r >> 3) & 1) << 2);
            tr[j] = r * BN + swz * 8 + (i & 1) * 4;
        }
    }
    auto step = [&](bf16_t *src, bool refill) __attribute__((always_inline)) {
        bf16x8 fa[U][MB], fw[U][NB];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const bf16_t *from = src + u * (MB + NB) * BLK;
#pragma unroll
            for (int b = 0; b < MB; ++b) fa[u][b] = *reinterpret_cast<const bf16x8 *>(from + b * BLK + frag);
            from += MB * BLK;
#pragma unroll
            for (int j = 0; j < NB; ++j) {
                if constexpr (BT) {
                    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(from + tr[j]));
                    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(from + tr[j] + 4 * BN));
                    fw[u][j] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                } else fw[u][j] = *reinterpret_cast<const bf16x8 *>(from + j * BLK + frag);
            }
        }
        wait_lgkmcnt0();                          // the slot's operands are in registers: it may be refilled
        __builtin_amdgcn_sched_barrier(0);
        if (refill) issue(src);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int b = 0; b < MB; ++b)
#pragma unroll
                for (int j = 0; j < NB; ++j) acc[b][j] = PLANES ? __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[u][b], fw[u][j], acc[b][j], 0, 0, 0)
                                             : __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[u][j], fa[u][b], acc[b][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    // gr.turns sets, of which the last NS are not followed by a refill.  Loads retire in order, so all but the youngest (NS - 1)*L
    // being done means that the oldest set has landed.
    const int ahead = min(gr.turns, NS);
#pragma unroll
    for (int q = 0; q < NS; ++q)
        if (q < ahead) issue(mine + q * SET);
    int slot = 0;
    for (int t = gr.turns; t > NS; --t) {
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

    // ---- results: this lane's columns n0 + 16*j + 4*g .. + 3 of pixel m0 + 16*b + i -------------------------------------
    const bool whole = NB > 1 && (p.Co & 7) == 0;     // uniform: results leave 16 bytes at a time
    const bool masked = p.mask != nullptr && (!CLASSES || gr.Kd > 0);      // (what no tap reaches is 0 whatever the mask says)
    const out_rsrc_t rs_bias = make_out_rsrc(const_cast<float *>(p.bias), p.bias != nullptr ? (unsigned)p.Cw * 4u : 0u);
    float bias[4 * NB];
    u32x4 mask[NB > 1 ? NB / 2 : 1];
    long long at;                                     // the pixel's first element in the result, or -1
    // of blocks j and j + 1, 16 bytes leave as columns n0 + col16(j) .. + 7: the lanes of odd g take block j + 1
    auto col16 = [&](int j) __attribute__((always_inline)) { return 16 * (j + (g & 1)) + 8 * (g >> 1); };
    // PLANES: pixels m0 + 16*b + 4*g .. + 3, element 0's place in the first plane of its image, or -1
    const int plane = PLANES ? gr.by_mw.d * gr.by_mh.d : 0;
    int pix = 0;
    auto image_of = [&](int m) __attribute__((always_inline)) { return gr.by_mh.div(gr.by_mw.div(m)); };
    auto store_planes = [&](const f32x4 (&v)[NB]) __attribute__((always_inline)) {
        if (pix >= gr.M) return;
        const bool quad = (plane & 3) == 0;            // (then the four are of one image, and lie on 8 bytes)
        const int n0_img = image_of(pix), n3_img = quad ? n0_img : image_of(pix + 3);
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int col = n0 + 16 * j + i;
            if (col >= p.cols) continue;
            uint32_t k[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                k[h] = pack_bf16x2(v[j][2 * h] + bias[j], v[j][2 * h + 1] + bias[j]);
                if (p.relu) k[h] = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2, k[h]), s16x2{0, 0}));
            }
            if (quad) {
                const long long to = ((long long)n0_img * p.cols + col) * plane + (pix - n0_img * plane);
                uint2 o = make_uint2(k[0], k[1]);
                if (p.mask != nullptr) {
                    const uint2 mk = *reinterpret_cast<const uint2 *>(p.mask + to);
                    o = make_uint2(mask_bf16x2(o.x, mk.x), mask_bf16x2(o.y, mk.y));
                }
                *reinterpret_cast<uint2 *>(p.out + to) = o;
                continue;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int m = pix + e, n = n0_img == n3_img ? n0_img : image_of(m);
                if (m >= gr.M) break;
                const long long to = ((long long)n * p.cols + col) * plane + (m - n * plane);
                const bf16_t r = (bf16_t)(k[e >> 1] >> ((e & 1) * 16));
                p.out[to] = (p.mask == nullptr || mask_keeps(p.mask + to)) ? r : (bf16_t)0;
            }
        }
    };
    // everything that does not depend on the sums
    auto locate = [&](int b) __attribute__((always_inline)) {
        if constexpr (PLANES) {
            pix = m0 + 16 * b + 4 * g;
            return;
        }
        const int m = m0 + 16 * b + i;
        at = (long long)m * p.Co + n0;
        if (!p.linear_out) {
            const int t = gr.by_mw.div(m), col = m - t * gr.by_mw.d, n = gr.by_mh.div(t), row = t - n * gr.by_mh.d;
            at = (((long long)n * p.Ho + (row * p.out_mul_h + gr.out_off_h)) * p.Wo + (col * p.out_mul_w + gr.out_off_w)) * p.Co + n0;
        }
        if (m >= gr.M) at = -1;
        if (whole && masked) {
#pragma unroll
            for (int j = 0; j < NB; j += 2)
                mask[j / 2] = at >= 0 && n0 + col16(j) < p.Co ? *reinterpret_cast<const u32x4 *>(p.mask + at + col16(j)) : u32x4{0, 0, 0, 0};
        }
    };
    auto fetch_bias = [&]() __attribute__((always_inline)) {
        if constexpr (PLANES) {
#pragma unroll
            for (int j = 0; j < NB; ++j)
                bias[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs_bias, (n0 + 16 * j + i) * 4, 0, 0));
            return;
        }
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                bias[4 * j + e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rs_bias, (n0 + 16 * j + 4 * g + e) * 4, 0, 0));
    };
    struct __attribute__((packed)) Packed8 { uint32_t lo, hi; };
    auto store = [&](const f32x4 (&v)[NB]) __attribute__((always_inline)) {
        if constexpr (PLANES) return store_planes(v);
        float r[4 * NB];
#pragma unroll
        for (int c = 0; c < 4 * NB; ++c) {
            r[c] = v[c / 4][c % 4] + bias[c];
            if (p.relu && !whole) r[c] = fmaxf(r[c], 0.f);
        }
        if (whole) {
            auto pair = [&](int c) __attribute__((always_inline)) {        // ReLU as a 16-bit integer maximum on the rounded pair
                const uint32_t k = pack_bf16x2(r[c], r[c + 1]);
                return p.relu ? __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2, k), s16x2{0, 0})) : k;
            };
#pragma unroll
            for (int j = 0; j + 1 < NB; j += 2) {
                // lanes of even g keep block j and get the next four columns of it, those of odd g likewise of block j + 1
                typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
                const u32x2 s0 = __builtin_amdgcn_permlane16_swap(pair(4 * j), pair(4 * j + 4), false, false);
                const u32x2 s1 = __builtin_amdgcn_permlane16_swap(pair(4 * j + 2), pair(4 * j + 6), false, false);
                u32x4 o = {s0.x, s1.x, s0.y, s1.y};
                if (masked) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = mask_bf16x2(o[e], mask[j / 2][e]);
                }
                if (at >= 0 && n0 + col16(j) < p.Co) *reinterpret_cast<u32x4 *>(p.out + at + col16(j)) = o;
            }
            return;
        }
        if (at < 0) return;
        // four columns at a time (8 bytes at any alignment), the last ones element by element
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int c = 16 * j + 4 * g;
            if (n0 + c + 4 <= p.Co) {
                Packed8 o{pack_bf16x2(r[4 * j], r[4 * j + 1]), pack_bf16x2(r[4 * j + 2], r[4 * j + 3])};
                if (p.mask != nullptr) {
                    const Packed8 mk = *reinterpret_cast<const Packed8 *>(p.mask + at + c);
                    o = Packed8{mask_bf16x2(o.lo, mk.lo), mask_bf16x2(o.hi, mk.hi)};
                }
                *reinterpret_cast<Packed8 *>(p.out + at + c) = o;
            } else {
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if (n0 + c + e < p.Co)
                        p.out[at + c + e] = (p.mask == nullptr || mask_keeps(p.mask + at + c + e)) ? f32_to_bf16(r[4 * j + e]) : (bf16_t)0;
            }
        }
    };
    if constexpr (KG == 1) {
        fetch_bias();
#pragma unroll
        for (int b = 0; b < MB; ++b) { locate(b); store(acc[b]); }
    } else {
        static_assert(MB <= KG || MB % KG == 0, "wave kg finishes pixel blocks kg, kg + KG, ...");
        // partial tiles in the waves' own rings (nothing is landing there any more)
        f32x4 *part = reinterpret_cast<f32x4 *>(ring);
        constexpr int PITCH = RING / 8;
#pragma unroll
        for (int b = 0; b < MB; ++b)
#pragma unroll
            for (int j = 0; j < NB; ++j) part[wave * PITCH + (b * NB + j) * 64 + lane] = acc[b][j];
        if (kg < MB) { fetch_bias(); locate(kg); }
        __syncthreads();
        if (kg < MB) {
#pragma unroll
            for (int b0 = 0; b0 < MB; b0 += KG) {
                const int b = b0 + kg;
                if (b0 > 0) locate(b);
                f32x4 v[NB];
#pragma unroll
                for (int j = 0; j < NB; ++j) v[j] = part[mg * KG * PITCH + (b * NB + j) * 64 + lane];
#pragma unroll
                for (int z = 1; z < KG; ++z)
#pragma unroll
                    for (int j = 0; j < NB; ++j) v[j] += part[(mg * KG + z) * PITCH + (b * NB + j) * 64 + lane];
                store(v);
            }
        }
    }
}

// The shapes and, for each, the time model that picks one (us, fitted to 828 GEMMs of 16 to 656 thousand rows on the device,
// 5-13% off): fixed + kb * (100 KB that the CU with most tiles loads) + round * (rounds of workgroups that fit a CU)
// + turn * (rounds times sets of loads) + out * (MB written, and of the mask read) + area * (thousand results of that CU).
struct WaveShape { int mb, nb, kg, mg, u, ns; const char *name; float fixed, kb, round, turn, out, area; };
#define SHAPES(X) \
    X(0, 1, 1, 8, 1, 2, 3, "igemm_wave_16x16_split8", 3.00f, 0.f, 0.185f, 0.320f, 2.01f, 0.f) \
    X(1, 1, 2, 8, 1, 2, 2, "igemm_wave_16x32_split8", 2.83f, 0.f, 0.386f, 0.447f, 0.962f, 0.f) \
    X(2, 2, 2, 8, 1, 1, 4, "igemm_wave_32x32_split8", 2.53f, 0.f, 0.f, 0.291f, 0.403f, 0.806f) \
    X(3, 4, 2, 8, 1, 1, 3, "igemm_wave_64x32_split8", 1.85f, 0.f, 0.f, 0.416f, 0.205f, 0.755f) \
    X(4, 4, 4, 8, 1, 1, 2, "igemm_wave_64x64_split8", 1.48f, 0.f, 0.f, 0.585f, 0.195f, 0.570f) \
    X(5, 4, 2, 4, 2, 1, 3, "igemm_wave_128x32_split4", 1.63f, 0.f, 0.f, 0.422f, 0.162f, 0.420f) \
    X(6, 2, 2, 2, 4, 1, 2, "igemm_wave_128x32_split2", 2.31f, 0.847f, 0.851f, 0.f, 0.110f, 0.032f) \
    X(7, 2, 2, 1, 4, 1, 2, "igemm_wave_128x32", 2.80f, 0.883f, 0.575f, 0.022f, 0.125f, 0.f) \
    X(8, 2, 4, 1, 4, 1, 2, "igemm_wave_128x64", 2.87f, 0.741f, 0.566f, 0.075f, 0.149f, 0.f) \
    X(9, 4, 4, 1, 4, 1, 2, "igemm_wave_256x64", 3.24f, 0.847f, 0.668f, 0.096f, 0.177f, 0.f)
#define X(I, MB, NB, KG, MG, U, NS, NAME, ...) {MB, NB, KG, MG, U, NS, NAME, __VA_ARGS__},
const WaveShape kShapes[] = {SHAPES(X)};
#undef X
constexpr int N_SHAPES = sizeof(kShapes) / sizeof(kShapes[0]);
// those that strided backward-data is built in
#define CLASS_SHAPES(X) X(2, 2, 2, 8, 1, 1, 4) X(3, 4, 2, 8, 1, 1, 3) X(5, 4, 2, 4, 2, 1, 3) X(7, 2, 2, 1, 4, 1, 2) X(8, 2, 4, 1, 4, 1, 2)
static bool has_classes(int shape) { return shape == 2 || shape == 3 || shape == 5 || shape == 7 || shape == 8; }

template <int MB, int NB, int KG, int MG, int U, int NS, bool BT, bool PLANES>
void launch_step(const WaveParams &p, int step, hipStream_t st)
{
    const dim3 grid((unsigned)((p.units + 7) / 8 * 8)), block(64 * KG * MG);
    if (step == STEP_1X1) hipLaunchKernelGGL((wave_kernel<MB, NB, KG, MG, U, NS, BT, STEP_1X1, PLANES, false>), grid, block, 0, st, p);
    else if (step == STEP_TAP) hipLaunchKernelGGL((wave_kernel<MB, NB, KG, MG, U, NS, BT, STEP_TAP, PLANES, false>), grid, block, 0, st, p);
    else hipLaunchKernelGGL((wave_kernel<MB, NB, KG, MG, U, NS, BT, STEP_ANY, PLANES, false>), grid, block, 0, st, p);
}

// strided backward-data: all residue classes in one launch, those no tap reaches with a reduction of nothing
template <int MB, int NB, int KG, int MG, int U, int NS>
int launch_classes(WaveClassParams &p, bool bt, hipStream_t st)
{
    long long m_tiles = 0;
    for (int c = 0; c < p.n_cls; ++c) {
        p.cls[c].tile0 = (int)m_tiles;
        p.cls[c].turns = (p.cls[c].Kd + 32 * KG * U - 1) / (32 * KG * U);
        m_tiles += ((long long)p.cls[c].M + 16 * MB * MG - 1) / (16 * MB * MG);
    }
    const int n_tiles = (p.Co + 16 * NB - 1) / (16 * NB);
    if (m_tiles * n_tiles > 0x3FFFFFFFll || m_tiles * 16 * MB * MG > 0x7FFFFFFFll) return MXC_ERR_SHAPE;
    p.units = (int)(m_tiles * n_tiles);
    p.by_inner = FastDiv(n_tiles);
    p.kq = 32 * KG / p.Ci; p.kr = 32 * KG % p.Ci;
    const dim3 grid((unsigned)((p.units + 7) / 8 * 8)), block(64 * KG * MG);
    const bool tap = p.Ci % 32 == 0;
    if (bt && tap) hipLaunchKernelGGL((wave_kernel<MB, NB, KG, MG, U, NS, true, STEP_TAP, false, true>), grid, block, 0, st, p);
    else if (bt) hipLaunchKernelGGL((wave_kernel<MB, NB, KG, MG, U, NS, true, STEP_ANY, false, true>), grid, block, 0, st, p);
    else if (tap) hipLaunchKernelGGL((wave_kernel<MB, NB, KG, MG, U, NS, false, STEP_TAP, false, true>), grid, block, 0, st, p);
    else hipLaunchKernelGGL((wave_kernel<MB, NB, KG, MG, U, NS, false, STEP_ANY, false, true>), grid, block, 0, st, p);
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
}

template <int MB, int NB, int KG, int MG, int U, int NS>
int launch(WaveParams &p, int step, bool bt, hipStream_t st)
{
    const long long m_tiles = ((long long)p.grid.M + 16 * MB * MG - 1) / (16 * MB * MG);
    const int n_tiles = (p.Co + 16 * NB - 1) / (16 * NB);
    if (m_tiles * n_tiles > 0x3FFFFFFFll || m_tiles * 16 * MB * MG > 0x7FFFFFFFll) return MXC_ERR_SHAPE;
    p.units = (int)(m_tiles * n_tiles);
    // A pixel's channels are read by all its taps, a filter row T times as long by one tile of columns.  Column tiles followed each other
    // before: 128 x 4096 to 1000 classes 11.9 us, now 7.1 (each XCD read all of the filter); 8x7x7 512 to 512 3x3 forward 11.4 -> 8.6,
    // dx 15.0 -> 10.1.
    p.rows_inner = rows_inner((p.units + 7) / 8, m_tiles, 16.0 * MB * MG * (p.T > 1 ? 2 : 1), n_tiles, 16.0 * NB * p.T);
    p.by_inner = FastDiv(p.rows_inner ? (int)m_tiles : n_tiles);
    p.grid.turns = (p.grid.Kd + 32 * KG * U - 1) / (32 * KG * U);
    p.kq = 32 * KG / p.Ci; p.kr = 32 * KG % p.Ci;
    if constexpr (NB >= 2) {
        if (bt && p.cols == 0) launch_step<MB, NB, KG, MG, U, NS, true, false>(p, step, st);
    }
    if (bt && (NB < 2 || p.cols != 0)) return MXC_ERR_UNSUPPORTED;
    if (!bt && p.cols == 0) launch_step<MB, NB, KG, MG, U, NS, false, false>(p, step, st);
    if (!bt && p.cols != 0) launch_step<MB, NB, KG, MG, U, NS, false, true>(p, step, st);
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
}

}  // namespace

const char *wave_name(int shape) { return shape >= 0 && shape < N_SHAPES ? kShapes[shape].name : nullptr; }

int wave_forced(const char *name, bool bwd)
{
    for (int i = 0; i < N_SHAPES; ++i)
        if (!strcmp(name, kShapes[i].name) && !(bwd && kShapes[i].nb == 1)) return i;
    return -1;
}

int wave_best(long long M, int Co, int Kd, bool bwd, bool masked, double *us)
{
    int best = -1;
    if (M > 1 << 30) return -1;            // row numbers up to a tile beyond M stay below 2^31
    for (int i = bwd ? 1 : 0; i < N_SHAPES; ++i) {
        const WaveShape &s = kShapes[i];
        const int bm = 16 * s.mb * s.mg, bn = 16 * s.nb, nw = s.kg * s.mg;
        const long long per_cu = ((M + bm - 1) / bm * ((Co + bn - 1) / bn) + 255) / 256;
        const int turns = (Kd + 32 * s.kg * s.u - 1) / (32 * s.kg * s.u), slots = 160 / (nw * s.ns * s.u * (s.mb + s.nb));
        const double rounds = (double)((per_cu + slots - 1) / slots);
        const double t = s.fixed + s.kb * per_cu * nw * turns * s.u * (s.mb + s.nb) * 0.01 + s.round * rounds + s.turn * rounds * turns +
                         s.out * (masked ? 4e-6 : 2e-6) * M * Co + s.area * per_cu * bm * bn * 1e-3;
        if (best < 0 || t < *us) { best = i; *us = t; }
    }
    return best;
}

// what the launches of all forms share
static void fill_common(WaveParams &p, const IgemmParams &q)
{
    p.in = q.in; p.wm = q.wm; p.out = q.out; p.bias = q.bias; p.mask = q.mask; p.relu = q.relu;
    p.Co = q.Co; p.Cw = q.Cw ? q.Cw : q.Co; p.Ci = q.Ci;
    p.in_bytes = (unsigned)((long long)q.N * q.Hi * q.Wi * q.pix * 2);
    p.hw_lim = ((q.Hi - 1) & 0xFFFF) | ((q.Wi - 1) << 16);
    p.px2 = q.pix * 2; p.row2 = q.Wi * p.px2; p.img2 = q.Hi * p.row2;
    p.mul_h = q.in_mul_h; p.mul_w = q.in_mul_w;
    p.row_inner = q.tap_row_inner;
    p.tap_h = q.tstep_h; p.tap_w = q.tstep_w;
    p.th2 = q.tstep_h * p.row2; p.tv2 = q.tstep_w * p.px2;
    p.by_ci = FastDiv(q.Ci);
    p.Ho = q.Ho; p.Wo = q.Wo; p.out_mul_h = q.out_mul_h; p.out_mul_w = q.out_mul_w;
}

int wave_launch(int shape, const IgemmParams &q, hipStream_t st, bool bt, PlaneOut *planes)
{
    WaveParams p{};
    fill_common(p, q);
    p.T = q.TR * q.TS;
    WaveGrid &gr = p.grid;
    gr.M = (int)((long long)q.N * q.Mh * q.Mw);
    gr.Kd = p.T * q.Ci;
    gr.off_h = q.in_off_h; gr.off_w = q.in_off_w; gr.out_off_h = q.out_off_h; gr.out_off_w = q.out_off_w;
    gr.TS = q.tap_row_inner ? q.TR : q.TS;
    gr.ts_magic = small_magic(gr.TS);
    gr.by_mw = FastDiv(q.Mw); gr.by_mh = FastDiv(q.Mh);
    p.wm_bytes = bt ? q.bt_w_bytes : (unsigned)((long long)p.Cw * gr.Kd * 2);
    p.linear_out = (q.out_mul_h == 1 && q.out_mul_w == 1 && q.out_off_h == 0 && q.out_off_w == 0 && q.Mh == q.Ho && q.Mw == q.Wo) ? 1 : 0;
    if (planes != nullptr && p.linear_out && !bt) {
        p.out = (bf16_t *)planes->out; p.mask = (const bf16_t *)planes->mask; p.cols = planes->cols;
        planes->stored = true;
    }
    const bool inside = p.T == 1 && q.in_off_h >= 0 && q.in_off_w >= 0 && (q.Mh - 1) * q.in_mul_h + q.in_off_h < q.Hi && (q.Mw - 1) * q.in_mul_w + q.in_off_w < q.Wi;
    const int step = q.Ci % 32 != 0 ? STEP_ANY : inside ? STEP_1X1 : STEP_TAP;
    switch (shape) {
#define X(I, MB, NB, KG, MG, U, NS, ...) case I: return launch<MB, NB, KG, MG, U, NS>(p, step, bt, st);
    SHAPES(X)
#undef X
    default: return MXC_ERR_UNSUPPORTED;
    }
}

bool wave_has_classes(int shape) { return has_classes(shape); }

// The residue classes of dx at stride 2, in the order (ph, pw): rows of the GEMM and the taps of each.
struct ClassDims { int Mh, Mw, TR, TS, off_h, off_w, out_off_h, out_off_w; };
static ClassDims class_dims(const ConvShape &s, int ph, int pw)
{
    ClassDims c{};
    c.TR = ph < s.R ? (s.R - ph + s.stride - 1) / s.stride : 0; c.TS = pw < s.S ? (s.S - pw + s.stride - 1) / s.stride : 0;
    // output rows h = ph - pad + stride*hh >= 0, h < H
    c.off_h = ph >= s.pad ? 0 : (s.pad - ph + s.stride - 1) / s.stride;
    c.off_w = pw >= s.pad ? 0 : (s.pad - pw + s.stride - 1) / s.stride;
    c.out_off_h = ph - s.pad + s.stride * c.off_h; c.out_off_w = pw - s.pad + s.stride * c.off_w;
    c.Mh = c.out_off_h < s.H ? (s.H - 1 - c.out_off_h) / s.stride + 1 : 0;
    c.Mw = c.out_off_w < s.W ? (s.W - 1 - c.out_off_w) / s.stride + 1 : 0;
    return c;
}

// The shape for dx at stride 2 and its modelled time (us, fitted to 160 layers of up to 20 GFLOP, 9-13% off): fixed + turn * (tiles times
// steps per wave and CU, at least the longest class's) + longest * (the longest class's steps) + tile * (tiles per CU) + mb * (MB written and
// of the mask read, which is where a tap reaches); and that of the re-packed filter and the tile kernel's launch over the classes (8%
// off).  A 1x1 filter reaches one class of four and zeros are a launch of their own: a fit of its own, to 294 layers with and without a
// mask, 9% off.  (With the mask of all pixels counted in a fit for both it was a quarter too long for masked layers, and layers went to the
// wave kernel that take longer there: 63 images of 29x29, 216 to 176 channels 15.7 us and 26.6, 146 of 42x42, 192 to 176 37.5 and 67.7.)
int wave_best_classes(const ConvShape &s, bool masked, double *us, double *other)
{
    static const struct { int shape; float fixed, turn, longest, tile, mb; } kUs[] = {
        {2, 2.44f, 0.492f, 0.114f, 1.28f, 1.20f}, {3, 2.57f, 0.603f, 0.f, 1.34f, 1.00f}, {5, 2.71f, 0.538f, 0.f, 1.28f, 0.809f},
        {7, 3.24f, 0.258f, 0.112f, 0.611f, 0.046f}, {8, 3.32f, 0.353f, 0.197f, 0.856f, 0.098f}};
    // 1x1 filters, of which three classes have no tap: fitted to 5386 layers, those below 16 us, 3% off (8 waves a tile) and 5-6%.  Their tiles of
    // zeros count like the others where a CU holds one workgroup at a time: one tile more than the chip has CUs is 1.7 to 2.5 us (12 images
    // of 16x16, 96 to 448 channels: 288 tiles of 32x32 7.1 us, 144 of 64x32 5.1).  Of 3007 layers the shape chosen takes 0.5% more than the
    // fastest; with tiles counted in fractions of the chip 1.5%, and a tenth to 1.42 times as long in 125.
    static const struct { int shape; float fixed, longest, round, work, tile, mb; } kUs1x1[] = {
        {2, 3.93f, 0.227f, 1.70f, 1.22f, 0.f, 0.f}, {3, 4.21f, 0.325f, 2.18f, 1.50f, 0.f, 0.f}, {5, 4.29f, 0.373f, 2.46f, 1.77f, 0.f, 0.f},
        {7, 3.91f, 0.301f, 0.962f, 0.399f, 0.165f, 0.177f}, {8, 4.33f, 0.468f, 1.91f, 0.390f, 0.173f, 0.150f}};
    const bool one = s.R * s.S == 1;
    double gflop = 0, zeros = 0, longest = 0, mb = 0;
    int best = -1;
    for (int i = 0; i < 5; ++i) {
        const WaveShape &w = kShapes[one ? kUs1x1[i].shape : kUs[i].shape];
        const int bm = 16 * w.mb * w.mg, n_tiles = (s.C + 16 * w.nb - 1) / (16 * w.nb);
        double tiles = 0, steps = 0, most = 0;
        gflop = zeros = longest = mb = 0;
        for (int ph = 0; ph < s.stride; ++ph)
            for (int pw = 0; pw < s.stride; ++pw) {
                const ClassDims c = class_dims(s, ph, pw);
                if (c.Mh <= 0 || c.Mw <= 0) continue;
                const double rows = (double)s.N * c.Mh * c.Mw, t = (double)(long long)((rows + bm - 1) / bm);
                const int Kd = c.TR * c.TS * s.K, turns = (Kd + 32 * w.kg - 1) / (32 * w.kg);
                tiles += t * n_tiles / 256; steps += t * n_tiles * turns / 256;
                if (turns > most) most = turns;
                if (Kd > longest) longest = Kd;
                gflop += 2e-9 * rows * Kd * ((s.C + 63) / 64 * 64);
                if (Kd == 0) zeros += 2e-6 * rows * s.C;
                else mb += 2e-6 * rows * s.C * (masked ? 2 : 1);
            }
        double t;
        if (one) {
            const auto &u = kUs1x1[i];
            const int slots = 160 / (w.kg * w.mg * w.ns * w.u * (w.mb + w.nb));
            t = u.fixed + u.longest * most + u.round * (ceil(ceil(tiles) / slots) - 1) + u.work * steps + u.tile * tiles + u.mb * (mb + zeros);
        } else {
            const auto &u = kUs[i];
            t = u.fixed + u.turn * (steps > most ? steps : most) + u.longest * most + u.tile * (tiles > 1 ? tiles : 1) + u.mb * (mb + zeros);
        }
        if (best < 0 || t < *us) { best = one ? kUs1x1[i].shape : kUs[i].shape; *us = t; }
    }
    if (one) *other = 9.28 + 0.902 * gflop + 0.125 * mb + 0.206 * zeros + 0.133 * 2e-6 * s.N * s.P * s.Q * s.K;
    else *other = 8.45 + 0.774 * gflop + 0.385 * (mb + zeros) + 0.127 * zeros + 0.00668 * longest + 0.52 * 2e-6 * s.K * s.C * s.R * s.S;
    return best;
}

int wave_launch_classes(int shape, const ConvShape &s, const IgemmParams &q, hipStream_t st, bool bt)
{
    WaveClassParams p{};
    fill_common(p, q);
    p.T = s.R * s.S;
    size_t wt_off = 0;
    for (int ph = 0; ph < s.stride; ++ph)
        for (int pw = 0; pw < s.stride; ++pw) {
            const ClassDims c = class_dims(s, ph, pw);
            WaveGrid g{};
            g.off_h = c.off_h; g.off_w = c.off_w; g.out_off_h = c.out_off_h; g.out_off_w = c.out_off_w;
            g.Kd = c.TR * c.TS * s.K;
            g.wm_off = (unsigned)(wt_off * 2);
            wt_off += (size_t)s.C * g.Kd;
            if (c.Mh <= 0 || c.Mw <= 0) continue;
            g.M = s.N * c.Mh * c.Mw;
            g.by_mw = FastDiv(c.Mw); g.by_mh = FastDiv(c.Mh);
            g.TS = c.TS > 0 ? c.TS : 1;
            g.ts_magic = small_magic(g.TS);
            g.tap0 = ph * s.S + pw; g.tap_row = s.stride * s.S; g.tap_col = s.stride;
            // most taps first: the longest reductions start first
            int at = p.n_cls++;
            for (; at > 0 && p.cls[at - 1].Kd < g.Kd; --at) p.cls[at] = p.cls[at - 1];
            p.cls[at] = g;
        }
    p.wm_bytes = bt ? (unsigned)((long long)s.K * s.R * s.S * s.C * 2) : (unsigned)(wt_off * 2);
    switch (shape) {
#define X(I, MB, NB, KG, MG, U, NS) case I: return launch_classes<MB, NB, KG, MG, U, NS>(p, bt, st);
    CLASS_SHAPES(X)
#undef X
    default: return MXC_ERR_UNSUPPORTED;
    }
}

}  // namespace mxc
