// bf16 implicit-GEMM convolution on the gfx950 matrix cores.
//
// One kernel family serves forward and backward-data.  The GEMM view is
//     Out[m][co] = sum_{t,ci} In[pixel(m) + tap(t)][ci] * Wm[co][t*Ci + ci]
// with m running over (image, output row, output column) of the launch's output grid, t over a
// TR x TS grid of filter taps, ci over input channels.  Both operands are contiguous along the
// reduction index (NHWC activations, filter rows of length T*Ci), which is the operand order the
// MFMA instructions want: every lane feeds 8 consecutive reduction elements of one row.
//
//   forward:        In = x,  Wm = w (KRSC),  pixel = (p*stride-pad, q*stride-pad), tap step +1
//   backward-data:  In = dy, Wm = per-phase re-packed filter [C][taps*K], one launch per residue
//                   class of (h+pad, v+pad) mod stride, tap step -1, strided output addressing.
//
// Tiling: a workgroup of 4 or 8 waves owns a BM x BN output tile; each wave accumulates a
// (BM/WR) x (BN/WC) sub-tile with v_mfma_f32_32x32x16_bf16 in fp32.  The reduction advances in
// steps of BKT (32 or 64) through a ring of NS LDS stages that are filled by direct global->LDS
// loads issued NS stages ahead of their use; 16-byte chunks are XOR-swizzled by row so that the
// ds_read_b128 operand fetches are bank-conflict free.
//
// Reduction order: tap-major as the filter matrix is laid out, or, when Ci is a multiple of the
// step, channel-block-major (all taps of a 64-channel block back to back: better L2 reuse).
// Problems with few tiles and a long reduction (FullyConnected shapes) split the reduction over
// workgroups into fp32 partial tiles that a finishing kernel adds in a fixed order.  A large 1x1
// filter can be read in place for backward-data (BT kernels: transposed LDS tiles).  The epilogue
// can add a bias, apply ReLU, and zero results under a mask.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <type_traits>

#include "mxc_internal.h"
#include "plan_cache.h"

namespace mxc {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef bf16x4 __attribute__((address_space(3))) * lds_bf16x4_ptr;

typedef __attribute__((address_space(3))) void *lds_vptr;
typedef short s16x2 __attribute__((ext_vector_type(2)));

constexpr unsigned OOB = 0x80000000u;   // a buffer offset no operand reaches: the load returns zeros


template <int N> __device__ __forceinline__ void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ void wait_lgkmcnt0() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void pin() { __builtin_amdgcn_sched_barrier(0); }   // nothing is scheduled across
// Workgroup barrier of the ring: the bare instruction, with the counters it needs waited for by hand just before
// it.  __syncthreads() would add a release fence, which the compiler turns into a wait for every outstanding
// global->LDS load (vmcnt(0)) - that empties a ring of more than two stages at every stage.
__device__ __forceinline__ void ring_barrier() { pin(); __builtin_amdgcn_s_barrier(); pin(); }

template <int I> using IC = std::integral_constant<int, I>;

// Transposed filter tiles (BT kernels): XOR applied to the chunk index of tile row `row` (RC chunks of
// 16 bytes per row) so that the four rows touched by one transposing read fall into different banks.
template <int RC> __device__ __forceinline__ int bt_row_swz(int row)
{
    if constexpr (RC >= 16) return (row & 3) << 2;
    else if constexpr (RC == 8) return ((row >> 1) & 1) << 2;
    else return 0;
}
template <class F, int... I> __device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>) { (f(IC<I>{}), ...); }
template <int N, class F> __device__ __forceinline__ void static_for(F &&f) { static_for_impl(f, std::make_integer_sequence<int, N>{}); }

// Position of a GEMM row in the launch's output grid, advanced by a fixed step without a division.
struct GridPos {
    int n, a, b;
    __device__ __forceinline__ GridPos(int m, int Mh, int Mw)
    {
        const unsigned t = (unsigned)m / (unsigned)Mw;
        b = (int)((unsigned)m - t * (unsigned)Mw);
        n = (int)(t / (unsigned)Mh);
        a = (int)(t - (unsigned)n * (unsigned)Mh);
    }
    // one step further; returns the change of an address that grows by n_len per image, a_len per grid row, b_len per column
    __device__ __forceinline__ int advance(const RowStep &s, int Mh, int Mw, int n_len, int a_len, int b_len)
    {
        int d = s.n * n_len + s.a * a_len + s.b * b_len;
        b += s.b;
        const bool cb = b >= Mw;
        b -= cb ? Mw : 0;
        a += s.a + (cb ? 1 : 0);
        d += cb ? a_len - Mw * b_len : 0;
        const bool ca = a >= Mh;
        a -= ca ? Mh : 0;
        n += s.n + (ca ? 1 : 0);
        d += ca ? n_len - Mh * a_len : 0;
        return d;
    }
};

// BM x BN output tile, BKT reduction elements per stage, NS stages, WR x WC waves.  The register
// budget is set for two waves per SIMD when the workgroup has 4 waves and its LDS lets two of them
// share a CU.
// BT = true: the filter operand is read transposed, straight from w[K][Co] (1x1 filters): its LDS tile is
// [reduction row][BN output columns] and its MFMA fragments come from ds_read_b64_tr_b16.
// TI = true: channel-block-major reduction order (see tap_inner_order); a compile-time choice so that the
// stage body is one basic block and the pinned interleave of address work and MFMAs survives.
// ZR = true: dx of a 1x1 filter at stride 2.  The rows of the GEMM are the pixels of even row and column; the other three of each 2x2
// block, which no tap reaches, are written as zeros beside them.  What bounds it is writing dx, of which the GEMM by itself
// has a quarter in pieces of one pixel.  us, the zeros as a launch of their own -> here, tensors coming from memory: 512 to 256 channels at
// 56x56, batch 256, 149 -> 143 (4.3 TB/s), with a mask 172 -> 156; 240 to 320, batch 128 86 -> 61 and 106 -> 88; 176 to 176 at 70x70,
// batch 100, 69 -> 56; small layers lose the launch: 256 to 128 at 28x28, batch 64, 12.6 -> 9.2.  (Half of the workgroups writing
// their zeros before the reduction, so that not all write at once: 0.98 to 1.25 of this.)
// Runs the output tile whose first row is m0 and first column n0 (split_z: its share of a split reduction).
template <int BM, int BN, int BKT, int NS, int WR, int WC, bool BT, bool TI, bool ZR = false>
__device__ __forceinline__ void igemm_tile(const IgemmParams &p, const int m0, const int n0, const int split_z)
{
    constexpr int NW = WR * WC, NT = 64 * NW;
    constexpr int WM = BM / WR, WN = BN / WC;     // wave tile
    constexpr int MI = WM / 32, NI = WN / 32;     // 32x32 MFMA blocks per wave
    constexpr int NMF = MI * NI;                  // MFMAs per k-step
    constexpr int CH = BKT / 8;                   // 16-byte chunks per tile row
    constexpr int RPL = 64 / CH;                  // tile rows filled by one wave-wide load
    constexpr int RB = 256 / (BKT * 2);           // tile rows per 256-byte span of LDS banks
    constexpr int A_LD = BM / RPL / NW;           // wave-wide loads per wave per stage
    constexpr int B_LD = BN / RPL / NW;
    constexpr int L = A_LD + B_LD;
    constexpr int KS = BKT / 16;                  // MFMA k-steps per stage
    static_assert(BKT == 32 || BKT == 64, "BKT");
    static_assert(NS >= 2 && NS <= 4, "NS");
    static_assert(NW % 2 == 0 && BM % (RPL * NW) == 0 && BN % (RPL * NW) == 0, "tile/wave mismatch");
    static_assert(L * (NS - 1) < 64, "vmcnt range");
    static_assert(KS % 2 == 0, "fragment ping-pong assumes an even number of k-steps");
    constexpr int RCB = BN / 8;                   // BT: 16-byte chunks per filter-tile row
    constexpr int RPLB = 64 / RCB;                // BT: filter-tile rows filled by one wave-wide load
    static_assert(!BT || (BKT == 64 && RCB >= 4 && RCB <= 32 && BKT % (RPLB * NW) == 0 && BKT / RPLB / NW == B_LD), "BT tile/wave mismatch");

    // Every stage is its own LDS object (not one array indexed by the stage): the compiler can then
    // see that the direct loads filling one stage never alias the operand reads of another and does
    // not serialise them.
    constexpr int SZA = BM * BKT, SZB = BN * BKT;
    __shared__ __attribute__((aligned(1024))) bf16_t sa0[SZA];
    __shared__ __attribute__((aligned(1024))) bf16_t sa1[SZA];
    __shared__ __attribute__((aligned(1024))) bf16_t sa2[NS > 2 ? SZA : 8];
    __shared__ __attribute__((aligned(1024))) bf16_t sa3[NS > 3 ? SZA : 8];
    __shared__ __attribute__((aligned(1024))) bf16_t sb0[SZB];
    __shared__ __attribute__((aligned(1024))) bf16_t sb1[SZB];
    __shared__ __attribute__((aligned(1024))) bf16_t sb2[NS > 2 ? SZB : 8];
    __shared__ __attribute__((aligned(1024))) bf16_t sb3[NS > 3 ? SZB : 8];
    // per tap: .x = byte offset of the tap relative to tap 0, .y = (dh, dv) packed as two int16
    __shared__ int2 tap_tab[MAX_TAPS + 1];
    auto stage_a = [&](auto s) __attribute__((always_inline)) -> bf16_t * {
        constexpr int S = decltype(s)::value;
        if constexpr (S == 0) return sa0; else if constexpr (S == 1) return sa1; else if constexpr (S == 2) return sa2; else return sa3;
    };
    auto stage_b = [&](auto s) __attribute__((always_inline)) -> bf16_t * {
        constexpr int S = decltype(s)::value;
        if constexpr (S == 0) return sb0; else if constexpr (S == 1) return sb1; else if constexpr (S == 2) return sb2; else return sb3;
    };

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // uniform: keeps LDS targets in SGPRs
    const int wave_m = (wave / WC) * WM, wave_n = (wave % WC) * WN;

    const int T = p.TR * p.TS;
    const int Kd = T * p.Ci;
    const int KT = TI ? T * ((p.Ci + BKT - 1) / BKT) : (Kd + BKT - 1) / BKT;

    // ---- tap table -------------------------------------------------------------------------------
    // Entry T is a sentinel whose row offset lies far outside any image: every chunk past the end
    // of the reduction fails the bounds test and is filled with zeros.
    for (int t = tid; t <= T; t += NT) {
        int2 e;
        if (t < T) {
            const int dh = (p.tap_row_inner ? t % p.TR : t / p.TS) * p.tstep_h;
            const int dv = (p.tap_row_inner ? t / p.TR : t % p.TS) * p.tstep_w;
            e.x = ((dh * p.Wi + dv) * p.pix) * 2;
            e.y = (dh & 0xFFFF) | (dv << 16);
        } else {
            e.x = 0;
            e.y = (-16384) & 0xFFFF;
        }
        tap_tab[t] = e;
    }

    // ---- load bookkeeping --------------------------------------------------------------------
    // Wave-wide load number i fills tile rows RPL*i .. RPL*i+RPL-1: lane l -> row RPL*i + l/CH, chunk
    // position l%CH.  Chunk c of row r lives at position c ^ ((r/RB) % CH), which spreads any 16
    // consecutive rows of one logical chunk over all 64 banks.  This wave issues loads wave, wave+NW,
    // ...; (RPL/RB)*NW is a multiple of CH, so the logical chunk (= reduction offset) a lane fetches is
    // the same for all of them.
    const int ld_sub = lane / CH;
    const int ld_chunk = (lane % CH) ^ (((RPL / RB) * wave + ld_sub / RB) % CH);

    const buf_rsrc_t rs_in = make_buf_rsrc(p.in, p.in_bytes);
    const buf_rsrc_t rs_wm = make_buf_rsrc(p.wm, p.wm_bytes);

    int a_off[A_LD];     // byte offset of (n, base_h, base_w, 0) in `in` (wraps below zero in the padding)
    int a_hw[A_LD];      // base_h (low 16 bits) and base_w (high 16), signed; invalid row: h = -16384
    {
        const int m = m0 + RPL * wave + ld_sub;                    // this lane's row of the first load; RPL*NW further for each next
        GridPos g(m, p.Mh, p.Mw);
        const int px2 = p.pix * 2, row2 = p.Wi * px2;
        int off = ((g.n * p.Hi + g.a * p.in_mul_h + p.in_off_h) * p.Wi + g.b * p.in_mul_w + p.in_off_w) * px2;
#pragma unroll
        for (int i = 0; i < A_LD; ++i) {
            a_off[i] = off;
            const int h = g.a * p.in_mul_h + p.in_off_h, w = g.b * p.in_mul_w + p.in_off_w;
            a_hw[i] = m + RPL * NW * i < p.m_end ? (h & 0xFFFF) | (w << 16) : (-16384) & 0xFFFF;
            if (i + 1 < A_LD) off += g.advance(p.in_step, p.Mh, p.Mw, p.Hi * row2, p.in_mul_h * row2, p.in_mul_w * px2);
        }
    }
    unsigned b_off[B_LD];   // byte offset of the filter row, OOB for rows past Co
    // BT: lane -> row RPLB*i' + lane/RCB of the stage's 64 reduction rows, output-column chunk lane%RCB (swizzled).  A
    // reduction row is (tap, k) and lies at row k*T + tap of the filter; b_off = byte offset of the lane's column chunk,
    // plus (channel-block-major order) that of the row within the stage's channel block
    [[maybe_unused]] const int lb_sub = lane / RCB;
    [[maybe_unused]] const int lb_chunk = (lane % RCB) ^ bt_row_swz<RCB>(RPLB * wave + lb_sub);   // RPLB*NW*i never changes the swizzle
    [[maybe_unused]] const bool bt_col_ok = n0 + lb_chunk * 8 < p.Co;
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
        if constexpr (BT) {
            b_off[i] = (unsigned)((TI ? (RPLB * (wave + NW * i) + lb_sub) * T * p.Co * 2 : 0) + (n0 + lb_chunk * 8) * 2);
        } else {
            const int co = n0 + RPL * (wave + NW * i) + ld_sub;
            b_off[i] = co < p.Co ? (unsigned)co * (unsigned)Kd * 2u : OOB;
        }
    }
    // Reduction position of this lane's chunk: kd = stage*BKT + ld_chunk*8 = tap*Ci + ci, kept as
    // (tap, ci) and advanced without branches: BKT = kq*Ci + kr.
    const int kq = BKT / p.Ci, kr2 = (BKT % p.Ci) * 2, Ci2 = p.Ci * 2, Kd2 = Kd * 2;
    // first stage and number of stages of this workgroup (all of them unless the reduction is split)
    const int k_lo = p.splits > 1 ? split_z * p.split_stages : 0;
    const int k_cnt = p.splits > 1 ? min(KT - k_lo, p.split_stages) : KT;
    const int kd0 = k_lo * BKT + ld_chunk * 8;     // this lane's reduction position in the first stage (tap-major order)
    int kd2 = kd0 * 2;                             // byte offset within a filter row
    int ci2 = (kd0 % p.Ci) * 2, tap = kd0 / p.Ci;
    if constexpr (TI) {                            // stage s = (channel block s / T, tap s % T)
        ci2 = (k_lo / T) * (BKT * 2) + ld_chunk * 16;
        tap = ci2 < Ci2 ? k_lo % T : T;            // past the channels of a last block that is not whole: the sentinel tap
    }
    // BT in that order: the stage's tap and first channel (a lane's own `tap` follows the chunk it brings of the other operand)
    [[maybe_unused]] int bt_t = TI ? k_lo % T : 0, bt_c0 = TI ? k_lo / T * BKT : 0;
    const int lim_hw = ((p.Hi - 1) & 0xFFFF) | ((p.Wi - 1) << 16);
    // BT, tap-major order: (tap, k) of this lane's filter rows in the next stage
    [[maybe_unused]] int bt_tap[B_LD], bt_k[B_LD];
    if constexpr (BT && !TI) {
#pragma unroll
        for (int i = 0; i < B_LD; ++i) {
            const int kd = k_lo * BKT + RPLB * (wave + NW * i) + lb_sub;
            bt_tap[i] = kd / p.Ci;
            bt_k[i] = kd - bt_tap[i] * p.Ci;
        }
    }

    unsigned va[A_LD], vb[B_LD];   // byte offsets of the next stage's loads

    // address generation for the next stage, split in A_LD + 1 small tasks so that it can be spread
    // between MFMAs.  tap_e is the tap-table entry of the stage the addresses are for; the last task
    // advances the reduction position and fetches the entry of the stage after, a whole stage before
    // the first task that reads it.
    int2 tap_e = make_int2(0, 0);
    auto fetch_tap = [&]() __attribute__((always_inline)) { tap_e = tap_tab[tap < T ? tap : T]; };
    auto addr_task = [&](auto t) __attribute__((always_inline)) {
        constexpr int Tk = decltype(t)::value;
        if constexpr (Tk < A_LD) {
            constexpr int i = Tk;
            const s16x2 hw = __builtin_bit_cast(s16x2, a_hw[i]) + __builtin_bit_cast(s16x2, tap_e.y);
            const s16x2 d = __builtin_bit_cast(s16x2, lim_hw) - hw;
            const int bad = (__builtin_bit_cast(int, hw) | __builtin_bit_cast(int, d)) & (int)0x80008000;
            va[i] = bad == 0 ? (unsigned)(a_off[i] + tap_e.x + ci2) : OOB;
        } else {
            if constexpr (BT && !TI) {
#pragma unroll
                for (int i = 0; i < B_LD; ++i) {
                    vb[i] = bt_col_ok && bt_tap[i] < T ? b_off[i] + (unsigned)(bt_k[i] * T + bt_tap[i]) * (unsigned)(p.Co * 2) : OOB;
                    bt_k[i] += kr2 / 2;
                    const int carry = bt_k[i] >= p.Ci ? 1 : 0;
                    bt_k[i] -= carry ? p.Ci : 0;
                    bt_tap[i] += kq + carry;
                }
                ci2 += kr2;
                const int carry = ci2 >= Ci2 ? 1 : 0;
                ci2 -= carry ? Ci2 : 0;
                tap += kq + carry;
            } else if constexpr (TI) {
                // Order (channel block, tap): the pixels a workgroup reads for one channel block serve all
                // its taps back to back, so they are still in the XCD's L2 when the next tap asks for them.
                if constexpr (BT) {
                    const unsigned base = (unsigned)(bt_c0 * T + bt_t) * (unsigned)(p.Co * 2);
                    const int rows = p.Ci - bt_c0;                // of the block that are there: none past the last block
#pragma unroll
                    for (int i = 0; i < B_LD; ++i) vb[i] = bt_col_ok && RPLB * (wave + NW * i) + lb_sub < rows ? b_off[i] + base : OOB;
                    const bool wrap = bt_t + 1 >= T;
                    bt_t = wrap ? 0 : bt_t + 1;
                    bt_c0 += wrap ? BKT : 0;
                } else {
                    const bool k_ok = tap < T;
                    const unsigned kd = (unsigned)(tap * Ci2 + ci2);
#pragma unroll
                    for (int i = 0; i < B_LD; ++i) vb[i] = k_ok ? b_off[i] + kd : OOB;
                }
                const int last = tap + 1 >= T ? 1 : 0;           // wrap to the next channel block
                tap = last ? 0 : tap + 1;
                ci2 += last ? BKT * 2 : 0;
                tap = ci2 >= Ci2 ? T : tap;                       // past the last block: the sentinel tap, for good
            } else {
                const bool k_ok = kd2 < Kd2;
#pragma unroll
                for (int i = 0; i < B_LD; ++i) vb[i] = k_ok ? b_off[i] + (unsigned)kd2 : OOB;
                // advance (tap, ci) and kd by one stage
                kd2 += BKT * 2;
                ci2 += kr2;
                const int carry = ci2 >= Ci2 ? 1 : 0;
                ci2 -= carry ? Ci2 : 0;
                tap += kq + carry;
            }
            fetch_tap();
        }
    };
    constexpr int N_ADDR = A_LD + 1;
    auto load_task = [&](auto t, bf16_t *dst_a, bf16_t *dst_b) __attribute__((always_inline)) {
        constexpr int Tk = decltype(t)::value;
        if constexpr (Tk < A_LD) lds_dma16(rs_in, va[Tk], dst_a + (wave + NW * Tk) * RPL * BKT);
        else lds_dma16(rs_wm, vb[Tk - A_LD], dst_b + (wave + NW * (Tk - A_LD)) * (BT ? RPLB * BN : RPL * BKT));
    };

    // this thread's share of the tile's bias vector (column n0 + tid), requested now, used after the loop
    static_assert(NT >= BN, "one bias value per thread");
    const float bias_t = (p.bias != nullptr && tid < BN && n0 + tid < p.Cw) ? p.bias[n0 + tid] : 0.f;

    f32x16 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    // operand fetch: lane -> tile row lane%32 of a 32-row block, 8-element group lane/32 of a 16-wide k-step
    const int frag_row = lane & 31, frag_kg = lane >> 5;
    const int frag_swz = (frag_row / RB) % CH;     // block bases are multiples of 32 rows
    const int a_lane = (wave_m + frag_row) * BKT, b_lane = (wave_n + frag_row) * BKT;

    // BT: transposing-read geometry (16-lane group g, lane j16 within it; one read covers 4 reduction rows x
    // 16 output columns): element offsets of the two reads of a 16-row k-step for each of the NI column blocks
    [[maybe_unused]] int bt_lo[NI], bt_hi[NI];
    if constexpr (BT) {
        const int g = lane >> 4, j16 = lane & 15;
        const int tr_row = (g >> 1) * 8 + (j16 >> 2);
        const int tr_ch = (g & 1) * 16 + (j16 & 3) * 4;
        auto tr_off = [&](int ch_base, int row) __attribute__((always_inline)) {
            const int ch = ch_base + tr_ch;
            return row * BN + (((ch >> 3) ^ bt_row_swz<RCB>(row)) << 3) + (ch & 7);
        };
#pragma unroll
        for (int j = 0; j < NI; ++j) { bt_lo[j] = tr_off(wave_n + j * 32, tr_row); bt_hi[j] = tr_off(wave_n + j * 32, tr_row + 4); }
    }
    struct Frags { bf16x8 a[MI], b[NI]; };
    auto read_task = [&](auto t, Frags &f, const bf16_t *src_a, const bf16_t *src_b, int ks) __attribute__((always_inline)) {
        constexpr int Tk = decltype(t)::value;
        const int pos = ((ks * 2 + frag_kg) ^ frag_swz) << 3;
        if constexpr (Tk < MI) f.a[Tk] = *reinterpret_cast<const bf16x8 *>(src_a + a_lane + Tk * 32 * BKT + pos);
        else if constexpr (BT) {
            const bf16_t *q = src_b + ks * 16 * BN;
            const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(q + bt_lo[Tk - MI]));
            const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(q + bt_hi[Tk - MI]));
            f.b[Tk - MI] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        } else f.b[Tk - MI] = *reinterpret_cast<const bf16x8 *>(src_b + b_lane + (Tk - MI) * 32 * BKT + pos);
    };
    constexpr int N_READ = MI + NI;

    // NMF MFMAs of one k-step with `NTASK` side tasks spread between them (program order is pinned:
    // the matrix pipe executes one MFMA while the wave issues the side work behind it)
    // The first NFRONT tasks (operand fetches, which the next k-step waits for) go behind the first half
    // of the MFMAs, the rest behind the second half.
    auto mfma_with = [&](const Frags &f, auto nfront, auto ntask, auto &&task) __attribute__((always_inline)) {
        constexpr int NFRONT = decltype(nfront)::value, NTASK = decltype(ntask)::value;
        constexpr int H1 = NMF > 1 ? NMF / 2 : 1, H2 = NMF - H1 > 0 ? NMF - H1 : 1;
        static_for<NMF>([&](auto s) __attribute__((always_inline)) {
            constexpr int S = decltype(s)::value;
            // filter fragment first: the product is formed transposed, D[co][pixel] (see the epilogue)
            acc[S / NI][S % NI] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f.b[S % NI], f.a[S / NI], acc[S / NI][S % NI], 0, 0, 0);
            static_for<NTASK>([&](auto t) __attribute__((always_inline)) {
                constexpr int Tk = decltype(t)::value;
                constexpr int slot = Tk < NFRONT ? Tk * H1 / NFRONT
                                                 : (NMF > 1 ? H1 + (Tk - NFRONT) * H2 / (NTASK - NFRONT > 0 ? NTASK - NFRONT : 1) : 0);
                if constexpr (slot == S) task(t);
            });
            pin();
        });
    };

    // ---- pipeline ------------------------------------------------------------------------------
    // Stage s lives in ring slot s % NS.  While stage kt is being multiplied, stages kt+1..kt+NS-1
    // are landing.  Per stage: k-steps 0..KS-2 fetch the next k-step's operands, and the one before
    // last also computes the addresses of the refill; then this wave's loads of stage kt+1 are
    // awaited (all but the (NS-2)*L youngest), one barrier publishes stage kt+1 and frees slot
    // kt % NS, and the last k-step's MFMAs run interleaved with the refill loads (stage kt+NS) and the
    // first operand fetch of stage kt+1 - the matrix pipe has work across the barrier.
    Frags f0, f1;
    __syncthreads();   // tap table visible
    fetch_tap();
    static_for<NS>([&](auto s) __attribute__((always_inline)) {
        static_for<N_ADDR>([&](auto t) __attribute__((always_inline)) { addr_task(t); });
        static_for<L>([&](auto t) __attribute__((always_inline)) { load_task(t, stage_a(s), stage_b(s)); });
    });
    wait_vmcnt<L * (NS - 1)>();
    ring_barrier();
    static_for<N_READ>([&](auto t) __attribute__((always_inline)) { read_task(t, f0, sa0, sb0, 0); });

    auto run_stage = [&](auto s) __attribute__((always_inline)) {
        constexpr int S = decltype(s)::value;
        constexpr int S1 = (S + 1) % NS;
        bf16_t *ca = stage_a(s), *cb = stage_b(s);
        static_for<KS - 1>([&](auto k) __attribute__((always_inline)) {
            constexpr int ks = decltype(k)::value;
            Frags &cur = (ks & 1) ? f1 : f0;
            Frags &nxt = (ks & 1) ? f0 : f1;
            // this k-step's share of the address tasks, spread evenly over k-steps 0..KS-2
            constexpr int a0 = ks * N_ADDR / (KS - 1), a1 = (ks + 1) * N_ADDR / (KS - 1);
            mfma_with(cur, IC<N_READ>{}, IC<N_READ + (a1 - a0)>{}, [&](auto t) __attribute__((always_inline)) {
                constexpr int Tk = decltype(t)::value;
                if constexpr (Tk < N_READ) read_task(t, nxt, ca, cb, ks + 1); else addr_task(IC<a0 + Tk - N_READ>{});
            });
        });
        // the last k-step's operands are in f1; all reads of this slot must have returned before it is refilled
        wait_lgkmcnt0();
        wait_vmcnt<L * (NS - 2)>();
        ring_barrier();
        mfma_with(f1, IC<N_READ>{}, IC<N_READ + L>{}, [&](auto t) __attribute__((always_inline)) {
            constexpr int Tk = decltype(t)::value;
            if constexpr (Tk < N_READ) read_task(t, f0, stage_a(IC<S1>{}), stage_b(IC<S1>{}), 0);
            else load_task(IC<Tk - N_READ>{}, ca, cb);
        });
    };

    // Whole turns of the ring in a loop whose body is one basic block (the compiler's own wait insertion for
    // LDS reads against in-flight global->LDS loads merges states at every control-flow join; a join inside
    // the loop makes it wait for all loads at the loop head), then the remaining stages.
    int kt = 0;
    for (; kt + NS <= k_cnt; kt += NS) static_for<NS>([&](auto s) __attribute__((always_inline)) { run_stage(s); });
    const int rem = k_cnt - kt;
    if (rem >= 1) run_stage(IC<0>{});
    if constexpr (NS > 2) if (rem >= 2) run_stage(IC<1>{});
    if constexpr (NS > 3) if (rem >= 3) run_stage(IC<2>{});
    wait_vmcnt<0>();   // drain the zero-fill loads of the stages past the end before the tile's LDS is abandoned

    // ---- epilogue: fp32 -> bf16 (RNE), to the output pixels ------------------------------------
    // The product was formed transposed (filter fragment as the first MFMA operand): accumulator element e of a
    // 32x32 block belongs to tile row lane%32 and column 8*(e/4) + 4*(lane/32) + e%4, so a lane holds runs of four
    // neighbouring output columns of one pixel.
    auto out_pixel = [&](int m) __attribute__((always_inline)) -> long long {
        if (p.linear_out) return m;
        const unsigned b = (unsigned)m % (unsigned)p.Mw, t2 = (unsigned)m / (unsigned)p.Mw;
        const unsigned a = t2 % (unsigned)p.Mh, n = t2 / (unsigned)p.Mh;
        return ((long long)n * p.Ho + ((int)a * p.out_mul_h + p.out_off_h)) * p.Wo + ((int)b * p.out_mul_w + p.out_off_w);
    };
    if (p.splits > 1 || p.f32_out) {
        // split reduction, or a caller that wants the fp32 sums themselves: accumulators to partial[z][m][co]
        // (row-major like the output; Co % 8 == 0), 16 bytes at a time
        float *part = p.partial + (size_t)split_z * p.M * p.Co;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int m = m0 + wave_m + i * 32 + frag_row;
            if (m >= p.m_end) continue;
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4) {
                    const int co = n0 + wave_n + j * 32 + 8 * g4 + 4 * frag_kg;
                    if (co < p.Co)
                        *reinterpret_cast<float4 *>(part + (size_t)m * p.Co + co) =
                            make_float4(acc[i][j][4 * g4], acc[i][j][4 * g4 + 1], acc[i][j][4 * g4 + 2], acc[i][j][4 * g4 + 3]);
                }
        }
        return;
    }
    if ((p.Co & 7) == 0) {
        // Through LDS, one 32-row block of the wave tile at a time, so that global stores are 16 bytes per lane and
        // a row's WN channels leave as one contiguous run.  Staged rows are padded by 16 bytes, and 8-byte unit u of
        // row r sits at u ^ ((r >> 3) % 4): the 32 rows that one 8-byte write instruction covers then fall on 16
        // different bank pairs (two rows each: the least 256 bytes over 128 bytes of banks allow).  A 16-byte chunk c
        // of row r is therefore found at chunk c ^ ((r >> 4) % 2), its halves exchanged when bit 3 of r is set.
        constexpr int CPR = WN / 8;                   // 16-byte chunks per staged row
        constexpr int PW = WN + 8;                    // staged row pitch, elements
        constexpr int RS = 32 * PW;                   // staging elements per wave
        constexpr bool USE_A = SZA >= SZB;
        constexpr int SZ = USE_A ? SZA : SZB;
        constexpr int WPB = SZ / RS;                  // waves whose staging fits one stage buffer
        static_assert(WPB >= 1 && NW <= WPB * NS, "epilogue staging must fit the stage buffers of one operand");
        static_assert((USE_A ? SZB : SZA) * 2 >= BN * 4, "the bias vector must fit a stage buffer of the other operand");
        wait_lgkmcnt0();
        __syncthreads();                              // every wave is done reading operands: LDS is free
        const int bi = wave / WPB;
        bf16_t *stg = bi == 0 ? (USE_A ? sa0 : sb0) : bi == 1 ? (USE_A ? sa1 : sb1) : bi == 2 ? (USE_A ? sa2 : sb2) : (USE_A ? sa3 : sb3);
        stg += (wave % WPB) * RS;
        float *s_bias = reinterpret_cast<float *>(USE_A ? sb0 : sa0);
        const bool has_bias = p.bias != nullptr;
        if (has_bias) {                               // uniform
            if (tid < BN) s_bias[tid] = bias_t;
            __syncthreads();
        }
        // conversion and staging of block (i, *): + bias, ReLU as a 16-bit integer maximum on the rounded pair
        auto stage_block = [&](int i, auto bias_c, auto relu_c) __attribute__((always_inline)) {
            constexpr bool BIAS = decltype(bias_c)::value, RELU = decltype(relu_c)::value;
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4) {
                    float v0 = acc[i][j][4 * g4], v1 = acc[i][j][4 * g4 + 1], v2 = acc[i][j][4 * g4 + 2], v3 = acc[i][j][4 * g4 + 3];
                    if (BIAS) {
                        const float4 b4 = *reinterpret_cast<const float4 *>(s_bias + wave_n + j * 32 + 8 * g4 + 4 * frag_kg);
                        v0 += b4.x; v1 += b4.y; v2 += b4.z; v3 += b4.w;
                    }
                    uint2 pk = make_uint2(pack_bf16x2(v0, v1), pack_bf16x2(v2, v3));
                    if (RELU) {
                        pk.x = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2, pk.x), s16x2{0, 0}));
                        pk.y = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2, pk.y), s16x2{0, 0}));
                    }
                    *reinterpret_cast<uint2 *>(stg + frag_row * PW + 4 * ((j * 8 + 2 * g4 + frag_kg) ^ ((frag_row >> 3) & 3))) = pk;
                }
        };
        // Outputs below 2 GiB whose staged rows one store instruction covers whole: one buffer store per 64/CPR rows;
        // rows past the end and columns past Co get an offset the resource rejects, which takes the place of a bounds
        // branch.  A mask is fetched the same way and all of it before the first conversion, so that its latency lies
        // under the staging.
        constexpr bool ROWS_PER_STORE_OK = 64 % CPR == 0;
        constexpr int RPI = ROWS_PER_STORE_OK ? 64 / CPR : 1;
        constexpr int NST = ROWS_PER_STORE_OK ? 32 / RPI : 1;
        const bool fast_store = ROWS_PER_STORE_OK && p.out_bytes != 0;
        const out_rsrc_t rs_out = make_out_rsrc(p.out, p.out_bytes);
        const int st_r = lane / CPR, st_c = lane % CPR;
        unsigned st_off[MI][NST];
        uint4 st_mask[MI][NST];
        // ZR: whether the pixel to the right of the store's is in the image (bit of z_right), and the one below (z_below)
        static_assert(MI * NST <= 32, "a bit per store");
        [[maybe_unused]] unsigned z_right = 0, z_below = 0;
        if (fast_store) {
            const bool col_ok = n0 + wave_n + st_c * 8 < p.Co;
            const int m = m0 + wave_m + st_r, co2 = p.Co * 2;      // this lane's row of the first store; RPI further for each next
            unsigned off = (unsigned)((n0 + wave_n + st_c * 8) * 2);
            if (p.linear_out) {
                off += (unsigned)m * (unsigned)co2;                // below 2^32: the output is below 2^31 and a tile adds little
#pragma unroll
                for (int k = 0; k < MI * NST; ++k) st_off[k / NST][k % NST] = col_ok && m + k * RPI < p.m_end ? off + (unsigned)(k * RPI * co2) : OOB;
            } else {
                GridPos g(m, p.Mh, p.Mw);
                off += (unsigned)(((g.n * p.Ho + g.a * p.out_mul_h + p.out_off_h) * p.Wo + g.b * p.out_mul_w + p.out_off_w) * co2);
#pragma unroll
                for (int k = 0; k < MI * NST; ++k) {
                    st_off[k / NST][k % NST] = col_ok && m + k * RPI < p.m_end ? off : OOB;
                    if constexpr (ZR) {
                        z_right |= 2 * g.b + 1 < p.Wo ? 1u << k : 0u;
                        z_below |= 2 * g.a + 1 < p.Ho ? 1u << k : 0u;
                    }
                    if (k + 1 < MI * NST)
                        off += (unsigned)g.advance(p.out_step, p.Mh, p.Mw, p.Ho * p.Wo * co2, p.out_mul_h * p.Wo * co2, p.out_mul_w * co2);
                }
            }
            if (p.mask != nullptr) {
                const out_rsrc_t rs_mask = make_out_rsrc(const_cast<bf16_t *>(p.mask), p.out_bytes);
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int k = 0; k < NST; ++k) st_mask[i][k] = buffer_load16(rs_mask, st_off[i][k]);
            }
        }
        auto staged_chunk = [&](int r, int c) __attribute__((always_inline)) {
            const uint4 v = *reinterpret_cast<const uint4 *>(stg + r * PW + ((c ^ ((r >> 4) & 1)) << 3));
            return ((r >> 3) & 1) ? make_uint4(v.z, v.w, v.x, v.y) : v;
        };
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            if (has_bias) { if (p.relu) stage_block(i, std::true_type{}, std::true_type{}); else stage_block(i, std::true_type{}, std::false_type{}); }
            else { if (p.relu) stage_block(i, std::false_type{}, std::true_type{}); else stage_block(i, std::false_type{}, std::false_type{}); }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
            if (fast_store) {
#pragma unroll
                for (int k = 0; k < NST; ++k) {
                    uint4 v = staged_chunk(st_r + k * RPI, st_c);
                    if (p.mask != nullptr) v = mask_bf16x8(v, st_mask[i][k]);
                    if (p.nt_out) buffer_store16_nt(rs_out, st_off[i][k], v);
                    else buffer_store16(rs_out, st_off[i][k], v);
                    if constexpr (ZR) {            // (an offset that the resource rejects stays one: the output is below 2^31)
                        const int at = i * NST + k;
                        const unsigned right = (unsigned)(p.Co * 2), below = (unsigned)p.Wo * right;
                        const unsigned o1 = (z_right >> at) & 1 ? st_off[i][k] + right : OOB, o2 = (z_below >> at) & 1 ? st_off[i][k] + below : OOB;
                        const unsigned o3 = (z_below >> at) & 1 ? o1 + below : OOB;
                        const uint4 z = make_uint4(0, 0, 0, 0);
                        if (p.nt_out) { buffer_store16_nt(rs_out, o1, z); buffer_store16_nt(rs_out, o2, z); buffer_store16_nt(rs_out, o3, z); }
                        else { buffer_store16(rs_out, o1, z); buffer_store16(rs_out, o2, z); buffer_store16(rs_out, o3, z); }
                    }
                }
            } else {
#pragma unroll
                for (int k = 0; k < 32 * CPR / 64; ++k) {
                    const int idx = k * 64 + lane;
                    const int r = idx / CPR, c = idx % CPR;
                    const int m = m0 + wave_m + i * 32 + r, co = n0 + wave_n + c * 8;
                    uint4 v = staged_chunk(r, c);
                    if (m < p.m_end && co < p.Co) {
                        const long long off = out_pixel(m) * p.Co + co;
                        if (p.mask != nullptr) {
                            const uint4 mk = *reinterpret_cast<const uint4 *>(p.mask + off);
                            v = mask_bf16x8(v, mk);
                        }
                        typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
                        const u32x4 vv = {v.x, v.y, v.z, v.w};
                        if (p.nt_out) __builtin_nontemporal_store(vv, reinterpret_cast<u32x4 *>(p.out + off));
                        else *reinterpret_cast<u32x4 *>(p.out + off) = vv;
                    }
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        }
    } else {
        // output channel counts that are not a multiple of 8: four neighbouring columns at a time (8 bytes at any
        // alignment), the last ones element by element
        struct __attribute__((packed)) Packed8 { uint32_t lo, hi; };
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int m = m0 + wave_m + i * 32 + frag_row;
            if (m >= p.m_end) continue;
            const long long orow = out_pixel(m) * p.Co;
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int g4 = 0; g4 < 4; ++g4) {
                    const int co = n0 + wave_n + j * 32 + 8 * g4 + 4 * frag_kg;
                    if (co >= p.Co) continue;
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        v[e] = acc[i][j][4 * g4 + e];
                        if (p.bias != nullptr && co + e < p.Cw) v[e] += p.bias[co + e];
                        if (p.relu) v[e] = fmaxf(v[e], 0.f);
                    }
                    if (co + 4 <= p.Co) {
                        Packed8 o{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
                        if (p.mask != nullptr) {
                            const Packed8 mk = *reinterpret_cast<const Packed8 *>(p.mask + orow + co);
                            o = Packed8{mask_bf16x2(o.lo, mk.lo), mask_bf16x2(o.hi, mk.hi)};
                        }
                        *reinterpret_cast<Packed8 *>(p.out + orow + co) = o;
                    } else {
#pragma unroll
                        for (int e = 0; e < 3; ++e)
                            if (co + e < p.Co)
                                p.out[orow + co + e] = (p.mask == nullptr || mask_keeps(p.mask + orow + co + e)) ? f32_to_bf16(v[e]) : (bf16_t)0;
                    }
                }
        }
    }
}

// Workgroup -> tile.  Consecutive workgroup ids are dealt round-robin to the 8 XCDs; give each XCD a contiguous range of
// tiles, n-tile fastest, so that tiles sharing an activation tile meet in one L2.
__device__ __forceinline__ int tile_unit(int units)
{
    const int per_xcd = (units + 7) / 8;
    return (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
}

template <int BM, int BN, int BKT, int NS, int WR, int WC>
constexpr int tile_min_blocks = (WR * WC == 4 && NS * (BM + BN) * BKT * 2 <= 80 * 1024) ? 2 : 1;

template <int BM, int BN, int BKT, int NS, int WR, int WC, bool BT, bool TI, bool ZR = false>
__global__ __launch_bounds__(64 * WR * WC, (tile_min_blocks<BM, BN, BKT, NS, WR, WC>)) void igemm_kernel(const IgemmParams p)
{
    const int total = p.m_tiles * p.n_tiles;
    const int units = total * (p.splits > 1 ? p.splits : 1);
    const int unit = tile_unit(units);
    if (unit >= units) return;
    const int logical = unit % total;
    igemm_tile<BM, BN, BKT, NS, WR, WC, BT, TI, ZR>(p, p.m_begin + (logical / p.n_tiles) * BM, (logical % p.n_tiles) * BN, unit / total);
}

// Strided backward-data: all residue classes of (h+pad, v+pad) mod stride that some tap reaches in one launch, the classes
// of one stretch of rows next to each other - they read the same dy rows and together write whole stretches of dx.  One
// launch per class ran them one after another, each with its own start, drain and part-filled last round (3x3 stride 2,
// 40->256 at 20x20, batch 12: 42 us in four launches, 14 in one).
struct IgemmClass {
    const bf16_t *wm;
    unsigned wm_bytes;
    int TR, TS, Mh, Mw, in_off_h, in_off_w, out_off_h, out_off_w;
    RowStep in_step, out_step;
};
struct IgemmClasses {
    IgemmParams p;       // what the classes share
    IgemmClass c[16];
    int n, max_m_tiles;
};

template <int BM, int BN, int BKT, int NS, int WR, int WC, bool TI>
__global__ __launch_bounds__(64 * WR * WC, (tile_min_blocks<BM, BN, BKT, NS, WR, WC>)) void igemm_classes_kernel(const IgemmClasses q)
{
    const int units = q.max_m_tiles * q.n * q.p.n_tiles;
    const int unit = tile_unit(units);
    if (unit >= units) return;
    const int n_tile = unit % q.p.n_tiles, t2 = unit / q.p.n_tiles;
    const IgemmClass &c = q.c[t2 % q.n];
    const int m0 = t2 / q.n * BM;
    IgemmParams p = q.p;
    p.wm = c.wm; p.wm_bytes = c.wm_bytes;
    p.TR = c.TR; p.TS = c.TS; p.Mh = c.Mh; p.Mw = c.Mw;
    p.in_off_h = c.in_off_h; p.in_off_w = c.in_off_w; p.out_off_h = c.out_off_h; p.out_off_w = c.out_off_w;
    p.in_step = c.in_step; p.out_step = c.out_step;
    p.M = p.N * c.Mh * c.Mw;
    p.m_end = p.M;
    if (m0 >= p.M) return;
    igemm_tile<BM, BN, BKT, NS, WR, WC, false, TI>(p, m0, n_tile * BN, 0);
}

// Whether the reduction runs over all taps of a block of bk channels before the next block: what the tiles of an XCD read of
// a block then stays in its L2 from tap to tap.  Where the last block is not whole its empty chunks cost stages, which narrow tiles
// of many channels repay (94864 pixels, 400 to 32 channels 3x3 94.9 -> 66.4 us, 151230, 288 to 32 5x5 240 -> 156, 20480, 352 to 24
// 5x5 53.4 -> 38.9): their many workgroups read the same pixels T times, and all channels of those do not fit the L2.  Wider tiles
// gain nothing, small problems fit it anyway (3969 pixels, 400 to 440: 65.9 against 69.6).
const bool tap_outer_forced = getenv("MXC_TAP_OUTER") != nullptr;       // tuning sweeps only; read once
inline bool tap_inner_order(int T, int Ci, int bk, int bn, long long M)
{
    if (T == 1 || tap_outer_forced) return false;
    return Ci % bk == 0 || (bn <= 64 && Ci >= 256 && M >= 1 << 14 && (Ci + bk - 1) / bk * bk <= Ci * 1.15);
}
inline int stages_of(int T, int Ci, int bk, int bn, long long M)
{
    return tap_inner_order(T, Ci, bk, bn, M) ? T * ((Ci + bk - 1) / bk) : (T * Ci + bk - 1) / bk;
}

// the kernel's row steps: from load to load of a wave, and from store to store (64 lanes of 16 bytes over the wave's columns)
template <int BN, int BKT, int WR, int WC>
void set_steps(RowStep &in, RowStep &out, int Mh, int Mw)
{
    constexpr int CPR = BN / WC / 8;
    in = row_step(64 / (BKT / 8) * WR * WC, Mh, Mw);
    out = row_step(64 % CPR == 0 ? 64 / CPR : 1, Mh, Mw);
}

// the tiles that are built with ZR: those that read the filter in place as well (has_bt)
template <int BM, int BN, int NW>
constexpr bool tile_zeroes = (BM == 128 && BN <= 128 && NW == 4) || (BM == 256 && BN == 256) || (BM == 64 && BN == 128);

// Launches the tile shape on GEMM rows [m_begin, m_end) of the problem (m_end < 0: to the last row).
template <int BM, int BN, int BKT, int NS, int WR, int WC, bool BT = false>
int launch(IgemmParams p, hipStream_t st, long long m_begin = 0, long long m_end = -1)
{
    const long long M = (long long)p.N * p.Mh * p.Mw;
    if (m_end < 0 || m_end > M) m_end = M;
    if (m_begin >= m_end) return MXC_OK;
    const long long mt = (m_end - m_begin + BM - 1) / BM;
    p.n_tiles = (p.Co + BN - 1) / BN;
    if (mt * p.n_tiles > 0x3FFFFFFFll) return MXC_ERR_SHAPE;
    set_steps<BN, BKT, WR, WC>(p.in_step, p.out_step, p.Mh, p.Mw);
    p.M = (int)M;
    p.m_begin = (int)m_begin;
    p.m_end = (int)m_end;
    p.m_tiles = (int)mt;
    p.in_bytes = (unsigned)((long long)p.N * p.Hi * p.Wi * p.pix * 2);
    if (p.Cw == 0) p.Cw = p.Co;
    p.wm_bytes = BT ? p.bt_w_bytes : (unsigned)((long long)p.Cw * p.TR * p.TS * p.Ci * 2);
    p.tap_inner = tap_inner_order(p.TR * p.TS, p.Ci, BKT, BN, M) ? 1 : 0;
    p.linear_out = (p.out_mul_h == 1 && p.out_mul_w == 1 && p.out_off_h == 0 && p.out_off_w == 0 && p.Mh == p.Ho && p.Mw == p.Wo) ? 1 : 0;
    // results of a large layer leave as non-temporal stores: the caches keep serving this kernel's operand reads
    static const char *nt_forced = getenv("MXC_NT_OUT");                      // tuning sweeps only; read once
    const long long out_bytes = (long long)p.N * p.Ho * p.Wo * p.Co * 2;
    p.out_bytes = out_bytes < 0x7FFF0000ll ? (unsigned)out_bytes : 0u;
    p.nt_out = nt_forced ? atoi(nt_forced) : ((long long)p.N * p.Ho * p.Wo * p.Co * 2 >= (128ll << 20) ? 1 : 0);
    if (p.splits > 1) {
        // even stage ranges; the last split may be shorter, none is empty
        const int KT = stages_of(p.TR * p.TS, p.Ci, BKT, BN, M);
        p.split_stages = (KT + p.splits - 1) / p.splits;
        p.splits = (KT + p.split_stages - 1) / p.split_stages;
        if (!p.linear_out || !p.partial || m_begin != 0 || m_end != M) return MXC_ERR_UNSUPPORTED;
    }
    const long long total = (long long)p.m_tiles * p.n_tiles * (p.splits > 1 ? p.splits : 1);
    if (total > 0x3FFFFFFFll) return MXC_ERR_SHAPE;
    const int grid = (int)((total + 7) / 8) * 8;
    if (p.zero_rest) {
        if constexpr (tile_zeroes<BM, BN, WR * WC>) {
            if (p.out_bytes == 0 || (p.Co & 7) != 0) return MXC_ERR_UNSUPPORTED;      // the buffer stores write them
            // Non-temporal stores reach memory as they are: of rows that are no multiple of 64 bytes in pieces of less (dx of 1-900 MB, 176
            // channels 71-350 us against 30-200, 80 channels 40-60 against 30-40; multiples of 32 channels gain from 200 MB on, 320 of them 1.3 times)
            if (p.Co % 32 != 0) p.nt_out = 0;
            hipLaunchKernelGGL((igemm_kernel<BM, BN, BKT, NS, WR, WC, BT, false, true>), dim3((unsigned)grid), dim3(64 * WR * WC), 0, st, p);
            return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
        } else return MXC_ERR_UNSUPPORTED;
    }
    if (p.tap_inner) {
        hipLaunchKernelGGL((igemm_kernel<BM, BN, BKT, NS, WR, WC, BT, true>), dim3((unsigned)grid), dim3(64 * WR * WC), 0, st, p);
        return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
    }
    hipLaunchKernelGGL((igemm_kernel<BM, BN, BKT, NS, WR, WC, BT, false>), dim3((unsigned)grid), dim3(64 * WR * WC), 0, st, p);
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
}

template <int BM, int BN, int BKT, int NS, int WR, int WC>
int launch_classes(IgemmClasses &q, hipStream_t st)
{
    IgemmParams &p = q.p;
    p.n_tiles = (p.Co + BN - 1) / BN;
    long long most = 0;
    for (int i = 0; i < q.n; ++i) {
        const long long mt = ((long long)p.N * q.c[i].Mh * q.c[i].Mw + BM - 1) / BM;
        if (mt > most) most = mt;
        set_steps<BN, BKT, WR, WC>(q.c[i].in_step, q.c[i].out_step, q.c[i].Mh, q.c[i].Mw);
    }
    const long long total = most * q.n * p.n_tiles;
    if (total > 0x3FFFFFFFll) return MXC_ERR_SHAPE;
    q.max_m_tiles = (int)most;
    const dim3 grid((unsigned)((total + 7) / 8 * 8)), block(64 * WR * WC);
    p.tap_inner = p.Ci % BKT == 0 ? 1 : 0;
    if (p.tap_inner) hipLaunchKernelGGL((igemm_classes_kernel<BM, BN, BKT, NS, WR, WC, true>), grid, block, 0, st, q);
    else hipLaunchKernelGGL((igemm_classes_kernel<BM, BN, BKT, NS, WR, WC, false>), grid, block, 0, st, q);
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
}

// A tile shape the launcher can pick: output tile, workgroups that fit one CU at a time (LDS and
// register budget) and the matrix-pipe utilisation it reaches relative to the 256x256 tile when the
// chip is full (fitted to per-layer times of the AlexNet- and VGG-style stacks run back to back).
struct TileChoice { int bm, bn, bk, slots; float util; const char *name; };   // bk: reduction elements per stage
const TileChoice kTiles[] = {
    {128, 128, 64, 2, 0.91f, "igemm_128x128_k64s2_w4"},
    {256, 256, 64, 1, 1.15f, "igemm_256x256_k64s2_w8"},
    {256, 128, 64, 1, 0.95f, "igemm_256x128_k64s3_w8"},
    {128, 256, 64, 1, 0.97f, "igemm_128x256_k64s3_w8"},
    {128, 64, 64, 3, 0.65f, "igemm_128x64_k64s2_w4"},
    {256, 64, 32, 2, 0.60f, "igemm_256x64_k32s3_w4"},
    {128, 32, 64, 4, 0.33f, "igemm_128x32_k64s2_w4"},
    {256, 32, 64, 2, 0.33f, "igemm_256x32_k64s2_w4"},
    {256, 192, 64, 1, 1.05f, "igemm_256x192_k64s2_w8"},
    {192, 256, 64, 1, 1.05f, "igemm_192x256_k64s2_w8"},
    {64, 256, 64, 1, 0.55f, "igemm_64x256_k64s3_w8"},
    {64, 128, 64, 2, 0.45f, "igemm_64x128_k64s3_w4"},
    {192, 128, 64, 1, 0.90f, "igemm_192x128_k64s3_w8"},
};
constexpr int N_TILE_CHOICES = sizeof(kTiles) / sizeof(kTiles[0]);
// plan index of the streaming kernel (stream.hip): not a tile of this file's kernel, one launch for all rows
constexpr int STREAM_TILE = N_TILE_CHOICES;
const char *const kStreamName = "igemm_stream";
// ... and of the window kernel (window.hip), likewise
constexpr int WINDOW_TILE = N_TILE_CHOICES + 1;
const char *const kWindowName = "igemm_window";
// ... whose form with a mask in the epilogue is a plan of its own: the same kernel instantiated for masks, under another name,
// because the tuning hook's and the measured tables' "igemm_window" was timed without a mask, and a forced "igemm_window" leaves
// masked launches to the tiled kernel (as the hook's users, the tests among them, expect).  Forced by its own name; the table
// entries of a masked launch mean it.
constexpr int MASKED_WINDOW_TILE = N_TILE_CHOICES + 2;
const char *const kMaskedWindowName = "igemm_patch_masked";
inline bool whole_launch(int idx) { return idx == STREAM_TILE || idx == WINDOW_TILE || idx == MASKED_WINDOW_TILE; }

// the tiles that also exist reading the filter in place (transposed tiles)
bool has_bt(int idx) { return idx == 0 || idx == 1 || idx == 4 || idx == 6 || idx == 11; }

int launch_choice(int idx, const IgemmParams &p, hipStream_t st, bool bt = false, long long m_begin = 0, long long m_end = -1)
{
    if (bt) {
        switch (idx) {
        case 0: return launch<128, 128, 64, 2, 2, 2, true>(p, st, m_begin, m_end);
        case 1: return launch<256, 256, 64, 2, 2, 4, true>(p, st, m_begin, m_end);
        case 4: return launch<128, 64, 64, 2, 2, 2, true>(p, st, m_begin, m_end);
        case 6: return launch<128, 32, 64, 2, 4, 1, true>(p, st, m_begin, m_end);
        case 11: return launch<64, 128, 64, 3, 2, 2, true>(p, st, m_begin, m_end);
        default: return MXC_ERR_UNSUPPORTED;
        }
    }
    switch (idx) {
    case 0: return launch<128, 128, 64, 2, 2, 2>(p, st, m_begin, m_end);
    case 1: return launch<256, 256, 64, 2, 2, 4>(p, st, m_begin, m_end);
    case 2: return launch<256, 128, 64, 3, 4, 2>(p, st, m_begin, m_end);
    case 3: return launch<128, 256, 64, 3, 2, 4>(p, st, m_begin, m_end);
    case 4: return launch<128, 64, 64, 2, 2, 2>(p, st, m_begin, m_end);
    case 5: return launch<256, 64, 32, 3, 4, 1>(p, st, m_begin, m_end);
    case 6: return launch<128, 32, 64, 2, 4, 1>(p, st, m_begin, m_end);
    case 7: return launch<256, 32, 64, 2, 4, 1>(p, st, m_begin, m_end);
    case 8: return launch<256, 192, 64, 2, 4, 2>(p, st, m_begin, m_end);
    case 9: return launch<192, 256, 64, 2, 2, 4>(p, st, m_begin, m_end);
    case 10: return launch<64, 256, 64, 3, 2, 4>(p, st, m_begin, m_end);
    case 11: return launch<64, 128, 64, 3, 2, 2>(p, st, m_begin, m_end);
    default: return launch<192, 128, 64, 3, 2, 4>(p, st, m_begin, m_end);
    }
}

int launch_classes_choice(int idx, IgemmClasses &q, hipStream_t st)
{
    switch (idx) {
    case 0: return launch_classes<128, 128, 64, 2, 2, 2>(q, st);
    case 1: return launch_classes<256, 256, 64, 2, 2, 4>(q, st);
    case 2: return launch_classes<256, 128, 64, 3, 4, 2>(q, st);
    case 3: return launch_classes<128, 256, 64, 3, 2, 4>(q, st);
    case 4: return launch_classes<128, 64, 64, 2, 2, 2>(q, st);
    case 5: return launch_classes<256, 64, 32, 3, 4, 1>(q, st);
    case 6: return launch_classes<128, 32, 64, 2, 4, 1>(q, st);
    case 7: return launch_classes<256, 32, 64, 2, 4, 1>(q, st);
    case 8: return launch_classes<256, 192, 64, 2, 4, 2>(q, st);
    case 9: return launch_classes<192, 256, 64, 2, 2, 4>(q, st);
    case 10: return launch_classes<64, 256, 64, 3, 2, 4>(q, st);
    case 11: return launch_classes<64, 128, 64, 3, 2, 2>(q, st);
    default: return launch_classes<192, 128, 64, 3, 2, 4>(q, st);
    }
}

// How a GEMM of M rows is run: every row by tile shape `main`, or - when the last round of main tiles would
// leave most CUs idle - rows [0, rows_main) by `main` in whole rounds over the chip and the rest by a second
// launch of the smaller shape `tail` (tail < 0: one launch).
struct Plan { int main, tail; long long rows_main; };

int tile_index(const char *name, size_t len)
{
    for (int i = 0; i < N_TILE_CHOICES; ++i)
        if (strlen(kTiles[i].name) == len && !strncmp(name, kTiles[i].name, len)) return i;
    if (strlen(kStreamName) == len && !strncmp(name, kStreamName, len)) return STREAM_TILE;
    if (strlen(kWindowName) == len && !strncmp(name, kWindowName, len)) return WINDOW_TILE;
    if (strlen(kMaskedWindowName) == len && !strncmp(name, kMaskedWindowName, len)) return MASKED_WINDOW_TILE;
    return -1;
}

// rows covered by the whole rounds of shape t over the chip's workgroup slots
long long whole_round_rows(const TileChoice &t, long long M, int Co)
{
    const long long n_tiles = (Co + t.bn - 1) / t.bn, slots = 256LL * t.slots;
    const long long tiles = ((M + t.bm - 1) / t.bm) * n_tiles;
    const long long rows = (tiles / slots) * slots / n_tiles * t.bm;
    return rows < M ? rows : M;
}

// Modelled time of shape t on M rows.  Tiles are dealt evenly to the 256 CUs, so a CU works through
// ceil(tiles/256) tiles, `slots` at a time; a tile costs its area over the utilisation the shape reaches,
// which drops when fewer workgroups than `slots` share the CU (less latency hiding).  Padding waste and the
// partly filled last round are what differ between shapes.
double model_time(const TileChoice &t, long long M, int Co, int KT, double fixed)
{
    const long long tiles = ((M + t.bm - 1) / t.bm) * ((Co + t.bn - 1) / t.bn);
    const long long per_cu = (tiles + 255) / 256;
    const double resident = per_cu < t.slots ? (double)per_cu : (double)t.slots;
    const double util = t.util * (0.6 + 0.4 * resident / t.slots);
    return (double)per_cu * ((double)t.bm * t.bn / util * KT + fixed / resident);
}

#include "tuned_igemm.inc"

// Plan choice, in this order: MXC_FORCE_VARIANT=<name> or <main>+<tail> (tuning sweeps only); the table of
// measured best plans (tuned_igemm.inc, written by the tuning script from timings on the device) when it
// holds this GEMM; else the least modelled time over single shapes and main+tail pairs.
// allow_stream = false: callers that need a tile of this file's kernel, not one of the whole-launch kernels (split
// reductions, in-place filters).
thread_local long long g_key_M = 0;
thread_local int g_key_Co = 0, g_key_Kd = 0;

Plan search_plan(long long M, int Co, int Kd, bool allow_stream, bool masked)
{
    ++g_plan_searches;
    if (const char *f = getenv("MXC_FORCE_VARIANT")) {
        const char *plus = strchr(f, '+'), *slash = strchr(f, '/');
        const int a = tile_index(f, plus ? (size_t)(plus - f) : slash ? (size_t)(slash - f) : strlen(f));
        const int b = plus ? tile_index(plus + 1, strlen(plus + 1)) : -1;
        if (a >= 0 && whole_launch(a) && !plus && allow_stream && !(a == WINDOW_TILE && masked) && !(a == MASKED_WINDOW_TILE && !masked)) return Plan{a, -1, M};
        if (a >= 0 && !whole_launch(a) && !whole_launch(b) && (!plus || b >= 0)) {
            const long long rows = b >= 0 ? whole_round_rows(kTiles[a], M, Co) : M;
            return (b >= 0 && rows > 0 && rows < M) ? Plan{a, b, rows} : Plan{a, -1, M};
        }
    }
    for (const TunedIgemm &e : kTunedIgemm)
        if (e.M == M && e.Co == Co && e.Kd == Kd) {
            const int a = tile_index(e.main, strlen(e.main)), b = e.tail[0] ? tile_index(e.tail, strlen(e.tail)) : -1;
            if (a < 0 || whole_launch(b) || (whole_launch(a) && !allow_stream)) break;
            if (whole_launch(a)) return Plan{a == WINDOW_TILE && masked ? MASKED_WINDOW_TILE : a, -1, M};
            const long long rows = b >= 0 ? whole_round_rows(kTiles[a], M, Co) : M;
            return (b >= 0 && rows > 0 && rows < M) ? Plan{a, b, rows} : Plan{a, -1, M};
        }
    // Reductions of one or two stages (first layers): a workgroup's fixed cost (launch, pipeline fill,
    // epilogue: about 4 us, shared by the workgroups resident on the CU) outweighs its matrix work, so
    // fewer, larger tiles win.  In the model's units (tile area x stages at 256x256 speed) that cost
    // is about 150000; a second launch costs about 200000 (5 us of drain, launch and refill).
    const int KT = (Kd + 63) / 64;
    const double fixed = KT <= 2 ? 150000.0 : 0.0, second_launch = 200000.0;
    Plan best{0, -1, M};
    double best_t = 1e300;
    for (int i = 0; i < N_TILE_CHOICES; ++i) {
        const double t1 = model_time(kTiles[i], M, Co, KT, fixed);
        if (t1 < best_t) { best_t = t1; best = Plan{i, -1, M}; }
        const long long rows = whole_round_rows(kTiles[i], M, Co);
        if (rows <= 0 || rows >= M) continue;
        const double t_main = model_time(kTiles[i], rows, Co, KT, fixed);
        for (int j = 0; j < N_TILE_CHOICES; ++j) {
            if (j == i) continue;
            const double t2 = t_main + model_time(kTiles[j], M - rows, Co, KT, fixed) + second_launch;
            if (t2 < best_t) { best_t = t2; best = Plan{i, j, rows}; }
        }
    }
    return best;
}

// What a thread's plans are kept by; flags hold what else the answer depends on.
struct GemmKey { long long M; int Co, Kd; long long flags; };

// The search walks the table and every pair of shapes: the calling thread keeps its answers.
Plan choose_plan(long long M, int Co, int Kd, bool allow_stream = true, bool masked = false)
{
    g_key_M = M; g_key_Co = Co; g_key_Kd = Kd;
    if (getenv("MXC_FORCE_VARIANT")) return search_plan(M, Co, Kd, allow_stream, masked);
    static thread_local PlanCache<GemmKey, Plan> cache;
    return cache.get(GemmKey{M, Co, Kd, (allow_stream ? 1 : 0) + (masked ? 2 : 0)}, [&] { return search_plan(M, Co, Kd, allow_stream, masked); });
}

int choose_tile(long long M, int Co, int Kd) { return choose_plan(M, Co, Kd, false).main; }

// the plan for one launch site: the streaming or the window kernel only where it can run the problem
Plan plan_for(const IgemmParams &p, long long M, int Co, int Kd, bool tiles_only = false)
{
    const Plan pl = choose_plan(M, Co, Kd, !tiles_only, p.mask != nullptr);
    if (pl.main == STREAM_TILE && !stream_applicable(p)) return choose_plan(M, Co, Kd, false);
    if ((pl.main == WINDOW_TILE || pl.main == MASKED_WINDOW_TILE) && !window_applicable(p)) return choose_plan(M, Co, Kd, false);
    return pl;
}

// runs the plan: one or two launches on the stream
int launch_plan(const Plan &pl, const IgemmParams &p, hipStream_t st, bool bt = false)
{
    if (pl.main == STREAM_TILE) return stream_launch(p, st);
    if (pl.main == WINDOW_TILE || pl.main == MASKED_WINDOW_TILE) return window_launch(p, st);
    if (pl.tail < 0) return launch_choice(pl.main, p, st, bt);
    const int rc = launch_choice(pl.main, p, st, bt, 0, pl.rows_main);
    if (rc != MXC_OK) return rc;
    return launch_choice(pl.tail, p, st, bt, pl.rows_main, -1);
}

// name of a plan for mxc_last_variant(): "<main>" or "<main>+<tail>"
const char *plan_name(const Plan &pl)
{
    static thread_local char name[96];
    if (pl.main == STREAM_TILE) return kStreamName;
    if (pl.main == WINDOW_TILE) return kWindowName;
    if (pl.main == MASKED_WINDOW_TILE) return kMaskedWindowName;
    if (pl.tail < 0) return kTiles[pl.main].name;
    snprintf(name, sizeof(name), "%s+%s", kTiles[pl.main].name, kTiles[pl.tail].name);
    return name;
}

// The kernel addresses both operands with signed 32-bit byte offsets, packs tile-row coordinates
// into 16 bits and holds at most MAX_TAPS filter taps in its tap table.
bool igemm_dims_ok(long long in_elems, long long wm_elems, long long M, int Hi, int Wi, int span, int taps)
{
    return in_elems * 2 < 0x7FFF0000ll && wm_elems * 2 < 0x7FFF0000ll && M < 0x7FFFFFFFll && Hi + span <= 8192 &&
           Wi + span <= 8192 && taps <= MAX_TAPS;
}

// dx of the residue classes that no tap reaches: zeros, where neither the tiles of a 1x1 filter at stride 2 write them beside their results
// (ZR) nor the wave kernel, whose classes they are.  What is left: strides of 3 and 4 with filters of fewer rows or columns, odd padding,
// channels that are no multiple of 8, dx of 2 GiB and more, tiles without ZR.  One workgroup per image row; `zero_h` / `zero_w`: bit
// (coordinate + pad) % stride of the rows / columns without a tap.
template <int V>      // channels per store: 8 (16 bytes) or 1
__global__ __launch_bounds__(256) void zero_classes_kernel(bf16_t *__restrict__ dx, int H, int W, int C, int stride, int pad, unsigned zero_h,
                                                           unsigned zero_w)
{
    const int h = blockIdx.x % H, per_pix = C / V;
    const bool whole = (zero_h >> ((h + pad) % stride)) & 1;
    if (!whole && zero_w == 0) return;
    bf16_t *row = dx + (size_t)blockIdx.x * W * C;
    for (int i = threadIdx.x; i < W * per_pix; i += 256) {
        const unsigned w = (unsigned)i / (unsigned)per_pix;
        if (whole || ((zero_w >> ((w + pad) % stride)) & 1)) {
            typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
            if constexpr (V == 8) __builtin_nontemporal_store(u32x4{0, 0, 0, 0}, reinterpret_cast<u32x4 *>(row) + i);
            else row[i] = 0;
        }
    }
}

// How many ways to split the reduction of a GEMM whose tiles would leave most of the chip idle
// (FullyConnected-shaped and small-batch problems): enough workgroups to fill the slots, at least 8
// stages per split, at most 32 splits.  1 = no split (every layer of the benchmark stacks).
int split_count(long long M, int Co, int Kd)
{
    const TileChoice &t = kTiles[choose_tile(M, Co, Kd)];
    if (const char *f = getenv("MXC_FORCE_VARIANT"))
        if (const char *slash = strchr(f, '/')) {
            const int most = (Kd + t.bk - 1) / t.bk, sp = atoi(slash + 1);
            return sp < 1 ? 1 : sp < most ? sp : most;
        }
    const long long tiles = ((M + t.bm - 1) / t.bm) * ((Co + t.bn - 1) / t.bn);
    const long long slots = 256LL * t.slots;
    if (tiles * 2 > slots) return 1;
    long long sp = slots / tiles;
    const long long KT = (Kd + 63) / 64;
    if (sp > KT / 8) sp = KT / 8;
    if (sp > 32) sp = 32;
    return sp >= 2 ? (int)sp : 1;
}

// Modelled time (us, fitted to the 828 GEMMs of wave.hip's model, 9% off) of one tile shape on all rows in `splits` ranges of
// the reduction: launch, the CU's share of padded tile area, partial tiles, rounds, results and mask.
double tile_us(const TileChoice &t, long long M, int Co, int Kd, int splits, bool masked)
{
    const long long tiles = ((M + t.bm - 1) / t.bm) * ((Co + t.bn - 1) / t.bn) * splits, per_cu = (tiles + 255) / 256;
    const long long resident = per_cu < t.slots ? per_cu : t.slots, rounds = (per_cu + t.slots - 1) / t.slots;
    const int KT = ((Kd + 63) / 64 + splits - 1) / splits;
    const double util = t.util * (0.6 + 0.4 * resident / t.slots), mc = 1e-6 * M * Co;
    return 2.37 + 1.38 * per_cu * t.bm * t.bn / 65536.0 / util * KT + 2.14 * rounds + (splits > 1 ? 1.7 + 2.19 * splits * mc : 0) + (masked ? 0.92 : 0.46) * mc;
}

// ... of a plan: its main tile on the rows it takes, and a second launch for the rest
double plan_us(const Plan &pl, long long M, int Co, int Kd, int splits, bool masked)
{
    if (pl.tail < 0 || splits > 1) return tile_us(kTiles[pl.main], M, Co, Kd, splits, masked);
    return tile_us(kTiles[pl.main], pl.rows_main, Co, Kd, 1, masked) + tile_us(kTiles[pl.tail], M - pl.rows_main, Co, Kd, 1, masked);
}

// The shape of the wave kernel (wave.hip) that runs this GEMM, or -1: the planned kernel does.  Of 600 forward and dx passes of 300
// random layers (up to 60 GFLOP; 27% NCHW) it runs 478; those that the planned kernel takes below 8, 8-12, 12-20, 20-40 and more us
// run 1.48, 1.68, 1.58, 1.29 and 1.49 times as fast (four of them more than 2% slower, 14% at worst: 56000 pixels, 24 columns, Kd = 1008).
// The models must agree by a margin, larger from 18 and from 36 modelled us on, where what they miss weighs more.  Measured time over
// the planned kernel's, mean and worst, by the ratio of the models: below 18 us at 0.85-0.92 0.87 / 0.98, at 0.92-1 0.96 / 1.40; 18-36 us
// at 0.74-0.785 0.88 / 1.08, at 0.785-0.85 0.93 / 1.14, at 0.85-0.92 1.13 / 1.31; 36-60 us at 0.69-0.92 0.93 / 1.24; above 60 us
// at 0.85-1 1.18 / 1.60 (359464 pixels, 24 columns, 5x5 on 320 channels: 432 us measured against 290).
int wave_choice(long long M, int Co, int Kd, bool bwd, bool masked, bool can_split)
{
    g_key_M = M; g_key_Co = Co; g_key_Kd = Kd;
    if (const char *f = getenv("MXC_FORCE_VARIANT")) return wave_forced(f, bwd);
    static thread_local PlanCache<GemmKey, int> cache;
    return cache.get(GemmKey{M, Co, Kd, (bwd ? 1 : 0) + (masked ? 2 : 0) + (can_split ? 4 : 0)}, [&] {
        ++g_plan_searches;
        const Plan pl = choose_plan(M, Co, Kd, true, masked);
        double us = 0;
        const int wave = whole_launch(pl.main) ? -1 : wave_best(M, Co, Kd, bwd, masked, &us);
        if (wave < 0) return -1;
        const double other = plan_us(pl, M, Co, Kd, can_split ? split_count(M, Co, Kd) : 1, masked);
        return us > other * (us < 18 ? 0.92 : us < 36 ? 0.785 : 0.69) ? -1 : wave;
    });
}

// The shape of the run kernel (runs.hip) that runs this GEMM, or -1: the wave kernel or the plan does, whichever it is without the run
// kernel.  Of an NCHW problem the wave kernel stores the result to its planes, which is a re-layout less.  Measured time over the other
// kernel's, mean and worst, by the ratio of the models (12685 layers of 0.3 to 300 GFLOP, forward and dx): others below 60 us at 0.8-0.85 0.82 /
// 1.11, at 0.85-0.9 0.86 / 1.16; from 60 us on at 0.85-0.9 0.86 / 1.16, at 0.9-0.95 0.89 / 1.12, at 0.95-1 0.91 / 1.07; 320 earlier layers had 1.2
// and more above 1.  Wave kernels below 8 modelled us, whose launch weighs most, at 0.85-0.875 0.84 / 1.01, at 0.875-0.9 1.01 / 1.15 (201
// layers, half of them more than 3% slower); plans of a split reduction 0.95 / 1.08 and 1.00 / 1.16.  Plans of the streaming and window
// kernels come from the measured table and stay.
int run_choice(const IgemmParams &p, bool bwd, bool masked, bool can_split, bool planes)
{
    if (!run_applicable(p)) return -1;
    const long long M = (long long)p.N * p.Mh * p.Mw;
    const int Kd = p.TR * p.TS * p.Ci;
    g_key_M = M; g_key_Co = p.Co; g_key_Kd = Kd;
    if (const char *f = getenv("MXC_FORCE_VARIANT")) return run_forced(f, p);
    struct Key { long long M; int Co, Ci, TR, TS; long long flags; };
    static thread_local PlanCache<Key, int> cache;
    return cache.get(Key{M, p.Co, p.Ci, p.TR, p.TS, (bwd ? 1 : 0) + (masked ? 2 : 0) + (can_split ? 4 : 0) + (planes ? 8 : 0)}, [&] {
        ++g_plan_searches;
        double us = 0, other = 0;
        const int run = run_best(M, p.Co, p.Ci, p.TR, p.TS, masked, &us);
        const int wave = wave_choice(M, p.Co, Kd, bwd, masked, can_split);
        const Plan pl = choose_plan(M, p.Co, Kd, true, masked);
        if (whole_launch(pl.main) || (wave >= 0 && planes)) return -1;
        if (wave >= 0) wave_best(M, p.Co, Kd, bwd, masked, &other);
        const int splits = wave < 0 && can_split ? split_count(M, p.Co, Kd) : 1;
        if (wave < 0) other = plan_us(pl, M, p.Co, Kd, splits, masked);
        // two launches take longer than modelled, at 0.9-1 0.87 / 0.98 (9 layers), but not with tiles of 256x256: 0.97 / 1.15 (5)
        const bool largest = wave < 0 && pl.main == 1, two = wave < 0 && pl.tail >= 0;
        const bool close = splits > 1 || (wave >= 0 && other < 8);
        return us < (close ? 0.875 : largest ? 0.9 : two ? 1. : other >= 60 ? 0.95 : 0.9) * other ? run : -1;
    });
}

// Whether the streaming kernel runs a 1x1 filter at stride 1 that the measured table does not hold, in the wave kernel's or the plan's place (of
// an NCHW problem the wave kernel stays, see run_choice), by the models of both (stream_pays).  What the tiles lose is that a CU's loads
// wait while it stores.
bool stream_choice(const IgemmParams &p, bool bwd, bool masked, bool can_split, bool planes)
{
    if (p.TR * p.TS != 1 || p.in_mul_h != 1 || p.in_mul_w != 1 || getenv("MXC_FORCE_VARIANT") || !stream_applicable(p)) return false;
    const long long M = (long long)p.N * p.Mh * p.Mw;
    g_key_M = M; g_key_Co = p.Co; g_key_Kd = p.Ci;
    static thread_local PlanCache<GemmKey, bool> cache;
    return cache.get(GemmKey{M, p.Co, p.Ci, (bwd ? 1 : 0) + (masked ? 2 : 0) + (can_split ? 4 : 0) + (planes ? 8 : 0)}, [&] {
        ++g_plan_searches;
        double other = 0;
        const int wave = wave_choice(M, p.Co, p.Ci, bwd, masked, can_split);
        const Plan pl = choose_plan(M, p.Co, p.Ci, true, masked);
        if (whole_launch(pl.main) || (wave >= 0 && planes)) return false;
        if (wave >= 0) wave_best(M, p.Co, p.Ci, bwd, masked, &other);
        else other = plan_us(pl, M, p.Co, p.Ci, can_split ? split_count(M, p.Co, p.Ci) : 1, masked);
        return stream_pays(p, masked, other);
    });
}

// out[m][co] = act(sum_z partial[z][m][co] + bias[co]) in ascending z (fixed order), 4 columns per thread
__global__ __launch_bounds__(256) void split_finish_kernel(const float *__restrict__ partial, bf16_t *__restrict__ out, long long MC,
                                                           int Co, int Cw, int splits, const float *__restrict__ bias, int relu,
                                                           const bf16_t *__restrict__ mask)
{
    const long long i4 = ((long long)blockIdx.x * blockDim.x + threadIdx.x) * 4;
    if (i4 >= MC) return;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int z = 0; z < splits; ++z) {
        const float4 v = *reinterpret_cast<const float4 *>(partial + (size_t)z * MC + i4);
        acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
    }
    if (bias != nullptr) {
        const int co = (int)(i4 % Co);          // Co % 8 == 0: the four columns share a row
        if (co + 4 <= Cw) { acc.x += bias[co]; acc.y += bias[co + 1]; acc.z += bias[co + 2]; acc.w += bias[co + 3]; }
        else { if (co < Cw) acc.x += bias[co]; if (co + 1 < Cw) acc.y += bias[co + 1]; if (co + 2 < Cw) acc.z += bias[co + 2]; }
    }
    if (relu) { acc.x = fmaxf(acc.x, 0.f); acc.y = fmaxf(acc.y, 0.f); acc.z = fmaxf(acc.z, 0.f); acc.w = fmaxf(acc.w, 0.f); }
    uint2 o = make_uint2((uint32_t)f32_to_bf16(acc.x) | ((uint32_t)f32_to_bf16(acc.y) << 16),
                         (uint32_t)f32_to_bf16(acc.z) | ((uint32_t)f32_to_bf16(acc.w) << 16));
    if (mask != nullptr) {
        const uint2 mk = *reinterpret_cast<const uint2 *>(mask + i4);
        o = make_uint2(mask_bf16x2(o.x, mk.x), mask_bf16x2(o.y, mk.y));
    }
    *reinterpret_cast<uint2 *>(out + i4) = o;
}

// One GEMM (output pixels numbered like the GEMM rows, Co % 8 == 0) run as `sp` splits of the reduction
// plus the finishing kernel, which applies `post`.
int launch_split(int tc, IgemmParams p, long long M, int sp, void *split_ws, void *out, const PostOp &post, hipStream_t st,
                 const char **variant, bool bt = false)
{
    p.splits = sp;
    p.partial = (float *)split_ws;
    p.bias = nullptr; p.relu = 0; p.mask = nullptr;      // applied by the finishing kernel
    const int rc = launch_choice(tc, p, st, bt);
    if (rc != MXC_OK) return rc;
    const long long MC = M * p.Co;
    if ((MC / 4 + 255) / 256 > 0x7FFFFFFFll) return MXC_ERR_SHAPE;
    // the launcher evens out the stage ranges, which can lower the split count: recompute it the same way
    const int bk = kTiles[tc].bk;
    const int KT = stages_of(p.TR * p.TS, p.Ci, bk, kTiles[tc].bn, M), per = (KT + sp - 1) / sp, used = (KT + per - 1) / per;
    static thread_local char split_name[64];
    snprintf(split_name, sizeof(split_name), "%s%s_split%d", kTiles[tc].name, bt ? "_inplace" : "", used);
    *variant = split_name;
    hipLaunchKernelGGL(split_finish_kernel, dim3((unsigned)((MC / 4 + 255) / 256)), dim3(256), 0, st, (const float *)split_ws,
                       (bf16_t *)out, MC, p.Co, p.Cw ? p.Cw : p.Co, used, post.bias, post.relu, (const bf16_t *)post.mask);
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
}

}  // namespace

const char *igemm_tile_name(int index) { return index >= 0 && index < N_TILE_CHOICES ? kTiles[index].name : nullptr; }
const char *igemm_stream_name(int index) { return index == 0 ? kStreamName : index == 1 ? kWindowName : nullptr; }
void igemm_last_plan_key(long long *M, int *Co, int *Kd) { *M = g_key_M; *Co = g_key_Co; *Kd = g_key_Kd; }

size_t igemm_bwd_data_split_bytes(const ConvShape &s)
{
    if (s.stride != 1 || s.C % 8 != 0) return 0;       // one residue class, output numbered like the GEMM rows
    const long long M = (long long)s.N * s.H * s.W;
    const int sp = split_count(M, s.C, s.R * s.S * s.K);
    return sp > 1 ? (size_t)sp * M * s.C * sizeof(float) : 0;
}

size_t igemm_fwd_split_bytes(const ConvShape &s)
{
    if (s.K % 8 != 0) return 0;
    const long long M = (long long)s.N * s.P * s.Q;
    const int sp = split_count(M, s.K, s.R * s.S * s.C);
    return sp > 1 ? (size_t)sp * M * s.K * sizeof(float) : 0;
}

bool igemm_fwd_supported(const ConvShape &s)
{
    return s.C % 8 == 0 && igemm_dims_ok((long long)s.N * s.H * s.W * s.C, (long long)s.K * s.R * s.S * s.C,
                                         (long long)s.N * s.P * s.Q, s.H, s.W, s.pad + s.R + s.S + s.stride, s.R * s.S);
}

int igemm_fwd(const ConvShape &s, const void *x, const void *w, void *y, hipStream_t st, const char **variant, const PostOp &post,
              void *split_ws)
{
    IgemmParams p{};
    p.bias = post.bias; p.relu = post.relu; p.copied = post.copied;
    p.in = (const bf16_t *)x; p.wm = (const bf16_t *)w; p.out = (bf16_t *)y;
    p.N = s.N; p.Hi = s.H; p.Wi = s.W; p.Ci = s.C; p.pix = s.C; p.Co = s.K; p.Cw = real_k(s);
    p.TR = s.R; p.TS = s.S; p.tstep_h = 1; p.tstep_w = 1;
    p.Mh = s.P; p.Mw = s.Q;
    p.in_mul_h = s.stride; p.in_mul_w = s.stride; p.in_off_h = -s.pad; p.in_off_w = -s.pad;
    p.Ho = s.P; p.Wo = s.Q; p.out_mul_h = 1; p.out_mul_w = 1; p.out_off_h = 0; p.out_off_w = 0;
    const long long M = (long long)s.N * s.P * s.Q;
    if (const int rv = run_choice(p, false, false, split_ws != nullptr && s.K % 8 == 0, post.planes != nullptr); rv >= 0) {
        *variant = run_name(rv);
        return run_launch(rv, p, st);
    }
    if (stream_choice(p, false, false, split_ws != nullptr && s.K % 8 == 0, post.planes != nullptr)) {
        *variant = kStreamName;
        return stream_launch(p, st);
    }
    if (const int wv = wave_choice(M, s.K, s.R * s.S * s.C, false, false, split_ws != nullptr && s.K % 8 == 0); wv >= 0) {
        *variant = wave_name(wv);
        return wave_launch(wv, p, st, false, post.planes);
    }
    const int sp = (split_ws != nullptr && s.K % 8 == 0) ? split_count(M, s.K, s.R * s.S * s.C) : 1;
    const Plan pl = plan_for(p, M, s.K, s.R * s.S * s.C, sp > 1);
    *variant = plan_name(pl);
    if (sp > 1) return launch_split(pl.main, p, M, sp, split_ws, y, post, st, variant);
    return launch_plan(pl, p, st);
}

// Plain GEMM on the same kernels: out[m][n] = sum_k a[m][k] * b[n][k], a and b bf16 (row-major, k contiguous, k % 8 == 0),
// out fp32, n % 8 == 0.  It is the 1x1 convolution of an M-image batch of 1x1 images whose fp32 accumulators are
// stored unrounded (the transform-domain convolution multiplies its 16 planes with it).
bool igemm_gemm_f32_supported(long long M, int Kd, int Nn)
{
    return Kd % 8 == 0 && Nn % 8 == 0 && igemm_dims_ok(M * Kd, (long long)Nn * Kd, M, 1, 1, 4, 1) && M * Nn * 4 < (1ll << 40);
}

int igemm_gemm_f32(long long M, int Kd, int Nn, const void *a, const void *b, float *out, hipStream_t st, const char **variant)
{
    IgemmParams p{};
    p.in = (const bf16_t *)a; p.wm = (const bf16_t *)b; p.out = nullptr;
    p.partial = out; p.f32_out = 1;
    p.N = (int)M; p.Hi = 1; p.Wi = 1; p.Ci = Kd; p.pix = Kd; p.Co = Nn;
    p.TR = 1; p.TS = 1; p.tstep_h = 1; p.tstep_w = 1;
    p.Mh = 1; p.Mw = 1;
    p.in_mul_h = 1; p.in_mul_w = 1; p.in_off_h = 0; p.in_off_w = 0;
    p.Ho = 1; p.Wo = 1; p.out_mul_h = 1; p.out_mul_w = 1; p.out_off_h = 0; p.out_off_w = 0;
    const Plan pl = choose_plan(M, Nn, Kd, false);
    *variant = plan_name(pl);
    return launch_plan(pl, p, st);
}

bool igemm_fwd_smallc_supported(const ConvShape &s)
{
    const SmallCGeom g = smallc_geom(s);
    return s.C <= 4 && igemm_dims_ok((long long)s.N * g.Hp * g.Wp * g.pix, (long long)s.K * s.R * g.run,
                                     (long long)s.N * s.P * s.Q, g.Hp, g.Wp, s.R + s.S + s.stride, s.R);
}

// Forward for a small-C image packed by smallc_pack_x / smallc_pack_w: R taps (filter rows), each a
// contiguous run of S*pix elements of the zero-bordered image.
int igemm_fwd_smallc(const ConvShape &s, const void *xp, const void *wp, void *y, hipStream_t st, const char **variant,
                     const PostOp &post)
{
    const SmallCGeom g = smallc_geom(s);
    IgemmParams p{};
    p.bias = post.bias; p.relu = post.relu;
    p.in = (const bf16_t *)xp; p.wm = (const bf16_t *)wp; p.out = (bf16_t *)y;
    p.N = s.N; p.Hi = g.Hp; p.Wi = g.Wp; p.Ci = g.run; p.pix = g.pix; p.Co = s.K; p.Cw = real_k(s);
    p.TR = s.R; p.TS = 1; p.tstep_h = 1; p.tstep_w = 1;
    p.Mh = s.P; p.Mw = s.Q;
    p.in_mul_h = s.stride; p.in_mul_w = s.stride; p.in_off_h = 0; p.in_off_w = 0;
    p.Ho = s.P; p.Wo = s.Q; p.out_mul_h = 1; p.out_mul_w = 1; p.out_off_h = 0; p.out_off_w = 0;
    if (const int wv = wave_choice((long long)s.N * s.P * s.Q, s.K, s.R * g.run, false, false, false); wv >= 0) {
        *variant = wave_name(wv);
        return wave_launch(wv, p, st, false, post.planes);
    }
    const Plan pl = plan_for(p, (long long)s.N * s.P * s.Q, s.K, s.R * g.run);
    *variant = plan_name(pl);
    return launch_plan(pl, p, st);
}

bool igemm_bwd_data_supported(const ConvShape &s)
{
    return s.K % 8 == 0 && s.stride <= 4 &&
           igemm_dims_ok((long long)s.N * s.P * s.Q * s.K, (long long)s.K * s.R * s.S * s.C, (long long)s.N * s.H * s.W, s.P,
                         s.Q, s.pad + s.R + s.S + s.stride, s.R * s.S);
}

size_t igemm_bwd_data_workspace(const ConvShape &s) { return (size_t)s.K * s.R * s.S * s.C * sizeof(bf16_t); }

namespace {
// stride 1: the one launch of the pass
IgemmParams bwd_data_params(const ConvShape &s)
{
    IgemmParams p{};
    p.N = s.N; p.Hi = s.P; p.Wi = s.Q; p.Ci = s.K; p.pix = s.K; p.Co = s.C; p.Cw = real_c(s);
    p.tstep_h = -1; p.tstep_w = -1;
    p.in_mul_h = 1; p.in_mul_w = 1;
    p.Ho = s.H; p.Wo = s.W; p.out_mul_h = s.stride; p.out_mul_w = s.stride;
    if (s.stride == 1) {
        // one class: rows h = hh - pad of hh = pad, pad + 1, ...
        p.TR = s.R; p.TS = s.S; p.Mh = s.H; p.Mw = s.W; p.in_off_h = s.pad; p.in_off_w = s.pad;
        p.bt_w_bytes = (unsigned)((long long)real_k(s) * s.R * s.S * s.C * 2);
    }
    return p;
}

// whether the whole pass is one launch of the streaming kernel, which then can take the filter as it is
bool bwd_data_streams_filter(const ConvShape &s, bool masked)
{
    const long long M = (long long)s.N * s.H * s.W;
    const int Kd = s.R * s.S * s.K;
    return s.stride == 1 && choose_plan(M, s.C, Kd, true, masked).main == STREAM_TILE && split_count(M, s.C, Kd) == 1 &&
           stream_applicable(bwd_data_params(s));
}
}  // namespace

// Needs columns of one staging pass and every image pixel inside some block of the packed grid (one that is not has a zero
// that nobody would write).
ImageStore igemm_bwd_data_image_store(const ConvShape &s2, const S2DStore &q)
{
    if (s2.stride != 1 || s2.C > 64 || s2.H * q.s - q.pad < q.H || s2.W * q.s - q.pad < q.W || q.H >= 16384 || q.W >= 16384 ||
        (long long)s2.N * q.H * q.W * q.C * 2 >= 0x7FFF0000ll || bwd_data_reads_filter_in_place(s2))
        return IMAGE_NONE;
    IgemmParams p = bwd_data_params(s2);
    p.s2d = q;
    const long long M = (long long)s2.N * s2.H * s2.W;
    const int Kd = s2.R * s2.S * s2.K;
    const bool stream = stream_applicable(p), window = window_applicable(p);
    if (getenv("MXC_FORCE_VARIANT")) {
        const int f = choose_plan(M, s2.C, Kd).main;
        return f == STREAM_TILE && stream ? IMAGE_STREAM : f == WINDOW_TILE && window ? IMAGE_WINDOW : IMAGE_NONE;
    }
    // Against the planned kernel with the separate un-packing (20 us for 128 224x224x3 images), input gradients in us, before ->
    // streaming / window: Kd = 64 (3x3 stride 2, K = 16, 200 100x100 images) 38 -> 27 / 37; Kd = 128 33 -> 30 / 29; Kd = 256 38 ->
    // 38 / 33; Kd = 320 36 -> 35 / -; Kd = 384 60 -> 65 / -; 11x11 stride 4, K = 64, batch 128 (Kd = 576) 66 -> 104 / 62; 7x7
    // stride 2, K = 64, batch 64 (Kd = 1024) 127 -> 256 / 88; with patches half empty (35x35 blocks) or too few the window
    // kernel loses up to 1 us of 18.
    if (Kd <= 64 && stream) return IMAGE_STREAM;
    if (window && window_fills_chip(p)) return IMAGE_WINDOW;
    return Kd <= 320 && stream ? IMAGE_STREAM : IMAGE_NONE;
}

int igemm_bwd_data_image(ImageStore kind, const ConvShape &s2, const S2DStore &q, const void *dy, const void *w2, const void *wt, void *dx, hipStream_t st,
                         const char **variant)
{
    IgemmParams p = bwd_data_params(s2);
    p.in = (const bf16_t *)dy; p.out = (bf16_t *)dx; p.s2d = q;
    p.wm = (const bf16_t *)(w2 != nullptr ? w2 : wt);
    p.wm_by_k = w2 != nullptr;
    g_key_M = (long long)s2.N * s2.H * s2.W; g_key_Co = s2.C; g_key_Kd = s2.R * s2.S * s2.K;      // (chosen without a plan)
    *variant = kind == IMAGE_STREAM ? kStreamName : kWindowName;
    return kind == IMAGE_STREAM ? stream_launch(p, st) : window_launch(p, st);
}

// Whether a call that is handed the KRSC filter itself reads it in place although a prepared filter would be re-packed:
// the re-pack is a launch of 4-5 us, which a small problem's slower operand fetch does not cost.  Same tile, same order
// of the reduction, same bits.  Measured over 60 shapes, masked or not: below 2 GFLOP every tile with the variant gains
// (64x128 2 us, 128x32 and 128x64 3.6 us of 12), at 4-10 GFLOP 2-3 us of 25-35, and from 12 GFLOP on it loses with
// 64x128 (15%) and breaks even with the others, which is where the line lies.
// The streaming kernel transposes the filter into its resident copy at any size, and the run kernel reads it in place (72 layers of up to 170 GFLOP:
// 1.01 of the time with a re-packed filter, which takes 4 to 5 us to make; 1.12 at worst).
bool bwd_data_small_in_place(const ConvShape &s, bool masked)
{
    if (real_c(s) != s.C || s.C % 8 != 0 || s.stride != 1 || bwd_data_reads_filter_in_place(s)) return false;
    const long long M = (long long)s.N * s.H * s.W;
    const int Kd = s.R * s.S * s.K;
    const IgemmParams p = bwd_data_params(s);
    if (run_choice(p, true, masked, true, false) >= 0 || stream_choice(p, true, masked, true, false)) return true;
    if (wave_choice(M, s.C, Kd, true, masked, true) >= 0 || bwd_data_streams_filter(s, masked)) return true;
    const Plan pl = choose_plan(M, s.C, Kd, true, masked);
    if (whole_launch(pl.main) || !has_bt(pl.main) || (pl.tail >= 0 && !has_bt(pl.tail))) return false;
    return 2.0 * M * s.C * Kd < 1e10;
}

// Whether the launch of the GEMM can write the zeros too (ZR): dx of a 1x1 filter at stride 2
static bool zeroes_rest(const ConvShape &s)
{
    return s.R * s.S == 1 && s.stride == 2 && s.pad % 2 == 0 && s.C % 8 == 0 && (long long)s.N * s.H * s.W * s.C * 2 < 0x7FFF0000ll;
}
static long long even_pixels(const ConvShape &s) { return (long long)s.N * ((s.H + 1) / 2) * ((s.W + 1) / 2); }

// ... and the tile that runs it.  Time models (us, fitted to 580 such layers of up to 900 MB of dx, 6-10% off; of another 193 the chosen
// tile takes 1.5% more than the fastest): launch, and the root of the squares of the CU's share of work (rounds of workgroups, stages,
// tiles) and of the MB that are moved (dx, mask, dy once per column tile), which run beside each other.  The tiles' general model
// knows no dx of four times its rows: 40071 pixels, 80 to 16 channels 14.2 -> 6.5 us.
static int zeroing_tile(const ConvShape &s, bool masked, double *us)
{
    static const struct { int tile; float fixed, round, stage, area, out, mask, in; } kUs[] = {
        {0, 4.16f, 0.903f, 0.563f, 1.69f, 0.144f, 0.171f, 0.052f}, {1, 1.12f, 9.03f, 0.294f, 0.267f, 0.165f, 0.205f, 0.165f},
        {4, 3.20f, 1.52f, 0.732f, 1.34f, 0.227f, 0.090f, 0.f},     {6, 4.12f, 0.f, 1.149f, 1.84f, 0.200f, 0.058f, 0.014f},
        {11, 3.44f, 0.559f, 0.724f, 3.27f, 0.104f, 0.294f, 0.022f}};
    const long long M = even_pixels(s);
    const int KT = (s.K + 63) / 64;
    int best = -1;
    for (const auto &u : kUs) {
        const TileChoice &t = kTiles[u.tile];
        const long long n_tiles = (s.C + t.bn - 1) / t.bn, per_cu = ((M + t.bm - 1) / t.bm * n_tiles + 255) / 256, rounds = (per_cu + t.slots - 1) / t.slots;
        const double work = u.round * rounds + (u.stage * KT + u.area) * per_cu * t.bm * t.bn / 16384.0;
        const double moved = 2e-6 * (u.out * s.N * s.H * s.W * s.C + (masked ? u.mask * M * s.C : 0.) + (double)u.in * M * s.K * n_tiles);
        const double v = u.fixed + sqrt(work * work + moved * moved);
        if (best < 0 || v < *us) { best = u.tile; *us = v; }
    }
    return best;
}

// The wave kernel's shape that runs dx of a layer of stride 2, all residue classes in one launch that reads the KRSC filter as it is, or -1.
// Filters of several taps: against re-packed filter, tile kernel and zeros, each its own launch; of the layers it is chosen for none runs
// slower: 9x10x10 128 to 128 channels 3x3 12.5 -> 4.7 us.  A prepared filter saves the other path its first launch, and has to give the
// same bits: six of 175 layers more than 3% slower (15% at worst).  The margin is larger from 10 modelled us on.  Measured time over the
// other path's by the ratio of the models: 10-20 us at 0.5-0.6 0.55, with a prepared filter up to 1.37, at 0.6-0.8 0.98 (1.27).
// 1x1 filters: against the tile that writes the zeros too, one launch as well.  Of 5386 layers of up to 80 MB the kernel chosen takes 1.4% more than
// the fastest of the five wave shapes and five tiles (1.27 times as long at worst), as much with a line at 1.03 or 1.1, 1.9% with one at 0.95.
static int classes_wave(const ConvShape &s, bool masked)
{
    if (s.stride != 2 || s.C % 8 != 0) return -1;
    if (const char *f = getenv("MXC_FORCE_VARIANT")) {
        const int wv = wave_forced(f, true);
        return wv >= 0 && wave_has_classes(wv) ? wv : -1;
    }
    struct Key { ConvShape s; int masked; };
    static thread_local PlanCache<Key, int> cache;
    return cache.get(Key{s, masked}, [&] {
        ++g_plan_searches;
        double us = 0, other = 0, tile_us = 0;
        const int wv = (long long)s.N * s.H * s.W <= 1 << 30 ? wave_best_classes(s, masked, &us, &other) : -1;
        if (wv >= 0 && zeroes_rest(s)) return zeroing_tile(s, masked, &tile_us) >= 0 && us < 1.06 * tile_us ? wv : -1;
        return wv >= 0 && us < (us < (s.R * s.S == 1 ? 7.5 : 10) ? 0.8 : 0.5) * other ? wv : -1;
    });
}

// The plan of a 1x1 filter at stride 2: see zeroing_tile; the tuning hook's where it is set
static Plan zeroing_plan(const ConvShape &s, bool masked)
{
    const long long M = even_pixels(s);
    if (getenv("MXC_FORCE_VARIANT")) return choose_plan(M, s.C, s.K, true, masked);
    g_key_M = M; g_key_Co = s.C; g_key_Kd = s.K;
    double us = 0;
    return Plan{zeroing_tile(s, masked, &us), -1, M};
}

// Whether dx at stride 2 of a call that is handed the KRSC filter itself reads it in place: the wave kernel always, and the tiles that
// write the zeros: bound by what they write, they take 0.98 of the time on a filter that was re-packed first (90 layers of 10 to 84 GFLOP,
// 0.92 to 1.02), 2 us less on small ones.
bool bwd_data_classes_in_place(const ConvShape &s, bool masked)
{
    if (real_c(s) != s.C || real_k(s) != s.K) return false;
    if (classes_wave(s, masked) >= 0) return true;
    if (!zeroes_rest(s)) return false;
    const Plan pl = zeroing_plan(s, masked);
    return has_bt(pl.main) && (pl.tail < 0 || has_bt(pl.tail));
}

// whether dx of an NCHW problem, its filter re-packed, goes straight to its planes (see PlaneOut)
bool igemm_bwd_data_planes(const ConvShape &s, bool masked)
{
    return s.stride == 1 && wave_choice((long long)s.N * s.H * s.W, s.C, s.R * s.S * s.K, true, masked, s.C % 8 == 0) >= 0;
}

// A large 1x1 filter at stride 1 (FullyConnected) is read in place, as transposed tiles, when the chosen
// tile has that variant: copying it would cost more than the slower operand fetch.
bool bwd_data_reads_filter_in_place(const ConvShape &s)
{
    return real_c(s) == s.C && real_k(s) == s.K && s.R == 1 && s.S == 1 && s.stride == 1 && s.K % 64 == 0 && (long long)s.K * s.C * 2 >= (4ll << 20) &&
           has_bt(choose_tile((long long)s.N * s.H * s.W, s.C, s.K));
}

int igemm_bwd_data_prepare(const ConvShape &s, const void *w, void *wt, hipStream_t st, bool copy_in_place_filter, bool kcrs)
{
    if (bwd_data_reads_filter_in_place(s))
        return copy_in_place_filter ? launch_copy(w, wt, (size_t)s.K * s.C * sizeof(bf16_t), st) : MXC_OK;
    const RelayJob job = relay_bwd_filter(s, w, wt, kcrs);
    return relayout(&job, 1, st);
}

// wt: the filter as igemm_bwd_data_prepare left it; w_in_place: if not null, the KRSC filter that the in-place variant reads
int igemm_bwd_data(const ConvShape &s, const void *dy, const void *w_in_place, void *dx, const void *wt, hipStream_t st,
                   const char **variant, const PostOp &post, void *split_ws)
{
    const bool bt = w_in_place != nullptr;
    IgemmParams p = bwd_data_params(s);
    p.in = (const bf16_t *)dy; p.out = (bf16_t *)dx;
    p.mask = (const bf16_t *)post.mask; p.copied = post.copied;
    if (s.stride == 1) {
        p.wm = bt ? (const bf16_t *)w_in_place : (const bf16_t *)wt;
        p.wm_by_k = bt && !bwd_data_reads_filter_in_place(s) && bwd_data_streams_filter(s, p.mask != nullptr);
        const long long M = (long long)s.N * s.H * s.W;
        const int Kd = s.R * s.S * s.K;
        if (const int rv = run_choice(p, true, p.mask != nullptr, s.C % 8 == 0, post.planes != nullptr); rv >= 0) {
            *variant = run_name(rv);
            return run_launch(rv, p, st, bt);
        }
        if (!bwd_data_reads_filter_in_place(s) && stream_choice(p, true, p.mask != nullptr, s.C % 8 == 0, post.planes != nullptr)) {
            *variant = kStreamName;
            p.wm_by_k = bt;
            return stream_launch(p, st);
        }
        if (const int wv = wave_choice(M, s.C, Kd, true, p.mask != nullptr, s.C % 8 == 0); wv >= 0) {
            *variant = wave_name(wv);
            return wave_launch(wv, p, st, bt, post.planes);
        }
        const int sp = (split_ws != nullptr && s.C % 8 == 0) ? split_count(M, s.C, Kd) : 1;
        Plan pl = plan_for(p, M, s.C, Kd, (bt && !p.wm_by_k) || sp > 1);
        if (bt && !p.wm_by_k && !has_bt(pl.tail)) pl = Plan{pl.main, -1, 0};
        *variant = plan_name(pl);
        if (sp > 1) return launch_split(pl.main, p, M, sp, split_ws, dx, post, st, variant, bt);
        return launch_plan(pl, p, st, bt);
    }
    if (const int wv = classes_wave(s, p.mask != nullptr); wv >= 0) {
        p.wm = (const bf16_t *)(bt ? w_in_place : wt);
        *variant = wave_name(wv);
        return wave_launch_classes(wv, s, p, st, bt);
    }
    IgemmClasses q{};
    bool zeros = false, zeroed = false;
    size_t wt_off = 0;
    long long rows = 0, area = 0;          // GEMM rows with taps, and their taps
    for (int ph = 0; ph < s.stride; ++ph) {
        for (int pw = 0; pw < s.stride; ++pw) {
            IgemmClass c{};
            c.TR = ph < s.R ? (s.R - ph + s.stride - 1) / s.stride : 0;
            c.TS = pw < s.S ? (s.S - pw + s.stride - 1) / s.stride : 0;
            // output rows h = ph - pad + stride*hh >= 0, h < H
            c.in_off_h = ph >= s.pad ? 0 : (s.pad - ph + s.stride - 1) / s.stride;
            c.in_off_w = pw >= s.pad ? 0 : (s.pad - pw + s.stride - 1) / s.stride;
            c.out_off_h = ph - s.pad + s.stride * c.in_off_h; c.out_off_w = pw - s.pad + s.stride * c.in_off_w;
            c.Mh = c.out_off_h < s.H ? (s.H - 1 - c.out_off_h) / s.stride + 1 : 0;
            c.Mw = c.out_off_w < s.W ? (s.W - 1 - c.out_off_w) / s.stride + 1 : 0;
            c.wm = (const bf16_t *)wt + wt_off;
            c.wm_bytes = (unsigned)((long long)p.Cw * c.TR * c.TS * s.K * 2);
            wt_off += (size_t)s.C * c.TR * c.TS * s.K;
            if (c.Mh <= 0 || c.Mw <= 0) continue;
            if (c.TR * c.TS == 0) { zeros = true; continue; }
            IgemmParams one = p;
            one.wm = c.wm; one.TR = c.TR; one.TS = c.TS; one.Mh = c.Mh; one.Mw = c.Mw;
            one.in_off_h = c.in_off_h; one.in_off_w = c.in_off_w; one.out_off_h = c.out_off_h; one.out_off_w = c.out_off_w;
            const bool rest = zeroes_rest(s);
            const Plan pl = rest && !getenv("MXC_FORCE_VARIANT") ? zeroing_plan(s, p.mask != nullptr) : plan_for(one, (long long)s.N * c.Mh * c.Mw, s.C, c.TR * c.TS * s.K);
            if (pl.main == STREAM_TILE || (s.R == 1 && s.S == 1)) {
                // one class alone (1x1), or one that the plan gives to the streaming kernel (short reductions): a launch of its own
                zeroed = rest && has_bt(pl.main) && (pl.tail < 0 || has_bt(pl.tail));
                one.zero_rest = zeroed;
                if (bt) { one.wm = (const bf16_t *)w_in_place; one.bt_w_bytes = (unsigned)((long long)s.K * s.C * 2); }
                const int rc = launch_plan(pl, one, st, bt);
                if (rc != MXC_OK) return rc;
                *variant = plan_name(pl);
                continue;
            }
            rows += (long long)s.N * c.Mh * c.Mw;
            area += (long long)s.N * c.Mh * c.Mw * c.TR * c.TS;
            // most taps first: the longest reductions start first
            int at = q.n++;
            for (; at > 0 && q.c[at - 1].TR * q.c[at - 1].TS < c.TR * c.TS; --at) q.c[at] = q.c[at - 1];
            q.c[at] = c;
        }
    }
    if (zeros && !zeroed) {
        unsigned zh = 0, zw = 0;
        for (int c = 0; c < s.stride; ++c) {
            zh |= c >= s.R ? 1u << c : 0u;
            zw |= c >= s.S ? 1u << c : 0u;
        }
        if ((long long)s.N * s.H > 0x7FFFFFFFll) return MXC_ERR_SHAPE;
        const dim3 grid((unsigned)(s.N * s.H)), block(256);
        if (s.C % 8 == 0) hipLaunchKernelGGL(zero_classes_kernel<8>, grid, block, 0, st, (bf16_t *)dx, s.H, s.W, s.C, s.stride, s.pad, zh, zw);
        else hipLaunchKernelGGL(zero_classes_kernel<1>, grid, block, 0, st, (bf16_t *)dx, s.H, s.W, s.C, s.stride, s.pad, zh, zw);
        if (hipGetLastError() != hipSuccess) return MXC_ERR_LAUNCH;
    }
    if (q.n == 0) return MXC_OK;
    p.in_bytes = (unsigned)((long long)s.N * s.P * s.Q * s.K * 2);
    const long long out_bytes = (long long)s.N * s.H * s.W * s.C * 2;
    p.out_bytes = out_bytes < 0x7FFF0000ll ? (unsigned)out_bytes : 0u;
    p.nt_out = out_bytes >= (128ll << 20) ? 1 : 0;
    q.p = p;
    const int tile = choose_tile(rows, s.C, (int)(area / rows * s.K));
    *variant = kTiles[tile].name;
    return launch_classes_choice(tile, q, st);
}

// ---- backward-data for small C (first layers) ------------------------------------------------
// With C <= 4 output channels the GEMM's N dimension would be almost empty.  Instead G consecutive
// output columns form one GEMM row: N' = G*4 (channels padded to 4), and the reduction runs over the
// U columns of dy that reach any of the G pixels.  Per residue class ph of (h+pad) mod stride:
//     dx4[n][h][b*G+g][c] = sum_{j,u,k} dy[n][hh-j][b*G/stride + uoff + u][k] * W2[(g,c)][(j,u,k)]
//     W2[(g,c)][(j,u,k)]  = w[k][ph+stride*j][s][c],  s = g + pad - stride*(u + uoff), zero if s outside [0,S)
// dx4 is then compacted to the caller's C channels.

namespace {

struct SmallCBwd { int G, U, uoff, Wg; };

SmallCBwd smallc_bwd_geom(const ConvShape &s)
{
    SmallCBwd g;
    g.G = 8;
    // floor((pad - S + 1) / stride)
    const int num = s.pad - s.S + 1;
    g.uoff = num >= 0 ? num / s.stride : -((-num + s.stride - 1) / s.stride);
    g.U = (g.G - 1 + s.pad) / s.stride - g.uoff + 1;
    g.Wg = (s.W + g.G - 1) / g.G;
    return g;
}

// all residue classes one after another; class ph holds [G*4][TR_ph*U*K]
__global__ __launch_bounds__(256) void smallc_bwd_pack_w_kernel(const bf16_t *__restrict__ w, bf16_t *__restrict__ w2, int K,
                                                               int Kr, int C, int R, int S, int stride, int pad, int G, int U,
                                                               int uoff)
{
    const int rows = G * 4;
    int gid = blockIdx.x * blockDim.x + threadIdx.x;
    int ph = 0, TRp = 0;
    for (; ph < stride; ++ph) {
        TRp = ph < R ? (R - ph + stride - 1) / stride : 0;
        const int sz = rows * TRp * U * K;
        if (gid < sz) break;
        gid -= sz;
    }
    if (ph == stride) return;
    // reduction order (u, j, k): the row taps of one dy column are consecutive stages, so the dy row a
    // GEMM row reads at row tap j is the one its neighbour one image row down reads at j+1, one stage
    // later, while it is still in the L2 (with j outermost the reuse came 10 stages later and missed)
    const int k = gid % K; int t = gid / K;
    const int j = t % TRp; t /= TRp;
    const int u = t % U; t /= U;
    const int c = t & 3, g = t >> 2;
    const int r = ph + stride * j;
    const int sidx = g + pad - stride * (u + uoff);
    bf16_t v = 0;
    if (k < Kr && c < C && sidx >= 0 && sidx < S) v = w[(((size_t)k * R + r) * S + sidx) * C + c];
    const size_t phase_base = (size_t)(blockIdx.x * blockDim.x + threadIdx.x) - gid;
    w2[phase_base + gid] = v;
}

// dx[n][h][w][c] = dx4[n][h][w][c], c < C; dx4 rows are Wg*G pixels wide
__global__ __launch_bounds__(256) void smallc_compact_kernel(const uint2 *__restrict__ dx4, bf16_t *__restrict__ dx, long long rows,
                                                            int W, int W4, int C, const bf16_t *__restrict__ mask)
{
    const long long total = rows * W;
    const long long gid = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= total) return;
    const long long row = gid / W;
    const int wv = (int)(gid % W);
    const uint2 v = dx4[row * W4 + wv];
    bf16_t *d = dx + gid * C;
    const bf16_t e[4] = {(bf16_t)(v.x & 0xFFFF), (bf16_t)(v.x >> 16), (bf16_t)(v.y & 0xFFFF), (bf16_t)(v.y >> 16)};
#pragma unroll
    for (int c = 0; c < 4; ++c)
        if (c < C) d[c] = (mask == nullptr || mask_keeps(mask + gid * C + c)) ? e[c] : (bf16_t)0;
}

}  // namespace

bool igemm_bwd_data_smallc_supported(const ConvShape &s)
{
    const SmallCBwd g = smallc_bwd_geom(s);
    return s.C <= 4 && s.K % 8 == 0 && (s.stride == 1 || s.stride == 2 || s.stride == 4) &&
           igemm_dims_ok((long long)s.N * s.P * s.Q * s.K, (long long)g.G * 4 * s.R * g.U * s.K, (long long)s.N * s.H * g.Wg, s.P,
                         s.Q, s.pad + s.R + s.S + s.stride + g.U, s.R * g.U) &&
           (long long)s.N * s.H * g.Wg * g.G * 4 * 2 < 0x7FFF0000ll;
}

void igemm_bwd_data_smallc_workspace(const ConvShape &s, size_t *w2_bytes, size_t *dx4_bytes)
{
    const SmallCBwd g = smallc_bwd_geom(s);
    size_t taps = 0;
    for (int ph = 0; ph < s.stride; ++ph) taps += ph < s.R ? (s.R - ph + s.stride - 1) / s.stride : 0;
    *w2_bytes = (size_t)g.G * 4 * taps * g.U * s.K * 2;
    *dx4_bytes = (size_t)s.N * s.H * g.Wg * g.G * 4 * 2;
}

int igemm_bwd_data_smallc_columns(const ConvShape &s) { return smallc_bwd_geom(s).U; }

int igemm_bwd_data_smallc_prepare(const ConvShape &s, const void *w, void *w2, hipStream_t st)
{
    const SmallCBwd g = smallc_bwd_geom(s);
    size_t w2_bytes, dx4_bytes;
    igemm_bwd_data_smallc_workspace(s, &w2_bytes, &dx4_bytes);
    const int total = (int)(w2_bytes / 2);
    hipLaunchKernelGGL(smallc_bwd_pack_w_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, st, (const bf16_t *)w,
                       (bf16_t *)w2, s.K, real_k(s), s.C, s.R, s.S, s.stride, s.pad, g.G, g.U, g.uoff);
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
}

// w2: the filter as igemm_bwd_data_smallc_prepare packed it
int igemm_bwd_data_smallc(const ConvShape &s, const void *dy, const void *w2, void *dx, void *dx4, hipStream_t st,
                          const char **variant, const PostOp &post)
{
    const SmallCBwd g = smallc_bwd_geom(s);
    size_t w2_off = 0;
    Plan pl{0, -1, 0};
    for (int ph = 0; ph < s.stride; ++ph) {
        const int TR = ph < s.R ? (s.R - ph + s.stride - 1) / s.stride : 0;
        const int hh0 = ph >= s.pad ? 0 : (s.pad - ph + s.stride - 1) / s.stride;
        const int h_first = ph - s.pad + s.stride * hh0;
        const int Mh = h_first < s.H ? (s.H - 1 - h_first) / s.stride + 1 : 0;
        IgemmParams p{};
        p.in = (const bf16_t *)dy; p.wm = (const bf16_t *)w2 + w2_off; p.out = (bf16_t *)dx4;
        p.N = s.N; p.Hi = s.P; p.Wi = s.Q; p.Ci = s.K; p.pix = s.K; p.Co = g.G * 4;
        p.TR = TR; p.TS = g.U; p.tstep_h = -1; p.tstep_w = 1; p.tap_row_inner = 1;
        p.Mh = Mh; p.Mw = g.Wg;
        p.in_mul_h = 1; p.in_mul_w = g.G / s.stride; p.in_off_h = hh0; p.in_off_w = g.uoff;
        p.Ho = s.H; p.Wo = g.Wg; p.out_mul_h = s.stride; p.out_mul_w = 1; p.out_off_h = h_first; p.out_off_w = 0;
        w2_off += (size_t)g.G * 4 * TR * g.U * s.K;
        if (Mh <= 0) continue;
        pl = plan_for(p, (long long)s.N * Mh * g.Wg, p.Co, TR * g.U * s.K);
        const int rc = launch_plan(pl, p, st);
        if (rc != MXC_OK) return rc;
    }
    const long long rows = (long long)s.N * s.H;
    const long long blocks = (rows * s.W + 255) / 256;
    if (blocks > 0x7FFFFFFFll) return MXC_ERR_SHAPE;
    hipLaunchKernelGGL(smallc_compact_kernel, dim3((unsigned)blocks), dim3(256), 0, st, (const uint2 *)dx4, (bf16_t *)dx, rows,
                       s.W, g.Wg * g.G, s.C, (const bf16_t *)post.mask);
    *variant = plan_name(pl);
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
}

}  // namespace mxc
