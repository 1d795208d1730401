// fp32 convolution on the gfx950 fp32 matrix cores, all three passes, both layouts, any channel count.
//
// One kernel template runs the three passes as GEMMs  D[i][j] = sum_k A[i][k] * B[k][j]  (fp32 operands, fp32
// accumulation, v_mfma_f32_32x32x2_f32):
//   forward:          i = output pixel, j = output channel, k = (tap, c) in NHWC / (c, tap) in NCHW
//   backward-data:    i = input pixel of one stride residue class, j = input channel, k over (tap, output channel);
//                     every residue class is part of the one launch, one that no tap reaches has an empty sum
//   backward-weight:  i = output channel, j = filter element in the filter's own order, k = output pixel
// The instruction takes ONE float per lane and operand, so an operand tile can sit in LDS with either index
// contiguous: k-contiguous ("KC", [i][16 k]) or k-slow ("KS", [16 k][i]).  Each operand is laid the way it lies in
// memory, and therefore no pass needs a transposed or re-packed copy of anything, in NHWC or NCHW:
//                     A                      B
//   fwd  NHWC         x gather, KC           w rows, KC
//   fwd  NCHW         x gather, KS           w rows, KC
//   bwd  NHWC         dy gather, KC          w, KS (input channels contiguous)
//   bwd  NCHW         dy gather, KS          w, KC (taps contiguous)
//   dw   NHWC         dy, KS                 x gather, KS
//   dw   NCHW         dy, KC                 x gather, KC (pixels contiguous)
//
// What bounds it: a SIMD runs either an fp32 MFMA or a vector instruction, never both (the coexecution counter reads 0; bf16
// MFMAs hide half of theirs), so the time is the matrix time (64 flop per clock and SIMD, 1/16 of bf16) plus the address
// arithmetic.  192->384 3x3 at 13x13, batch 32, NCHW forward: 57 vector instructions per 8 MFMAs, 56% + 36% of the SIMD
// cycles.  A larger wave tile has fewer of them per MFMA, a smaller one fills the chip.  Transfers are 4 bytes per lane, which
// is what makes every channel count, alignment and layout run alike (16 bytes where the reduction comes in aligned fours).
// Tiles are filled by direct global->LDS loads through a ring of NS stages, one barrier per stage; lanes that fall
// into padding, past a ragged edge or past the reduction end get an offset the buffer rejects, which deposits zeros.
//
// Small problems: Z groups of waves of one workgroup take the 16-element stages in turn (group z runs stages z, z+Z,
// ...), each with a ring of its own, and the Z partial tiles are added in ascending z through LDS: a 32x32 tile with
// eight one-wave groups (no barrier inside the loop) turns a single-layer problem into many short chains.
#include <stdlib.h>
#include <string.h>

#include <type_traits>

#include "mxc_internal.h"
#include "plan_cache.h"

namespace mxc {

namespace {

typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x2 __attribute__((ext_vector_type(2)));

constexpr unsigned OOB = 0x80000000u;   // a buffer offset no operand reaches: the load returns zeros
constexpr int BK = 16;                  // reduction elements per stage
constexpr int MAX_CLASSES = 16;         // stride residue classes of backward-data (stride <= 4)
enum { OP_FWD = 0, OP_BWD = 1, OP_WGRAD = 2 };

template <int N> __device__ __forceinline__ void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ void wait_lgkmcnt0() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void pin() { __builtin_amdgcn_sched_barrier(0); }

template <int I> using IC = std::integral_constant<int, I>;
template <class F, int... I> __device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>) { (f(IC<I>{}), ...); }
template <int N, class F> __device__ __forceinline__ void static_for(F &&f) { static_for_impl(f, std::make_integer_sequence<int, N>{}); }

// A stride residue class of backward-data; forward has one, the whole problem.
struct F32Class {
    int tile0;              // first row tile
    int TR, TS;             // tap grid
    int Mh, Mw;             // pixel grid of the rows
    int off_h, off_w;       // gathered position of row (0, 0), tap 0
    int ph, pw;             // first filter row / column
    int h_first, v_first;   // output position of row (0, 0)
    FastDiv mw, mh, t, ts;
    int ts_magic;           // see small_div
};

struct F32Params {
    const float *a, *b;     // the two operands as the table above names them
    float *out;             // y, dx, dw or the first split's partial dw
    unsigned a_bytes, b_bytes;
    ConvShape s;
    int M;                  // forward: N*P*Q; backward-weight: the reduction length N*P*Q
    int n_tiles, tiles, units;      // tiles: per split; units: tiles * splits
    int span;               // backward-weight: pixels per split (a multiple of 16 * Z)
    F32Class cls[MAX_CLASSES];
    int n_cls;
    FastDiv by_ntiles, by_tiles, by_ci, by_c, by_rs, by_s, by_pq, by_q, by_p;
    const float *bias;      // forward, or null
    int relu;
    const float *mask;      // backward-data, or null: the result is 0 where mask <= 0
    int outside;            // whether any result has a tap outside the gathered tensor
};

__device__ __forceinline__ int pack_hw(int h, int w) { return (h & 0xFFFF) | (w << 16); }
// nonzero where (h, w) + (dh, dw) leaves the image; all packed as two 16-bit integers
__device__ __forceinline__ int outside(int hw, int d, int lim)
{
    const s16x2 v = __builtin_bit_cast(s16x2, hw) + __builtin_bit_cast(s16x2, d);
    const s16x2 e = __builtin_bit_cast(s16x2, lim) - v;
    return (__builtin_bit_cast(int, v) | __builtin_bit_cast(int, e)) & (int)0x80008000;
}
constexpr int FAR = (-16384) & 0xFFFF;  // a packed position that is outside whatever is added to it

// Result (i, j) over the taps inside the gathered tensor and nothing else, in the order tap, channel or pixel; a sum that turns
// NaN ends there.  (The matrix-core kernels multiply a deposited zero for a tap outside, and that is NaN where the other operand is
// infinite or NaN: such a result is itself NaN, nothing else is wrong about it, and one lane sums it once more with this.)
template <int OP, bool NCHW>
__device__ float sum_inside(const F32Params &p, const F32Class &cls, int i, int j, int k_lo, int k_hi)
{
    const ConvShape &s = p.s;
    const int RS = s.R * s.S, PQ = s.P * s.Q;
    const int Ci = OP == OP_BWD ? s.K : s.C, Hi = OP == OP_BWD ? s.P : s.H, Wi = OP == OP_BWD ? s.Q : s.W, plane = Hi * Wi;
    float acc = 0.f;
    if constexpr (OP == OP_WGRAD) {
        const int hi = NCHW ? p.by_rs.div(j) : p.by_c.div(j), lo = j - hi * (NCHW ? RS : s.C);
        const int tap = NCHW ? lo : hi, c = NCHW ? hi : lo, r = p.by_s.div(tap), t = tap - r * s.S;
        for (int m = k_lo; m < k_hi && acc == acc;) {
            const int end = min(m + 64, k_hi);
#pragma unroll 4
            for (; m < end; ++m) {
                const int row = p.by_q.div(m), n = p.by_p.div(row), q = m - row * s.Q;
                const int h = (row - n * s.P) * s.stride - s.pad + r, w = q * s.stride - s.pad + t;
                const bool in = (unsigned)h < (unsigned)s.H && (unsigned)w < (unsigned)s.W;
                const float dy = p.a[NCHW ? (n * s.K + i) * PQ + m - n * PQ : m * s.K + i];
                const float x = p.b[!in ? 0 : NCHW ? (n * s.C + c) * plane + h * s.W + w : ((n * s.H + h) * s.W + w) * s.C + c];
                if (in) acc = fmaf(dy, x, acc);
            }
        }
    } else {
        const int t2 = cls.mw.div(i), b = i - t2 * cls.Mw, n = cls.mh.div(t2), a = t2 - n * cls.Mh;
        const int mul = OP == OP_FWD ? s.stride : 1, sgn = OP == OP_FWD ? 1 : -1;
        for (int tr = 0; tr < cls.TR; ++tr)
            for (int ts = 0; ts < cls.TS; ++ts) {
                const int h = a * mul + cls.off_h + sgn * tr, w = b * mul + cls.off_w + sgn * ts;
                if ((unsigned)h >= (unsigned)Hi || (unsigned)w >= (unsigned)Wi) continue;
                const int rs = OP == OP_FWD ? tr * s.S + ts : (cls.ph + s.stride * tr) * s.S + cls.pw + s.stride * ts;
                const float *x = p.a + (NCHW ? n * Ci * plane + h * Wi + w : ((n * Hi + h) * Wi + w) * Ci);
                const float *f = p.b + (OP == OP_FWD ? (NCHW ? j * Ci * RS + rs : (j * RS + rs) * Ci) : NCHW ? j * RS + rs : rs * s.C + j);
                const int xs = NCHW ? plane : 1, fs = OP == OP_BWD ? s.C * RS : NCHW ? RS : 1;
#pragma unroll 4
                for (int c = 0; c < Ci; ++c) acc = fmaf(x[c * xs], f[c * fs], acc);
                if (acc != acc) return acc;
            }
    }
    return acc;
}

// OP, layout; VA / VB: floats per lane and transfer of the two operands (4 only for KC operands); the workgroup has Z
// groups of WR x WC waves, a wave MI x NI blocks of 32x32.
template <int OP, bool NCHW, int VA, int VB, int WR, int WC, int MI, int NI, int Z, int NS>
__global__ __launch_bounds__(64 * WR * WC * Z, MI * NI == 4 ? 2 : 1) void f32_conv_kernel(const F32Params p)
{
    constexpr int NG = WR * WC, NT = 64 * NG * Z;
    constexpr int BM = 32 * MI * WR, BN = 32 * NI * WC;
    constexpr bool A_KC = OP == OP_WGRAD ? NCHW : !NCHW;
    constexpr bool B_KC = OP == OP_FWD || NCHW;
    constexpr bool SWAP = NCHW && OP != OP_WGRAD;       // which operand's index runs along the lanes of the result
    static_assert((VA == 1 || A_KC) && (VB == 1 || B_KC), "16-byte transfers are for k-contiguous operands");
    constexpr int A_LD = BM * BK / (64 * VA) / NG, B_LD = BN * BK / (64 * VB) / NG;     // transfers per wave and stage
    constexpr int L = A_LD + B_LD;
    static_assert(A_LD >= 1 && B_LD >= 1 && A_LD * NG * 64 * VA == BM * BK && B_LD * NG * 64 * VB == BN * BK, "tile/wave mismatch");
    static_assert(L * (NS - 1) < 64 && NS >= 3, "ring depth against the range of the load counter");
    static_assert(NG == 1 || NG == 4, "group size");
    constexpr int STG = (BM + BN) * BK;                 // floats per stage
    constexpr int RED = Z > 1 ? Z * BM * BN : 0;        // floats of the partial tiles that meet at the end
    constexpr int SMEM = Z * NS * STG > RED ? Z * NS * STG : RED;
    __shared__ __attribute__((aligned(1024))) float smem[SMEM];
    __shared__ int2 tap_tab[MAX_TAPS + 1];

    const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int zg = wave / NG, gw = wave & (NG - 1);
    const int wave_m = (gw / WC) * (32 * MI), wave_n = (gw % WC) * (32 * NI);

    // workgroup -> unit: a contiguous range of units per XCD, column tile fastest
    const int per_xcd = (p.units + 7) / 8;
    const int unit = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (unit >= p.units) return;
    const int split = p.by_tiles.div(unit), tile = unit - split * p.tiles;
    const ConvShape &s = p.s;
    const int RS = s.R * s.S;
    int mt = p.by_ntiles.div(tile);
    const int n0 = (tile - mt * p.n_tiles) * BN;

    // ---- geometry of this unit ---------------------------------------------------------------------------
    int ci = 0;
    if constexpr (OP == OP_BWD) {
        while (ci + 1 < p.n_cls && mt >= p.cls[ci + 1].tile0) ++ci;
        mt -= p.cls[ci].tile0;
    }
    const F32Class &cls = p.cls[ci];
    const int m0 = mt * BM;
    // gathered tensor (x, dy, x), tap grid and direction, pixel grid of the rows
    const int Ci = OP == OP_BWD ? s.K : s.C, Hi = OP == OP_BWD ? s.P : s.H, Wi = OP == OP_BWD ? s.Q : s.W;
    const int TS = cls.TS, Mh = cls.Mh, Mw = cls.Mw;
    [[maybe_unused]] const int ph = cls.ph, pw = cls.pw, h_first = cls.h_first, v_first = cls.v_first;
    const int T = cls.TR * TS;
    const int rows = OP == OP_FWD ? p.M : OP == OP_BWD ? s.N * Mh * Mw : s.K;       // extent of i
    const int cols = OP == OP_FWD ? s.K : OP == OP_BWD ? s.C : s.C * RS;            // extent of j
    const int k_lo = OP == OP_WGRAD ? split * p.span : 0;
    const int k_hi = OP == OP_WGRAD ? min(k_lo + p.span, p.M) : T * Ci;
    const int KT = k_hi > k_lo ? (k_hi - k_lo + BK * Z - 1) / (BK * Z) : 0;         // stages per group
    const int k0 = k_lo + zg * BK;                      // first reduction element of this group
    constexpr int KSTEP = BK * Z;
    const int lim_hw = pack_hw(Hi - 1, Wi - 1);
    const int plane = Hi * Wi, PQ = s.P * s.Q;

    // ---- tap table: .x = offset (floats), .y = packed (dh, dv).  Forward and backward-data in NHWC: the gathered
    // tensor's; backward-data in NCHW: .x = the filter element (its gather works the taps out itself).  Entry T: outside.
    constexpr bool TABLE = OP != OP_WGRAD && (A_KC || (OP == OP_BWD && B_KC));
    if constexpr (TABLE) {
        for (int t = tid; t <= T; t += NT) {
            const int j = t < T ? cls.ts.div(t) : 0, i = t < T ? t - j * TS : 0;
            const int sgn = OP == OP_BWD ? -1 : 1;
            int2 e = make_int2(sgn * (j * Wi + i) * Ci, pack_hw(sgn * j, sgn * i));
            if constexpr (OP == OP_BWD && NCHW) e.x = (ph + s.stride * j) * s.S + pw + s.stride * i;
            if (t == T) e = make_int2(0, FAR);
            tap_tab[t] = e;
        }
    }
    const int ts_magic = cls.ts_magic;

    const buf_rsrc_t rs_a = make_buf_rsrc(p.a, p.a_bytes), rs_b = make_buf_rsrc(p.b, p.b_bytes);

    // position of output-grid row m: offset of its tap-0 element in the gathered tensor, and packed (h, w)
    auto pixel = [&](int m, int &off, int &hw) __attribute__((always_inline)) {
        off = 0; hw = FAR;
        if (m < rows) {
            const int t2 = cls.mw.div(m), b = m - t2 * Mw, n = cls.mh.div(t2), a = t2 - n * Mh;
            const int mul = OP == OP_FWD ? s.stride : 1;
            const int h = a * mul + cls.off_h, w = b * mul + cls.off_w;
            off = NCHW ? n * Ci * plane + h * Wi + w : ((n * Hi + h) * Wi + w) * Ci;
            hw = pack_hw(h, w);
        }
    };
    // the k-slow operands' transfer i of this wave: reduction row and column it covers (a column's 32-float half is
    // exchanged in every second group of four rows: the two halves of a wave read rows 4 apart)
    auto ks_row = [&](int BX, int i) __attribute__((always_inline)) { return BX >= 64 ? (gw + NG * i) / (BX / 64) : (gw + NG * i) * 2 + half; };
    auto ks_col = [&](int BX, int i) __attribute__((always_inline)) {
        if (BX < 64) return lane & 31;
        const int r = (gw + NG * i) / (BX / 64);
        return (((gw + NG * i) % (BX / 64)) * 64 + lane) ^ (((r >> 2) & 1) * 32);
    };
    // ... and the k-contiguous operands': tile row, and the lane's reduction element within a stage
    auto kc_row = [&](int V, int i) __attribute__((always_inline)) { return V == 4 ? 16 * (gw + NG * i) + (lane >> 2) : 4 * (gw + NG * i) + (lane >> 4); };
    auto kc_k = [&](int V) __attribute__((always_inline)) {
        return V == 4 ? ((lane & 3) ^ ((lane >> 4) & 3)) * 4 : ((((lane & 15) >> 2) ^ (gw & 3)) << 2) + (lane & 3);
    };
    // one-wave groups with 4-byte transfers: the swizzle changes with the transfer (row / 4 = i), the element does too
    constexpr bool A_VARK = A_KC && VA == 1 && NG == 1, B_VARK = B_KC && VB == 1 && NG == 1;
    auto kc_k_var = [&](int i) __attribute__((always_inline)) { return ((((lane & 15) >> 2) ^ (i & 3)) << 2) + (lane & 3); };
    constexpr int NKA = A_VARK ? 4 : 1, NKB = B_VARK ? 4 : 1;   // distinct reduction elements a lane handles per stage

    // ---- positions ------------------------------------------------------------------------------------------
    // Each transfer has a fixed part (its tile row or column: byte offset, packed position) and a moving one (the
    // reduction element).  A lane of a k-contiguous operand handles one reduction element per stage (NKA / NKB where the
    // swizzle makes it four) and keeps it itself.  A k-slow operand has 16 reduction rows per stage, each shared by all
    // lanes of a transfer: lane r keeps row r % 16, works out its share of the addresses once per stage, and every
    // transfer picks its row's up with a lane read.  (Kept per transfer, the same arithmetic was eight times as much and
    // most of a small tile's time.)  An invalid part is 2^31, which no operand reaches; sums saturate.
    unsigned a_off[A_LD], b_off[B_LD];
    int a_hw[A_LD], b_hw[B_LD];
    int a_k[NKA], a_t[NKA], a_c[NKA];               // element; tap, or pixel within the image; channel, or image
    int b_k[NKB], b_t[NKB], b_c[NKB];
    [[maybe_unused]] int b_q[NKB];                  // backward-weight: b_c image, b_t row, b_q column
    [[maybe_unused]] unsigned ar_off = 0, br_off = 0;       // this lane's reduction row: byte offset and packed position
    [[maybe_unused]] int ar_d = 0, br_d = 0;

    const int adv_n = p.by_pq.div(KSTEP), adv_pq = KSTEP - adv_n * PQ;          // NCHW backward-weight
    const int adv_row = p.by_q.div(KSTEP), adv_q = KSTEP - adv_row * s.Q, adv_n3 = p.by_p.div(adv_row), adv_p = adv_row - adv_n3 * s.P;
    const int adv_tq = cls.t.div(KSTEP), adv_tr = KSTEP - adv_tq * T;           // (c, tap) order
    const int adv_cq = p.by_ci.div(KSTEP), adv_cr = KSTEP - adv_cq * Ci;        // (tap, c) order
    auto pixel_of = [&](int m, int &k, int &q, int &row, int &n) __attribute__((always_inline)) {
        const int t = p.by_q.div(m);
        k = m; q = m - t * s.Q; n = p.by_p.div(t); row = t - n * s.P;
    };
#pragma unroll
    for (int i = 0; i < A_LD; ++i) {
        a_hw[i] = 0;
        if constexpr (OP == OP_WGRAD) {                 // dy[m][k] or dy[n][k][pq]
            const int row = m0 + (NCHW ? kc_row(VA, i) : ks_col(BM, i));
            a_off[i] = row < rows ? (unsigned)(NCHW ? row * PQ : row) * 4u : OOB;
        } else {
            int off;
            pixel(m0 + (A_KC ? kc_row(VA, i) : ks_col(BM, i)), off, a_hw[i]);
            a_off[i] = (unsigned)off * 4u;
        }
    }
#pragma unroll
    for (int v = 0; v < NKA; ++v) {
        const int kd = k0 + (!A_KC ? lane & 15 : A_VARK ? kc_k_var(v) : kc_k(VA));
        a_k[v] = kd;
        if constexpr (OP == OP_WGRAD) { a_c[v] = p.by_pq.div(kd); a_t[v] = kd - a_c[v] * PQ; }
        else if constexpr (A_KC) { a_t[v] = p.by_ci.div(kd); a_c[v] = kd - a_t[v] * Ci; }
        else { a_c[v] = cls.t.div(kd); a_t[v] = kd - a_c[v] * T; }
    }
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
        b_hw[i] = 0;
        const int j = n0 + (B_KC ? kc_row(VB, i) : ks_col(BN, i));
        if constexpr (OP == OP_FWD) b_off[i] = j < cols ? (unsigned)(j * (T * Ci)) * 4u : OOB;         // w[co][kd]
        else if constexpr (OP == OP_BWD) b_off[i] = j < cols ? (unsigned)(NCHW ? j * RS : j) * 4u : OOB;  // w[k][c][rs] or w[k][rs][c]
        else {                                          // x gather: column = (c, tap) or (tap, c)
            const int hi = NCHW ? p.by_rs.div(j) : p.by_c.div(j), lo = j - hi * (NCHW ? RS : s.C);
            const int tap = NCHW ? lo : hi, c = NCHW ? hi : lo;
            const int tr = p.by_s.div(tap), r = tr - s.pad, q = tap - tr * s.S - s.pad;
            b_off[i] = (unsigned)(NCHW ? c * plane + r * s.W + q : (r * s.W + q) * s.C + c) * 4u;
            b_hw[i] = j < cols ? pack_hw(r, q) : FAR;
        }
    }
#pragma unroll
    for (int v = 0; v < NKB; ++v) {
        const int kd = k0 + (!B_KC ? lane & 15 : B_VARK ? kc_k_var(v) : kc_k(VB));
        b_k[v] = kd;
        if constexpr (OP == OP_WGRAD) pixel_of(kd, b_k[v], b_q[v], b_t[v], b_c[v]);
        else if constexpr (OP == OP_BWD && B_KC) { b_c[v] = cls.t.div(kd); b_t[v] = kd - b_c[v] * T; }
        else if constexpr (OP == OP_BWD) { b_t[v] = p.by_ci.div(kd); b_c[v] = kd - b_t[v] * Ci; }
    }

    float *ring = smem + zg * (NS * STG);
    // The transfers of one stage as L tasks (A's, then B's), each with its address arithmetic, so that they can be spread
    // between matrix instructions; `advance` moves the reduction positions one stage further, `fetch_rows` works out
    // what the coming stage's tasks share.
    [[maybe_unused]] int2 te[NKA];
    [[maybe_unused]] unsigned we[NKB];
    auto fetch_rows = [&]() __attribute__((always_inline)) {
        if constexpr (OP != OP_WGRAD && A_KC) {
#pragma unroll
            for (int v = 0; v < NKA; ++v) te[v] = tap_tab[a_t[v] < T ? a_t[v] : T];
        }
        if constexpr (OP == OP_WGRAD && !NCHW) ar_off = a_k[0] < k_hi ? (unsigned)(a_k[0] * s.K) * 4u : OOB;
        if constexpr (OP != OP_WGRAD && !A_KC) {
            const int j = small_div(a_t[0], ts_magic), q = a_t[0] - j * TS;
            const int dh = OP == OP_BWD ? -j : j, dv = OP == OP_BWD ? -q : q;
            ar_off = (unsigned)(a_c[0] * plane + dh * Wi + dv) * 4u;
            ar_d = a_k[0] < k_hi ? pack_hw(dh, dv) : FAR;
        }
        if constexpr (OP == OP_BWD && B_KC) {
#pragma unroll
            for (int v = 0; v < NKB; ++v) we[v] = b_k[v] < k_hi ? (unsigned)(b_c[v] * s.C * RS + tap_tab[b_t[v]].x) * 4u : OOB;
        } else if constexpr (OP == OP_BWD) {
            const int j = small_div(b_t[0], ts_magic), q = b_t[0] - j * TS;
            const int rs = (ph + s.stride * j) * s.S + pw + s.stride * q;
            br_off = b_k[0] < k_hi ? (unsigned)((b_c[0] * RS + rs) * s.C) * 4u : OOB;
        } else if constexpr (OP == OP_FWD) {
#pragma unroll
            for (int v = 0; v < NKB; ++v) we[v] = b_k[v] < k_hi ? (unsigned)b_k[v] * 4u : OOB;
        } else {
            if constexpr (NCHW) {
#pragma unroll
                for (int v = 0; v < NKB; ++v) {
                    const int h = b_t[v] * s.stride, w = b_q[v] * s.stride;
                    we[v] = (unsigned)(b_c[v] * s.C * plane + h * s.W + w) * 4u;
                    te[v & (NKA - 1)].y = b_k[v] < k_hi ? pack_hw(h, w) : FAR;      // NKA == NKB here
                    te[v & (NKA - 1)].x = b_k[v] < k_hi ? (a_c[v & (NKA - 1)] * s.K * PQ + a_t[v & (NKA - 1)]) * 4 : (int)OOB;
                }
            } else {
                const int h = b_t[0] * s.stride, w = b_q[0] * s.stride;
                br_off = (unsigned)(((b_c[0] * s.H + h) * s.W + w) * s.C) * 4u;
                br_d = b_k[0] < k_hi ? pack_hw(h, w) : FAR;
            }
        }
    };
    // reduction row r's value, held by lane r: the row is the same for the whole wave, or one per half of it
    auto of_row = [&](int BX, int i, int v) __attribute__((always_inline)) -> int {
        if (BX >= 64) return __builtin_amdgcn_readlane(v, ks_row(BX, i));
        const int r = (gw + NG * i) * 2, lo = __builtin_amdgcn_readlane(v, r), hi = __builtin_amdgcn_readlane(v, r + 1);
        return half ? hi : lo;
    };
    auto add_sat = [](unsigned x, unsigned y) __attribute__((always_inline)) { return __builtin_elementwise_add_sat(x, y); };
    auto task = [&](auto tc, int slot) __attribute__((always_inline)) {
        constexpr int Tk = decltype(tc)::value;
        unsigned off;
        if constexpr (Tk < A_LD) {
            constexpr int i = Tk, v = A_VARK ? i & 3 : 0;
            if constexpr (OP == OP_WGRAD && !NCHW) off = add_sat(a_off[i], (unsigned)of_row(BM, i, (int)ar_off));
            else if constexpr (OP == OP_WGRAD) off = add_sat(a_off[i], (unsigned)te[v].x);
            else if constexpr (A_KC) off = outside(a_hw[i], te[v].y, lim_hw) == 0 ? a_off[i] + (unsigned)(te[v].x + a_c[v]) * 4u : OOB;
            else {
                const unsigned to = a_off[i] + (unsigned)of_row(BM, i, (int)ar_off);      // lane reads: never under a condition
                off = outside(a_hw[i], of_row(BM, i, ar_d), lim_hw) == 0 ? to : OOB;
            }
            float *d = ring + slot * STG + (gw + NG * i) * (64 * VA);
            if constexpr (VA == 4) lds_dma16(rs_a, off, d); else lds_dma4(rs_a, off, d);
        } else {
            constexpr int i = Tk - A_LD, v = B_VARK ? i & 3 : 0;
            if constexpr (OP == OP_FWD || (OP == OP_BWD && NCHW)) off = add_sat(b_off[i], we[v]);
            else if constexpr (OP == OP_BWD) off = add_sat(b_off[i], (unsigned)of_row(BN, i, (int)br_off));
            else if constexpr (NCHW) off = outside(te[v].y, b_hw[i], lim_hw) == 0 ? b_off[i] + we[v] : OOB;
            else {
                const unsigned to = b_off[i] + (unsigned)of_row(BN, i, (int)br_off);
                off = outside(of_row(BN, i, br_d), b_hw[i], lim_hw) == 0 ? to : OOB;
            }
            float *d = ring + slot * STG + BM * BK + (gw + NG * i) * (64 * VB);
            if constexpr (VB == 4) lds_dma16(rs_b, off, d); else lds_dma4(rs_b, off, d);
        }
    };
    auto advance = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < NKA; ++v) {
            a_k[v] += KSTEP;
            if constexpr (OP == OP_WGRAD) {
                const int t = a_t[v] + adv_pq, carry = t >= PQ ? 1 : 0;
                a_t[v] = t - (carry ? PQ : 0);
                a_c[v] += adv_n + carry;
            } else if constexpr (A_KC) {
                const int c = a_c[v] + adv_cr, carry = c >= Ci ? 1 : 0;
                a_c[v] = c - (carry ? Ci : 0);
                a_t[v] += adv_cq + carry;
            } else {
                const int t = a_t[v] + adv_tr, carry = t >= T ? 1 : 0;
                a_t[v] = t - (carry ? T : 0);
                a_c[v] += adv_tq + carry;
            }
        }
#pragma unroll
        for (int v = 0; v < NKB; ++v) {
            b_k[v] += KSTEP;
            if constexpr (OP == OP_WGRAD) {
                const int q = b_q[v] + adv_q, cq = q >= s.Q ? 1 : 0;
                b_q[v] = q - (cq ? s.Q : 0);
                const int pr = b_t[v] + adv_p + cq, cp = pr >= s.P ? 1 : 0;
                b_t[v] = pr - (cp ? s.P : 0);
                b_c[v] += adv_n3 + cp;
            } else if constexpr (OP == OP_BWD && B_KC) {
                const int t = b_t[v] + adv_tr, carry = t >= T ? 1 : 0;
                b_t[v] = t - (carry ? T : 0);
                b_c[v] += adv_tq + carry;
            } else if constexpr (OP == OP_BWD) {
                const int c = b_c[v] + adv_cr, carry = c >= Ci ? 1 : 0;
                b_c[v] = c - (carry ? Ci : 0);
                b_t[v] += adv_cq + carry;
            }
        }
        fetch_rows();
    };

    f32x16 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    // one stage: two groups of 8 reduction elements; lanes of half h hold elements 4h..4h+3 of the group, so matrix
    // step j multiplies elements j and 4+j
    const int l32 = lane & 31;
    auto frag = [&](auto kc, auto bx, const float *src, int base, int g, float (&f)[4]) __attribute__((always_inline)) {
        constexpr bool KC = decltype(kc)::value;
        constexpr int BX = decltype(bx)::value;
        if constexpr (KC) {
            const float4 v = *reinterpret_cast<const float4 *>(src + (base + l32) * BK + (((2 * g + half) ^ ((l32 >> 2) & 3)) << 2));
            f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
        } else {
            const int col = BX >= 64 ? (base + l32) ^ (half * 32) : base + l32;
#pragma unroll
            for (int j = 0; j < 4; ++j) f[j] = src[(8 * g + 4 * half + j) * BX + col];
        }
    };
    struct Frags { float a[MI][4], b[NI][4]; };
    constexpr int N_READ = MI + NI, NMF = 4 * MI * NI;
    auto read_task = [&](auto tc, Frags &f, int slot, int g) __attribute__((always_inline)) {
        constexpr int Tk = decltype(tc)::value;
        const float *sa = ring + slot * STG, *sb = sa + BM * BK;
        if constexpr (Tk < MI) frag(std::integral_constant<bool, A_KC>{}, IC<BM>{}, sa, wave_m + 32 * Tk, g, f.a[Tk]);
        else frag(std::integral_constant<bool, B_KC>{}, IC<BN>{}, sb, wave_n + 32 * (Tk - MI), g, f.b[Tk - MI]);
    };
    // the matrix instructions of one group of 8 reduction elements with N side tasks spread between them, in pinned
    // order: the wave issues a task while the matrix pipe works on the instruction before it
    auto mfma_with = [&](const Frags &f, auto n, auto &&side) __attribute__((always_inline)) {
        constexpr int N = decltype(n)::value;
        static_for<NMF>([&](auto sc) __attribute__((always_inline)) {
            constexpr int S = decltype(sc)::value, q = S / (MI * NI), i = S / NI % MI, j = S % NI;
            acc[i][j] = SWAP ? __builtin_amdgcn_mfma_f32_32x32x2f32(f.b[j][q], f.a[i][q], acc[i][j], 0, 0, 0)
                             : __builtin_amdgcn_mfma_f32_32x32x2f32(f.a[i][q], f.b[j][q], acc[i][j], 0, 0, 0);
            static_for<N>([&](auto tc) __attribute__((always_inline)) {
                if constexpr (decltype(tc)::value * NMF / N == S) side(tc);
            });
            pin();
        });
    };

    // Pipeline.  Stage kt lives in slot kt % NS.  Its first group of 8 runs beside the fetch of the second group's
    // operands and the second half of the transfers of stage kt+NS-1; then the wave waits for its reads of this slot and
    // its transfers of stage kt+1, one barrier publishes stage kt+1 and frees this slot, and the second group runs beside
    // the first operand fetch of stage kt+1 and the first half of the transfers of stage kt+NS into the freed slot.
    constexpr int L1 = (L + 1) / 2, L2 = L - L1;
    if constexpr (TABLE) __syncthreads();
    fetch_rows();
    static_for<NS - 1>([&](auto sc) __attribute__((always_inline)) {
        static_for<L>([&](auto tc) __attribute__((always_inline)) { task(tc, decltype(sc)::value); });
        advance();
    });
    static_for<L1>([&](auto tc) __attribute__((always_inline)) { task(tc, NS - 1); });
    wait_vmcnt<L * (NS - 2) + L1>();
    if constexpr (NG > 1) { pin(); __builtin_amdgcn_s_barrier(); pin(); }
    Frags f0, f1;
    static_for<N_READ>([&](auto tc) __attribute__((always_inline)) { read_task(tc, f0, 0, 0); });
    int slot = 0;
    for (int kt = 0; kt < KT; ++kt) {
        const int prev = slot == 0 ? NS - 1 : slot - 1, next = slot + 1 == NS ? 0 : slot + 1;
        mfma_with(f0, IC<N_READ + L2 + 1>{}, [&](auto tc) __attribute__((always_inline)) {
            constexpr int Tk = decltype(tc)::value;
            if constexpr (Tk < N_READ) read_task(tc, f1, slot, 1);
            else if constexpr (Tk < N_READ + L2) task(IC<L1 + Tk - N_READ>{}, prev);
            else advance();
        });
        wait_lgkmcnt0();
        wait_vmcnt<L * (NS - 2)>();
        if constexpr (NG > 1) { pin(); __builtin_amdgcn_s_barrier(); pin(); }
        mfma_with(f1, IC<N_READ + L1>{}, [&](auto tc) __attribute__((always_inline)) {
            constexpr int Tk = decltype(tc)::value;
            if constexpr (Tk < N_READ) read_task(tc, f0, next, 0);
            else task(IC<Tk - N_READ>{}, slot);
        });
        slot = next;
    }
    wait_vmcnt<0>();                        // zero-fill transfers of the stages past the end

    // ---- results ---------------------------------------------------------------------------------------------
    float *out = p.out;
    if constexpr (OP == OP_WGRAD) out += (size_t)split * ((size_t)rows * cols);
    // offset of result row i (without the column's share), or -1 past the end
    auto row_off = [&](int i) __attribute__((always_inline)) -> long long {
        if (i >= rows) return -1;
        if constexpr (OP == OP_WGRAD) return (long long)i * cols;
        else if constexpr (OP == OP_FWD) {
            if (!NCHW) return (long long)i * cols;
            const int n = p.by_pq.div(i);
            return (long long)n * cols * PQ + (i - n * PQ);
        } else {
            int pix = i;
            if (NCHW || s.stride != 1) {
                const int t2 = cls.mw.div(i), b = i - t2 * Mw, n = cls.mh.div(t2), a = t2 - n * Mh;
                const int hw = (h_first + s.stride * a) * s.W + v_first + s.stride * b;
                if (NCHW) return (long long)n * cols * (s.H * s.W) + hw;
                pix = n * (s.H * s.W) + hw;
            }
            return (long long)pix * cols;
        }
    };
    const int col_stride = !NCHW || OP == OP_WGRAD ? 1 : OP == OP_FWD ? PQ : s.H * s.W;
    auto put = [&](long long ro, int j, float v) __attribute__((always_inline)) {
        if (ro < 0 || j >= cols) return;
        const long long o = ro + (long long)j * col_stride;
        if constexpr (OP == OP_FWD) {
            if (p.bias != nullptr) v += p.bias[j];
            if (p.relu) v = fmaxf(v, 0.f);
        }
        if constexpr (OP == OP_BWD) {
            if (p.mask != nullptr && !(p.mask[o] > 0.f)) v = 0.f;
        }
        out[o] = v;
    };
    // row and column of this lane's result number `at`: element (block, e) of its wave's tile, or (Z > 1) of the workgroup's
    // summed tile, which the threads share out
    auto place = [&](int at, int &row, int &col) __attribute__((always_inline)) {
        const int idx = Z == 1 ? (gw * MI * NI * 16 + at) * 64 + lane : at * NT + tid;
        const int ln = idx & 63, e = (idx >> 6) & 15, blk = idx >> 10;
        const int wv = blk / (MI * NI), bi = blk % (MI * NI) / NI, bj = blk % NI;
        const int reg = 8 * (e >> 2) + 4 * (ln >> 5) + (e & 3), al = ln & 31;
        row = m0 + (wv / WC) * (32 * MI) + 32 * bi + (SWAP ? al : reg);
        col = n0 + (wv % WC) * (32 * NI) + 32 * bj + (SWAP ? reg : al);
    };
    // A result that is NaN is noted (bit `at`; one comparison a result) and summed once more: see sum_inside.
    unsigned long long noted = 0;
    auto finish = [&](int at, long long ro, int j, float v) __attribute__((always_inline)) {
        if (v != v) noted |= 1ull << at;
        put(ro, j, v);
    };
    // accumulator element e of a block: index along the registers 8*(e/4) + 4*half + e%4, along the lanes lane%32
    if constexpr (Z == 1) {
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            if constexpr (SWAP) {
                const long long ro = row_off(m0 + wave_m + 32 * i + l32);
#pragma unroll
                for (int j = 0; j < NI; ++j)
#pragma unroll
                    for (int e = 0; e < 16; ++e) finish((i * NI + j) * 16 + e, ro, n0 + wave_n + 32 * j + 8 * (e >> 2) + 4 * half + (e & 3), acc[i][j][e]);
            } else {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const long long ro = row_off(m0 + wave_m + 32 * i + 8 * (e >> 2) + 4 * half + (e & 3));
#pragma unroll
                    for (int j = 0; j < NI; ++j) finish((i * NI + j) * 16 + e, ro, n0 + wave_n + 32 * j + l32, acc[i][j][e]);
                }
            }
        }
    } else {
        __syncthreads();                    // every group is done with its ring
        constexpr int WT = MI * NI * 1024;  // floats of a wave's tile: [block][e][lane]
        float *mine = smem + (zg * NG + gw) * WT;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int e = 0; e < 16; ++e) mine[(i * NI + j) * 1024 + e * 64 + lane] = acc[i][j][e];
        __syncthreads();
#pragma unroll
        for (int q = 0; q < NG * WT / NT; ++q) {
            float v = 0.f;
#pragma unroll
            for (int z = 0; z < Z; ++z) v += smem[z * NG * WT + q * NT + tid];
            int row, col;
            place(q, row, col);
            finish(q, row_off(row), col, v);
        }
    }
    if (p.outside)
        while (noted != 0) {
            int row, col;
            place(__ffsll(noted) - 1, row, col);
            noted &= noted - 1;
            if (row < rows && col < cols) put(row_off(row), col, sum_inside<OP, NCHW>(p, cls, row, col, k_lo, k_hi));
        }
}

// ---- NHWC, whole 16-byte chunks of channels: waves that share a tile's reduction ------------------------------------------------
// The fp32 counterparts of wave.hip and wave_dw.hip (see there for the scheme): a wave reduces its whole tile over every KG-th
// step of 16 elements through a ring of its own, no barrier before the KG partial tiles meet in LDS.  v_mfma_f32_16x16x4_f32 with
// the operand first whose index is contiguous in the result: lane 16*g + i holds columns 4*g .. 4*g + 3 of row i, 16 bytes of it.
// A block of 16 rows x 16 reduction elements is one direct global->LDS load of 16 bytes per lane and one ds_read_b128, whose
// four elements serve four MFMAs.  Operands that lie the other way round (the KRSC filter in backward-data, both in
// backward-weight) land as 16 reduction rows of 16*B floats and are fetched with ds_read_b32.
//
// What bounds it: 1024 multiply-adds per 32 clocks of a SIMD, and beside them (fp32 MFMAs never overlap vector instructions) the
// address arithmetic, which here is per 16-byte chunk and not per element: 64 MFMAs to some 90 vector instructions in the 64x64
// tiles, where the kernel above has 8 to 57.  Measured (us, kernel above -> here; forward, dx, dw): 512 pixels 16->32
// 3x3 4.7 -> 3.8, 7.1 -> 5.1, 9.6 -> 5.9; 4096 pixels 64->96 3x3 11.6 -> 9.0, 10.9 -> 9.8, 21.0 -> 12.0; 392 pixels 448->112 3x3
// 23.0 -> 15.1, 12.0 -> 10.6, 18.4 -> 9.2.  Which layers these get: wave_rows, wave_wgrad.

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Tile of 16 reduction rows x 16*B floats: row r lies at row_at(r), its 16-byte chunks exchanged by chunk_swz(r), so that the four
// rows that one fetch touches (4*g + s, g = 0..3) fall on different banks.
template <int B> __device__ __forceinline__ int row_at(int r) { return B == 2 ? r ^ ((r >> 3) & 1) : r; }
template <int B> __device__ __forceinline__ int chunk_swz(int r) { return ((r >> 2) & (B - 1)) << 2; }

// the ring of a wave: `turns` steps through NS slots of L loads each
template <int L, int NS, class I, class S> __device__ __forceinline__ void run_ring(float *ring, int slot_floats, int turns, I &&issue, S &&step)
{
    const int ahead = min(turns, NS);
#pragma unroll
    for (int q = 0; q < NS; ++q)
        if (q < ahead) issue(ring + q * slot_floats);
    int slot = 0;
    for (int t = turns; t > NS; --t) {
        wait_vmcnt<L * (NS - 1)>();
        step(ring + slot * slot_floats, true);
        slot = slot + 1 == NS ? 0 : slot + 1;
    }
#pragma unroll
    for (int q = NS; q > 0; --q)
        if (q <= ahead) {
            if (q == 4) wait_vmcnt<L * 3>();
            else if (q == 3) wait_vmcnt<L * 2>();
            else if (q == 2) wait_vmcnt<L>();
            else wait_vmcnt<0>();
            step(ring + slot * slot_floats, false);
            slot = slot + 1 == NS ? 0 : slot + 1;
        }
}

// MB x NB blocks of 16 pixels x 16 columns; KG waves share a tile's reduction, MG stand side by side along the pixels.
// TAP: a step lies in one tap (channels % 16 == 0), whose arithmetic is scalar.  PLANES: the operands are NHWC copies of an NCHW
// problem and the result goes straight to its planes: the product is formed the other way round, lane 16*g + i holds pixels
// 4*g .. 4*g + 3 of column i.
template <int OP, int MB, int NB, int KG, int MG, int NS, bool TAP, bool PLANES>
__global__ __launch_bounds__(64 * KG * MG) void f32_wave_kernel(const F32Params p)
{
    constexpr int BM = 16 * MB * MG, BN = 16 * NB, BLK = 256, SLOT = (MB + NB) * BLK, RING = NS * SLOT, L = MB + NB;
    static_assert(L * (NS - 1) < 64 && (KG == 1 || MB * NB * 256 <= RING), "vmcnt range; a wave's partial tile must fit its ring");
    static_assert(MB <= KG || MB % KG == 0, "wave kg finishes pixel blocks kg, kg + KG, ...");
    static_assert(OP == OP_FWD || NB == 2 || NB == 4, "rows of a transposed filter tile");
    __shared__ __attribute__((aligned(1024))) float ring[KG * MG * RING];

    const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int kg = wave % KG, mg = wave / KG;
    const int per_xcd = (p.units + 7) / 8;
    const int unit = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (unit >= p.units) return;
    int mt = p.by_ntiles.div(unit), ci = 0;
    const int n0 = (unit - mt * p.n_tiles) * BN;
    const ConvShape &s = p.s;
    if constexpr (OP == OP_BWD) {
        while (ci + 1 < p.n_cls && mt >= p.cls[ci + 1].tile0) ++ci;
        mt -= p.cls[ci].tile0;
    }
    const F32Class &cls = p.cls[ci];
    const int m0 = mt * BM + mg * 16 * MB;
    const int Ci = OP == OP_BWD ? s.K : s.C, Hi = OP == OP_BWD ? s.P : s.H, Wi = OP == OP_BWD ? s.Q : s.W, RS = s.R * s.S;
    const int TS = cls.TS, T = cls.TR * TS, Kd = T * Ci;
    const int rows = OP == OP_FWD ? p.M : s.N * cls.Mh * cls.Mw, cols = OP == OP_FWD ? s.K : s.C;
    const int turns = (Kd + 16 * KG - 1) / (16 * KG);
    const int px4 = Ci * 4, row4 = Wi * px4, lim_hw = pack_hw(Hi - 1, Wi - 1), ts_magic = cls.ts_magic;
    const buf_rsrc_t rs_a = make_buf_rsrc(p.a, p.a_bytes), rs_b = make_buf_rsrc(p.b, p.b_bytes);

    // ---- what this lane loads: row l/4 of every block, chunk (l%4) ^ (l/16) of its step
    const int ld_row = lane >> 2, chunk = ((lane & 3) ^ (lane >> 4)) * 4;
    int a_off[MB], a_hw[MB];
#pragma unroll
    for (int b = 0; b < MB; ++b) {
        const int m = m0 + 16 * b + ld_row, t = cls.mw.div(m), col = m - t * cls.Mw, n = cls.mh.div(t), row = t - n * cls.Mh;
        const int mul = OP == OP_FWD ? s.stride : 1, h = row * mul + cls.off_h, w = col * mul + cls.off_w;
        a_off[b] = (n * Hi + h) * row4 + w * px4;
        a_hw[b] = m < rows ? pack_hw(h, w) : FAR;
    }
    const int in_kd = TAP ? 0 : chunk, in_off = chunk - in_kd;
    int kd = kg * 16 + in_kd, tap = p.by_ci.div(kd), c = kd - tap * Ci, first = kg * 16;     // first: the step's
    const int adv_t = p.by_ci.div(16 * KG), adv_c = 16 * KG - adv_t * Ci;
    constexpr int BCH = 4 * NB, BROWS = 64 / BCH;
    unsigned f_off[NB];
    int f_row[NB];                       // backward: the reduction row of load j
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        if constexpr (OP == OP_BWD) {
            const int at = BROWS * j + lane / BCH, r = row_at<NB>(at), col = n0 + ((lane % BCH) ^ chunk_swz<NB>(r)) * 4;
            f_row[j] = r;
            f_off[j] = col < cols ? (unsigned)col * 4u : OOB;
        } else {
            const int co = n0 + 16 * j + ld_row;
            f_row[j] = 0;
            f_off[j] = co < cols ? ((unsigned)co * (unsigned)Kd + (unsigned)in_off) * 4u : OOB;
        }
    }
    auto filter_tap = [&](int t) __attribute__((always_inline)) {
        const int j = small_div(t, ts_magic), q = t - j * TS;
        return (cls.ph + s.stride * j) * s.S + cls.pw + s.stride * q;
    };
    auto issue = [&](float *dst) __attribute__((always_inline)) {
        const bool k_ok = kd < Kd;
        const int j = small_div(tap, ts_magic), q = tap - j * TS;
        const int dh = OP == OP_BWD ? -j : j, dw = OP == OP_BWD ? -q : q;
        const int t_hw = k_ok ? pack_hw(dh, dw) : FAR, base = dh * row4 + dw * px4 + (c + in_off) * 4;
#pragma unroll
        for (int b = 0; b < MB; ++b) lds_dma16(rs_a, outside(a_hw[b], t_hw, lim_hw) == 0 ? (unsigned)(a_off[b] + base) : OOB, dst + b * BLK);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            unsigned off;
            if constexpr (OP == OP_BWD) {
                const int at = first + f_row[b];
                int t = tap, k = c + f_row[b];
                if constexpr (!TAP) { t = p.by_ci.div(at); k = at - t * Ci; }
                off = at < Kd && f_off[b] != OOB ? f_off[b] + (unsigned)((k * RS + filter_tap(t)) * s.C) * 4u : OOB;
            } else off = k_ok && f_off[b] != OOB ? f_off[b] + (unsigned)kd * 4u : OOB;
            lds_dma16(rs_b, off, dst + (MB + b) * BLK);
        }
        kd += KG * 16; first += KG * 16;
        c += adv_c;
        const int carry = c >= Ci ? 1 : 0;
        c -= carry ? Ci : 0;
        tap += adv_t + carry;
    };
    f32x4 acc[MB][NB];
#pragma unroll
    for (int b = 0; b < MB; ++b)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[b][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int frag = i * 16 + ((g ^ (i >> 2)) & 3) * 4;
    auto step = [&](float *src, bool refill) __attribute__((always_inline)) {
        f32x4 fa[MB], fw[NB];
#pragma unroll
        for (int b = 0; b < MB; ++b) fa[b] = *reinterpret_cast<const f32x4 *>(src + b * BLK + frag);
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            if constexpr (OP == OP_BWD) {
#pragma unroll
                for (int e = 0; e < 4; ++e) fw[j][e] = src[MB * BLK + row_at<NB>(4 * g + e) * BN + ((16 * j) ^ (chunk_swz<NB>(4 * g) * 4)) + i];
            } else fw[j] = *reinterpret_cast<const f32x4 *>(src + (MB + j) * BLK + frag);
        }
        wait_lgkmcnt0();
        pin();
        if (refill) issue(src);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int b = 0; b < MB; ++b)
#pragma unroll
                for (int j = 0; j < NB; ++j) {
                    if constexpr (PLANES) acc[b][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fa[b][e], fw[j][e], acc[b][j], 0, 0, 0);
                    else acc[b][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[j][e], fa[b][e], acc[b][j], 0, 0, 0);
                }
        pin();
    };
    run_ring<L, NS>(ring + wave * RING, SLOT, turns, issue, step);

    // ---- results: columns n0 + 16*j + 4*g .. + 3 of pixel m0 + 16*b + i
    const bool whole = (cols & 3) == 0;
    auto store_planes = [&](int b, const f32x4 (&v)[NB]) __attribute__((always_inline)) {
        const int m = m0 + 16 * b + 4 * g, plane = OP == OP_FWD ? s.P * s.Q : s.H * s.W;
        if (m >= rows) return;
        const bool unit = OP == OP_FWD || s.stride == 1, quad = unit && (plane & 3) == 0;      // four pixels of one image, 16 bytes
        int img[4], at[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int t = cls.mw.div(m + e), n = cls.mh.div(t);
            img[e] = n;
            if (unit) at[e] = m + e - n * plane;
            else at[e] = (cls.h_first + s.stride * (t - n * cls.Mh)) * s.W + cls.v_first + s.stride * (m + e - t * cls.Mw);
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int col = n0 + 16 * j + i;
            if (col >= cols) continue;
            f32x4 r = v[j];
            const bool nan = r.x != r.x || r.y != r.y || r.z != r.z || r.w != r.w;
            if (p.outside && nan)
#pragma unroll 1
                for (int e = 0; e < 4; ++e)
                    if (m + e < rows) {
                        const float x = e == 0 ? r.x : e == 1 ? r.y : e == 2 ? r.z : r.w;
                        const float y = x != x ? sum_inside<OP, false>(p, cls, m + e, col, 0, 0) : x;
                        if (e == 0) r.x = y; else if (e == 1) r.y = y; else if (e == 2) r.z = y; else r.w = y;
                    }
            if (OP == OP_FWD && p.bias != nullptr) r += p.bias[col];
            long long off[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                off[e] = ((long long)img[e] * cols + col) * plane + at[e];
                if (OP == OP_FWD && p.relu) r[e] = fmaxf(r[e], 0.f);
                if (OP == OP_BWD && p.mask != nullptr && m + e < rows && !(p.mask[off[e]] > 0.f)) r[e] = 0.f;
            }
            if (quad) *reinterpret_cast<f32x4 *>(p.out + off[0]) = r;      // (rows are a multiple of plane)
            else
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (m + e < rows) p.out[off[e]] = r[e];
        }
    };
    auto store = [&](int b, const f32x4 (&v)[NB]) __attribute__((always_inline)) {
        if constexpr (PLANES) return store_planes(b, v);
        const int m = m0 + 16 * b + i;
        if (m >= rows) return;
        long long pix = m;
        if (OP == OP_BWD && s.stride != 1) {
            const int t = cls.mw.div(m), col = m - t * cls.Mw, n = cls.mh.div(t), row = t - n * cls.Mh;
            pix = ((long long)n * s.H + cls.h_first + s.stride * row) * s.W + cls.v_first + s.stride * col;
        }
        float *out = p.out + pix * cols;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const int col = n0 + 16 * j + 4 * g;
            if (col >= cols) continue;
            f32x4 r = v[j];
            const bool nan = r.x != r.x || r.y != r.y || r.z != r.z || r.w != r.w;
            if (p.outside && nan)
#pragma unroll 1
                for (int e = 0; e < 4; ++e)
                    if (col + e < cols) {
                        const float x = e == 0 ? r.x : e == 1 ? r.y : e == 2 ? r.z : r.w;
                        const float y = x != x ? sum_inside<OP, false>(p, cls, m, col + e, 0, 0) : x;
                        if (e == 0) r.x = y; else if (e == 1) r.y = y; else if (e == 2) r.z = y; else r.w = y;
                    }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (OP == OP_FWD && p.bias != nullptr && col + e < cols) r[e] += p.bias[col + e];
                if (OP == OP_FWD && p.relu) r[e] = fmaxf(r[e], 0.f);
                if (OP == OP_BWD && p.mask != nullptr && col + e < cols && !(p.mask[pix * cols + col + e] > 0.f)) r[e] = 0.f;
            }
            if (whole) *reinterpret_cast<f32x4 *>(out + col) = r;
            else
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (col + e < cols) out[col + e] = r[e];
        }
    };
    if constexpr (KG == 1) {
#pragma unroll
        for (int b = 0; b < MB; ++b) store(b, acc[b]);
    } else {
        f32x4 *part = reinterpret_cast<f32x4 *>(ring);
        constexpr int PITCH = RING / 4;
#pragma unroll
        for (int b = 0; b < MB; ++b)
#pragma unroll
            for (int j = 0; j < NB; ++j) part[wave * PITCH + (b * NB + j) * 64 + lane] = acc[b][j];
        __syncthreads();
        if (kg >= MB) return;
#pragma unroll
        for (int b0 = 0; b0 < MB; b0 += KG) {
            const int b = b0 + kg;
            f32x4 v[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) v[j] = part[mg * KG * PITCH + (b * NB + j) * 64 + lane];
#pragma unroll
            for (int z = 1; z < KG; ++z)
#pragma unroll
                for (int j = 0; j < NB; ++j) v[j] += part[(mg * KG + z) * PITCH + (b * NB + j) * 64 + lane];
            store(b, v);
        }
    }
}

// dw[k][col] over one pixel range per unit, MB x NB blocks of 16 filters x 16 columns, KG waves.  LINEAR: a 1x1 filter at stride 1
// without padding.
template <int MB, int NB, int KG, int NS, bool LINEAR>
__global__ __launch_bounds__(64 * KG) void f32_wave_dw_kernel(const F32Params p)
{
    constexpr int BLK = 256, SLOT = (MB + NB) * BLK, RING = NS * SLOT, L = MB + NB;
    static_assert((MB == 2 || MB == 4) && (NB == 2 || NB == 4) && L * (NS - 1) < 64 && MB * NB * 256 <= RING, "config");
    __shared__ __attribute__((aligned(1024))) float ring[KG * RING];
    const int lane = threadIdx.x & 63, i = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int per_xcd = (p.units + 7) / 8;
    const int unit = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (unit >= p.units) return;
    const ConvShape &s = p.s;
    const int z = p.by_tiles.div(unit), tile = unit - z * p.tiles, kt = p.by_ntiles.div(tile);
    const int k0 = kt * 16 * MB, n0 = (tile - kt * p.n_tiles) * 16 * NB, cols = s.C * s.R * s.S;
    const int m_lo = z * p.span, m_end = min(m_lo + p.span, p.M);
    const int turns = (m_end - m_lo + 16 * KG - 1) / (16 * KG);
    const int px4 = s.C * 4, row4 = s.W * px4, img4 = s.H * row4, lim_hw = pack_hw(s.H - 1, s.W - 1);
    const buf_rsrc_t rs_a = make_buf_rsrc(p.a, p.a_bytes), rs_b = make_buf_rsrc(p.b, p.b_bytes);

    constexpr int ACH = 4 * MB, AROWS = 64 / ACH, BCH = 4 * NB, BROWS = 64 / BCH;
    const int m_first = m_lo + wave * 16;
    int a_m[MB], b_m[NB];                // pixel of load j
    unsigned a_off[MB];
    int b_off[NB], b_q[NB], b_p[NB], b_tap[NB];
#pragma unroll
    for (int j = 0; j < MB; ++j) {
        const int r = row_at<MB>(AROWS * j + lane / ACH), k = k0 + ((lane % ACH) ^ chunk_swz<MB>(r)) * 4;
        a_m[j] = m_first + r;
        a_off[j] = k < s.K ? ((unsigned)a_m[j] * (unsigned)s.K + (unsigned)k) * 4u : OOB;
    }
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int r = row_at<NB>(BROWS * j + lane / BCH), col = n0 + ((lane % BCH) ^ chunk_swz<NB>(r)) * 4, m = m_first + r;
        b_m[j] = m;
        if constexpr (LINEAR) {
            b_off[j] = col < cols ? m * px4 + col * 4 : (int)OOB;
        } else {
            const int tap = p.by_c.div(col), fr = p.by_s.div(tap), fs = tap - fr * s.S, t = p.by_q.div(m), n = p.by_p.div(t);
            b_q[j] = m - t * s.Q; b_p[j] = t - n * s.P;
            b_off[j] = n * img4 + (b_p[j] * s.stride + fr - s.pad) * row4 + (b_q[j] * s.stride + fs - s.pad) * px4 + (col - tap * s.C) * 4;
            b_tap[j] = col < cols ? pack_hw(fr - s.pad, fs - s.pad) : FAR;
        }
    }
    const unsigned a_adv = (unsigned)(KG * 16) * (unsigned)(s.K * 4);
    const int adv_row = p.by_q.div(KG * 16), adv_q = KG * 16 - adv_row * s.Q, adv_n = p.by_p.div(adv_row), adv_p = adv_row - adv_n * s.P;
    const int sp = s.stride * px4, sr = s.stride * row4;
    auto issue = [&](float *dst) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < MB; ++j) {
            lds_dma16(rs_a, a_m[j] < m_end && a_off[j] < OOB ? a_off[j] : OOB, dst + j * BLK);
            a_off[j] += a_off[j] < OOB ? a_adv : 0u;
            a_m[j] += KG * 16;
        }
#pragma unroll
        for (int j = 0; j < NB; ++j) {
            const bool in = b_m[j] < m_end;
            b_m[j] += KG * 16;
            if constexpr (LINEAR) {
                lds_dma16(rs_b, in ? (unsigned)b_off[j] : OOB, dst + (MB + j) * BLK);
                b_off[j] += (unsigned)b_off[j] < OOB ? KG * 16 * px4 : 0;
            } else {
                const bool ok = in && outside(pack_hw(b_p[j] * s.stride, b_q[j] * s.stride), b_tap[j], lim_hw) == 0;
                lds_dma16(rs_b, ok ? (unsigned)b_off[j] : OOB, dst + (MB + j) * BLK);
                int off = b_off[j] + adv_n * img4 + adv_p * sr + adv_q * sp, q = b_q[j] + adv_q;
                const bool cq = q >= s.Q;
                q -= cq ? s.Q : 0;
                off += cq ? sr - s.Q * sp : 0;
                int pr = b_p[j] + adv_p + (cq ? 1 : 0);
                const bool cp = pr >= s.P;
                pr -= cp ? s.P : 0;
                off += cp ? img4 - s.P * sr : 0;
                b_q[j] = q; b_p[j] = pr; b_off[j] = off;
            }
        }
    };
    f32x4 acc[MB][NB];
#pragma unroll
    for (int b = 0; b < MB; ++b)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[b][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto step = [&](float *src, bool refill) __attribute__((always_inline)) {
        float fa[MB][4], fb[NB][4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
#pragma unroll
            for (int b = 0; b < MB; ++b) fa[b][e] = src[row_at<MB>(4 * g + e) * (16 * MB) + ((16 * b) ^ (chunk_swz<MB>(4 * g) * 4)) + i];
#pragma unroll
            for (int j = 0; j < NB; ++j) fb[j][e] = src[MB * BLK + row_at<NB>(4 * g + e) * (16 * NB) + ((16 * j) ^ (chunk_swz<NB>(4 * g) * 4)) + i];
        }
        wait_lgkmcnt0();
        pin();
        if (refill) issue(src);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int b = 0; b < MB; ++b)
#pragma unroll
                for (int j = 0; j < NB; ++j) acc[b][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(fb[j][e], fa[b][e], acc[b][j], 0, 0, 0);
        pin();
    };
    run_ring<L, NS>(ring + wave * RING, SLOT, turns, issue, step);

    f32x4 *part = reinterpret_cast<f32x4 *>(ring);
    constexpr int PITCH = RING / 4;
#pragma unroll
    for (int b = 0; b < MB; ++b)
#pragma unroll
        for (int j = 0; j < NB; ++j) part[wave * PITCH + (b * NB + j) * 64 + lane] = acc[b][j];
    __syncthreads();
    float *out = p.out + (size_t)z * ((size_t)s.K * cols);
    for (int blk = wave; blk < MB * NB; blk += KG) {
        f32x4 v = part[blk * 64 + lane];
#pragma unroll
        for (int w = 1; w < KG; ++w) v += part[w * PITCH + blk * 64 + lane];
        const int k = k0 + blk / NB * 16 + i, col = n0 + blk % NB * 16 + 4 * g;
        if (k >= s.K || col >= cols) continue;
        const bool nan = v.x != v.x || v.y != v.y || v.z != v.z || v.w != v.w;
        if (p.outside && nan)
#pragma unroll 1
            for (int e = 0; e < 4; ++e) {
                const float x = e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w;
                const float y = x != x ? sum_inside<OP_WGRAD, false>(p, p.cls[0], k, col + e, m_lo, m_end) : x;
                if (e == 0) v.x = y; else if (e == 1) v.y = y; else if (e == 2) v.z = y; else v.w = y;
            }
        *reinterpret_cast<f32x4 *>(out + (size_t)k * cols + col) = v;
    }
}

// The shapes and the time models that pick one (us, fitted to 260 layers of 0.001 to 25 GFLOP on the device, 3-10% off):
// {fixed, mfma, turn, round, mb, area}: fixed + mfma * (hundred 16x16x16 products of the CU with most tiles) + turn * (rounds of
// workgroups that fit a CU, times steps per wave) + round * rounds + mb * (MB written, and of the mask read) + area * (ten blocks of
// that CU); backward-weight's {fixed, mfma, turn, round, mb, ranges, part}: with several pixel ranges + ranges + part * (MB of partial tensors).
struct F32Wave { int mb, nb, kg, mg, ns; const char *name; float us[2][6]; };     // us: forward, backward-data
#define F32_WAVES(X) \
    X(0, 1, 2, 8, 1, 4, "f32_wave_16x32_split8", {{1.78f, 0.f, 0.387f, 1.43f, 0.740f, 0.f}, {2.69f, 0.f, 0.546f, 1.48f, 0.613f, 0.f}}) \
    X(1, 2, 2, 8, 1, 4, "f32_wave_32x32_split8", {{1.72f, 0.f, 0.642f, 1.67f, 0.473f, 0.f}, {2.38f, 0.f, 0.790f, 2.19f, 0.231f, 0.f}}) \
    X(2, 4, 2, 8, 1, 3, "f32_wave_64x32_split8", {{1.52f, 0.f, 1.14f, 2.22f, 0.299f, 0.f}, {2.36f, 0.f, 1.28f, 2.52f, 0.177f, 0.f}}) \
    X(3, 4, 4, 8, 1, 2, "f32_wave_64x64_split8", {{1.82f, 1.60f, 0.f, 0.f, 0.501f, 1.49f}, {1.93f, 1.77f, 0.f, 0.f, 0.343f, 2.01f}}) \
    X(4, 2, 2, 4, 2, 3, "f32_wave_64x32_split4", {{1.83f, 0.f, 0.631f, 1.61f, 0.362f, 0.f}, {2.43f, 0.f, 0.787f, 1.97f, 0.173f, 0.f}}) \
    X(5, 2, 2, 2, 4, 2, "f32_wave_128x32_split2", {{2.96f, 1.56f, 0.148f, 0.f, 0.222f, 0.327f}, {3.83f, 1.42f, 0.322f, 0.f, 0.161f, 0.700f}}) \
    X(6, 2, 2, 1, 4, 2, "f32_wave_128x32", {{3.87f, 1.59f, 0.223f, 0.f, 0.239f, 0.038f}, {3.99f, 1.43f, 0.310f, 0.f, 0.084f, 0.926f}})
#define X(I, MB, NB, KG, MG, NS, NAME, ...) {MB, NB, KG, MG, NS, NAME, __VA_ARGS__},
const F32Wave kWaves[] = {F32_WAVES(X)};
#undef X
constexpr int N_WAVES = sizeof(kWaves) / sizeof(kWaves[0]);

struct F32WaveDw { int mb, nb, kg, ns; const char *name; float us[7]; };
#define F32_DW_WAVES(X) \
    X(0, 2, 2, 8, 4, "f32_wave_dw_32x32_w8", {1.52f, 0.f, 0.720f, 1.40f, 0.475f, 3.94f, 0.f}) \
    X(1, 4, 2, 8, 3, "f32_wave_dw_64x32_w8", {1.69f, 0.f, 1.34f, 1.25f, 0.398f, 3.43f, 0.431f}) \
    X(2, 4, 4, 8, 2, "f32_wave_dw_64x64_w8", {1.89f, 1.81f, 0.f, 1.52f, 0.454f, 2.97f, 0.677f})
#define X(I, MB, NB, KG, NS, NAME, ...) {MB, NB, KG, NS, NAME, __VA_ARGS__},
const F32WaveDw kDwWaves[] = {F32_DW_WAVES(X)};
#undef X
constexpr int N_DW_WAVES = sizeof(kDwWaves) / sizeof(kDwWaves[0]);

template <int OP, int MB, int NB, int KG, int MG, int NS, bool PLANES>
void launch_wave(const F32Params &p, bool tap, hipStream_t st)
{
    const dim3 grid((unsigned)((p.units + 7) / 8 * 8)), block(64 * KG * MG);
    if (tap) hipLaunchKernelGGL((f32_wave_kernel<OP, MB, NB, KG, MG, NS, true, PLANES>), grid, block, 0, st, p);
    else hipLaunchKernelGGL((f32_wave_kernel<OP, MB, NB, KG, MG, NS, false, PLANES>), grid, block, 0, st, p);
}
template <int MB, int NB, int KG, int NS>
void launch_wave_dw(const F32Params &p, bool linear, hipStream_t st)
{
    const dim3 grid((unsigned)((p.units + 7) / 8 * 8)), block(64 * KG);
    if (linear) hipLaunchKernelGGL((f32_wave_dw_kernel<MB, NB, KG, NS, true>), grid, block, 0, st, p);
    else hipLaunchKernelGGL((f32_wave_dw_kernel<MB, NB, KG, NS, false>), grid, block, 0, st, p);
}

int launch_wave_op(int op, bool planes, int t, const F32Params &p, hipStream_t st)
{
    const bool tap = (op == OP_BWD ? p.s.K : p.s.C) % 16 == 0;
    switch (t) {
#define X(I, MB, NB, KG, MG, NS, ...) \
    case I: \
        if (op == OP_FWD) planes ? launch_wave<OP_FWD, MB, NB, KG, MG, NS, true>(p, tap, st) : launch_wave<OP_FWD, MB, NB, KG, MG, NS, false>(p, tap, st); \
        else planes ? launch_wave<OP_BWD, MB, NB, KG, MG, NS, true>(p, tap, st) : launch_wave<OP_BWD, MB, NB, KG, MG, NS, false>(p, tap, st); \
        break;
    F32_WAVES(X)
#undef X
    default: return MXC_ERR_UNSUPPORTED;
    }
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
}
int launch_wave_dw_op(int t, const F32Params &p, hipStream_t st)
{
    const ConvShape &s = p.s;
    const bool linear = s.R * s.S == 1 && s.stride == 1 && s.pad == 0;
    switch (t) {
#define X(I, MB, NB, KG, NS, ...) case I: launch_wave_dw<MB, NB, KG, NS>(p, linear, st); break;
    F32_DW_WAVES(X)
#undef X
    default: return MXC_ERR_UNSUPPORTED;
    }
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
}

// ---- tile choice ------------------------------------------------------------------------------------------------
// bm x bn tile, z groups of waves; eff: share of the fp32 matrix rate (256 flop per clock and CU) the tile sustains with one
// workgroup on a CU, and with several.  Timed on 16 layers (1x1 to 5x5, 3 to 512 channels, 0.03 to 30 GFLOP, NHWC and NCHW), forward
// and dx at 2.1 GHz less the fixed clocks below, median / best share: 128x128 .67/.90 alone, .72/.93 with several; 128x64
// .49/.76, .61/.87; 64x64 .54/.76, .61/.88; 128x32 .33/.56, .52/.81; 32x128 .39/.55, .63/.81; 32x32 .30/.66, .32/.70.  The
// values are fitted to the choices rather than to single times: against each of the six tiles forced, the chosen one is within
// 5% of the best in 90 of the 96 passes and within 8% in 93; dw of a 512->1000 head is the worst, 10.4 us against 8.2.
struct F32Tile { int bm, bn, z; float eff1, eff; const char *name; };
const F32Tile kTiles[] = {
    {128, 128, 1, 0.62f, 0.88f, "f32_128x128"},
    {128, 64, 1, 0.55f, 0.80f, "f32_128x64"},
    {64, 64, 2, 0.55f, 0.72f, "f32_64x64_z2"},
    {128, 32, 1, 0.40f, 0.70f, "f32_128x32"},
    {32, 128, 1, 0.40f, 0.70f, "f32_32x128"},
    {32, 32, 8, 0.40f, 0.50f, "f32_32x32_z8"},
};
constexpr int N_TILES = sizeof(kTiles) / sizeof(kTiles[0]);

template <int OP, bool NCHW, int VA, int VB, int WR, int WC, int MI, int NI, int Z, int NS>
int launch(const F32Params &p, hipStream_t st)
{
    hipLaunchKernelGGL((f32_conv_kernel<OP, NCHW, VA, VB, WR, WC, MI, NI, Z, NS>), dim3((unsigned)((p.units + 7) / 8 * 8)),
                       dim3(64 * WR * WC * Z), 0, st, p);
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
}

template <int OP, bool NCHW, int VA, int VB>
int launch_tile(int t, const F32Params &p, hipStream_t st)
{
    switch (t) {
    case 0: return launch<OP, NCHW, VA, VB, 2, 2, 2, 2, 1, 3>(p, st);
    case 1: return launch<OP, NCHW, VA, VB, 2, 2, 2, 1, 1, 3>(p, st);
    case 2: return launch<OP, NCHW, VA, VB, 2, 2, 1, 1, 2, 3>(p, st);
    // 32 rows of an operand are too few 16-byte transfers for four waves
    case 3: return launch<OP, NCHW, VA, 1, 4, 1, 1, 1, 1, 3>(p, st);
    case 4: return launch<OP, NCHW, 1, VB, 1, 4, 1, 1, 1, 3>(p, st);
    default: return launch<OP, NCHW, VA, VB, 1, 1, 1, 1, 8, 3>(p, st);
    }
}

int launch_op(int op, bool nchw, int t, const F32Params &p, hipStream_t st)
{
    const ConvShape &s = p.s;
    if (op == OP_FWD) {
        if (!nchw) return s.C % 4 == 0 ? launch_tile<OP_FWD, false, 4, 4>(t, p, st) : launch_tile<OP_FWD, false, 1, 1>(t, p, st);
        return (s.C * s.R * s.S) % 4 == 0 ? launch_tile<OP_FWD, true, 1, 4>(t, p, st) : launch_tile<OP_FWD, true, 1, 1>(t, p, st);
    }
    if (op == OP_BWD) {
        if (!nchw) return s.K % 4 == 0 ? launch_tile<OP_BWD, false, 4, 1>(t, p, st) : launch_tile<OP_BWD, false, 1, 1>(t, p, st);
        return launch_tile<OP_BWD, true, 1, 1>(t, p, st);
    }
    return nchw ? launch_tile<OP_WGRAD, true, 1, 1>(t, p, st) : launch_tile<OP_WGRAD, false, 1, 1>(t, p, st);
}

// forced tile (tests and tuning sweeps): MXC_FORCE_VARIANT for forward and backward-data, MXC_FORCE_WGRAD=<tile>[/<splits>]
int forced_tile(const char *env, int *splits)
{
    const char *f = getenv(env);
    if (f == nullptr) return -1;
    const char *slash = strchr(f, '/');
    const size_t len = slash ? (size_t)(slash - f) : strlen(f);
    for (int t = 0; t < N_TILES; ++t)
        if (strlen(kTiles[t].name) == len && !strncmp(f, kTiles[t].name, len)) {
            if (splits && slash) *splits = atoi(slash + 1);
            return t;
        }
    return -1;
}

// Modelled clocks of `tiles` workgroups of tile t that each reduce `k` elements: a CU's workgroups share its matrix
// pipes.  4000 clocks of pipeline fill and result stores, 1500 for every further workgroup of a CU, whose fill the others hide in
// part: with the shares above they rank the tiles as measured.  A fit of the single times of one workgroup per CU, the gap between
// launches included, gives 8 to 15 thousand clocks and shares of .43 (128x32) to .75 (128x128).
double model_clocks(const F32Tile &t, long long tiles, long long k)
{
    const long long per_cu = (tiles + 255) / 256;
    const double stages = (double)((k + BK * t.z - 1) / (BK * t.z)) * t.z;
    const double work = stages * (double)t.bm * t.bn * BK * 2.0 / 256.0;
    return (double)per_cu * work / (per_cu > 1 ? t.eff : t.eff1) + 4000.0 + 1500.0 * (per_cu - 1);
}

struct F32Plan { int tile, splits, span; };

// Time (us) of a tile beside the wave kernel's, fitted to the layers of its models, 2-6% off: {fixed, tile, first, work, mb} of
// forward, backward-data and backward-weight, by the CU with most tiles: fixed + tile * tiles + first * (65536 multiply-adds of one
// tile) + work * (of all) + mb * (MB written, and of the mask read; of all partial tensors), and 3 for the summing launch.  Zeros: a
// tile that those layers did not get, which keeps what it has.
const float kTileUs[N_TILES][3][5] = {
    {{9.53f, 2.36f, 0.747f, 3.64f, 0.128f}, {5.35f, 0.f, 0.f, 3.61f, 0.435f}, {}},
    {{6.53f, 0.886f, 1.91f, 3.71f, 0.192f}, {6.12f, 3.86f, 1.52f, 4.37f, 0.f}, {0.f, 8.10f, 0.f, 5.69f, 0.047f}},
    {{3.45f, 0.708f, 0.987f, 4.02f, 0.245f}, {4.97f, 0.501f, 1.06f, 5.04f, 0.153f}, {2.02f, 1.79f, 1.91f, 5.24f, 0.628f}},
    {{4.99f, 0.440f, 1.79f, 4.50f, 0.171f}, {5.29f, 1.27f, 3.79f, 4.71f, 0.082f}, {2.23f, 1.54f, 3.75f, 5.35f, 0.561f}},
    {{}, {}, {3.62f, 0.817f, 4.20f, 6.48f, 0.596f}},
    {{1.89f, 1.75f, 0.f, 5.00f, 0.466f}, {2.08f, 2.62f, 0.f, 7.40f, 0.181f}, {1.22f, 3.00f, 1.30f, 9.73f, 0.736f}},
};
// The same for forward and backward-data of NCHW problems read in place (1218 passes of 440 layers; 2-5% off, dx 5-13%).  The first
// tile's fixed time in forward is 8.0 and not the fit's 11.8: of the layers that get another kernel by it, 40 random ones run in 0.82 of the
// time (0.62 to 1.08; 20x41x41 1x1 20 to 68 on 30 images 14.5 us against 19.5).
const float kPlaneTileUs[N_TILES][2][5] = {
    {{8.0f, 0.682f, 0.513f, 4.33f, 0.277f}, {6.07f, 0.f, 4.23f, 2.47f, 0.513f}},
    {{8.07f, 1.13f, 1.66f, 5.17f, 0.142f}, {6.30f, 0.f, 3.25f, 4.71f, 0.327f}},
    {{3.62f, 1.34f, 1.29f, 5.27f, 0.217f}, {4.19f, 1.90f, 1.93f, 5.55f, 0.224f}},
    {{6.31f, 0.f, 3.74f, 6.58f, 0.263f}, {5.65f, 0.328f, 4.85f, 6.38f, 0.232f}},
    {{}, {}},
    {{1.63f, 2.97f, 0.239f, 9.21f, 0.438f}, {1.30f, 5.39f, 1.18f, 10.78f, 0.469f}},
};
double tile_us(int tile, int op, bool nchw, long long i, long long j, long long k, int splits, bool masked)
{
    const F32Tile &t = kTiles[tile];
    const float *c = nchw ? kPlaneTileUs[tile][op] : kTileUs[tile][op];
    const double per_cu = (double)(((i + t.bm - 1) / t.bm * ((j + t.bn - 1) / t.bn) * splits + 255) / 256);
    const double work = (double)((k + BK * t.z - 1) / (BK * t.z)) * t.z * t.bm * t.bn / 65536.0;
    return c[0] + c[1] * per_cu + (c[2] + c[3] * per_cu) * work + c[4] * (masked ? 8e-6 : 4e-6) * i * j * splits + (splits > 1 ? 3.0 : 0.0);
}

F32Class residue_class(const ConvShape &s, int ph, int pw)
{
    F32Class c{};
    c.ph = ph; c.pw = pw;
    c.TR = ph < s.R ? (s.R - ph + s.stride - 1) / s.stride : 0;
    c.TS = pw < s.S ? (s.S - pw + s.stride - 1) / s.stride : 0;
    c.off_h = ph >= s.pad ? 0 : (s.pad - ph + s.stride - 1) / s.stride;
    c.off_w = pw >= s.pad ? 0 : (s.pad - pw + s.stride - 1) / s.stride;
    c.h_first = ph - s.pad + s.stride * c.off_h; c.v_first = pw - s.pad + s.stride * c.off_w;
    c.Mh = c.h_first < s.H ? (s.H - 1 - c.h_first) / s.stride + 1 : 0;
    c.Mw = c.v_first < s.W ? (s.W - 1 - c.v_first) / s.stride + 1 : 0;
    return c;
}

void set_divisors(F32Class &c)
{
    c.mw = FastDiv(c.Mw); c.mh = FastDiv(c.Mh); c.t = FastDiv(c.TR * c.TS); c.ts = FastDiv(c.TS);
    c.ts_magic = small_magic(c.TS > 0 ? c.TS : 1);
}

F32Plan plan_rows(const ConvShape &s, int op)
{
    int t = forced_tile("MXC_FORCE_VARIANT", nullptr);
    if (t >= 0) return F32Plan{t, 1, 0};
    ++g_plan_searches;
    double best = 1e300;
    F32Plan pl{0, 1, 0};
    for (t = 0; t < N_TILES; ++t) {
        const long long cols = op == OP_FWD ? s.K : s.C, nt = (cols + kTiles[t].bn - 1) / kTiles[t].bn;
        const long long k = op == OP_FWD ? (long long)s.R * s.S * s.C
                                         : (long long)((s.R + s.stride - 1) / s.stride) * ((s.S + s.stride - 1) / s.stride) * s.K;
        const long long m = op == OP_FWD ? (long long)s.N * s.P * s.Q : (long long)s.N * s.H * s.W;
        const double c = model_clocks(kTiles[t], (m + kTiles[t].bm - 1) / kTiles[t].bm * nt, k);
        if (c < best) { best = c; pl.tile = t; }
    }
    return pl;
}

// Backward-weight: tile and number of pixel ranges; every range beyond the first writes and re-reads one fp32 dw
// (8 bytes per element at about 3 TB/s) and makes the summing launch necessary (5000 clocks: 2.2 us where it is all launch).
F32Plan search_wgrad(const ConvShape &s, int ft, int fs)
{
    ++g_plan_searches;
    const long long M = (long long)s.N * s.P * s.Q, cols = (long long)s.C * s.R * s.S;
    double best = 1e300;
    F32Plan pl{0, 1, (int)M};
    for (int t = 0; t < N_TILES; ++t) {
        if (ft >= 0 && t != ft) continue;
        const F32Tile &tc = kTiles[t];
        const long long tiles = ((s.K + tc.bm - 1) / tc.bm) * ((cols + tc.bn - 1) / tc.bn), q = (long long)BK * tc.z;
        long long max_sp = M / (4 * q);
        if (max_sp > 512) max_sp = 512;
        if (max_sp < 1) max_sp = 1;
        for (long long sp = 1; sp <= max_sp; sp += 1 + sp / 16) {
            if (fs > 0 && sp > 1) break;
            long long want = fs > 0 ? (fs < max_sp ? fs : max_sp) : sp;
            const long long span = ((M + want - 1) / want + q - 1) / q * q, used = (M + span - 1) / span;
            double c = model_clocks(tc, tiles * used, span);
            if (used > 1) c += 5000.0 + (double)used * s.K * cols * 8.0 / 3e12 * 2.1e9;
            if (c < best) { best = c; pl = F32Plan{t, (int)used, (int)span}; }
        }
    }
    return pl;
}

}  // namespace

const char *f32_wave_name(int index)
{
    return index < 0 ? nullptr : index < N_WAVES ? kWaves[index].name : index - N_WAVES < N_DW_WAVES ? kDwWaves[index - N_WAVES].name : nullptr;
}
const char *f32_tile_name(int index) { return index >= 0 && index < N_TILES ? kTiles[index].name : nullptr; }

// The kernel addresses its operands with 31-bit byte offsets, packs positions into 16 bits and holds MAX_TAPS taps.
bool f32_supported(const ConvShape &s)
{
    const long long lim = 0x7FFF0000ll, x = (long long)s.N * s.C * s.H * s.W * 4, y = (long long)s.N * s.K * s.P * s.Q * 4,
                    w = (long long)s.K * s.C * s.R * s.S * 4;
    return x < lim && y < lim && w < lim && s.R * s.S <= MAX_TAPS && s.stride <= 4 && s.H + s.pad + s.R <= 8192 && s.W + s.pad + s.S <= 8192 &&
           (long long)s.P * s.stride <= 8192 && (long long)s.Q * s.stride <= 8192;
}

// The wave kernel's shape for forward or backward-data, or -1: whole 16-byte chunks of channels (of backward-data's filter too),
// and less modelled time than tile `other`.  Chosen so, of those 260 NHWC layers forward runs 1.18 times as fast
// (1.19 below 7 us, 1.09 above 40), backward-data 1.19; strided backward-data, whose classes differ in length, must gain more.
// NCHW problems pay for the launch that copies their operands, the copies (3 TB/s) and, where planes are no whole groups of four
// pixels, results that leave one by one: of 440 layers forward takes them in 190 and runs those 1.37 times as fast, dx 1.34 (strided included).
int wave_rows(const ConvShape &s, int op, bool nchw, int other, bool masked)
{
    if (s.C % 4 != 0 || (op == OP_BWD && s.K % 4 != 0)) return -1;
    if (const char *f = getenv("MXC_FORCE_VARIANT")) {
        for (int i = 0; i < N_WAVES; ++i)
            if (!strcmp(f, kWaves[i].name)) return i;
        return -1;
    }
    ++g_plan_searches;
    const long long m = op == OP_FWD ? (long long)s.N * s.P * s.Q : (long long)s.N * s.H * s.W, cols = op == OP_FWD ? s.K : s.C;
    const int taps = op == OP_FWD ? s.R * s.S : ((s.R + s.stride - 1) / s.stride) * ((s.S + s.stride - 1) / s.stride);
    const long long k = (long long)taps * (op == OP_FWD ? s.C : s.K);
    const bool classes = op == OP_BWD && s.stride > 1;
    double most = tile_us(other, op, nchw, m, cols, k, 1, masked) * (classes ? 0.75 : nchw ? 0.93 : 0.95);
    if (nchw) {
        const int RS = s.R * s.S, plane = op == OP_FWD ? s.P * s.Q : s.H * s.W;
        const long long from = op == OP_FWD ? (long long)s.N * s.C * s.H * s.W : (long long)s.N * s.K * s.P * s.Q;
        most -= 3.3 + 0.33 * 4e-6 * (from + (RS > 1 ? (long long)s.K * s.C * RS : 0)) + (classes || plane % 4 != 0 ? 0.22 * 4e-6 * m * cols : 0.0);
        if (op == OP_FWD) most -= 0.00047 * s.N * ((s.C + 63) / 64) * ((s.H * s.W + 63) / 64);
    }
    double best = 0;
    int shape = -1;
    for (int i = 0; i < N_WAVES; ++i) {
        const F32Wave &w = kWaves[i];
        const float *c = w.us[op == OP_FWD ? 0 : 1];
        const int nw = w.kg * w.mg, slots = 160 / (nw * w.ns * (w.mb + w.nb));
        const long long per_cu = ((m + 16 * w.mb * w.mg - 1) / (16 * w.mb * w.mg) * ((cols + 16 * w.nb - 1) / (16 * w.nb)) + 255) / 256;
        const double rounds = (double)((per_cu + slots - 1) / slots), turns = (double)((k + 16 * w.kg - 1) / (16 * w.kg));
        const double t = c[0] + c[1] * per_cu * turns * nw * w.mb * w.nb * 0.01 + c[2] * rounds * turns + c[3] * rounds +
                         c[4] * (masked ? 8e-6 : 4e-6) * m * cols + c[5] * per_cu * w.mb * w.nb * w.mg * 0.1;
        if (shape < 0 || t < best) { best = t; shape = i; }
    }
    return best < most ? shape : -1;
}

// t: a tile of the general kernel, or -1 - (a shape of the wave kernel)
static int run(int op, bool nchw, int t, F32Params &p, long long row_tiles, long long cols, int splits, hipStream_t st)
{
    const int bn = t < 0 ? 16 * (op == OP_WGRAD ? kDwWaves[-1 - t].nb : kWaves[-1 - t].nb) : kTiles[t].bn;
    const long long nt = (cols + bn - 1) / bn;
    if (row_tiles * nt * splits > 0x3FFFFFFFll) return MXC_ERR_SHAPE;
    p.n_tiles = (int)nt;
    p.tiles = (int)(row_tiles * nt);
    p.units = p.tiles * splits;
    const ConvShape &s = p.s;
    p.by_ntiles = FastDiv(p.n_tiles); p.by_tiles = FastDiv(p.tiles);
    p.by_ci = FastDiv(op == OP_BWD ? s.K : s.C); p.by_c = FastDiv(s.C); p.by_rs = FastDiv(s.R * s.S); p.by_s = FastDiv(s.S);
    p.by_pq = FastDiv(s.P * s.Q); p.by_q = FastDiv(s.Q); p.by_p = FastDiv(s.P);
    if (t < 0) return op == OP_WGRAD ? launch_wave_dw_op(-1 - t, p, st) : launch_wave_op(op, nchw, -1 - t, p, st);
    return launch_op(op, nchw, t, p, st);
}

// The tile that runs forward or backward-data, and the wave kernel's shape that runs it instead, or -1.  The calling thread keeps its
// answers: with them the host's part of a call (2x16x16x16 to 32, 3x3) is 0.40 us forward and 0.42 for dx, searched anew 0.62 and 0.67.
struct F32Rows { int tile, wave; };
static F32Rows choose_rows(const ConvShape &s, int op, bool nchw, bool masked)
{
    const auto search = [&] {
        const int tile = plan_rows(s, op).tile;
        return F32Rows{tile, wave_rows(s, op, nchw, tile, masked)};
    };
    if (getenv("MXC_FORCE_VARIANT")) return search();
    struct Key { ConvShape s; int op, nchw, masked; };
    static thread_local PlanCache<Key, F32Rows> cache;
    return cache.get(Key{s, op, nchw, masked}, search);
}

// The wave kernel's shape that runs an NCHW problem on NHWC copies of its operands, or -1: the operands are read in place.
int f32_copies(const ConvShape &s, bool bwd, bool masked) { return choose_rows(s, bwd ? OP_BWD : OP_FWD, true, masked).wave; }

int f32_fwd(const ConvShape &s, bool nchw, int copies, const void *x, const void *w, void *y, hipStream_t st, const char **variant, const PostOp &post)
{
    const F32Rows rows = choose_rows(s, OP_FWD, nchw, false);
    const int wv = nchw ? copies : rows.wave, t = wv >= 0 ? -1 - wv : rows.tile;
    const int bm = wv >= 0 ? 16 * kWaves[wv].mb * kWaves[wv].mg : kTiles[t].bm;
    F32Params p{};
    p.a = (const float *)x; p.b = (const float *)w; p.out = (float *)y;
    p.a_bytes = (unsigned)((long long)s.N * s.C * s.H * s.W * 4);
    p.b_bytes = (unsigned)((long long)s.K * s.C * s.R * s.S * 4);
    p.s = s;
    p.M = s.N * s.P * s.Q;
    p.bias = post.bias; p.relu = post.relu;
    p.outside = s.pad > 0;
    F32Class &c = p.cls[0];
    c.TR = s.R; c.TS = s.S; c.Mh = s.P; c.Mw = s.Q; c.off_h = c.off_w = -s.pad;
    set_divisors(c);
    *variant = wv >= 0 ? kWaves[wv].name : kTiles[t].name;
    return run(OP_FWD, nchw, t, p, ((long long)p.M + bm - 1) / bm, s.K, 1, st);
}

int f32_bwd_data(const ConvShape &s, bool nchw, int copies, const void *dy, const void *w, void *dx, hipStream_t st, const char **variant,
                 const PostOp &post)
{
    const F32Rows rows = choose_rows(s, OP_BWD, nchw, post.mask != nullptr);
    const int wv = nchw ? copies : rows.wave, t = wv >= 0 ? -1 - wv : rows.tile;
    const int bm = wv >= 0 ? 16 * kWaves[wv].mb * kWaves[wv].mg : kTiles[t].bm;
    F32Params p{};
    p.a = (const float *)dy; p.b = (const float *)w; p.out = (float *)dx;
    p.a_bytes = (unsigned)((long long)s.N * s.K * s.P * s.Q * 4);
    p.b_bytes = (unsigned)((long long)s.K * s.C * s.R * s.S * 4);
    p.s = s;
    p.mask = (const float *)post.mask;
    p.outside = s.pad > 0 || s.R > 1 || s.S > 1;
    p.n_cls = s.stride * s.stride;
    long long tiles = 0;
    for (int c = 0; c < p.n_cls; ++c) {
        F32Class &f = p.cls[c];
        f = residue_class(s, c / s.stride, c % s.stride);
        set_divisors(f);
        f.tile0 = (int)tiles;
        tiles += ((long long)s.N * f.Mh * f.Mw + bm - 1) / bm;
    }
    *variant = wv >= 0 ? kWaves[wv].name : kTiles[t].name;
    return run(OP_BWD, nchw, t, p, tiles, s.C, 1, st);
}

// The wave kernel's shape (tile), pixel ranges and their length for backward-weight of an NHWC problem, or splits 0: the plan.  Never
// more ranges than the plan has: the workspace is sized for those.  Of those 260 gradients 1.38 times as fast.
static F32Plan wave_wgrad(const ConvShape &s, const F32Plan &pl)
{
    if (s.C % 4 != 0 || s.K % 4 != 0) return F32Plan{0, 0, 0};
    const long long M = (long long)s.N * s.P * s.Q, cols = (long long)s.C * s.R * s.S;
    auto ranges = [&](int shape, long long want) {
        if (want > pl.splits) want = pl.splits;
        if (want < 1) want = 1;
        const long long span = ((M + want - 1) / want + 15) / 16 * 16;
        return F32Plan{shape, (int)((M + span - 1) / span), (int)span};
    };
    if (const char *f = getenv("MXC_FORCE_WGRAD")) {
        const char *slash = strchr(f, '/');
        const size_t len = slash ? (size_t)(slash - f) : strlen(f);
        for (int i = 0; i < N_DW_WAVES; ++i)
            if (strlen(kDwWaves[i].name) == len && !strncmp(f, kDwWaves[i].name, len)) return ranges(i, slash ? atoi(slash + 1) : 1);
        return F32Plan{0, 0, 0};
    }
    ++g_plan_searches;
    double best = 0.95 * tile_us(pl.tile, OP_WGRAD, false, s.K, cols, pl.span, pl.splits, false);
    F32Plan chosen{0, 0, 0};
    for (int i = 0; i < N_DW_WAVES; ++i) {
        const F32WaveDw &w = kDwWaves[i];
        const long long tiles = ((s.K + 16 * w.mb - 1) / (16 * w.mb)) * ((cols + 16 * w.nb - 1) / (16 * w.nb));
        const int slots = 160 / (w.kg * w.ns * (w.mb + w.nb));
        for (int fill = 64; fill <= 512; fill *= 2) {           // one range, then as many as give 128, 256 and 512 workgroups
            const F32Plan p = ranges(i, fill == 64 ? 1 : fill / tiles);
            const double per_cu = (double)((tiles * p.splits + 255) / 256), rounds = (double)(((long long)per_cu + slots - 1) / slots);
            const double turns = (double)((p.span + 16 * w.kg - 1) / (16 * w.kg)), mb = 4e-6 * s.K * cols;
            const double t = w.us[0] + w.us[1] * per_cu * turns * w.kg * w.mb * w.nb * 0.01 + w.us[2] * rounds * turns + w.us[3] * rounds + w.us[4] * mb +
                             (p.splits > 1 ? w.us[5] + w.us[6] * p.splits * mb : 0.0);
            if (t < best) { best = t; chosen = p; }
        }
    }
    return chosen;
}

// Both answers for backward-weight.  A call asks three times, at up to 7 us a search: the calling thread keeps them (with the wave
// kernel's shape searched for on every call, that layer's call was 0.68 us of host time instead of 0.48).
struct F32Dw { F32Plan plan, wave; };
static F32Dw plan_wgrad(const ConvShape &s)
{
    const auto search = [&] {
        int fs = 0;
        const int ft = forced_tile("MXC_FORCE_WGRAD", &fs);
        const F32Plan pl = search_wgrad(s, ft, fs);
        return F32Dw{pl, wave_wgrad(s, pl)};
    };
    if (getenv("MXC_FORCE_WGRAD")) return search();
    struct Key { long long M; int K, C, R, S; };
    static thread_local PlanCache<Key, F32Dw> cache;
    return cache.get(Key{(long long)s.N * s.P * s.Q, s.K, s.C, s.R, s.S}, search);
}

size_t f32_wgrad_workspace(const ConvShape &s) { return (size_t)plan_wgrad(s).plan.splits * s.K * s.C * s.R * s.S * sizeof(float); }

int f32_wgrad(const ConvShape &s, bool nchw, const void *x, const void *dy, void *dw, float *partial, hipStream_t st, const char **variant)
{
    const F32Dw both = plan_wgrad(s);
    F32Plan pl = both.plan;
    const char *name = kTiles[pl.tile].name;
    int bm = kTiles[pl.tile].bm;
    if (const F32Plan wv = both.wave; !nchw && wv.splits > 0) {
        name = kDwWaves[wv.tile].name;
        bm = 16 * kDwWaves[wv.tile].mb;
        pl = F32Plan{-1 - wv.tile, wv.splits, wv.span};
    }
    F32Params p{};
    p.a = (const float *)dy; p.b = (const float *)x; p.out = pl.splits > 1 ? partial : (float *)dw;
    p.a_bytes = (unsigned)((long long)s.N * s.K * s.P * s.Q * 4);
    p.b_bytes = (unsigned)((long long)s.N * s.C * s.H * s.W * 4);
    p.s = s;
    p.M = s.N * s.P * s.Q;
    p.span = pl.span;
    p.outside = s.pad > 0;
    const long long cols = (long long)s.C * s.R * s.S;
    *variant = name;
    const int rc = run(OP_WGRAD, nchw, pl.tile, p, (s.K + bm - 1) / bm, cols, pl.splits, st);
    if (rc != MXC_OK || pl.splits == 1) return rc;
    return sum_splits(partial, dw, false, s.K * cols, pl.splits, st);
}

}  // namespace mxc
