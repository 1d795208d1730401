// bf16 backward-weight for filters of 3 or 5 columns at stride 1 whose output rows are as wide as the input's.
//
//     dw[k][r][s][c] = sum_m dy[m][k] * x[m + (r,s)][c],   m = (n,p,q)
//
// wgrad.hip's tiles take their columns (r,s,c) as they come: x is fetched into LDS once per tap, and the waves' 64x64 products read 1 KB of
// operands from LDS per MFMA, which is all that LDS gives at the full rate of the MFMAs.  Here a wave computes all TS taps of a filter row
// for 32*MI output channels and 32 input channels: one run of pixels of x serves the taps at shifted rows, as in runs.hip, and an
// operand of dy serves TS MFMAs, one of x MI (5 columns, 64 channels: 0.7 KB per MFMA).  Pixels that the shift takes across an image row's end
// are zeros: the lane reads zeros instead.  (A run that ends with the tensor needs nothing else: what lies past its end in a row that
// begins there lies past the tensor.)
//
// A workgroup's waves are WK blocks of output channels, WC of input channels and WP shares of the pixels of each stage, whose sums meet in LDS in
// ascending order at the end.  Tiles lie in LDS in panels of 32 channels, 64 bytes a pixel, so that the four pixel rows of a transposing read
// are in different banks whatever row comes first.
//
// Measured (us with the sum of the pixel ranges, the tile that ran it before -> this kernel): 128x27x27, 5x5, 64 to 192 channels 75 -> 57 (1009
// TFLOP/s, the matrix pipe 0.60 busy); 105x40x56, 3x3, 256 to 192 235 -> 182; 99x72x72, 5x5, 128 to 32 294 -> 181; 70x40x77, 3x3, 176 to 32 78 -> 40; 163x19x19, 3x3,
// 224 to 144 71 -> 52.  64x28x28, 3x3, 512 to 512 203 -> 213: whole 256x256 tiles stay the faster ones there, and the wave
// kernel below some 12 us.
#include <stdlib.h>
#include <string.h>

#include <type_traits>
#include <utility>

#include "mxc_internal.h"

namespace mxc {

namespace {

typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef bf16x4 __attribute__((address_space(3))) * lds_bf16x4_ptr;

constexpr unsigned OOB = 0x80000000u;   // a buffer offset no operand reaches: the load returns zeros
constexpr int ROW = 64;                 // bytes of a pixel in a panel
constexpr int RPL = 16;                 // pixels that one wave-wide load fills

struct RunDwParams {
    const bf16_t *x, *dy;
    float *partial;      // [splits][K][ncols]
    int H, W, P, Q, C, K, R, pad, M;      // M: positions, rows of W
    int c_tiles, tiles, n_wg, span, rows, ncols;
    int step_p, step_q;  // a stage's pixels as images (in step_off alone), rows and columns, and as bytes of x
    unsigned step_off, dy_step, dy_wrap;   // ... of dy, and from a row's last position to the next row's first
    int inc0, inc1;      // 16 pixels, and those from a wave's second k-step to the next stage's first, modulo W
    unsigned x_bytes, dy_bytes;
};

template <int N> __device__ __forceinline__ void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ void wait_lgkmcnt0() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void pin() { __builtin_amdgcn_sched_barrier(0); }
__device__ __forceinline__ void ring_barrier() { pin(); __builtin_amdgcn_s_barrier(); pin(); }
template <int I> using IC = std::integral_constant<int, I>;
template <class F, int... I> __device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>) { (f(IC<I>{}), ...); }
template <int N, class F> __device__ __forceinline__ void static_for(F &&f) { static_for_impl(f, std::make_integer_sequence<int, N>{}); }

// IN: no padding, and dy rows of Q = W - TS + 1 (layers in space-to-depth form).  The positions are x's, rows of W; tap s reads s further on, and the
// last TS - 1 positions of a row have neither dy nor, so that nothing is multiplied with what is not there, x.
template <int MI, int TS, bool IN, int WK, int WC, int WP, int NS>
__global__ __launch_bounds__(64 * WK * WC * WP, 2) void run_dw_kernel(const RunDwParams p)
{
    constexpr int NW = WK * WC * WP, HALO = IN ? 0 : TS / 2, BP = 32 * WP;
    constexpr int NKP = MI * WK, NCP = WC;                         // panels
    constexpr int GROUPS = BP / RPL, SETS = NW / GROUPS;           // a wave loads pixels 16*(wave % GROUPS) ... of every SETS-th panel
    constexpr int DY_LD = (NKP + SETS - 1) / SETS, X_LD = (NCP + SETS - 1) / SETS, L = DY_LD + X_LD + 1;
    constexpr int DY_PANEL = BP * ROW, X_PANEL = (BP + RPL) * ROW, X_AT = NKP * DY_PANEL, Z_AT = X_AT + NCP * X_PANEL;
    constexpr int SLOT = Z_AT + 1280;                              // zeros: 16 pixels and a row, what a lane's two k-steps span
    constexpr int SCRATCH = NS * SLOT;                             // where loads of no panel go
    constexpr int STAGING = 2 * NW * 4096;                         // two 32x32 blocks of each wave
    constexpr int LDS = SCRATCH + 1024 > STAGING ? SCRATCH + 1024 : STAGING;
    static_assert(GROUPS <= NW && NW % GROUPS == 0 && NCP <= NW && NS >= 2 && L * (NS - 1) < 64, "config");
    static_assert(LDS <= 160 * 1024, "LDS");
    __shared__ __attribute__((aligned(1024))) char smem[LDS];

    const int per_xcd = (p.n_wg + 7) / 8, logical = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);     // tiles of one range of pixels: one L2
    if (logical >= p.n_wg) return;
    const int tile = logical % p.tiles, z = logical / p.tiles;
    const int c0 = tile % p.c_tiles * 32 * WC, t2 = tile / p.c_tiles, r = t2 % p.R, k0 = t2 / p.R * 32 * NKP;
    const int m_begin = z * p.span, m_end = min(m_begin + p.span, p.M);
    const int stages = (m_end - m_begin + BP - 1) / BP;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wp = wave % WP, wc = wave / WP % WC, wk = wave / WP / WC;
    for (int i = tid; i < NS * 80; i += 64 * NW) *reinterpret_cast<float4 *>(smem + i / 80 * SLOT + Z_AT + i % 80 * 16) = make_float4(0.f, 0.f, 0.f, 0.f);

    // ---- loads: lane l brings chunk l%4 of pixel l/4 -------------------------------------------------------
    const buf_rsrc_t rs_x = make_buf_rsrc(p.x, p.x_bytes), rs_dy = make_buf_rsrc(p.dy, p.dy_bytes);
    const int sub = lane >> 2, chunk = lane & 3, group = wave % GROUPS, set = wave / GROUPS;
    const int px2 = p.C * 2, k2 = p.K * 2;
    // dy of the lane's position; past the tensor's end the load returns zeros
    const int dy_m = m_begin + group * RPL + sub, dy_row = IN ? (int)((unsigned)dy_m / (unsigned)p.W) : 0;
    int dy_q = IN ? dy_m - dy_row * p.W : 0;
    unsigned dy_off = (unsigned)(IN ? dy_row * p.Q + dy_q : dy_m) * (unsigned)k2;
    unsigned dy_col[DY_LD], x_col[X_LD], e_col;
#pragma unroll
    for (int i = 0; i < DY_LD; ++i) {
        const int k = k0 + (set + SETS * i) * 32 + chunk * 8;
        dy_col[i] = set + SETS * i < NKP && k < p.K ? (unsigned)(k * 2) : OOB;
    }
    auto channel = [&](int panel) __attribute__((always_inline)) {
        const int c = c0 + panel * 32 + chunk * 8;
        return panel < NCP && c < p.C ? (unsigned)(c * 2) : OOB;
    };
#pragma unroll
    for (int i = 0; i < X_LD; ++i) x_col[i] = channel(set + SETS * i);
    e_col = channel(wave);
    // x: pixel (n, p + r - pad, q) of position m - HALO, walked by additions
    struct Pos { int h, q; unsigned off; } xp, ep;
    auto place = [&](int m) __attribute__((always_inline)) {
        // positions are counted from the image before: m may be up to HALO before the first; what lies before or past the tensor has an offset beyond its end
        const unsigned mm = (unsigned)(m + p.P * p.W), t = mm / (unsigned)p.W;
        const int n = (int)(t / (unsigned)p.P) - 1;
        Pos o;
        o.q = (int)(mm - t * (unsigned)p.W);
        o.h = (int)(t - (unsigned)(n + 1) * (unsigned)p.P) + r - p.pad;
        o.off = (unsigned)(((n * p.H + o.h) * p.W + o.q) * px2);
        return o;
    };
    xp = place(m_begin - HALO + group * RPL + sub);
    ep = place(m_begin - HALO + BP + sub);
    const int row2 = p.W * px2, skip2 = (p.H - p.P) * row2, h_end = p.P + r - p.pad;
    auto advance = [&](Pos &o) __attribute__((always_inline)) {
        o.q += p.step_q;
        const bool c = o.q >= p.W;
        o.q -= c ? p.W : 0;
        o.h += p.step_p + (c ? 1 : 0);
        const bool next = o.h >= h_end;
        o.h -= next ? p.P : 0;
        o.off += p.step_off + (next ? (unsigned)skip2 : 0u);
    };
    unsigned va[L];
    auto addr_task = [&](auto t) __attribute__((always_inline)) {
        constexpr int Tk = decltype(t)::value;
        if constexpr (Tk < DY_LD) {
            va[Tk] = (dy_col[Tk] & OOB) || (IN && dy_q >= p.Q) ? OOB : dy_off + dy_col[Tk];
            if constexpr (Tk + 1 == DY_LD) {
                dy_off += p.dy_step;
                if constexpr (IN) {
                    dy_q += p.step_q;
                    const bool c = dy_q >= p.W;
                    dy_q -= c ? p.W : 0;
                    dy_off -= c ? p.dy_wrap : 0u;
                }
            }
        } else if constexpr (Tk + 1 < L) {
            va[Tk] = (unsigned)xp.h < (unsigned)p.H ? (x_col[Tk - DY_LD] & OOB ? OOB : xp.off + x_col[Tk - DY_LD]) : OOB;
            if constexpr (Tk + 2 == L) advance(xp);
        } else {
            va[Tk] = (unsigned)ep.h < (unsigned)p.H ? (e_col & OOB ? OOB : ep.off + e_col) : OOB;
            advance(ep);
        }
    };
    auto load_task = [&](auto t, int slot) __attribute__((always_inline)) {
        constexpr int Tk = decltype(t)::value;
        if constexpr (Tk < DY_LD) {
            const int panel = set + SETS * Tk;
            lds_dma16(rs_dy, va[Tk], smem + (panel < NKP ? slot * SLOT + panel * DY_PANEL + group * RPL * ROW : SCRATCH));
        } else if constexpr (Tk + 1 < L) {
            const int panel = set + SETS * (Tk - DY_LD);
            lds_dma16(rs_x, va[Tk], smem + (panel < NCP ? slot * SLOT + X_AT + panel * X_PANEL + group * RPL * ROW : SCRATCH));
        } else lds_dma16(rs_x, va[Tk], smem + (wave < NCP ? slot * SLOT + X_AT + wave * X_PANEL + BP * ROW : SCRATCH));
    };

    // ---- operand fetches: 16-lane group g, lane j of it addresses 4 channels of pixel j/4 ---------------------
    const int g = lane >> 4, j16 = lane & 15;
    const int tr_row = wp * 32 + (g >> 1) * 8 + (j16 >> 2), tr_byte = ((g & 1) * 16 + (j16 & 3) * 4) * 2;
    const int a_at = wk * MI * DY_PANEL + tr_row * ROW + tr_byte, b_at = X_AT + wc * X_PANEL + tr_row * ROW + tr_byte;
    int q_lo = (int)((unsigned)(m_begin + tr_row) % (unsigned)p.W), q_hi = (int)((unsigned)(m_begin + tr_row + 4) % (unsigned)p.W);
    auto walk = [&](int by) __attribute__((always_inline)) {
        q_lo += by; q_lo -= q_lo >= p.W ? p.W : 0;
        q_hi += by; q_hi -= q_hi >= p.W ? p.W : 0;
    };
    auto read8 = [&](int slot, int lo, int hi, int off) __attribute__((always_inline)) {
        const bf16x4 l = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(smem + slot * SLOT + off + lo));
        const bf16x4 h = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(smem + slot * SLOT + off + hi));
        return __builtin_shufflevector(l, h, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    auto read_a = [&](int slot, int ks, int i) __attribute__((always_inline)) { return read8(slot, a_at + i * DY_PANEL, a_at + i * DY_PANEL + 4 * ROW, ks * 16 * ROW); };
    auto read_b = [&](int slot, int ks, auto s) __attribute__((always_inline)) {
        constexpr int D = decltype(s)::value - HALO;
        const int at = b_at + (D + HALO) * ROW;
        if constexpr (!IN && D == 0) return read8(slot, at, at + 4 * ROW, ks * 16 * ROW);
        if constexpr (IN) return read8(slot, q_lo < p.Q ? at : Z_AT + tr_byte, q_hi < p.Q ? at + 4 * ROW : Z_AT + tr_byte, ks * 16 * ROW);
        const bool lo = D < 0 ? q_lo >= -D : q_lo < p.W - D, hi = D < 0 ? q_hi >= -D : q_hi < p.W - D;
        return read8(slot, lo ? at : Z_AT + tr_byte, hi ? at + 4 * ROW : Z_AT + tr_byte, ks * 16 * ROW);
    };

    f32x16 acc[MI][TS];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int s = 0; s < TS; ++s)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][s][e] = 0.f;

    // ---- pipeline: two k-steps of 16 pixels per stage; a tap's operand of the next k-step is fetched when its MFMAs have issued --------
    static_for<NS>([&](auto s) __attribute__((always_inline)) {
        static_for<L>([&](auto t) __attribute__((always_inline)) { addr_task(t); });
        static_for<L>([&](auto t) __attribute__((always_inline)) { load_task(t, decltype(s)::value); });
    });
    wait_lgkmcnt0();                  // the zeros
    wait_vmcnt<L * (NS - 1)>();
    ring_barrier();
    bf16x8 a0[MI], a1[MI], b[TS];
#pragma unroll
    for (int i = 0; i < MI; ++i) a0[i] = read_a(0, 0, i);
    static_for<TS>([&](auto s) __attribute__((always_inline)) { b[decltype(s)::value] = read_b(0, 0, s); });

    auto mfmas = [&](const bf16x8 (&a)[MI], auto s) __attribute__((always_inline)) {
        constexpr int S = decltype(s)::value;
#pragma unroll
        for (int i = 0; i < MI; ++i) acc[i][S] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[S], acc[i][S], 0, 0, 0);
    };
    constexpr int MEET = TS / 2;      // the taps of the second k-step before the barrier: their MFMAs hide the fetches of the others
    auto run_stage = [&](auto sl) __attribute__((always_inline)) {
        constexpr int S0 = decltype(sl)::value, S1 = (S0 + 1) % NS;
        walk(p.inc0);
#pragma unroll
        for (int i = 0; i < MI; ++i) a1[i] = read_a(S0, 1, i);
        static_for<TS>([&](auto s) __attribute__((always_inline)) {
            constexpr int S = decltype(s)::value;
            mfmas(a0, s);
            b[S] = read_b(S0, 1, s);
            constexpr int t0 = S * L / TS, t1 = (S + 1) * L / TS;
            static_for<t1 - t0>([&](auto t) __attribute__((always_inline)) { addr_task(IC<t0 + decltype(t)::value>{}); });
            pin();
        });
        static_for<MEET>([&](auto s) __attribute__((always_inline)) { mfmas(a1, s); pin(); });
        wait_lgkmcnt0();              // every operand of this slot is in registers
        wait_vmcnt<L * (NS - 2)>();   // the next stage's have landed
        ring_barrier();
        walk(p.inc1);
#pragma unroll
        for (int i = 0; i < MI; ++i) a0[i] = read_a(S1, 0, i);
        static_for<TS - MEET>([&](auto d) __attribute__((always_inline)) {
            constexpr int D = decltype(d)::value;
            mfmas(a1, IC<MEET + D>{});
            constexpr int r0 = D * TS / (TS - MEET), r1 = (D + 1) * TS / (TS - MEET);       // taps whose operands are free by then: r1 <= MEET + D + 1
            static_for<r1 - r0>([&](auto t) __attribute__((always_inline)) { constexpr int S = r0 + decltype(t)::value; b[S] = read_b(S1, 0, IC<S>{}); });
            constexpr int t0 = D * L / (TS - MEET), t1 = (D + 1) * L / (TS - MEET);
            static_for<t1 - t0>([&](auto t) __attribute__((always_inline)) { load_task(IC<t0 + decltype(t)::value>{}, S0); });
            pin();
        });
    };
    int kt = 0;
    for (; kt + NS <= stages; kt += NS) static_for<NS>([&](auto s) __attribute__((always_inline)) { run_stage(s); });
    const int rem = stages - kt;
    if (rem >= 1) run_stage(IC<0>{});
    if constexpr (NS > 2) if (rem >= 2) run_stage(IC<1>{});
    if constexpr (NS > 3) if (rem >= 3) run_stage(IC<2>{});
    wait_vmcnt<0>();                  // the loads past the last stage
    wait_lgkmcnt0();
    __syncthreads();                  // LDS is free

    // ---- the pixel shares' sums meet block by block; a wave stores 32/WP rows of each -----------------------
    float *out = p.partial + (size_t)z * p.K * p.ncols;
    constexpr int RW = 32 / WP, NQ = RW * 8 / 64 > 0 ? RW * 8 / 64 : 1;
    static_for<MI * TS>([&](auto bi) __attribute__((always_inline)) {
        constexpr int B = decltype(bi)::value, I = B / TS, S = B % TS;
        float *stg = reinterpret_cast<float *>(smem + (B & 1) * NW * 4096);
        float *mine = stg + wave * 1024;
#pragma unroll
        for (int e = 0; e < 16; ++e) mine[(8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)) * 32 + (lane & 31)] = acc[I][S][e];
        __syncthreads();              // (the other half of the staging area is being read meanwhile; this one was, two blocks ago)
        const float *first = stg + (wave - wp) * 1024;
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int idx = q * 64 + lane, row = wp * RW + idx / 8, c4 = idx % 8;
            if (idx < RW * 8) {
                float4 v = *reinterpret_cast<const float4 *>(first + row * 32 + c4 * 4);
#pragma unroll
                for (int w = 1; w < WP; ++w) {
                    const float4 u = *reinterpret_cast<const float4 *>(first + w * 1024 + row * 32 + c4 * 4);
                    v.x += u.x; v.y += u.y; v.z += u.z; v.w += u.w;
                }
                const int k = k0 + (wk * MI + I) * 32 + row, c = c0 + wc * 32 + c4 * 4;
                if (k < p.rows && c < p.C) *reinterpret_cast<float4 *>(out + (size_t)k * p.ncols + (r * TS + S) * p.C + c) = v;
            }
        }
    });
}

// Of the shapes for 5 columns four hold more than 256 registers and keep some that the loop does not touch in scratch (128x32 six, 256x32 two,
// 128x64 and 256x64 one), written before it and read after it; their times below are with that.
// A shape and its time model (us, fitted to 340 layers of 0.6 to 400 GFLOP in up to five ranges each; 2 to 6% off, and the choice takes 0.3%
// more than the fastest): launch, a stage's MFMAs and its own time on the CU with most tiles, their results, a second launch and the partial
// tensors it adds, tiles, dw.
struct RunDwShape { int mi, wk, wc, wp; const char *name; float fixed, tap, stage, block, sum, parts, tile, out; };
const RunDwShape kShapes[] = {
    {1, 1, 2, 4, "wgrad_run_32x64", 2.2f, 0.0454f, 0.322f, 0.363f, 2.14f, 0.525f, 1.4f, 0.152f},
    {2, 1, 2, 4, "wgrad_run_64x64", 3.25f, 0.0907f, 0.328f, 0.224f, 1.71f, 0.589f, 1.65f, 0.135f},
    {2, 2, 1, 4, "wgrad_run_128x32", 3.24f, 0.128f, 0.283f, 0.292f, 1.48f, 0.676f, 0.826f, 0.162f},
    {2, 2, 2, 2, "wgrad_run_128x64", 3.58f, 0.0977f, 0.221f, 0.354f, 1.43f, 0.562f, 1.7f, 0.0942f},
    {2, 4, 2, 1, "wgrad_run_256x64", 4.7f, 0.101f, 0.197f, 0.28f, 1.63f, 0.451f, 1.93f, 0.124f},
    {3, 1, 2, 4, "wgrad_run_96x64", 4.17f, 0.248f, 0.f, 0.265f, 0.913f, 0.655f, 1.14f, 0.0475f},
    {3, 2, 2, 2, "wgrad_run_192x64", 4.27f, 0.221f, 0.f, 0.379f, 1.12f, 0.57f, 0.911f, 0.025f},
    {1, 1, 4, 2, "wgrad_run_32x128", 3.57f, 0.0506f, 0.263f, 0.347f, 2.f, 0.501f, 1.42f, 0.104f},
    {2, 1, 4, 2, "wgrad_run_64x128", 3.87f, 0.0936f, 0.223f, 0.303f, 1.63f, 0.567f, 1.29f, 0.132f},
    {2, 4, 1, 2, "wgrad_run_256x32", 4.55f, 0.0764f, 0.41f, 0.325f, 1.02f, 0.625f, 0.765f, 0.178f},
};
constexpr int N_SHAPES = sizeof(kShapes) / sizeof(kShapes[0]);

template <int TS, bool IN>
void launch(int shape, const RunDwParams &p, hipStream_t st)
{
    const dim3 grid((unsigned)((p.n_wg + 7) / 8 * 8)), block(512);
    switch (shape) {
    case 0: hipLaunchKernelGGL((run_dw_kernel<1, TS, IN, 1, 2, 4, 3>), grid, block, 0, st, p); break;
    case 1: hipLaunchKernelGGL((run_dw_kernel<2, TS, IN, 1, 2, 4, 3>), grid, block, 0, st, p); break;
    case 2: hipLaunchKernelGGL((run_dw_kernel<2, TS, IN, 2, 1, 4, 3>), grid, block, 0, st, p); break;
    case 3: hipLaunchKernelGGL((run_dw_kernel<2, TS, IN, 2, 2, 2, 4>), grid, block, 0, st, p); break;
    case 4: hipLaunchKernelGGL((run_dw_kernel<2, TS, IN, 4, 2, 1, 4>), grid, block, 0, st, p); break;
    case 5: if constexpr (TS == 3) hipLaunchKernelGGL((run_dw_kernel<3, TS, IN, 1, 2, 4, 3>), grid, block, 0, st, p); break;
    case 6: if constexpr (TS == 3) hipLaunchKernelGGL((run_dw_kernel<3, TS, IN, 2, 2, 2, 4>), grid, block, 0, st, p); break;
    case 7: hipLaunchKernelGGL((run_dw_kernel<1, TS, IN, 1, 4, 2, 4>), grid, block, 0, st, p); break;
    case 9: hipLaunchKernelGGL((run_dw_kernel<2, TS, IN, 4, 1, 2, 4>), grid, block, 0, st, p); break;
    case 8: hipLaunchKernelGGL((run_dw_kernel<2, TS, IN, 1, 4, 2, 4>), grid, block, 0, st, p); break;
    }
}

}  // namespace

const char *run_dw_name(int shape) { return shape >= 0 && shape < N_SHAPES ? kShapes[shape].name : nullptr; }

bool run_dw_applicable(const WgradGeom &g)
{
    const long long M = (long long)g.N * g.P * g.W;
    return (((g.TS == 3 || g.TS == 5) && g.Q == g.W && g.pad == g.TS / 2) || (g.TS == 3 && g.Q == g.W - 2 && g.pad == 0)) && g.stride == 1 && g.run == g.pix && g.pix % 8 == 0 && g.K % 8 == 0 &&
           M + (long long)g.P * g.W + 2048 < 0x7FFFFFFFll;
}

bool run_dw_has(int shape, int columns) { return columns == 3 || (columns == 5 && kShapes[shape].mi < 3); }

// ranges: at most so many; what comes of them and their length
int run_dw_ranges(int shape, long long M, int ranges, int *span)
{
    const long long bp = 32 * kShapes[shape].wp, most = (M + bp - 1) / bp;
    long long r = ranges < 1 ? 1 : ranges < most ? ranges : most;
    *span = (int)(((M + r - 1) / r + bp - 1) / bp * bp);
    return (int)((M + *span - 1) / *span);
}

// What a dw of so many MB costs besides, where its order is not the columns' (copies): the pass that sums its ranges finds every place, and of one
// range it is a pass that the wave kernel does without (4 images of 14x14, 491 to 300 channels, 3x3: 24 us).
double dw_places_us(int ranges, double mb) { return ranges == 1 ? 3 + 4 * mb : mb; }

int run_dw_best(const WgradGeom &g, int most_ranges, bool copies, int *ranges, int *span, double *us)
{
    const long long M = (long long)g.N * g.P * g.W;
    const double mb = 4e-6 * g.K * g.TR * g.TS * g.run;
    int best = -1;
    for (int i = 0; i < N_SHAPES; ++i) {
        const RunDwShape &s = kShapes[i];
        if (!run_dw_has(i, g.TS)) continue;
        const long long tiles = (long long)((g.K + 32 * s.mi * s.wk - 1) / (32 * s.mi * s.wk)) * g.TR * ((g.pix + 32 * s.wc - 1) / (32 * s.wc));
        for (int want = 1, last = 0; want <= most_ranges && tiles * want <= 4096 + tiles; ++want) {
            int len = 0;
            const int n = run_dw_ranges(i, M, want, &len);
            if (n == last) continue;
            last = n;
            const double rounds = (double)((tiles * n + 255) / 256), stages = (double)(len / (32 * s.wp));
            const double t = s.fixed + rounds * stages * (s.tap * g.TS + s.stage) + s.block * rounds * g.TS * s.mi + (n > 1 ? s.sum + s.parts * n * mb : 0) +
                             s.tile * tiles * n / 256.0 + s.out * mb + (copies ? dw_places_us(n, mb) : 0);
            if (best < 0 || t < *us) { best = i; *us = t; *ranges = n; *span = len; }
        }
    }
    return best;
}

int run_dw_launch(int shape, const WgradGeom &g, int ranges, int span, const void *x, const void *dy, float *out, int rows, hipStream_t st)
{
    if (!run_dw_applicable(g) || shape < 0 || shape >= N_SHAPES || !run_dw_has(shape, g.TS)) return MXC_ERR_UNSUPPORTED;
    const RunDwShape &s = kShapes[shape];
    RunDwParams p{};
    p.x = (const bf16_t *)x; p.dy = (const bf16_t *)dy; p.partial = out;
    p.H = g.H; p.W = g.W; p.P = g.P; p.Q = g.Q; p.C = g.pix; p.K = g.K; p.R = g.TR; p.pad = g.pad; p.M = g.N * g.P * g.W;
    p.c_tiles = (g.pix + 32 * s.wc - 1) / (32 * s.wc);
    const long long tiles = (long long)p.c_tiles * g.TR * ((g.K + 32 * s.mi * s.wk - 1) / (32 * s.mi * s.wk));
    if (tiles * ranges > 0x3FFFFFFFll) return MXC_ERR_SHAPE;
    p.tiles = (int)tiles; p.n_wg = (int)tiles * ranges; p.span = span; p.rows = rows; p.ncols = g.TR * g.TS * g.run;
    const int bp = 32 * s.wp;
    p.step_q = bp % g.W; p.step_p = bp / g.W % g.P;
    p.step_off = (unsigned)((bp + (long long)(bp / g.W / g.P) * (g.H - g.P) * g.W) * g.pix * 2);
    p.dy_step = (unsigned)((bp / g.W * g.Q + bp % g.W) * (long long)g.K * 2); p.dy_wrap = (unsigned)((g.W - g.Q) * g.K * 2);
    p.inc0 = 16 % g.W; p.inc1 = (bp - 16) % g.W;
    p.x_bytes = (unsigned)((long long)g.N * g.H * g.W * g.pix * 2);
    p.dy_bytes = (unsigned)((long long)g.N * g.P * g.Q * g.K * 2);
    if (g.Q != g.W) launch<3, true>(shape, p, st);
    else if (g.TS == 3) launch<3, false>(shape, p, st);
    else launch<5, false>(shape, p, st);
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
}

}  // namespace mxc
