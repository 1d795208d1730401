// bf16 backward-data of first layers (1 to 4 channels, 3x3 or 5x5 at stride 1): one launch that reads dy once.
//
//     G[y][q][(t,c)] = sum_k dy[y][q][k] * w[k][t][c]        a GEMM of R*S*C columns, 27 for 3x3 on RGB
//     dx[h][v][c]    = sum_t G[h + pad - r][v + pad - s][(t,c)]
//
// Gathered as an implicit GEMM over (tap, k), C columns use a fraction of a matrix instruction and every dy pixel is read R*S
// times through LDS.  Here each dy pixel is multiplied once and what is summed over the taps are the fp32 products in LDS, of which
// a tap outside the image is simply left out.
//
// A workgroup slides down a strip of TW columns: per step its four waves multiply one dy row each (32 pixels, 32 - (S-1) of them
// the strip's own), a ring per wave brings the rows of the steps ahead by direct global->LDS loads, and after a barrier all threads
// sum the four dx rows that are complete.  The filter lies in registers, fetched from the caller's KRSC tensor or the prepared form.
//
// What bounds it: the steps, of which the two barriers, the LDS reads of the taps and the latencies between them are most; dy itself comes
// at 4.2 TB/s.  The ring is never drained: the stores of a step are issued after its loads, and the waits of the next step count them
// as younger operations that may be open still.  (A wave's counter holds loads and stores alike and completion is reported in the order of
// issue: the AMDGPU backend's user guide, memory model of gfx90a and gfx942.)  Products of pixels outside dy are stored as zeros, so that
// the sum needs no condition (conditional reads, which became branches with a wait each, took 73 us where this takes 48).  Measured (us,
// packing + GEMM + compaction -> here): 32x224x224, 64 channels to 3, 3x3 69.8 -> 48.5; 3x115x70, 64 to 3 22.7 -> 5.6; 23x25x25, 112 to 3,
// 5x5 58.5 -> 12.3.
#include "mxc_internal.h"
#include "plan_cache.h"

namespace mxc {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr unsigned OOB = 0x80000000u;   // a buffer offset no operand reaches: loads return zeros, stores go nowhere
constexpr int POS = 32, ROWS = 4;       // dy pixels per strip row, dy rows (waves) per step

struct TapsDxParams {
    const bf16_t *dy, *w, *mask;
    bf16_t *dx;
    unsigned dy_bytes, dx_bytes;
    int P, Q, K, Kr, H, W, pad;
    int strips, segs, rows, units;      // rows: of a segment of a strip
    int w_k, w_c, w_r, w_s, w_0;        // element (k, r, s, c) of w lies at w_0 + k*w_k + r*w_r + s*w_s + c*w_c
};

template <int N> __device__ __forceinline__ void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ void wait_lgkmcnt0() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void step_barrier()
{
    wait_lgkmcnt0();
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

template <int C, int RS> struct TapsDx {
    static constexpr int COLS = RS * RS * C, NCB = (COLS + 15) / 16, PITCH = (COLS + 3) / 4 * 4, TW = POS - (RS - 1), NR = RS - 1 + ROWS;
    static constexpr int NS = 4, ITEM = POS * 32, L = 2, STORES = (ROWS * POS * C + 255) / 256;
    static constexpr int LDS = NR * POS * PITCH * 4 + ROWS * NS * ITEM * 2;
};

// KS: steps of 32 channels of dy
template <int C, int RS, int KS> __global__ __launch_bounds__(64 * ROWS) void taps_dx_kernel(const TapsDxParams p)
{
    using T = TapsDx<C, RS>;
    constexpr int COLS = T::COLS, NCB = T::NCB, PITCH = T::PITCH, TW = T::TW, NR = T::NR, NS = T::NS, ITEM = T::ITEM, L = T::L, STORES = T::STORES;
    static_assert(KS <= NS, "the stores of one step pass between the loads of an item and its wait");
    static_assert(KS * 32 * NCB * 16 * 2 <= NR * POS * PITCH * 4, "the filter is laid out where the products will lie");
    __shared__ __attribute__((aligned(1024))) float prod[NR * POS * PITCH];
    __shared__ __attribute__((aligned(1024))) bf16_t ring[ROWS * NS * ITEM];

    const int tid = threadIdx.x, lane = tid & 63, i = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int per_xcd = (p.units + 7) / 8;
    const int unit = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    if (unit >= p.units) return;
    const int strip = unit % p.strips, rest = unit / p.strips, seg = rest % p.segs, n = rest / p.segs;
    const int h_lo = seg * p.rows, h_hi = min(h_lo + p.rows, p.H), v0 = strip * TW;
    const int y0 = h_lo + p.pad - (RS - 1), q0 = v0 + p.pad - (RS - 1), steps = (h_hi - h_lo + RS - 1 + ROWS - 1) / ROWS;
    const buf_rsrc_t rs_dy = make_buf_rsrc(p.dy, p.dy_bytes);
    const out_rsrc_t rs_dx = make_out_rsrc(p.dx, p.dx_bytes);

    // ---- dy: item (step, 32 channels) of this wave's row; lane l brings chunk (l%4) ^ (l/16) of pixel l/4 of a block of 16 ----------
    const int chunk = ((lane & 3) ^ (lane >> 4)) * 8;
    bf16_t *mine = ring + wave * (NS * ITEM);
    int off[2];
    bool in_row[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const int q = q0 + 16 * b + (lane >> 2);
        in_row[b] = (unsigned)q < (unsigned)p.Q;
        off[b] = (q * p.K + chunk) * 2;
    }
    int it_y = y0 + wave, it_ks = 0, it_left = steps;
    auto issue = [&](bf16_t *dst) __attribute__((always_inline)) {
        const bool row_ok = it_left > 0 && (unsigned)it_y < (unsigned)p.P;
        const unsigned base = (unsigned)((n * p.P + it_y) * p.Q) * (unsigned)(p.K * 2) + (unsigned)(it_ks * 64);
        const bool k_ok = it_ks * 32 + chunk < p.K;
#pragma unroll
        for (int b = 0; b < 2; ++b) lds_dma16(rs_dy, row_ok && k_ok && in_row[b] ? base + (unsigned)off[b] : OOB, dst + b * 512);
        if (++it_ks == KS) { it_ks = 0; it_y += ROWS; --it_left; }
    };
#pragma unroll
    for (int q = 0; q < NS; ++q) issue(mine + q * ITEM);

    // ---- the filter: through LDS into fragments, lane 16*g + i holds channels 8*g .. 8*g + 7 of column i -----------------------------
    {
        bf16_t *lds_w = reinterpret_cast<bf16_t *>(prod);
        constexpr int TOTAL = KS * 32 * NCB * 16;
#pragma unroll 8
        for (int at = tid; at < TOTAL; at += 64 * ROWS) {
            const int k = at / (NCB * 16), col = at % (NCB * 16), t = col / C, c = col % C, r = t / RS, s = t % RS;
            bf16_t v = 0;
            if (k < p.Kr && col < COLS) v = p.w[p.w_0 + k * p.w_k + r * p.w_r + s * p.w_s + c * p.w_c];
            lds_w[(((k >> 5) * NCB + (col >> 4)) * 64 + ((k >> 3) & 3) * 16 + (col & 15)) * 8 + (k & 7)] = v;
        }
    }
    step_barrier();
    bf16x8 fw[KS][NCB];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
        for (int j = 0; j < NCB; ++j) fw[ks][j] = *reinterpret_cast<const bf16x8 *>(reinterpret_cast<bf16_t *>(prod) + ((ks * NCB + j) * 64 + lane) * 8);
    step_barrier();

    const int frag = i * 32 + ((g ^ (i >> 2)) & 3) * 8;
    int slot = 0, row0 = 0;              // ring slot of the next item; product row of the step's first dy row
    for (int t = 0; t < steps; ++t) {
        f32x4 acc[2][NCB];
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int j = 0; j < NCB; ++j) acc[b][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            // younger than the item: the NS - 1 items behind it and, from the second step on, the stores of at least one step
            if (t == 0) wait_vmcnt<L * (NS - 1)>();
            else wait_vmcnt<L * (NS - 1) + STORES>();
            bf16_t *src = mine + slot * ITEM;
            bf16x8 fa[2];
#pragma unroll
            for (int b = 0; b < 2; ++b) fa[b] = *reinterpret_cast<const bf16x8 *>(src + b * 512 + frag);
            wait_lgkmcnt0();
            __builtin_amdgcn_sched_barrier(0);
            issue(src);
            slot = slot + 1 == NS ? 0 : slot + 1;
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int j = 0; j < NCB; ++j) acc[b][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[ks][j], fa[b], acc[b][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        // columns 16*j + 4*g .. + 3 of pixel 16*b + i; a pixel outside dy adds nothing, whatever the filter holds
        int row = row0 + wave;
        row -= row >= NR ? NR : 0;
        const bool y_ok = (unsigned)(y0 + ROWS * t + wave) < (unsigned)p.P;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const bool in = y_ok && (unsigned)(q0 + 16 * b + i) < (unsigned)p.Q;
            float *to = prod + (row * POS + 16 * b + i) * PITCH + 4 * g;
#pragma unroll
            for (int j = 0; j < NCB; ++j) {
                const f32x4 v = in ? acc[b][j] : f32x4{0.f, 0.f, 0.f, 0.f};
                if (16 * j + 12 < PITCH || 16 * j + 4 * g < PITCH) *reinterpret_cast<f32x4 *>(to + 16 * j) = v;
            }
        }
        step_barrier();
#pragma unroll
        for (int it = 0; it < STORES; ++it) {
            const int e = it * 64 * ROWS + tid, rr = e / (POS * C), x = e % (POS * C) / C, c = e % C;
            const int h = h_lo + ROWS * t - (RS - 1) + rr, v = v0 + x;
            const bool ok = rr < ROWS && x < TW && h >= h_lo && h < h_hi && v < p.W;
            const float *from = prod + min(x, TW - 1) * PITCH + c;
            float sum = 0.f;
#pragma unroll
            for (int r = 0; r < RS; ++r) {
                int at = row0 + min(rr, ROWS - 1) - r;      // the step's dy rows are row0 .. row0 + 3, dx row rr needs row0 + rr and the RS - 1 before
                at += at < 0 ? NR : 0;
                at -= at >= NR ? NR : 0;
#pragma unroll
                for (int s = 0; s < RS; ++s) sum += from[at * (POS * PITCH) + (RS - 1 - s) * PITCH + (r * RS + s) * C];
            }
            const unsigned at = (unsigned)(((n * p.H + h) * p.W + v) * C + c);
            if (p.mask != nullptr && ok && !mask_keeps(p.mask + at)) sum = 0.f;
            __builtin_amdgcn_raw_buffer_store_b16((short)f32_to_bf16(sum), rs_dx, (int)(ok ? at * 2u : OOB), 0, 0);
        }
        step_barrier();                              // the rows are read: the next step overwrites the oldest
        row0 += ROWS;
        row0 -= row0 >= NR ? NR : 0;
    }
    wait_vmcnt<0>();
}

const char *const kName = "taps_dx";

template <int C, int RS, int KS> void launch(const TapsDxParams &p, hipStream_t st)
{
    hipLaunchKernelGGL((taps_dx_kernel<C, RS, KS>), dim3((unsigned)((p.units + 7) / 8 * 8)), dim3(64 * ROWS), 0, st, p);
}
template <int C, int RS> void launch_ks(const TapsDxParams &p, hipStream_t st)
{
    switch ((p.K + 31) / 32) {
    case 1: return launch<C, RS, 1>(p, st);
    case 2: return launch<C, RS, 2>(p, st);
    case 3: return launch<C, RS, 3>(p, st);
    default: return launch<C, RS, 4>(p, st);
    }
}
template <int RS> int lds_bytes(int C)
{
    return C == 1 ? TapsDx<1, RS>::LDS : C == 2 ? TapsDx<2, RS>::LDS : C == 3 ? TapsDx<3, RS>::LDS : TapsDx<4, RS>::LDS;
}
template <int RS> void launch_c(int C, const TapsDxParams &p, hipStream_t st)
{
    switch (C) {
    case 1: return launch_ks<1, RS>(p, st);
    case 2: return launch_ks<2, RS>(p, st);
    case 3: return launch_ks<3, RS>(p, st);
    default: return launch_ks<4, RS>(p, st);
    }
}

}  // namespace

const char *taps_dx_name() { return kName; }

// Segments of a strip: each repeats R - 1 rows and its start, which is worth some three steps; as many as let the chip's last round end
// soonest (32 images of 224x224, 3x3 on 3 channels: 8 strips each, so 256 strips on 768 places: three segments).
struct Cut { int strips, segs, rows, steps; long long units, rounds; };
static Cut cut(const ConvShape &s)
{
    ++g_plan_searches;
    const int slots = 256 * (160 * 1024 / (s.R == 3 ? lds_bytes<3>(s.C) : lds_bytes<5>(s.C)));
    Cut best{};
    const int strips = (s.W + POS - s.R) / (POS - (s.R - 1));
    for (int segs = 1; segs <= (s.H + ROWS - 1) / ROWS && segs <= 64; ++segs) {
        Cut c{strips, 0, (s.H + segs - 1) / segs, 0, 0, 0};
        c.segs = (s.H + c.rows - 1) / c.rows;
        c.steps = (c.rows + s.R - 1 + ROWS - 1) / ROWS;
        c.units = (long long)s.N * strips * c.segs;
        c.rounds = (c.units + slots - 1) / slots;
        if (best.units == 0 || c.rounds * (c.steps + 3) < best.rounds * (best.steps + 3)) best = c;
    }
    return best;
}

// Modelled times (us) of this kernel and of the packing, GEMM and compaction it replaces, fitted to 180 layers of up to 0.5 GB of dy, 7-9%
// and 12-17% off.  Of those 3x3 runs 2.99 times as fast as before and takes this kernel in 73 of 77, 5x5 2.65 times in 94 of 103:
// the rest have few channels of dy, large images and a filter of many products per pixel (131x91x91, 40 to 3, 5x5: 71 against 113).
static bool faster(const ConvShape &s, const Cut &c)
{
    const double per_cu = (double)((c.units + 255) / 256), ks = (s.K + 31) / 32, mb = 2e-6 * s.N * s.P * s.Q * s.K;
    const double gflop = 64e-9 * s.N * s.H * ((s.W + 7) / 8) * s.R * (s.S + 7) * s.K;
    if (s.R == 3)
        return 2.85 + per_cu * c.steps * (0.0285 + 0.126 * s.C + 0.063 * ks) + 0.165 * ks * s.C + 0.07 * mb < 6.1 + 2.44 * gflop + 6.42 * ks;
    return 2.05 + c.steps * (0.363 * c.rounds + per_cu * (0.247 * s.C + 0.1 * ks)) + 0.56 * ks * s.C + 0.101 * mb < 1.67 + 1.97 * gflop + 13.4 * ks;
}

// Both answers.  The calling thread keeps them: with up to 64 cuts looked at twice a call, the host's part of dx of 32 images of 224x224
// (3x3, 64 channels to 3) was 1.06 us instead of 0.38.
struct TapsPlan { Cut cut; bool faster; };
static TapsPlan plan(const ConvShape &s)
{
    static thread_local PlanCache<ConvShape, TapsPlan> cache;
    return cache.get(s, [&] {
        const Cut c = cut(s);
        return TapsPlan{c, faster(s, c)};
    });
}

bool taps_dx_faster(const ConvShape &s) { return plan(s).faster; }

bool taps_dx_supported(const ConvShape &s)
{
    const long long lim = 0x7FFF0000ll;
    return s.stride == 1 && s.R == s.S && (s.R == 3 || s.R == 5) && s.C >= 1 && s.C <= 4 && s.K % 8 == 0 && s.K <= 128 &&
           (long long)s.N * s.P * s.Q * s.K * 2 < lim && (long long)s.N * s.H * s.W * s.C * 2 < lim && (long long)s.N * s.H * ((s.W + 27) / 28) < lim;
}

// packed: w is the form igemm_bwd_data_smallc_prepare makes, [8 pixels][4][S + 7 dy columns][R][K], of which its first pixel's
// rows hold the whole filter (dy column S - 1 - s)
int taps_dx(const ConvShape &s, const void *dy, const void *w, bool packed, int packed_cols, void *dx, hipStream_t st, const PostOp &post)
{
    TapsDxParams p{};
    p.dy = (const bf16_t *)dy; p.w = (const bf16_t *)w; p.mask = (const bf16_t *)post.mask; p.dx = (bf16_t *)dx;
    p.dy_bytes = (unsigned)((long long)s.N * s.P * s.Q * s.K * 2);
    p.dx_bytes = (unsigned)((long long)s.N * s.H * s.W * s.C * 2);
    p.P = s.P; p.Q = s.Q; p.K = s.K; p.Kr = real_k(s); p.H = s.H; p.W = s.W; p.pad = s.pad;
    if (packed) { p.w_k = 1; p.w_c = packed_cols * s.R * s.K; p.w_r = s.K; p.w_s = -s.R * s.K; p.w_0 = (s.S - 1) * s.R * s.K; }
    else { p.w_k = s.R * s.S * s.C; p.w_c = 1; p.w_r = s.S * s.C; p.w_s = s.C; p.w_0 = 0; }
    const Cut c = plan(s).cut;
    p.strips = c.strips; p.segs = c.segs; p.rows = c.rows; p.units = (int)c.units;
    if (s.R == 3) launch_c<3>(s.C, p, st);
    else launch_c<5>(s.C, p, st);
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
}

}  // namespace mxc
