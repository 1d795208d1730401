// bf16 implicit GEMM for filters of 3 or 5 columns at stride 1 whose output rows are as wide as the input's.
//
//     Out[m][co] = sum_{r,s,ci} In[pixel(m) + (r,s)][ci] * Wm[co][(r*TS + s)*Ci + ci]
//
// What bounds igemm.hip's tiles on such layers is what they bring into LDS: a tile's rows are fetched once per tap, and where a tile has
// few columns those bytes (128x64: 96 bytes a clock and CU at the full rate of the MFMAs, of 64 that the cache gives) are more than
// the MFMAs hide.  Here the taps of one filter row share their pixels: where Q = W, GEMM row m reads at tap (r, s) what row m + s - pad reads
// at (r, pad), so one run of BM + TS - 1 consecutive pixels, brought into LDS once per (channel block, filter row), serves TS taps at
// shifted rows.  Pixels that the shift takes across an image row's end are zeros: the lane reads a row of zeros instead, at an
// address worked out once per tile.  A stage is a filter row's taps over 32 channels: 2*TS k-steps, with one barrier.
//
// Measured (us, the kernel that ran it before -> this one): 128x27x27, 5x5, 64 to 192 channels forward 70 -> 61 (935 TFLOP/s; 72 -> 65 on a
// slower box), its dx 77 -> 58; 56x63x63, 3x3, 160 to 80 95 -> 62; 206x21x21, 5x5, 288 to 24 100 -> 46; 101x49x49, 3x3, dx of 32 to 144 60 ->
// 43; 252x31x31, 3x3, dx of 56 to 224 118 -> 78.  What bounds it then are the operand fetches of narrow tiles (256x64: 1 KB per MFMA) and,
// for wide ones, the MFMAs (1100 to 1160 TFLOP/s, as igemm.hip's large tiles, which stay the faster ones there).  Counters: the matrix pipe
// is 0.37 to 0.62 busy; LDS bank conflicts cost 0.4 (images of 112 columns) to 1.35 cycles (27) per active one: lanes that read zeros read
// one address.
#include <stdlib.h>
#include <string.h>

#include <type_traits>
#include <utility>

#include "mxc_internal.h"

namespace mxc {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef short s16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef bf16x4 __attribute__((address_space(3))) * lds_bf16x4_ptr;

constexpr unsigned OOB = 0x80000000u;   // a buffer offset no operand reaches: the load returns zeros
constexpr int CB = 32;                  // channels per stage
constexpr int ROW = CB * 2;             // bytes of a row in LDS: four 16-byte chunks, chunk c of row r at c ^ ((r >> 2) % 4) (any 16
                                        // consecutive rows of one chunk lie in 64 different banks, whatever row comes first)
constexpr int RPL = 16;                 // rows that one wave-wide load fills

template <int N> __device__ __forceinline__ void wait_vmcnt() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ void wait_lgkmcnt0() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }
__device__ __forceinline__ void pin() { __builtin_amdgcn_sched_barrier(0); }
__device__ __forceinline__ void ring_barrier() { pin(); __builtin_amdgcn_s_barrier(); pin(); }
template <int I> using IC = std::integral_constant<int, I>;
template <class F, int... I> __device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>) { (f(IC<I>{}), ...); }
template <int N, class F> __device__ __forceinline__ void static_for(F &&f) { static_for_impl(f, std::make_integer_sequence<int, N>{}); }

template <int BM, int BN, int TS> constexpr int slot_bytes = (BM + RPL + TS * BN) * ROW + 256;      // rows, filter rows of TS taps, a row of zeros
template <int BM, int BN, int TS, int NS> constexpr int lds_bytes = NS * slot_bytes<BM, BN, TS>;
template <int BM, int BN, int TS, int NS, int NW>
constexpr int min_blocks = NW > 4 ? 2 : lds_bytes<BM, BN, TS, NS> <= 53 * 1024 ? 3 : lds_bytes<BM, BN, TS, NS> <= 80 * 1024 ? 2 : 1;      // waves per SIMD

// BM x BN output tile, WR x WC waves, TS filter columns, NS stages in the ring
// BT: backward-data from the KRSC filter itself, whose row (k, r, s) is a run of output columns: a tap's tile is panels of 32 columns, 32
// rows of 64 bytes each, fetched with ds_read_b64_tr_b16 (the four rows of one read lie in different banks).  Same products in the same
// order as with the re-packed filter, without the launch that makes it (4 to 5 us).
template <int BM, int BN, int TS, int NS, int WR, int WC, bool BT>
__global__ __launch_bounds__(64 * WR * WC, (min_blocks<BM, BN, TS, NS, WR * WC>)) void run_kernel(const IgemmParams p)
{
    constexpr int NW = WR * WC, NT = 64 * NW;
    constexpr int WM = BM / WR, WN = BN / WC, MI = WM / 32, NI = WN / 32, NMF = MI * NI;
    constexpr int A_ROWS = BM + RPL, A_SZ = A_ROWS * ROW, B_SZ = TS * BN * ROW, SLOT = slot_bytes<BM, BN, TS>;
    constexpr int A_LD = BM / RPL / NW + 1;                        // the last one: rows BM ..., by every wave (the same bytes)
    constexpr int B_LOADS = TS * BN / RPL, B_LD = (B_LOADS + NW - 1) / NW;
    constexpr int L = A_LD + B_LD;
    constexpr int KST = 2 * TS;                                    // MFMA k-steps per stage
    constexpr int HALO = TS / 2;
    static_assert(BM % (RPL * NW) == 0 && BN % 32 == 0 && WM % 32 == 0 && WN % 32 == 0 && NT >= BN, "tile/wave mismatch");
    static_assert(NS >= 2 && NS <= 3 && L * (NS - 1) < 64, "ring");
    constexpr int PW = WN + 8, STAGING = NW * 32 * PW * 2;         // epilogue: 32 rows of each wave, padded by 16 bytes
    static_assert(STAGING + BN * 4 <= NS * SLOT, "the staged results and the bias fit the ring");
    __shared__ __attribute__((aligned(1024))) char smem[NS * SLOT];

    const int units = p.m_tiles * p.n_tiles, per_xcd = (units + 7) / 8;
    const int unit = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);         // each XCD a contiguous range of tiles, column tiles fastest
    if (unit >= units) return;
    const int m0 = unit / p.n_tiles * BM, n0 = unit % p.n_tiles * BN;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wave_m = wave / WC * WM, wave_n = wave % WC * WN;
    if (tid < NS * 16) *reinterpret_cast<float4 *>(smem + (tid >> 4) * SLOT + A_SZ + B_SZ + (tid & 15) * 16) = make_float4(0.f, 0.f, 0.f, 0.f);

    // ---- loads: lane l of load i -> row 16*i + l/4, chunk (l%4) ^ (l/16) -----------------------------------
    const int ld_sub = lane >> 2, ld_chunk = (lane & 3) ^ (lane >> 4);
    const buf_rsrc_t rs_in = make_buf_rsrc(p.in, p.in_bytes), rs_wm = make_buf_rsrc(p.wm, p.wm_bytes);
    const int px2 = p.pix * 2, row2 = p.Wi * px2, Ci2 = p.Ci * 2, Kd2 = p.TR * TS * Ci2;
    int a_off[A_LD], a_h[A_LD];       // byte offset of the row's pixel (of tap row 0), and its image row
    auto place = [&](int i, int m) __attribute__((always_inline)) {
        // m may be up to HALO before the first row: positions are counted from the image before; what lies before or past the tensor has
        // an offset beyond its end as an unsigned number
        const unsigned mm = (unsigned)(m + p.Mh * p.Mw), t = mm / (unsigned)p.Mw;
        const int b = (int)(mm - t * (unsigned)p.Mw), n = (int)(t / (unsigned)p.Mh), a = (int)(t - (unsigned)n * (unsigned)p.Mh);
        a_h[i] = a + p.in_off_h;
        a_off[i] = (((n - 1) * p.Hi + a_h[i]) * p.Wi + b) * px2 + ld_chunk * 16;
    };
    static_for<A_LD>([&](auto i) __attribute__((always_inline)) {
        place(i, m0 - HALO + ld_sub + (decltype(i)::value + 1 < A_LD ? RPL * (wave + NW * decltype(i)::value) : BM));
    });
    unsigned b_off[B_LD];
    [[maybe_unused]] int b_rows = 0;  // BT: bit i: load i brings the second half of a panel's rows
    int b_at[B_LD];                   // where the load's rows lie in the slot
#pragma unroll
    for (int i = 0; i < B_LD; ++i) {
        int idx = wave + NW * i;
        if (idx > B_LOADS - 1) idx = B_LOADS - 1;                 // (the same bytes as another wave)
        if constexpr (BT) {           // half a panel
            const int s = idx / 2 / (BN / 32), co = n0 + idx / 2 % (BN / 32) * 32 + (lane & 3) * 8;
            b_off[i] = co < p.Co ? (unsigned)((((idx & 1) * RPL + ld_sub) * p.TR * TS + s) * p.Co + co) * 2u : OOB;
            b_rows |= (idx & 1) << i;
        } else {
            const int s = idx * RPL / BN, co = n0 + idx * RPL % BN + ld_sub;
            b_off[i] = co < p.Co ? (unsigned)(co * Kd2 + s * Ci2 + ld_chunk * 16) : OOB;
        }
        b_at[i] = A_SZ + idx * RPL * ROW;
    }
    // the stage that addresses are worked out for next: filter row st_r of channel block st_c
    int st_r = 0, st_c2 = 0;          // st_c2: bytes of the channels before the block
    const int step_h2 = p.tstep_h * row2;
    unsigned va[A_LD], vb[B_LD];
    auto addr_task = [&](auto t) __attribute__((always_inline)) {
        constexpr int Tk = decltype(t)::value;
        const bool c_ok = st_c2 + ld_chunk * 16 < Ci2;             // false past the last channel, and so past the last stage
        if constexpr (Tk < A_LD) {
            const int h = a_h[Tk] + st_r * p.tstep_h;
            va[Tk] = c_ok && (unsigned)h < (unsigned)p.Hi ? (unsigned)(a_off[Tk] + st_r * step_h2 + st_c2) : OOB;
        } else {
            if constexpr (BT) {
                const unsigned at = (unsigned)((st_c2 / 2 * p.TR + st_r) * TS * p.Co) * 2u;
                const int rows = p.Ci - st_c2 / 2;                 // of the block that are there: none past the last one
#pragma unroll
                for (int i = 0; i < B_LD; ++i) vb[i] = ld_sub + ((b_rows >> i) & 1) * RPL < rows && !(b_off[i] & OOB) ? b_off[i] + at : OOB;
            } else {
                const unsigned at = (unsigned)(st_r * TS * Ci2 + st_c2);
#pragma unroll
                for (int i = 0; i < B_LD; ++i) vb[i] = c_ok ? b_off[i] + at : OOB;
            }
            const bool wrap = st_r + 1 == p.TR;
            st_r = wrap ? 0 : st_r + 1;
            st_c2 += wrap ? ROW : 0;
        }
    };
    constexpr int N_ADDR = A_LD + 1;
    auto load_task = [&](auto t, int slot) __attribute__((always_inline)) {
        constexpr int Tk = decltype(t)::value;
        if constexpr (Tk < A_LD) lds_dma16(rs_in, va[Tk], smem + slot * SLOT + (Tk + 1 < A_LD ? (wave + NW * Tk) * RPL : BM) * ROW);
        else lds_dma16(rs_wm, vb[Tk - A_LD], smem + slot * SLOT + b_at[Tk - A_LD]);
    };

    // ---- operand fetches ---------------------------------------------------------------------------------
    const int frag_row = lane & 31, frag_kg = lane >> 5;
    int a_at[MI][TS];                 // this lane's first chunk of block i at tap column s, in a slot; the second k-step's is 32 bytes off by XOR
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int row = wave_m + i * 32 + frag_row, q = (int)((unsigned)(m0 + row) % (unsigned)p.Mw);
#pragma unroll
        for (int s = 0; s < TS; ++s) {
            const int shift = s * p.tstep_w + p.in_off_w, at = row + HALO + shift;
            a_at[i][s] = (unsigned)(q + shift) < (unsigned)p.Wi ? at * ROW + ((frag_kg ^ ((at >> 2) & 3)) << 4) : A_SZ + B_SZ + (frag_kg << 4);
        }
    }
    const int tr_at = A_SZ + wave_n * ROW + ((lane >> 5) * 8 + ((lane & 15) >> 2)) * ROW + (((lane >> 4) & 1) * 16 + (lane & 3) * 4) * 2;      // BT
    const int b_lane = A_SZ + (wave_n + frag_row) * ROW + ((frag_kg ^ ((frag_row >> 2) & 3)) << 4);
    struct Frags { bf16x8 a[MI], b[NI]; };
    auto read_task = [&](auto t, Frags &f, int slot, auto k) __attribute__((always_inline)) {
        constexpr int Tk = decltype(t)::value, S = decltype(k)::value / 2, X = (decltype(k)::value & 1) << 5;
        if constexpr (Tk < MI) f.a[Tk] = *reinterpret_cast<const bf16x8 *>(smem + slot * SLOT + (a_at[Tk][S] ^ X));
        else if constexpr (BT) {
            const char *q = smem + slot * SLOT + (S * BN + (Tk - MI) * 32) * ROW + (decltype(k)::value & 1) * 16 * ROW + tr_at;
            const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)q);
            const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(q + 4 * ROW));
            f.b[Tk - MI] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
        } else f.b[Tk - MI] = *reinterpret_cast<const bf16x8 *>(smem + slot * SLOT + (S * BN + (Tk - MI) * 32) * ROW + (b_lane ^ X));
    };
    constexpr int N_READ = MI + NI;
    const float bias_t = (p.bias != nullptr && tid < BN && n0 + tid < p.Cw) ? p.bias[n0 + tid] : 0.f;      // used after the loop

    f32x16 acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    // the MFMAs of a k-step with side tasks between them: the first NFRONT (operand fetches) behind the first half, the rest behind the second
    auto mfma_with = [&](const Frags &f, auto nfront, auto ntask, auto &&task) __attribute__((always_inline)) {
        constexpr int NFRONT = decltype(nfront)::value, NTASK = decltype(ntask)::value;
        constexpr int H1 = NMF > 1 ? NMF / 2 : 1, H2 = NMF - H1 > 0 ? NMF - H1 : 1;
        static_for<NMF>([&](auto s) __attribute__((always_inline)) {
            constexpr int S = decltype(s)::value;
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

    // ---- pipeline: as igemm.hip's, one barrier per stage before its last k-step ----------------------------
    const int stages = p.TR * ((p.Ci + CB - 1) / CB);
    Frags f0, f1;
    static_for<NS>([&](auto s) __attribute__((always_inline)) {
        static_for<N_ADDR>([&](auto t) __attribute__((always_inline)) { addr_task(t); });
        static_for<L>([&](auto t) __attribute__((always_inline)) { load_task(t, decltype(s)::value); });
    });
    wait_lgkmcnt0();                  // the zeros
    wait_vmcnt<L * (NS - 1)>();
    ring_barrier();
    static_for<N_READ>([&](auto t) __attribute__((always_inline)) { read_task(t, f0, 0, IC<0>{}); });
    auto run_stage = [&](auto s) __attribute__((always_inline)) {
        constexpr int S = decltype(s)::value, S1 = (S + 1) % NS;
        static_for<KST - 1>([&](auto k) __attribute__((always_inline)) {
            constexpr int ks = decltype(k)::value;
            Frags &cur = (ks & 1) ? f1 : f0;
            Frags &nxt = (ks & 1) ? f0 : f1;
            constexpr int a0 = ks * N_ADDR / (KST - 1), a1 = (ks + 1) * N_ADDR / (KST - 1);
            mfma_with(cur, IC<N_READ>{}, IC<N_READ + (a1 - a0)>{}, [&](auto t) __attribute__((always_inline)) {
                constexpr int Tk = decltype(t)::value;
                if constexpr (Tk < N_READ) read_task(t, nxt, S, IC<ks + 1>{}); else addr_task(IC<a0 + Tk - N_READ>{});
            });
        });
        wait_lgkmcnt0();              // every operand of this slot is in registers
        wait_vmcnt<L * (NS - 2)>();   // the next stage's have landed
        ring_barrier();
        mfma_with(f1, IC<N_READ>{}, IC<N_READ + L>{}, [&](auto t) __attribute__((always_inline)) {
            constexpr int Tk = decltype(t)::value;
            if constexpr (Tk < N_READ) read_task(t, f0, S1, IC<0>{}); else load_task(IC<Tk - N_READ>{}, S);
        });
    };
    int kt = 0;
    for (; kt + NS <= stages; kt += NS) static_for<NS>([&](auto s) __attribute__((always_inline)) { run_stage(s); });
    const int rem = stages - kt;
    if (rem >= 1) run_stage(IC<0>{});
    if constexpr (NS > 2) if (rem >= 2) run_stage(IC<1>{});
    wait_vmcnt<0>();                  // the zero-fill loads past the last stage
    wait_lgkmcnt0();
    __syncthreads();                  // LDS is free

    // ---- epilogue: as igemm.hip's, through LDS in blocks of 32 rows to 16-byte buffer stores -----------------
    constexpr int CPR = WN / 8, NST = 32 * CPR / 64;
    bf16_t *stg = reinterpret_cast<bf16_t *>(smem) + wave * 32 * PW;
    float *s_bias = reinterpret_cast<float *>(smem + STAGING);
    if (p.bias != nullptr) {
        if (tid < BN) s_bias[tid] = bias_t;
        __syncthreads();
    }
    const out_rsrc_t rs_out = make_out_rsrc(p.out, p.out_bytes), rs_mask = make_out_rsrc(const_cast<bf16_t *>(p.mask), p.mask != nullptr ? p.out_bytes : 0u);
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        unsigned off[NST];
        uint4 mask[NST];
#pragma unroll
        for (int k = 0; k < NST; ++k) {
            const int idx = k * 64 + lane, m = m0 + wave_m + i * 32 + idx / CPR, co = n0 + wave_n + idx % CPR * 8;
            off[k] = m < p.M && co < p.Co ? (unsigned)(m * p.Co + co) * 2u : OOB;
            if (p.mask != nullptr) mask[k] = buffer_load16(rs_mask, off[k]);
        }
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4) {
                float v0 = acc[i][j][4 * g4], v1 = acc[i][j][4 * g4 + 1], v2 = acc[i][j][4 * g4 + 2], v3 = acc[i][j][4 * g4 + 3];
                if (p.bias != nullptr) {
                    const float4 b4 = *reinterpret_cast<const float4 *>(s_bias + wave_n + j * 32 + 8 * g4 + 4 * frag_kg);
                    v0 += b4.x; v1 += b4.y; v2 += b4.z; v3 += b4.w;
                }
                uint2 pk = make_uint2(pack_bf16x2(v0, v1), pack_bf16x2(v2, v3));
                if (p.relu) {         // an integer maximum on the rounded pair
                    pk.x = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2, pk.x), s16x2{0, 0}));
                    pk.y = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(s16x2, pk.y), s16x2{0, 0}));
                }
                *reinterpret_cast<uint2 *>(stg + frag_row * PW + 4 * ((j * 8 + 2 * g4 + frag_kg) ^ ((frag_row >> 3) & 3))) = pk;
            }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int k = 0; k < NST; ++k) {
            const int idx = k * 64 + lane, r = idx / CPR, c = idx % CPR;
            const uint4 u = *reinterpret_cast<const uint4 *>(stg + r * PW + ((c ^ ((r >> 4) & 1)) << 3));
            uint4 v = ((r >> 3) & 1) ? make_uint4(u.z, u.w, u.x, u.y) : u;
            if (p.mask != nullptr) v = mask_bf16x8(v, mask[k]);
            if (p.nt_out) buffer_store16_nt(rs_out, off[k], v);
            else buffer_store16(rs_out, off[k], v);
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

// A shape and its time model (us, fitted to 320 layers of 0.4 to 400 GFLOP, forward and masked dx, 640 GEMMs; 3 to 9% off, and the shape
// chosen takes 1.5% more than the fastest): launch, the CU's share of tile area times taps and stages, the chain of stages of its rounds,
// rounds, area, results and mask, input.
struct RunShape { int bm, bn, waves, most_ts; const char *name; float fixed, work, stage, round, area, out, in; };
const RunShape kShapes[] = {
    {128, 32, 4, 5, "igemm_run_128x32", 2.57f, 0.233f, 0.132f, 0.287f, 1.4f, 0.18f, 0.124f},
    {256, 32, 4, 5, "igemm_run_256x32", 2.96f, 0.189f, 0.117f, 0.668f, 1.27f, 0.192f, 0.195f},
    {128, 64, 4, 5, "igemm_run_128x64", 2.7f, 0.198f, 0.0696f, 1.2f, 0.35f, 0.242f, 0.052f},
    {192, 64, 4, 5, "igemm_run_192x64", 3.37f, 0.175f, 0.0436f, 1.33f, 0.214f, 0.258f, 0.145f},
    {256, 64, 4, 5, "igemm_run_256x64", 3.1f, 0.147f, 0.111f, 2.17f, 0.f, 0.265f, 0.183f},
    {384, 64, 4, 5, "igemm_run_384x64", 3.05f, 0.16f, 0.0306f, 3.83f, 0.f, 0.217f, 0.168f},
    {256, 96, 4, 5, "igemm_run_256x96", 3.13f, 0.167f, 0.0135f, 4.16f, 0.f, 0.2f, 0.0205f},
    {192, 128, 4, 5, "igemm_run_192x128", 3.34f, 0.168f, 0.00117f, 3.59f, 0.f, 0.202f, 0.f},
    {256, 128, 8, 5, "igemm_run_256x128", 1.8f, 0.128f, 0.0328f, 0.f, 1.64f, 0.337f, 0.262f},
    {256, 192, 8, 5, "igemm_run_256x192", 2.07f, 0.13f, 0.f, 0.f, 1.65f, 0.309f, 0.222f},
    {256, 256, 8, 3, "igemm_run_256x256", 2.62f, 0.122f, 0.f, 0.f, 1.37f, 0.309f, 0.32f},
};
constexpr int N_SHAPES = sizeof(kShapes) / sizeof(kShapes[0]);

template <int BM, int BN, int TS, int NS, int WR, int WC>
int launch(IgemmParams p, hipStream_t st, bool bt)
{
    const long long mt = ((long long)p.M + BM - 1) / BM;
    p.n_tiles = (p.Co + BN - 1) / BN;
    if (mt * p.n_tiles > 0x3FFFFFFFll) return MXC_ERR_SHAPE;
    p.m_tiles = (int)mt;
    const int grid = (p.m_tiles * p.n_tiles + 7) / 8 * 8;
    if (bt) hipLaunchKernelGGL((run_kernel<BM, BN, TS, NS, WR, WC, true>), dim3((unsigned)grid), dim3(64 * WR * WC), 0, st, p);
    else hipLaunchKernelGGL((run_kernel<BM, BN, TS, NS, WR, WC, false>), dim3((unsigned)grid), dim3(64 * WR * WC), 0, st, p);
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
}

template <int TS>
int launch_shape(int shape, const IgemmParams &p, hipStream_t st, bool bt)
{
    switch (shape) {
    case 0: return launch<128, 32, TS, 2, 4, 1>(p, st, bt);
    case 1: return launch<256, 32, TS, 2, 4, 1>(p, st, bt);
    case 2: return launch<128, 64, TS, 2, 2, 2>(p, st, bt);
    case 3: return launch<192, 64, TS, 2, 2, 2>(p, st, bt);
    case 4: return launch<256, 64, TS, 2, 4, 1>(p, st, bt);
    case 5: return launch<384, 64, TS, 2, 4, 1>(p, st, bt);
    case 6: return launch<256, 96, TS, 2, 4, 1>(p, st, bt);
    case 7: return launch<192, 128, TS, 2, 2, 2>(p, st, bt);
    case 8: return launch<256, 128, TS, 2, 4, 2>(p, st, bt);
    case 9: return launch<256, 192, TS, 2, 4, 2>(p, st, bt);
    case 10: if constexpr (TS == 3) return launch<256, 256, TS, 2, 2, 4>(p, st, bt);
    }
    return MXC_ERR_UNSUPPORTED;
}

}  // namespace

const char *run_name(int shape) { return shape >= 0 && shape < N_SHAPES ? kShapes[shape].name : nullptr; }

int run_forced(const char *name, const IgemmParams &p)
{
    for (int i = 0; i < N_SHAPES; ++i)
        if (!strcmp(name, kShapes[i].name) && p.TS <= kShapes[i].most_ts) return i;
    return -1;
}

int run_best(long long M, int Co, int Ci, int TR, int TS, bool masked, double *us)
{
    int best = -1;
    for (int i = 0; i < N_SHAPES; ++i) {
        const RunShape &s = kShapes[i];
        if (TS > s.most_ts) continue;
        const int lds = 2 * ((s.bm + RPL + TS * s.bn) * ROW + 256);
        const int fit = 160 * 1024 / lds, slots = s.waves > 4 ? 1 : fit > 3 ? 3 : fit;
        const long long per_cu = ((M + s.bm - 1) / s.bm * ((Co + s.bn - 1) / s.bn) + 255) / 256, rounds = (per_cu + slots - 1) / slots;
        const int stages = TR * ((Ci + CB - 1) / CB);
        const double area = per_cu * s.bm * s.bn / 16384.0;
        const double t = s.fixed + s.work * area * stages * TS + s.stage * rounds * stages + s.round * rounds + s.area * area +
                         (masked ? 2e-6 : 1e-6) * s.out * M * Co + 1e-6 * s.in * M * Ci;
        if (best < 0 || t < *us) { best = i; *us = t; }
    }
    return best;
}

bool run_applicable(const IgemmParams &p)
{
    const long long M = (long long)p.N * p.Mh * p.Mw;
    return (p.TS == 3 || p.TS == 5) && p.in_mul_h == 1 && p.in_mul_w == 1 && p.Mw == p.Wi && p.pix == p.Ci && p.Ci % 8 == 0 && p.Co % 8 == 0 &&
           (p.tstep_w == 1 ? p.in_off_w == -(p.TS / 2) : p.tstep_w == -1 && p.in_off_w == p.TS / 2) && !p.tap_row_inner && p.splits <= 1 && !p.f32_out &&
           p.out_mul_h == 1 && p.out_mul_w == 1 && p.out_off_h == 0 && p.out_off_w == 0 && p.Mh == p.Ho && p.Mw == p.Wo && p.s2d.s == 0 &&
           M + (long long)p.Mh * p.Mw + 512 < 0x7FFFFFFFll && M * p.Co * 2 < 0x7FFF0000ll && (long long)p.N * p.Hi * p.Wi * p.pix * 2 < 0x7FFF0000ll;
}

int run_launch(int shape, IgemmParams p, hipStream_t st, bool bt)
{
    if (!run_applicable(p) || shape < 0 || shape >= N_SHAPES || p.TS > kShapes[shape].most_ts) return MXC_ERR_UNSUPPORTED;
    p.M = p.N * p.Mh * p.Mw;
    p.in_bytes = (unsigned)((long long)p.N * p.Hi * p.Wi * p.pix * 2);
    if (p.Cw == 0) p.Cw = p.Co;
    p.wm_bytes = bt ? p.bt_w_bytes : (unsigned)((long long)p.Cw * p.TR * p.TS * p.Ci * 2);
    p.out_bytes = (unsigned)((long long)p.M * p.Co * 2);
    p.nt_out = p.out_bytes >= 128u << 20 ? 1 : 0;
    return p.TS == 3 ? launch_shape<3>(shape, p, st, bt) : launch_shape<5>(shape, p, st, bt);
}

}  // namespace mxc
