// Layout conversion kernels: batched 2-D transposes through LDS.
//
// NCHW -> NHWC of an activation tensor is, per image, the transpose of a
// [C][H*W] matrix; KCRS -> KRSC of a filter bank is the same with [C][R*S].
// Pure data movement: 1 read + 1 write of every element, HBM-bound.
#include <type_traits>

#include "resum.h"

namespace mxc {

namespace {

constexpr int TILE = 64;

// The tile kernels run on a one-dimensional grid of batch x row tiles x column tiles workgroups (column tile
// fastest), so that neither the batch nor the row-tile count is bound by the 65535 limit of the grid's y and z.
struct TileId { unsigned bx, by, bz; };
__device__ __forceinline__ TileId tile_id(int rows, int cols)
{
    const unsigned gx = (unsigned)(cols + TILE - 1) / TILE, gy = (unsigned)(rows + TILE - 1) / TILE;
    const unsigned t = blockIdx.x / gx;
    return TileId{blockIdx.x % gx, t % gy, t / gy};
}

// One 64x64 tile per workgroup of 256 threads.  Reads are contiguous along
// `cols`, writes contiguous along `rows`; the +1 pad keeps the column reads of
// the LDS tile off a single bank.
template <typename T>
__global__ __launch_bounds__(256) void transpose_tile_kernel(const T *__restrict__ src, T *__restrict__ dst,
                                                             int rows, int cols)
{
    __shared__ T tile[TILE][TILE + 1];
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const TileId id = tile_id(rows, cols);
    const int c0 = id.bx * TILE, r0 = id.by * TILE;
    const size_t base = (size_t)id.bz * rows * cols;
#pragma unroll
    for (int i = 0; i < TILE; i += 4) {
        const int r = r0 + ty + i, c = c0 + tx;
        if (r < rows && c < cols) tile[ty + i][tx] = src[base + (size_t)r * cols + c];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < TILE; i += 4) {
        const int c = c0 + ty + i, r = r0 + tx;
        if (r < rows && c < cols) dst[base + (size_t)c * rows + r] = tile[tx][ty + i];
    }
}

// The same transpose at vector width for 2-byte elements: 16-byte global loads and stores on both sides.
// A workgroup moves a 64 x 64 tile; a thread loads the same 8 columns of two consecutive rows, pairs the
// elements of each column into one dword (byte permutes) and writes the 8 dwords into the transposed LDS tile
// [column][row pair]; then every thread gathers 8 consecutive rows of one column (4 dwords) and stores them as
// one 16-byte chunk of the destination row.  Needs rows % 8 == 0 and cols % 8 == 0 (16-byte alignment of
// every row on both sides); ragged tile edges are handled chunk-wise.
__global__ __launch_bounds__(256) void transpose_vec16_kernel(const uint16_t *__restrict__ src, uint16_t *__restrict__ dst,
                                                              int rows, int cols)
{
    constexpr int PITCH = 33;                              // dwords per LDS column: odd, conflict-free dword writes
    __shared__ uint32_t tile[TILE * PITCH];
    const int t = threadIdx.x;
    const TileId id = tile_id(rows, cols);
    const int c0 = id.bx * TILE, r0 = id.by * TILE;
    const size_t base = (size_t)id.bz * rows * cols;
    {
        const int cc = t & 7, rp = t >> 3;                 // 8-column chunk, row pair
        const int r = r0 + 2 * rp, c = c0 + cc * 8;
        uint4 a = make_uint4(0, 0, 0, 0), b = a;
        if (r < rows && c < cols) {                        // rows is even: r + 1 < rows as well
            a = *reinterpret_cast<const uint4 *>(src + base + (size_t)r * cols + c);
            b = *reinterpret_cast<const uint4 *>(src + base + (size_t)(r + 1) * cols + c);
        }
        const uint32_t av[4] = {a.x, a.y, a.z, a.w}, bv[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            // columns 2j and 2j+1: low halves and high halves of the two rows' dwords
            tile[(cc * 8 + 2 * j) * PITCH + rp] = __builtin_amdgcn_perm(bv[j], av[j], 0x05040100u);
            tile[(cc * 8 + 2 * j + 1) * PITCH + rp] = __builtin_amdgcn_perm(bv[j], av[j], 0x07060302u);
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int oc = (t >> 3) + 32 * i, q = t & 7;       // tile column, chunk of 8 rows
        const int c = c0 + oc, r = r0 + q * 8;
        if (c < cols && r < rows) {
            const uint32_t *l = tile + oc * PITCH + q * 4;
            *reinterpret_cast<uint4 *>(dst + base + (size_t)c * rows + r) = make_uint4(l[0], l[1], l[2], l[3]);
        }
    }
}

// ... and for 4-byte elements: 16-byte chunks hold 4 elements; 64 x 64 tile in four passes of 16 rows.
__global__ __launch_bounds__(256) void transpose_vec16_kernel(const uint32_t *__restrict__ src, uint32_t *__restrict__ dst,
                                                              int rows, int cols)
{
    constexpr int PITCH = 65;
    __shared__ uint32_t tile[TILE * PITCH];
    const int t = threadIdx.x;
    const TileId id = tile_id(rows, cols);
    const int c0 = id.bx * TILE, r0 = id.by * TILE;
    const size_t base = (size_t)id.bz * rows * cols;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int cc = t & 15, lr = (t >> 4) + 16 * i;
        const int r = r0 + lr, c = c0 + cc * 4;
        uint4 a = make_uint4(0, 0, 0, 0);
        if (r < rows && c < cols) a = *reinterpret_cast<const uint4 *>(src + base + (size_t)r * cols + c);
        tile[(cc * 4 + 0) * PITCH + lr] = a.x;
        tile[(cc * 4 + 1) * PITCH + lr] = a.y;
        tile[(cc * 4 + 2) * PITCH + lr] = a.z;
        tile[(cc * 4 + 3) * PITCH + lr] = a.w;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int oc = (t >> 4) + 16 * i, q = t & 15;
        const int c = c0 + oc, r = r0 + q * 4;
        if (c < cols && r < rows) {
            const uint32_t *l = tile + oc * PITCH + q * 4;
            *reinterpret_cast<uint4 *>(dst + base + (size_t)c * rows + r) = make_uint4(l[0], l[1], l[2], l[3]);
        }
    }
}

// ---- several 2-byte re-layouts in one launch ------------------------------------------------------------------
// What the bf16 kernels' operands need before they can run on a caller's NCHW tensors or on channel counts that are
// no multiple of 8: batched transposes whose destination runs are padded with zeros to whole 16-byte chunks, the
// filter of backward-data (transposed per stride residue class), and plain channel padding.  A call has two or three
// of them, each a few microseconds of work at ordinary sizes, so they share one launch: a workgroup finds its job by
// its index.  Rows of any length are read and written 16 bytes at a time (global memory takes unaligned vector
// accesses); only the last piece of a destination row goes element by element.  100x30x45x37 to [..][32]: 5.2 us against 6.9 + 5.2
// of a scalar transpose followed by a padding pass.
struct __attribute__((packed)) Packed16 { uint32_t v[4]; };

__device__ __forceinline__ uint4 load8(const uint16_t *p, int n)        // n >= 1 elements are there
{
    if (n >= 8) {
        const Packed16 v = *reinterpret_cast<const Packed16 *>(p);
        return make_uint4(v.v[0], v.v[1], v.v[2], v.v[3]);
    }
    uint32_t v[4] = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < 7; ++j)
        if (j < n) v[j >> 1] |= (uint32_t)p[j] << ((j & 1) * 16);
    return make_uint4(v[0], v[1], v[2], v[3]);
}

// eight elements at `at` of a tensor of `total`, whatever row they belong to; the tensor's very last go one by one.  The last
// piece of every row of 30 or 50 channels went element by element before, 7 loads under 7 conditions in every workgroup:
// 64x45x37 pixels of 30 channels to NCHW 6.2 us, now 5.3.
__device__ __forceinline__ uint4 load8_of(const uint16_t *src, long long at, long long total)
{
    return at < total ? load8(src + at, total - at >= 8 ? 8 : (int)(total - at)) : make_uint4(0, 0, 0, 0);
}

__device__ __forceinline__ uint4 keep_first(uint4 v, int n)             // the first n of 8 elements, zeros behind them
{
    const auto part = [n](uint32_t u, int at) { return n >= at + 2 ? u : n == at + 1 ? u & 0xFFFFu : 0u; };
    return make_uint4(part(v.x, 0), part(v.y, 2), part(v.z, 4), part(v.w, 6));
}

__device__ __forceinline__ void store8(uint16_t *p, uint4 v, int n)
{
    const uint32_t u[4] = {v.x, v.y, v.z, v.w};
    if (n >= 8) {
        *reinterpret_cast<Packed16 *>(p) = Packed16{{v.x, v.y, v.z, v.w}};
        return;
    }
#pragma unroll
    for (int j = 0; j < 7; ++j)
        if (j < n) p[j] = (uint16_t)(u[j >> 1] >> ((j & 1) * 16));
}

struct RelayJobs { RelayJob job[MAX_RELAY_JOBS]; int n; };

// NJ jobs: with a compile-time count the jobs' fields are fetched together instead of one search step after another.  R = Resum:
// the job brings dx to its NCHW place, and what is NaN is summed again.
struct NoResum {};
template <int NJ, class R = NoResum>
__global__ __launch_bounds__(256) void relayout_kernel(const RelayJobs jobs, const R rs)
{
    constexpr int PITCH = 33;                              // dwords per LDS column: odd, conflict-free dword writes
    __shared__ uint32_t tile[TILE * PITCH];
    unsigned blk = blockIdx.x;
    RelayJob q = jobs.job[0];
#pragma unroll
    for (int i = 1; i < NJ; ++i) {
        const unsigned before = i == 1 ? jobs.job[0].blocks : jobs.job[0].blocks + jobs.job[1].blocks;
        if (blockIdx.x >= before) { q = jobs.job[i]; blk = blockIdx.x - before; }
    }
    const int t = threadIdx.x;
    const uint16_t *src = (const uint16_t *)q.src;
    uint16_t *dst = (uint16_t *)q.dst;

    if (q.kind == RELAY_PAD) {                             // [batch][cols] -> [batch][run]
        const int chunks = q.run >> 3;
        const long long id = (long long)blk * 256 + t;
        const long long row = id / chunks;
        if (row >= q.batch) return;
        const int c = (int)(id % chunks) * 8;
        const uint4 v = c < q.cols ? keep_first(load8_of(src, row * q.cols + c, q.batch * q.cols), q.cols - c) : make_uint4(0, 0, 0, 0);
        *reinterpret_cast<uint4 *>(dst + row * q.run + c) = v;
        return;
    }
    const unsigned gx = (unsigned)(q.cols + TILE - 1) / TILE, gy = (unsigned)(q.run_tiles);
    const unsigned b2 = blk / gx;
    const int c0 = (int)(blk % gx) * TILE, r0 = (int)(b2 % gy) * TILE;
    const long long b = b2 / gy;
    {
        const int cc = t & 7, rp = t >> 3;                 // 8-column chunk, row pair
        const int r = r0 + 2 * rp, c = c0 + cc * 8;
        uint4 a = make_uint4(0, 0, 0, 0), d = a;
        const long long at = b * q.src_batch + (long long)r * q.src_pitch + c;
        const long long total = (q.batch - 1) * q.src_batch + (long long)q.rows * q.src_pitch;
        if (c < q.cols) {                                  // columns past the row's end are not stored
            if (r < q.rows) a = load8_of(src, at, total);
            if (r + 1 < q.rows) d = load8_of(src, at + q.src_pitch, total);
        }
        const uint32_t av[4] = {a.x, a.y, a.z, a.w}, dv[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            tile[(cc * 8 + 2 * j) * PITCH + rp] = __builtin_amdgcn_perm(dv[j], av[j], 0x05040100u);
            tile[(cc * 8 + 2 * j + 1) * PITCH + rp] = __builtin_amdgcn_perm(dv[j], av[j], 0x07060302u);
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int oc = (t >> 3) + 32 * i, part = t & 7;    // tile column, chunk of 8 rows
        const int c = c0 + oc, r = r0 + part * 8;
        if (c >= q.cols || r >= q.run) continue;
        long long off = b * q.dst_batch + (long long)c * q.dst_pitch;
        if (q.kind != RELAY_TRANSPOSE) {
            // filter of backward-data: column (rs, ci) or (ci, rs) of w goes to its residue class's row ci, tap (j, i)
            const int RS = q.R * q.S;
            const int rs = q.kind == RELAY_FILTER_KRSC ? c / q.C : c % RS, ci = q.kind == RELAY_FILTER_KRSC ? c % q.C : c / RS;
            const int fr = rs / q.S, fs = rs % q.S, ph = fr % q.stride, pw = fs % q.stride;
            int before_r = 0, before_s = 0;                // filter rows / columns of the classes before this one
            for (int a = 0; a < ph; ++a) before_r += (q.R - a + q.stride - 1) / q.stride;
            for (int a = 0; a < pw; ++a) before_s += (q.S - a + q.stride - 1) / q.stride;
            const int TR = (q.R - ph + q.stride - 1) / q.stride, TS = (q.S - pw + q.stride - 1) / q.stride;
            off = ((long long)q.class_C * (before_r * q.S + TR * before_s) + (long long)ci * (TR * TS) + fr / q.stride * TS + fs / q.stride) * q.dst_pitch;
        }
        const uint32_t *l = tile + oc * PITCH + part * 4;
        store8(dst + off + r, make_uint4(l[0], l[1], l[2], l[3]), q.run - r);
        if constexpr (std::is_same_v<R, Resum>)
            for (unsigned bad = nan_bits(make_uint4(l[0], l[1], l[2], l[3])); bad != 0; bad &= bad - 1) {
                const int pix = r + __ffs(bad) - 1;
                if (pix < q.run) store_f32(dst + off + pix, sum_dx<bf16_t, true>(rs.s, rs.a, rs.b, (int)b, pix / rs.s.W, pix % rs.s.W, c));
            }
    }
}

// The same for plain transposes of 4-byte elements, 64 x 64 a workgroup: reads and writes of 256 contiguous bytes per wave, the
// elements of a tile of fewer columns (the taps of a filter) in the order they lie.
template <int NJ>
__global__ __launch_bounds__(256) void relayout4_kernel(const RelayJobs jobs)
{
    constexpr int PITCH = TILE + 1;
    __shared__ uint32_t tile[TILE * PITCH];
    const bool second = NJ == 2 && blockIdx.x >= jobs.job[0].blocks;
    const RelayJob &q = jobs.job[second ? 1 : 0];
    const unsigned blk = blockIdx.x - (second ? jobs.job[0].blocks : 0u);
    const unsigned gx = (unsigned)(q.cols + TILE - 1) / TILE, gy = (unsigned)q.run_tiles, b2 = blk / gx;
    const int c0 = (int)(blk % gx) * TILE, r0 = (int)(b2 % gy) * TILE, nr = min(TILE, q.rows - r0), nc = min(TILE, q.cols - c0);
    const long long b = b2 / gy;
    const uint32_t *src = (const uint32_t *)q.src + b * q.src_batch + (long long)r0 * q.src_pitch + c0;
    uint32_t *dst = (uint32_t *)q.dst + b * q.dst_batch + (long long)c0 * q.dst_pitch + r0;
    const int t = threadIdx.x;
    // f(i, o, in) for the places of an outer x inner tile, inner padded to a power of two that the lanes share; all loads in flight at once
    auto each = [&](int outer, int inner, auto &&f) __attribute__((always_inline)) {
        const int lw = 32 - __clz(inner - 1 | 3), in = t & ((1 << lw) - 1);
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int o = (t >> lw) + (i << (8 - lw));
            if (o < outer && in < inner) f(i, o, in);
        }
    };
    uint32_t v[16];
    each(nr, nc, [&](int i, int r, int c) __attribute__((always_inline)) { v[i] = src[(long long)r * q.src_pitch + c]; });
    each(nr, nc, [&](int i, int r, int c) __attribute__((always_inline)) { tile[c * PITCH + r] = v[i]; });
    __syncthreads();
    each(nc, nr, [&](int, int c, int r) __attribute__((always_inline)) { dst[(long long)c * q.dst_pitch + r] = tile[c * PITCH + r]; });
}

// Few channels (c <= 8): one thread per pixel.  planar[b][c][pixels] <-> interleaved[b][pixels][c];
// both sides are contiguous across the lanes of a wave.
template <typename T, bool TO_INTERLEAVED>
__global__ __launch_bounds__(256) void small_c_kernel(const T *__restrict__ src, T *__restrict__ dst, int c, long long pixels)
{
    const long long pix = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (pix >= pixels) return;
    const size_t base = (size_t)blockIdx.y * c * pixels;
    for (int ch = 0; ch < c; ++ch) {
        if (TO_INTERLEAVED) dst[base + (size_t)pix * c + ch] = src[base + (size_t)ch * pixels + pix];
        else dst[base + (size_t)ch * pixels + pix] = src[base + (size_t)pix * c + ch];
    }
}

// Same permutation for 2-byte elements, C channels, 8 pixels per thread: C 16-byte accesses on the planar side, a
// register shuffle, and C 16-byte accesses on the interleaved side.  A thread's C interleaved chunks are
// neighbours in memory (a wave-wide access of "my i-th chunk" would touch 16 bytes of every 16*C), so they pass
// through LDS and each instruction of the interleaved side covers one contiguous span of the workgroup's pixels.
// Needs pixels % 8 == 0 (keeps every access 16-byte aligned).
template <int C, bool TO_INTERLEAVED>
__global__ __launch_bounds__(256) void small_c_vec_kernel(const uint16_t *__restrict__ src, uint16_t *__restrict__ dst,
                                                          long long pixels)
{
    __shared__ uint4 chunks[256 * C];
    const int t = threadIdx.x;
    const long long blk_pix0 = (long long)blockIdx.x * 2048;           // first pixel of this workgroup
    const long long pix0 = blk_pix0 + (long long)t * 8;
    const bool mine = pix0 < pixels;
    const size_t base = (size_t)blockIdx.y * C * pixels;
    const long long blk_chunks = (min(pixels - blk_pix0, 2048ll) / 8) * C;   // 16-byte chunks of this workgroup's span
    uint16_t *inter = const_cast<uint16_t *>(TO_INTERLEAVED ? dst : src) + base + (size_t)blk_pix0 * C;
    union V { uint4 v; uint16_t e[8]; };
    V in[C], out[C];
    if (TO_INTERLEAVED) {
        if (mine) {
#pragma unroll
            for (int ch = 0; ch < C; ++ch) in[ch].v = *reinterpret_cast<const uint4 *>(src + base + (size_t)ch * pixels + pix0);
#pragma unroll
            for (int j = 0; j < 8 * C; ++j) out[j / 8].e[j % 8] = in[j % C].e[j / C];
#pragma unroll
            for (int i = 0; i < C; ++i) chunks[t * C + i] = out[i].v;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < C; ++i)
            if (i * 256 + t < blk_chunks) reinterpret_cast<uint4 *>(inter)[i * 256 + t] = chunks[i * 256 + t];
    } else {
#pragma unroll
        for (int i = 0; i < C; ++i)
            if (i * 256 + t < blk_chunks) chunks[i * 256 + t] = reinterpret_cast<const uint4 *>(inter)[i * 256 + t];
        __syncthreads();
        if (mine) {
#pragma unroll
            for (int i = 0; i < C; ++i) in[i].v = chunks[t * C + i];
#pragma unroll
            for (int j = 0; j < 8 * C; ++j) out[j % C].e[j / C] = in[j / 8].e[j % 8];
#pragma unroll
            for (int ch = 0; ch < C; ++ch) *reinterpret_cast<uint4 *>(dst + base + (size_t)ch * pixels + pix0) = out[ch].v;
        }
    }
}

template <int C>
void launch_small_c_vec(const void *src, void *dst, int batch, long long pixels, bool to_inter, hipStream_t stream)
{
    dim3 grid((unsigned)((pixels / 8 + 255) / 256), (unsigned)batch), block(256);
    if (to_inter) hipLaunchKernelGGL((small_c_vec_kernel<C, true>), grid, block, 0, stream, (const uint16_t *)src, (uint16_t *)dst, pixels);
    else hipLaunchKernelGGL((small_c_vec_kernel<C, false>), grid, block, 0, stream, (const uint16_t *)src, (uint16_t *)dst, pixels);
}

// Plain copy: every workgroup owns one contiguous span of 4 x 256 chunks of 16 bytes; a thread issues its four
// loads before the first store, so four chunks per lane are in flight.
__global__ __launch_bounds__(256) void copy_kernel(const uint4 *__restrict__ src, uint4 *__restrict__ dst, size_t n16,
                                                   const unsigned char *__restrict__ tail_src,
                                                   unsigned char *__restrict__ tail_dst, int tail)
{
    typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 *s = reinterpret_cast<const u32x4 *>(src);
    u32x4 *d = reinterpret_cast<u32x4 *>(dst);
    const size_t i0 = (size_t)blockIdx.x * 1024 + threadIdx.x;
    u32x4 v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (i0 + 256 * j < n16) v[j] = __builtin_nontemporal_load(s + i0 + 256 * j);
#pragma unroll
    for (int j = 0; j < 4; ++j)
        if (i0 + 256 * j < n16) __builtin_nontemporal_store(v[j], d + i0 + 256 * j);
    if (blockIdx.x == 0 && (int)threadIdx.x < tail) tail_dst[threadIdx.x] = tail_src[threadIdx.x];
}

}  // namespace

bool transpose_launchable(long long batch, long long rows, long long cols)
{
    if (batch <= 0 || rows <= 0 || cols <= 0 || rows > 0x7FFFFFFFll || cols > 0x7FFFFFFFll) return false;
    const long long gx = (cols + TILE - 1) / TILE, gy = (rows + TILE - 1) / TILE;
    return gx * gy <= 0x7FFFFFFFll / batch;
}

int launch_transpose(const void *src, void *dst, int batch, int rows, int cols, int elem_bytes, hipStream_t stream)
{
    if (batch <= 0 || rows <= 0 || cols <= 0) return MXC_ERR_SHAPE;
    if ((rows <= 8 || cols <= 8) && batch <= 65535 && (elem_bytes == 2 || elem_bytes == 4)) {
        const bool to_inter = rows <= 8;           // [c][pixels] -> [pixels][c]
        const int c = to_inter ? rows : cols;
        const long long pixels = to_inter ? cols : rows;
        if (elem_bytes == 2 && pixels % 8 == 0 && c >= 2 && c <= 4) {
            if (c == 2) launch_small_c_vec<2>(src, dst, batch, pixels, to_inter, stream);
            else if (c == 3) launch_small_c_vec<3>(src, dst, batch, pixels, to_inter, stream);
            else launch_small_c_vec<4>(src, dst, batch, pixels, to_inter, stream);
            return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
        }
        dim3 grid((unsigned)((pixels + 255) / 256), (unsigned)batch), block(256);
        if (elem_bytes == 2) {
            if (to_inter) hipLaunchKernelGGL((small_c_kernel<uint16_t, true>), grid, block, 0, stream, (const uint16_t *)src, (uint16_t *)dst, c, pixels);
            else hipLaunchKernelGGL((small_c_kernel<uint16_t, false>), grid, block, 0, stream, (const uint16_t *)src, (uint16_t *)dst, c, pixels);
        } else {
            if (to_inter) hipLaunchKernelGGL((small_c_kernel<uint32_t, true>), grid, block, 0, stream, (const uint32_t *)src, (uint32_t *)dst, c, pixels);
            else hipLaunchKernelGGL((small_c_kernel<uint32_t, false>), grid, block, 0, stream, (const uint32_t *)src, (uint32_t *)dst, c, pixels);
        }
        return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
    }
    if (!transpose_launchable(batch, rows, cols)) return MXC_ERR_SHAPE;
    const long long gx = (cols + TILE - 1) / TILE, gy = (rows + TILE - 1) / TILE;
    dim3 grid((unsigned)(gx * gy * batch)), block(256);
    const int per16 = 16 / (elem_bytes > 0 ? elem_bytes : 1);
    const bool vec16 = rows % per16 == 0 && cols % per16 == 0 && ((uintptr_t)src % 16) == 0 && ((uintptr_t)dst % 16) == 0;
    if (elem_bytes == 2 && vec16)
        hipLaunchKernelGGL((void (*)(const uint16_t *, uint16_t *, int, int))transpose_vec16_kernel, grid, block, 0, stream,
                           (const uint16_t *)src, (uint16_t *)dst, rows, cols);
    else if (elem_bytes == 4 && vec16)
        hipLaunchKernelGGL((void (*)(const uint32_t *, uint32_t *, int, int))transpose_vec16_kernel, grid, block, 0, stream,
                           (const uint32_t *)src, (uint32_t *)dst, rows, cols);
    else if (elem_bytes == 2)
        hipLaunchKernelGGL(transpose_tile_kernel<uint16_t>, grid, block, 0, stream, (const uint16_t *)src,
                           (uint16_t *)dst, rows, cols);
    else if (elem_bytes == 4)
        hipLaunchKernelGGL(transpose_tile_kernel<uint32_t>, grid, block, 0, stream, (const uint32_t *)src,
                           (uint32_t *)dst, rows, cols);
    else
        return MXC_ERR_UNSUPPORTED;
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
}

RelayJob relay_to_nhwc(const void *src, void *dst, int n, int c, int hw, int c_pitch)
{
    RelayJob q{};
    q.kind = RELAY_TRANSPOSE; q.src = src; q.dst = dst; q.batch = n;
    q.rows = c; q.cols = hw; q.src_pitch = hw; q.src_batch = (long long)c * hw;
    q.run = c_pitch; q.dst_pitch = c_pitch; q.dst_batch = (long long)hw * c_pitch;
    return q;
}

RelayJob relay_to_nchw(const void *src, void *dst, int n, int c, int hw, int c_pitch)
{
    RelayJob q{};
    q.kind = RELAY_TRANSPOSE; q.src = src; q.dst = dst; q.batch = n;
    q.rows = hw; q.cols = c; q.src_pitch = c_pitch; q.src_batch = (long long)hw * c_pitch;
    q.run = hw; q.dst_pitch = hw; q.dst_batch = (long long)c * hw;
    return q;
}

RelayJob relay_pad(const void *src, void *dst, long long rows, int c, int c_pitch)
{
    RelayJob q{};
    q.kind = RELAY_PAD; q.src = src; q.dst = dst; q.batch = rows; q.cols = c; q.run = c_pitch;
    return q;
}

RelayJob relay_bwd_filter(const ConvShape &s, const void *w, void *wt, bool kcrs)
{
    RelayJob q{};
    q.kind = kcrs ? RELAY_FILTER_KCRS : RELAY_FILTER_KRSC; q.src = w; q.dst = wt; q.batch = 1;
    q.C = real_c(s); q.class_C = s.C; q.R = s.R; q.S = s.S; q.stride = s.stride;
    q.rows = real_k(s); q.cols = q.C * s.R * s.S; q.src_pitch = q.cols;
    q.run = s.K; q.dst_pitch = s.K;
    if (s.R == 1 && s.S == 1) {        // the one tap's matrix is the filter's transpose
        q.kind = RELAY_TRANSPOSE;
        q.src_batch = q.dst_batch = (long long)q.rows * q.cols;
    }
    return q;
}

static int launch_relayout(const RelayJobs &all, long long blocks, hipStream_t st, const Resum *resum)
{
    static_assert(MAX_RELAY_JOBS == 3, "job counts the kernel is built for");
    const dim3 grid((unsigned)blocks), block(256);
    const RelayJob &q = all.job[0];
    if (resum != nullptr) hipLaunchKernelGGL((relayout_kernel<1, Resum>), grid, block, 0, st, all, *resum);
    else if (all.n == 1 && q.kind == RELAY_TRANSPOSE && q.rows % 8 == 0 && q.cols % 8 == 0 && q.run == q.rows && q.src_pitch == q.cols &&
        q.dst_pitch == q.rows && q.src_batch == q.dst_batch)
        // one dense transpose of whole chunks: the plain kernel (half the time of the general one where it is all launch)
        hipLaunchKernelGGL((void (*)(const uint16_t *, uint16_t *, int, int))transpose_vec16_kernel, grid, block, 0, st, (const uint16_t *)q.src,
                           (uint16_t *)q.dst, q.rows, q.cols);
    else if (all.n == 1) hipLaunchKernelGGL(relayout_kernel<1>, grid, block, 0, st, all, NoResum{});
    else if (all.n == 2) hipLaunchKernelGGL(relayout_kernel<2>, grid, block, 0, st, all, NoResum{});
    else hipLaunchKernelGGL(relayout_kernel<3>, grid, block, 0, st, all, NoResum{});
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
}

int relayout4(const RelayJob *jobs, int n, hipStream_t st)
{
    if (n < 1 || n > 2) return MXC_ERR_UNSUPPORTED;
    RelayJobs all{};
    long long total = 0;
    for (all.n = 0; all.n < n; ++all.n) {
        RelayJob &q = all.job[all.n];
        q = jobs[all.n];
        q.run_tiles = (q.run + TILE - 1) / TILE;
        const long long blocks = (long long)((q.cols + TILE - 1) / TILE) * q.run_tiles * q.batch;
        if ((total += blocks) > 0x7FFFFFFFll) return MXC_ERR_SHAPE;
        q.blocks = (unsigned)blocks;
    }
    const dim3 grid((unsigned)total), block(256);
    if (n == 1) hipLaunchKernelGGL(relayout4_kernel<1>, grid, block, 0, st, all);
    else hipLaunchKernelGGL(relayout4_kernel<2>, grid, block, 0, st, all);
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
}

int relayout(const RelayJob *jobs, int n, hipStream_t st, const Resum *resum)
{
    RelayJobs all{};
    long long total = 0;
    for (int i = 0; i < n; ++i) {
        RelayJob &q = all.job[all.n];
        q = jobs[i];
        long long blocks;
        if (q.kind == RELAY_PAD) blocks = (q.batch * (q.run / 8) + 255) / 256;
        else {
            q.run_tiles = (q.run + TILE - 1) / TILE;
            blocks = (long long)((q.cols + TILE - 1) / TILE) * q.run_tiles * q.batch;
        }
        if (blocks > 0x7FFFFFFFll) return MXC_ERR_SHAPE;
        if (blocks == 0) continue;
        q.blocks = (unsigned)blocks;
        if (total + blocks > 0x7FFFFFFFll) {               // more workgroups than one launch holds: what there is goes first
            const RelayJob last = q;
            const int rc = launch_relayout(all, total, st, nullptr);
            if (rc != MXC_OK) return rc;
            all.job[0] = last;
            all.n = 0;
            total = 0;
        }
        total += blocks;
        ++all.n;
    }
    return all.n ? launch_relayout(all, total, st, resum) : MXC_OK;
}

int launch_copy(const void *src, void *dst, size_t bytes, hipStream_t stream)
{
    if (bytes == 0) return MXC_OK;
    const size_t n16 = bytes / 16;
    const int tail = (int)(bytes % 16);
    size_t blocks = (n16 + 1023) / 1024;
    if (blocks < 1) blocks = 1;
    if (blocks > 0x7FFFFFFFull) return MXC_ERR_SHAPE;
    hipLaunchKernelGGL(copy_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, (const uint4 *)src, (uint4 *)dst, n16,
                       (const unsigned char *)src + n16 * 16, (unsigned char *)dst + n16 * 16, tail);
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
}

}  // namespace mxc
