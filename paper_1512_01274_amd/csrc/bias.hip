// Bias gradient: db[k] = sum over images and pixels of dy[n, k, p, q], fp32, in a fixed order.
//
// HBM-bound (dy is read once).  Every workgroup adds up a share of the tensor into a partial vector, and a second
// kernel adds the partial vectors in ascending order; a tensor small enough for one share per group of columns needs
// no second kernel.  All global reads are 16 bytes per lane, four in flight, for every channel count and alignment.
#include "mxc_internal.h"

namespace mxc {
namespace {

constexpr int BT = 1024;
constexpr int SHORT_CHUNKS = 4096;   // 64 KB
constexpr int SHORT_CPB = 64;        // 256 threads are four row groups
constexpr int MAX_CPB = 256;      // 16-byte chunks of a row that a workgroup covers

template <typename T> constexpr int VEC = 16 / (int)sizeof(T);

template <typename T> __device__ __forceinline__ void add_vec(float (&acc)[VEC<T>], const uint4 v)
{
    if constexpr (sizeof(T) == 2) {
        const uint32_t u[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            acc[2 * e] += __uint_as_float(u[e] << 16);
            acc[2 * e + 1] += __uint_as_float(u[e] & 0xFFFF0000u);
        }
    } else {
        acc[0] += __uint_as_float(v.x); acc[1] += __uint_as_float(v.y);
        acc[2] += __uint_as_float(v.z); acc[3] += __uint_as_float(v.w);
    }
}

// NHWC.  dy as [rows][width]: a row is the fewest pixels whose channels fill whole 16-byte chunks (one pixel where K is
// a multiple of a chunk, else up to 8), so that a chunk covers the same channels in every row.  Workgroup (x, y) owns
// chunks [x*cpb, x*cpb + cpb) of the rows [y*rows_per_wg, + rows_per_wg); its 1024 threads form 1024/cpb row groups,
// whose sums meet in LDS (in two steps, each in ascending order).  out: [gridDim.y][width].  (1024 threads with four loads each in
// flight, or BT = 256 with eight for shares up to 64 KB of at most 64 chunks a row, where starting and joining sixteen waves is most of the
// time: 32 KB 3.4 -> 2.7 us, 55 shares of 33 KB 4.7 -> 4.1.)
template <typename T, int BT>
__global__ __launch_bounds__(BT) void bias_grad_rows_kernel(const uint4 *__restrict__ dy, float *__restrict__ out, long long rows, int chunks,
                                                            int cpb, int rows_per_wg)
{
    constexpr int V = VEC<T>;
    // Element e of thread t at [e][t], the rows `cpb` apart in their banks: the threads below that add up neighbouring (e, column)
    // read neighbouring banks (with rows of BT they met in cpb of the 64: 3.7 -> 3.4 us for one share of 32 KB).
    __shared__ float red[(BT + MAX_CPB) * V];
    const int pitch = BT + cpb;
    const int groups = BT / cpb, c = threadIdx.x % cpb, grp = threadIdx.x / cpb;
    const int chunk = blockIdx.x * cpb + c;
    const long long r0 = (long long)blockIdx.y * rows_per_wg, r1 = min(rows, r0 + rows_per_wg);
    float acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = 0.f;
    if (grp < groups && chunk < chunks) {
        const uint4 *base = dy + chunk;
        const long long step = (long long)groups * chunks;
        long long r = r0 + grp;
        const uint4 *p = base + r * chunks;
        if constexpr (BT == 256)
            for (; r + 7LL * groups < r1; r += 8LL * groups, p += 8 * step) {
                uint4 v[8];
#pragma unroll
                for (int q = 0; q < 8; ++q) v[q] = p[q * step];
#pragma unroll
                for (int q = 0; q < 8; ++q) add_vec<T>(acc, v[q]);
            }
        for (; r + 3LL * groups < r1; r += 4LL * groups, p += 4 * step) {
            const uint4 a = p[0], b = p[step], d = p[2 * step], f = p[3 * step];
            add_vec<T>(acc, a); add_vec<T>(acc, b); add_vec<T>(acc, d); add_vec<T>(acc, f);
        }
        for (; r < r1; r += groups, p += step) add_vec<T>(acc, *p);
    }
    // then thread (e, c, part) adds every PARTS-th row group
#pragma unroll
    for (int e = 0; e < V; ++e) red[e * pitch + threadIdx.x] = acc[e];
    __syncthreads();
    const int items = cpb * V;
    const int parts = items >= BT ? 1 : BT / items;      // at least 1 thread per output
    for (int i = threadIdx.x; i < items * parts; i += BT) {
        const int e = i / cpb % V, col = i % cpb, part = i / items;
        float s = 0.f;
        for (int g = part; g < groups; g += parts) s += red[e * pitch + g * cpb + col];
        acc[0] = s;                                      // items*parts <= BT where parts > 1: one value per thread
        if (parts == 1) { if (blockIdx.x * cpb + col < chunks) out[(size_t)blockIdx.y * chunks * V + (blockIdx.x * cpb + col) * V + e] = s; }
    }
    if (parts == 1) return;
    __syncthreads();
    if ((int)threadIdx.x < items * parts) red[threadIdx.x] = acc[0];
    __syncthreads();
    if ((int)threadIdx.x < items) {
        const int e = threadIdx.x / cpb, col = threadIdx.x % cpb;
        float s = 0.f;
        for (int q = 0; q < parts; ++q) s += red[q * items + threadIdx.x];
        if (blockIdx.x * cpb + col < chunks) out[(size_t)blockIdx.y * chunks * V + (blockIdx.x * cpb + col) * V + e] = s;
    }
}

// NCHW: dy is [N][K][PQ].  Workgroup (k, y) adds the planes (n, k) of images [y*n_per_wg, + n_per_wg), each plane a
// contiguous run read in 16-byte pieces at whatever alignment it has.  out: [gridDim.y][K].
template <typename T>
__global__ __launch_bounds__(256) void bias_grad_planes_kernel(const T *__restrict__ dy, float *__restrict__ out, int N, int K, int PQ, int n_per_wg)
{
    constexpr int V = VEC<T>;
    struct __attribute__((packed)) Packed16 { uint32_t v[4]; };
    __shared__ float red[4];
    const int k = blockIdx.x, n0 = blockIdx.y * n_per_wg, n1 = (int)min((long long)N, (long long)n0 + n_per_wg);
    const int full = PQ / V;
    float acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = 0.f;
    // Whole pieces first, without a branch between their loads, then what is left of each plane (with the two in one loop no
    // loads ran ahead of a branch: 64x50x23x19 bf16 9.1 us, now 4.3).
    const int total = (n1 - n0) * full, rest = PQ - full * V;      // below 2^30: see plan
    const long long tails = (long long)(n1 - n0) * rest;
#pragma unroll 4
    for (int i = threadIdx.x; i < total; i += 256) {
        const int n = (int)((unsigned)i / (unsigned)full), q = i - n * full;
        const Packed16 v = *reinterpret_cast<const Packed16 *>(dy + ((size_t)(n0 + n) * K + k) * PQ + (size_t)q * V);
        add_vec<T>(acc, make_uint4(v.v[0], v.v[1], v.v[2], v.v[3]));
    }
#pragma unroll 4
    for (long long i = threadIdx.x; i < tails; i += 256) {
        const int n = (int)((unsigned)i / (unsigned)rest), e = (int)((unsigned)i % (unsigned)rest);
        acc[0] += load_f32(dy + ((size_t)(n0 + n) * K + k) * PQ + (size_t)(full * V + e));
    }
    float s = acc[0];
#pragma unroll
    for (int e = 1; e < V; ++e) s += acc[e];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) s += __shfl_xor(s, d);
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) out[(size_t)blockIdx.y * K + k] = ((red[0] + red[1]) + red[2]) + red[3];
}

// db[k] = sum of the partial vectors' entries f*K + k, f < fold, and of the last `left` pixels of dy (those that fill no
// whole row): 32 columns per workgroup, 32 thread groups that each add every 32nd entry, then the 32 sums in order.
template <typename T>
__global__ __launch_bounds__(BT) void bias_grad_sum_kernel(const float *__restrict__ partial, float *__restrict__ db, int K, int entries,
                                                           const T *__restrict__ rest, int left)
{
    __shared__ float red[BT];
    constexpr int GROUPS = BT / 32;
    const int col = threadIdx.x % 32, grp = threadIdx.x / 32;
    const int k = blockIdx.x * 32 + col;
    float acc = 0.f;
    if (k < K) {
#pragma unroll 8
        for (int i = grp; i < entries; i += GROUPS) acc += partial[(size_t)i * K + k];
        if (grp < left) acc += load_f32(rest + (size_t)grp * K + k);
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    if (grp == 0 && k < K) {
        float s = 0.f;
        for (int g = 0; g < GROUPS; ++g) s += red[g * 32 + col];
        db[k] = s;
    }
}

// How the tensor is cut.  One share (no second kernel) up to about 256 KB per workgroup: there the second launch costs
// more than the rest of the chip would save.  Beyond that a workgroup per CU, in 1024 threads with 64 bytes each in
// flight, reads at the rate of the copy kernel; more partial vectors only make the second kernel longer (1024 of them
// cost it 9-12 us, 256 cost 3).
struct BiasPlan { int fold, chunks, cpb, parts; long long rows, left; };

BiasPlan plan(long long N, int K, long long PQ, int dtype, int layout)
{
    BiasPlan b{};
    const int V = dtype == MXC_BF16 ? 8 : 4;
    b.fold = 1;
    if (layout == MXC_NCHW) {
        // at least 512 workgroups, as far as there are images and 16 KB for each of them.  With below 2^40 elements, and
        // planes below 2^31, a workgroup's whole pieces are below 2^40 / (512 * 4) + 2^29, and its planes below 2^23.
        long long parts = (512 + K - 1) / K;
        const long long per_image = PQ * (16 / V);
        long long most = N * per_image / (16 << 10);
        if (most < 1) most = 1;
        if (parts > most) parts = most;
        if (parts > N) parts = N;
        // Up to 64 KB of a channel one workgroup is done before the second launch would be, if its threads have at most 20 loads; elements
        // behind a plane's last whole piece are loads of their own, and four at a time are in flight.  us, one launch / two, bf16, 16
        // channels: 48 KB of 8x8 planes, 12 loads 3.3 / 4.4; 64 KB, 16 loads 3.7 / 4.5, of 14x14 planes, 18 loads 4.8 / 4.8, of 5x5, 21 loads
        // 6.5 / 5.6, of 9 elements, 28 loads 7.8 / 5.7, of 15, 68 loads 9.2 / 6.6, of one, 128 loads 16.1 / 7.3.  Over 197 sizes of both types one
        // launch takes 0.83 of the time of two at 14-16 loads, 0.89 at 16-20, 1.05 at 20-24, 1.29 above 40.
        if (N * per_image <= 64 << 10 && N * (PQ / V + PQ % V) <= 20 * 256) parts = 1;
        b.parts = (int)(parts < 1 ? 1 : parts);
        return b;
    }
    while ((long long)K * b.fold % V != 0) b.fold *= 2;
    b.chunks = K * b.fold / V;
    b.rows = N * PQ / b.fold;
    b.left = N * PQ % b.fold;
    // One share in blocks of few columns: more workgroups, and with a block within SHORT_CHUNKS the kernel of 256 threads (see run), as long as not too
    // many of them fetch the same lines.  Time over that of 4 chunks, which from 1025 rows on are 1024 threads, in a graph, 3162 tensors, mean and
    // worst: 1025 to 2048 rows, 2 chunks: of rows of 3 to 20 chunks 0.88 / 1.11, of 21 to 63 1.01 / 1.30, of 64 1.34 / 1.46, of more 1.04 / 1.26; up
    // to 4096 rows, 1 chunk: of 2 to 10 0.86 / 1.13, of 11 to 15 0.99 / 1.23, of 16 1.39 / 1.49, of 17 to 24 1.09 / 1.38.
    const bool one = b.fold == 1 && b.rows <= SHORT_CHUNKS;
    const int within = b.rows <= SHORT_CHUNKS / 4 ? 4 : b.rows <= SHORT_CHUNKS / 2 ? 2 : 1, width = one ? (b.chunks <= 10 * within ? within : 4) : BT;
    b.cpb = b.chunks < width ? b.chunks : width;
    // wide rows: equal column blocks of at most 256 chunks, so that 1024 threads are four row groups with loads in flight
    if (!one && b.cpb > MAX_CPB) b.cpb = MAX_CPB;
    if (one) { b.parts = 1; return b; }
    const long long col_blocks = (b.chunks + b.cpb - 1) / b.cpb;
    long long parts = (256 + col_blocks - 1) / col_blocks;
    const long long most = (b.rows * b.cpb * 16 + (32 << 10) - 1) / (32 << 10);      // at least 32 KB per workgroup
    if (parts > most) parts = most;
    b.parts = (int)(parts < 1 ? 1 : parts);
    return b;
}

template <typename T>
int run(const BiasPlan &b, long long N, int K, long long PQ, int layout, const T *dy, float *db, float *partial, hipStream_t st)
{
    const bool one = b.parts == 1 && b.fold == 1;
    float *out = one ? db : partial;
    if (layout == MXC_NCHW) {
        const int per = (int)((N + b.parts - 1) / b.parts);
        hipLaunchKernelGGL(bias_grad_planes_kernel<T>, dim3((unsigned)K, (unsigned)((N + per - 1) / per)), dim3(256), 0, st, dy, out, (int)N, K,
                           (int)PQ, per);
        if (hipGetLastError() != hipSuccess) return MXC_ERR_LAUNCH;
        if (one) return MXC_OK;
        hipLaunchKernelGGL(bias_grad_sum_kernel<T>, dim3((unsigned)((K + 31) / 32)), dim3(BT), 0, st, partial, db, K, (int)((N + per - 1) / per), dy, 0);
        return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
    }
    const long long per = b.rows > 0 ? (b.rows + b.parts - 1) / b.parts : 1;
    if (per > 0x7FFFFFFFll) return MXC_ERR_SHAPE;
    const int used = (int)((b.rows + per - 1) / per);          // 0: only left-over pixels
    const dim3 grid((unsigned)((b.chunks + b.cpb - 1) / b.cpb), (unsigned)used);
    // Few long rows leave 256 threads one or two row groups and each a chain of loads.  Time with 256 threads over that with 1024, 438 tensors
    // of 8 to 1024 channels, by chunks a row: below 8 0.86, 8-64 0.95 (1.05 at worst), 64-128 1.01 (1.08), 128-256 1.09 (1.17).
    if (used > 0 && b.cpb <= SHORT_CPB && per * b.cpb <= SHORT_CHUNKS)
        hipLaunchKernelGGL((bias_grad_rows_kernel<T, 256>), grid, dim3(256), 0, st, (const uint4 *)dy, out, b.rows, b.chunks, b.cpb, (int)per);
    else if (used > 0)
        hipLaunchKernelGGL((bias_grad_rows_kernel<T, BT>), grid, dim3(BT), 0, st, (const uint4 *)dy, out, b.rows, b.chunks, b.cpb, (int)per);
    if (hipGetLastError() != hipSuccess) return MXC_ERR_LAUNCH;
    if (one) return MXC_OK;
    hipLaunchKernelGGL(bias_grad_sum_kernel<T>, dim3((unsigned)((K + 31) / 32)), dim3(BT), 0, st, partial, db, K, used * b.fold,
                       dy + (size_t)b.rows * b.fold * K, (int)b.left);
    return hipGetLastError() == hipSuccess ? MXC_OK : MXC_ERR_LAUNCH;
}

}  // namespace

size_t bias_grad_scratch(long long N, int K, long long PQ, int dtype, int layout)
{
    const BiasPlan b = plan(N, K, PQ, dtype, layout);
    return (size_t)b.parts * b.fold * K * sizeof(float);
}

int bias_grad(long long N, int K, long long PQ, int dtype, int layout, const void *dy, float *db, float *partial, hipStream_t st)
{
    if (layout == MXC_NCHW && (PQ > 0x7FFFFFFFll || N * K > 0x7FFFFFFFll)) return MXC_ERR_SHAPE;
    const BiasPlan b = plan(N, K, PQ, dtype, layout);
    if (dtype == MXC_BF16) return run(b, N, K, PQ, layout, (const bf16_t *)dy, db, partial, st);
    return run(b, N, K, PQ, layout, (const float *)dy, db, partial, st);
}

}  // namespace mxc
