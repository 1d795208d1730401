// C ABI entry points: argument validation, workspace carving, layout handling
// and kernel selection.  See include/mxc.h for the contract of every call.
#include <string.h>

#include <mutex>
#include <string>

#include "mxc_internal.h"
#include "plan_cache.h"

namespace mxc {

thread_local long long g_plan_searches = 0;

namespace {

thread_local char g_variant[128] = "";

void set_variant(const char *pass, const char *name)
{
    snprintf(g_variant, sizeof(g_variant), "%s:%s", pass, name);
}

// Sequential carve-out of the caller's workspace.  The same code path runs in
// "dry" mode (base == nullptr, nothing launched) to answer the size query, so
// the reported size is by construction what a real call consumes.
struct Carver {
    char *base;
    size_t used = 0;
    explicit Carver(void *b) : base((char *)b) {}
    void *take(size_t bytes)
    {
        const size_t off = used;
        used += align_up(bytes, 256);
        return base ? base + off : nullptr;
    }
};

int validate_shape(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, int dtype, int layout,
                   ConvShape *out)
{
    if (N <= 0 || C <= 0 || H <= 0 || W <= 0 || K <= 0 || R <= 0 || S <= 0 || stride <= 0 || pad < 0)
        return MXC_ERR_SHAPE;
    if ((long long)H + 2LL * pad < R || (long long)W + 2LL * pad < S) return MXC_ERR_SHAPE;
    if (dtype != MXC_F32 && dtype != MXC_BF16) return MXC_ERR_UNSUPPORTED;
    if (layout != MXC_NCHW && layout != MXC_NHWC) return MXC_ERR_UNSUPPORTED;
    ConvShape s{N, C, H, W, K, R, S, stride, pad, (H + 2 * pad - R) / stride + 1, (W + 2 * pad - S) / stride + 1};
    // Per-tensor element counts must stay below 2^40 (kernels index with 64 bits; this only
    // guards the size arithmetic) and the filter below 2^31 elements.
    const long double lim = 1099511627776.0L;
    if ((long double)N * C * H * W >= lim || (long double)N * K * s.P * s.Q >= lim ||
        (long double)K * C * R * S >= 2147483648.0L)
        return MXC_ERR_SHAPE;
    // NCHW operands are converted by batched transposes whose row and column counts are ints and whose grids
    // are bounded: refuse here, before anything is launched, what they could not run
    if (layout == MXC_NCHW) {
        const long long HW = (long long)H * W, PQ = (long long)s.P * s.Q, RS = (long long)R * S;
        if (!transpose_launchable(N, C, HW) || !transpose_launchable(N, HW, C) || !transpose_launchable(N, K, PQ) ||
            !transpose_launchable(N, PQ, K) || !transpose_launchable(K, C, RS) || !transpose_launchable(K, RS, C))
            return MXC_ERR_SHAPE;
    }
    *out = s;
    return MXC_OK;
}

bool misaligned(const void *p) { return ((uintptr_t)p & 15u) != 0; }

#define MXC_TRY(expr)                 \
    do {                              \
        const int rc_ = (expr);       \
        if (rc_ != MXC_OK) return rc_; \
    } while (0)

// Set while a call must get by with the least scratch (see mxc_conv2d_bwd_weight_static): no kernel that trades
// scratch for speed is chosen.
thread_local bool g_lean = false;
struct LeanScope {
    explicit LeanScope(bool on) { g_lean = on; }
    ~LeanScope() { g_lean = false; }
};

bool f32_in_place(const ConvShape &s, int dtype) { return dtype == MXC_F32 && !g_lean && f32_supported(s); }

// ---- passes in the working layout (NHWC / KRSC) --------------------------------
// dry == true: only account workspace.

ConvShape with_channels(const ConvShape &s, int C)
{
    ConvShape t = s;
    t.C = C;
    return t;
}

// How forward and backward-weight get their input.  Layers whose channel count is not a multiple of 8 first
// bring x into the form their GEMM reads (space-to-depth packed, zero-bordered with 4 channels per pixel, or
// channel-padded), the same form for both passes; a caller that runs both on one x can have that done once
// (INPUT_PREPARE_ONLY fills a buffer of the caller's, nothing else runs) and hand the buffer to both
// (INPUT_PREPARED).  The form is carved from `xws` - the ordinary workspace in INPUT_RAW mode, the caller's
// buffer in the other two.  Layers that read x as it is have an empty prepared form.
enum InputMode { INPUT_RAW = 0, INPUT_PREPARE_ONLY = 1, INPUT_PREPARED = 2 };
enum InputForm { FORM_AS_IS = 0, FORM_S2D = 1, FORM_SMALLC = 2, FORM_CHANPAD = 3 };
struct InputPrep {
    Carver *xws = nullptr;
    InputMode mode = INPUT_RAW;
    int *form = nullptr;       // out: the InputForm the pass reads (the two passes must agree before they share a buffer)
};
inline void note_form(const InputPrep &ip, int form) { if (ip.form) *ip.form = form; }

// ---- bf16 channel counts that are no multiple of 8 -----------------------------------------------------------------

ConvShape with_padded_k(const ConvShape &s)
{
    ConvShape t = s;
    t.K = (s.K + 7) / 8 * 8;
    if (t.K != s.K) t.Kr = s.K;
    return t;
}

// ... and the input's too, except for the first layers' (at most 4, which have packings of their own)
ConvShape with_padded_channels(const ConvShape &s)
{
    ConvShape t = with_padded_k(s);
    if (s.C > 4 && s.C % 8 != 0) { t.C = (s.C + 7) / 8 * 8; t.Cr = s.C; }
    return t;
}

// the problem without the padding
ConvShape without_padding(const ConvShape &s)
{
    ConvShape t = s;
    t.K = real_k(s); t.C = real_c(s);
    t.Kr = t.Cr = 0;
    return t;
}

// Whether the gradients of a layer of ragged K can have terms that are products with padding, so that resum_dx / resum_dw
// have to follow: taps outside dy, or the packings of first layers, which leave places empty; taps outside x.
bool padded_k_resums_dx(const ConvShape &s8) { return s8.Kr != 0 && (s8.C <= 4 || s8.pad > 0 || s8.R > 1 || s8.S > 1); }
bool padded_k_resums_dw(const ConvShape &s8) { return s8.Kr != 0 && s8.pad > 0; }

// NHWC gradients of ragged K that are so small that one thread per result, in one launch, is done before the padded path's
// launches are.  us, one thread / padded, launches of a graph:
// dx: the one-thread kernel takes 2.4 + 0.11 per step of its chain (K times the taps that reach a pixel, and two for every
// tap it looks at) up to 2^18 results and more beyond; padding dy and the GEMM take 5-6, with resum_dx 8-10, first layers
// 8-14 (where pixels of all stride classes share a wave, which then walks every tap).  128x4096 to 10 classes 5.7 / 5.6,
// 8x64x14x14 3x3 K=4 8.3 / 9.8, K=6 10.4 / 9.8, K=9 13.7 / 8.7; 3x32x32 3x3 K=10 11.7 / 7.8, K=20 20.1 / 8.3; with
// 400 thousand results 3x3 K=3 10.8 / 10.8, K=4 12.0 / 10.8, 1x1 K=20 6.6 / 5.5, K=28 7.5 / 5.5.  Over 390 layers the faster of the two would
// take 3.8% less than these lines' choices; no line moved by itself saves more than 0.2% of that.  Most of it is images of a few pixels,
// whose chain counts taps that no pixel has (4x256, one pixel, 5x5 K=2: 3.3 / 9.8).
bool small_ragged_dx(const ConvShape &s)
{
    const bool first = s.C <= 4, resums = padded_k_resums_dx(with_padded_k(s));
    const long long out = (long long)s.N * s.H * s.W * s.C;
    const long long taps = first ? (long long)s.R * s.S : (long long)((s.R + s.stride - 1) / s.stride) * ((s.S + s.stride - 1) / s.stride);
    const long long chain = s.K * taps + 2LL * s.R * s.S;
    if (out > (first ? 1 << 20 : 1 << 19)) return false;
    if (out > 1 << 18) return chain <= (resums && !first ? 45 : 30);
    return chain <= (first ? 108 : resums ? 78 : 42);
}
// dw, by its multiply-adds, while the pixels are few enough for the one-thread kernel's ranges: 8x512 to 10 classes 4.5 / 5.2,
// 32x512 to 10 5.5 / 5.2; 128x512 to 2 (131 thousand) 5.4 / 4.8, to 4 (262 thousand) 6.3 / 4.9; 28x28 64 to 1 channel 3x3 (451
// thousand) 7.1 / 8.6, to 2 (903 thousand) 8.3 / 8.7, 8x14x14 64 to 2 (1.8 million) 11.3 / 8.9; 8x28x28 16 to 1 (6272 pixels)
// 13.3 / 10.1.  Above 4 channels the line lies where heads break even; convolutions of 0.1-0.6 million, which the tests of ragged
// channels want on the matrix cores, lose up to 2.3 us by it, first layers up to 6 (over 243 layers the faster of the two would
// take 4% less).
bool small_ragged_dw(const ConvShape &s)
{
    const long long m = (long long)s.N * s.P * s.Q;
    if (m > 1600) return false;
    return m * s.K * s.C * s.R * s.S <= (s.K > 4 ? 3 << 15 : s.pad > 0 || m > 400 ? 1 << 20 : 1 << 17);
}

// whether a matrix-core path takes the (padded) problem, in the order the passes below try them
bool mfma_fwd_supported(const ConvShape &s)
{
    if (s.C % 8 == 0) return igemm_fwd_supported(s);
    return (s2d_applicable(s) && igemm_fwd_supported(s2d_shape(s))) || (s.C <= 4 && igemm_fwd_smallc_supported(s));
}
// ... by the general kernels on the re-packed filter, not by one of the first layers' packings or from the filter in place
bool mfma_bwd_data_plain(const ConvShape &s)
{
    return !(s2d_applicable(s) && igemm_bwd_data_supported(s2d_shape(s))) && !igemm_bwd_data_smallc_supported(s) && igemm_bwd_data_supported(s) &&
           !bwd_data_reads_filter_in_place(s);
}
bool mfma_bwd_data_supported(const ConvShape &s)
{
    return (s2d_applicable(s) && igemm_bwd_data_supported(s2d_shape(s))) || igemm_bwd_data_smallc_supported(s) || igemm_bwd_data_supported(s);
}
bool mfma_wgrad_supported(const ConvShape &s)
{
    if (s.C % 8 == 0) return wgrad_supported(wgrad_geom_plain(s));
    return (s2d_applicable(s) && wgrad_supported(wgrad_geom_s2d(s))) || (s.C <= 4 && wgrad_supported(wgrad_geom_smallc(s))) ||
           wgrad_supported(wgrad_geom_chanpad(s));
}

int fwd_nhwc(const ConvShape &s, int dtype, const void *x, const void *w, void *y, const PostOp &post, Carver &ws, hipStream_t st,
             bool dry, const InputPrep &ip = InputPrep())
{
    const char *v = "";
    Carver &xws = ip.xws ? *ip.xws : ws;
    const bool pack = ip.mode != INPUT_PREPARED, run = ip.mode != INPUT_PREPARE_ONLY;
    if (dtype == MXC_BF16 && s.C % 8 == 0 && igemm_fwd_supported(s)) {
        const size_t split_bytes = run ? igemm_fwd_split_bytes(s) : 0;
        void *split_ws = split_bytes ? ws.take(split_bytes) : nullptr;
        if (dry || !run) return MXC_OK;
        const int rc = igemm_fwd(s, x, w, y, st, &v, post, split_ws);
        set_variant("fwd", v);
        return rc;
    }
    if (dtype == MXC_BF16 && s2d_applicable(s) && igemm_fwd_supported(s2d_shape(s))) {
        // strided first layer: space-to-depth turns it into a stride-1 problem with stride^2*C channels
        const ConvShape s2 = s2d_shape(s);
        note_form(ip, FORM_S2D);
        void *x2 = xws.take((size_t)s2.N * s2.H * s2.W * s2.C * 2);
        void *w2 = run ? ws.take((size_t)s2.K * s2.R * s2.S * s2.C * 2) : nullptr;
        if (dry) return MXC_OK;
        if (pack) MXC_TRY(s2d_pack_x(s, x, x2, st));
        if (!run) return MXC_OK;
        MXC_TRY(s2d_pack_w(s, w, w2, st));
        const int rc = igemm_fwd(s2, x2, w2, y, st, &v, post);
        set_variant("fwd", (std::string("s2d+") + v).c_str());
        return rc;
    }
    if (dtype == MXC_BF16 && s.C <= 4 && igemm_fwd_smallc_supported(s)) {
        // first-layer style: zero-bordered image with 4 or 8 channels per pixel, filter rows as runs
        const SmallCGeom g = smallc_geom(s);
        note_form(ip, FORM_SMALLC);
        void *xp = xws.take((size_t)s.N * g.Hp * g.Wp * g.pix * 2);
        void *wp = run ? ws.take((size_t)s.K * s.R * g.run * 2) : nullptr;
        if (dry) return MXC_OK;
        if (pack) MXC_TRY(smallc_pack_x(s, x, xp, st));
        if (!run) return MXC_OK;
        MXC_TRY(smallc_pack_w(s, w, wp, st));
        const int rc = igemm_fwd_smallc(s, xp, wp, y, st, &v, post);
        set_variant("fwd", (std::string("smallc+") + v).c_str());
        return rc;
    }
    const int C8 = (s.C + 7) / 8 * 8;
    if (dtype == MXC_BF16 && s.C % 8 != 0 && igemm_fwd_supported(with_channels(s, C8))) {
        // other channel counts: zero-pad the channels of x and w to a multiple of 8
        note_form(ip, FORM_CHANPAD);
        void *xp = xws.take((size_t)s.N * s.H * s.W * C8 * 2);
        void *wp = run ? ws.take((size_t)s.K * s.R * s.S * C8 * 2) : nullptr;
        if (dry) return MXC_OK;
        RelayJob jobs[2];
        int nj = 0;
        if (pack) jobs[nj++] = relay_pad(x, xp, (long long)s.N * s.H * s.W, s.C, C8);
        if (run) jobs[nj++] = relay_pad(w, wp, (long long)s.K * s.R * s.S, s.C, C8);
        MXC_TRY(relayout(jobs, nj, st));
        if (!run) return MXC_OK;
        const int rc = igemm_fwd(with_channels(s, C8), xp, wp, y, st, &v, post);
        set_variant("fwd", (std::string("chanpad+") + v).c_str());
        return rc;
    }
    if (dry || !run) return MXC_OK;
    if (f32_in_place(s, dtype)) {
        const int rc = f32_fwd(s, false, -1, x, w, y, st, &v, post);
        set_variant("fwd", v);
        return rc;
    }
    set_variant("fwd", "direct");
    return direct_fwd(s, dtype, x, w, y, st, post);
}

// How backward-data gets its filter.  Every bf16 path first brings the filter into the form its GEMM reads
// (re-packed per stride residue class, transposed, space-to-depth or column-group packed); a caller whose
// weights change less often than it calls backward-data can have that done once (FILTER_PREPARE_ONLY fills
// a buffer of the caller's, nothing else runs) and hand the buffer in afterwards (FILTER_PREPARED).  The
// prepared forms are carved from `fws` - the ordinary workspace in FILTER_RAW mode, the caller's buffer in
// the other two - in one fixed order, so all three modes agree on where each form lies.
enum FilterMode { FILTER_RAW = 0, FILTER_PREPARE_ONLY = 1, FILTER_PREPARED = 2 };

int bwd_data_nhwc(const ConvShape &s, int dtype, const void *dy, const void *w, void *dx, const PostOp &post, Carver &fws,
                  Carver &ws, hipStream_t st, bool dry, FilterMode mode = FILTER_RAW, bool kcrs = false)
{
    const bool prep = mode != FILTER_PREPARED, run = mode != FILTER_PREPARE_ONLY;
    if (const ConvShape s8 = with_padded_k(s); dtype == MXC_BF16 && s8.K != s.K && !g_lean && !small_ragged_dx(s) && mfma_bwd_data_supported(s8)) {
        // the GEMM reduces over whole 16-byte chunks of dy: zero-pad its channels (the filter form follows, see real_k)
        const bool resum = padded_k_resums_dx(s8);
        const size_t wbytes = (size_t)s.K * s.R * s.S * s.C * 2;
        void *wc = resum && mode != FILTER_RAW ? fws.take(wbytes) : nullptr;        // a prepared filter brings the filter itself along
        if (wc != nullptr && mode == FILTER_PREPARE_ONLY && !dry) MXC_TRY(launch_copy(w, wc, wbytes, st));
        void *dy8 = run ? ws.take((size_t)s.N * s.P * s.Q * s8.K * 2) : nullptr;
        if (!dry && run) {
            RelayJob jobs[2] = {relay_pad(dy, dy8, (long long)s.N * s.P * s.Q, s.K, s8.K)};
            int nj = 1;
            if (mode == FILTER_RAW && mfma_bwd_data_plain(s8)) {        // its filter form in the same launch
                Carver peek = fws;
                jobs[nj++] = relay_bwd_filter(s8, w, peek.take(igemm_bwd_data_workspace(s8)), kcrs);
                MXC_TRY(relayout(jobs, nj, st));
                MXC_TRY(bwd_data_nhwc(s8, dtype, dy8, w, dx, post, fws, ws, st, dry, FILTER_PREPARED, kcrs));
                return resum ? resum_dx(Resum{s, false, (const bf16_t *)dy, (const bf16_t *)w}, dx, st) : MXC_OK;
            }
            MXC_TRY(relayout(jobs, nj, st));
        }
        MXC_TRY(bwd_data_nhwc(s8, dtype, dy8, w, dx, post, fws, ws, st, dry, mode, kcrs));
        return resum && run && !dry ? resum_dx(Resum{s, false, (const bf16_t *)dy, (const bf16_t *)(mode == FILTER_PREPARED ? wc : w)}, dx, st) : MXC_OK;
    }
    if (dtype == MXC_BF16 && s.K % 8 == 0 && s2d_applicable(s) && igemm_bwd_data_supported(s2d_shape(s))) {
        const ConvShape s2 = s2d_shape(s);
        void *w2 = fws.take((size_t)s2.K * s2.R * s2.S * s2.C * 2), *wt = fws.take(igemm_bwd_data_workspace(s2));
        // (not used where the image is stored directly: which kernel runs depends on the tuning hook, the size must not)
        void *dx2 = run ? ws.take((size_t)s2.N * s2.H * s2.W * s2.C * 2) : nullptr;
        if (dry) return MXC_OK;
        const char *v = "";
        const S2DStore image{s.stride, s.pad, s.C, s2d_geom(s).Cq, s.H, s.W};
        const ImageStore direct = post.mask == nullptr ? igemm_bwd_data_image_store(s2, image) : IMAGE_NONE;
        const void *in_place = nullptr;
        if (bwd_data_reads_filter_in_place(s2)) in_place = wt;
        else if (mode == FILTER_RAW && (direct == IMAGE_STREAM || (direct == IMAGE_NONE && bwd_data_small_in_place(s2, false)))) in_place = w2;
        if (prep) {
            if (in_place == nullptr) MXC_TRY(s2d_pack_wt(s, w, wt, st));
            else {
                MXC_TRY(s2d_pack_w(s, w, w2, st));
                if (in_place != w2) MXC_TRY(igemm_bwd_data_prepare(s2, w2, wt, st, true));
            }
        }
        if (!run) return MXC_OK;
        if (direct != IMAGE_NONE) MXC_TRY(igemm_bwd_data_image(direct, s2, image, dy, in_place, wt, dx, st, &v));
        else MXC_TRY(igemm_bwd_data(s2, dy, in_place, dx2, wt, st, &v));
        set_variant("bwd_data", (std::string("s2d+") + v).c_str());
        return direct != IMAGE_NONE ? MXC_OK : s2d_unpack_dx(s, dx2, dx, st, post.mask);      // the mask is applied where dx itself is written
    }
    if (dtype == MXC_BF16 && igemm_bwd_data_smallc_supported(s)) {
        size_t w2_bytes, dx4_bytes;
        igemm_bwd_data_smallc_workspace(s, &w2_bytes, &dx4_bytes);
        void *w2 = fws.take(w2_bytes), *dx4 = run ? ws.take(dx4_bytes) : nullptr;
        if (dry) return MXC_OK;
        const char *v = "";
        const char *forced = getenv("MXC_FORCE_VARIANT");
        const bool taps = taps_dx_supported(s) && (forced == nullptr ? taps_dx_faster(s) : !strcmp(forced, taps_dx_name()));
        if (prep && !(taps && mode == FILTER_RAW)) MXC_TRY(igemm_bwd_data_smallc_prepare(s, w, w2, st));
        if (!run) return MXC_OK;
        if (taps) {
            set_variant("bwd_data", (std::string("smallc+") + taps_dx_name()).c_str());
            return taps_dx(s, dy, mode == FILTER_RAW ? w : w2, mode != FILTER_RAW, igemm_bwd_data_smallc_columns(s), dx, st, post);
        }
        const int rc = igemm_bwd_data_smallc(s, dy, w2, dx, dx4, st, &v, post);
        set_variant("bwd_data", (std::string("smallc+") + v).c_str());
        return rc;
    }
    if (dtype == MXC_BF16 && igemm_bwd_data_supported(s)) {
        void *wt = fws.take(igemm_bwd_data_workspace(s));
        const size_t split_bytes = run ? igemm_bwd_data_split_bytes(s) : 0;
        void *split_ws = split_bytes ? ws.take(split_bytes) : nullptr;
        if (dry) return MXC_OK;
        const char *v = "";
        // a filter the kernel reads in place stays where it is unless the caller keeps a prepared copy
        const void *in_place = nullptr;
        if (bwd_data_reads_filter_in_place(s)) in_place = mode == FILTER_RAW ? w : wt;
        else if (mode == FILTER_RAW && (!kcrs || s.R * s.S == 1) &&
                 (bwd_data_small_in_place(s, post.mask != nullptr) || bwd_data_classes_in_place(s, post.mask != nullptr))) in_place = w;
        if (prep && !(in_place != nullptr && mode == FILTER_RAW)) MXC_TRY(igemm_bwd_data_prepare(s, w, wt, st, mode == FILTER_PREPARE_ONLY, kcrs));
        if (!run) return MXC_OK;
        const int rc = igemm_bwd_data(s, dy, in_place, dx, wt, st, &v, post, split_ws);
        set_variant("bwd_data", v);
        return rc;
    }
    // direct kernels read the KRSC filter itself: its prepared form is a copy
    const size_t wbytes = (size_t)s.K * s.R * s.S * s.C * elem_size(dtype);
    void *wc = mode != FILTER_RAW ? fws.take(wbytes) : nullptr;
    if (dry) return MXC_OK;
    if (mode == FILTER_PREPARE_ONLY) return launch_copy(w, wc, wbytes, st);
    set_variant("bwd_data", "direct");
    return direct_bwd_data(s, dtype, dy, mode == FILTER_PREPARED ? wc : w, dx, st, post);
}

// ip: see InputMode (the forms are those of fwd_nhwc, chosen by the same tests in the same order; only
// INPUT_RAW and INPUT_PREPARED reach this function).  resum: the caller's operands where x and dy are copies whose padding may
// have to be left out of dw (of operands padded here it is done anyway)
int bwd_weight_nhwc(const ConvShape &s_in, int dtype, const void *x, const void *dy, void *dw, bool dw_bf16, Carver &ws,
                    hipStream_t st, bool dry, const InputPrep &ip = InputPrep(), bool kcrs = false, const Resum *resum = nullptr)
{
    const char *v = "";
    Carver &xws = ip.xws ? *ip.xws : ws;
    const bool pack = ip.mode != INPUT_PREPARED;
    // dy's channels come in whole 16-byte chunks: zero-pad them where they do not (dw keeps its own rows, see real_k)
    ConvShape s = s_in;
    const Resum own{s_in, false, (const bf16_t *)x, (const bf16_t *)dy};
    RelayJob jobs[2];
    int nj = 0;
    if (const ConvShape s8 = with_padded_k(s); dtype == MXC_BF16 && s8.K != s.K && !g_lean && !small_ragged_dw(s) && mfma_wgrad_supported(s8)) {
        void *dy8 = ws.take((size_t)s.N * s.P * s.Q * s8.K * 2);
        jobs[nj++] = relay_pad(dy, dy8, (long long)s.N * s.P * s.Q, s.K, s8.K);
        dy = dy8;
        s = s8;
        if (padded_k_resums_dw(s8)) resum = &own;        // x is the caller's: a layer of ragged K has no prepared input
    }
    if (dtype == MXC_BF16 && s.C % 8 == 0 && wgrad_supported(wgrad_geom_plain(s))) {
        const WgradGeom g = wgrad_geom_plain(s);
        float *partial = (float *)ws.take(wgrad_workspace(g));
        if (dry) return MXC_OK;
        MXC_TRY(relayout(jobs, nj, st));
        const int rc = wgrad(g, x, dy, dw, dw_bf16, kcrs, partial, st, &v, resum);
        set_variant("bwd_weight", v);
        return rc;
    }
    if (dtype == MXC_BF16 && s2d_applicable(s) && wgrad_supported(wgrad_geom_s2d(s))) {
        const ConvShape s2 = s2d_shape(s);
        const WgradGeom g = wgrad_geom_s2d(s);
        note_form(ip, FORM_S2D);
        void *x2 = xws.take((size_t)s2.N * s2.H * s2.W * s2.C * 2);
        float *partial = (float *)ws.take(wgrad_workspace(g));
        if (dry) return MXC_OK;
        if (pack) MXC_TRY(s2d_pack_x(s, x, x2, st));
        MXC_TRY(relayout(jobs, nj, st));
        const int rc = wgrad(g, x2, dy, dw, dw_bf16, kcrs, partial, st, &v, resum);
        set_variant("bwd_weight", (std::string("s2d+") + v).c_str());
        return rc;
    }
    if (dtype == MXC_BF16 && s.C <= 4 && wgrad_supported(wgrad_geom_smallc(s))) {
        const SmallCGeom sg = smallc_geom(s);
        const WgradGeom g = wgrad_geom_smallc(s);
        note_form(ip, FORM_SMALLC);
        void *xp = xws.take((size_t)s.N * sg.Hp * sg.Wp * sg.pix * 2);
        float *partial = (float *)ws.take(wgrad_workspace(g));
        if (dry) return MXC_OK;
        if (pack) MXC_TRY(smallc_pack_x(s, x, xp, st));
        MXC_TRY(relayout(jobs, nj, st));
        const int rc = wgrad(g, xp, dy, dw, dw_bf16, kcrs, partial, st, &v, resum);
        set_variant("bwd_weight", (std::string("smallc+") + v).c_str());
        return rc;
    }
    if (dtype == MXC_BF16 && s.C % 8 != 0 && wgrad_supported(wgrad_geom_chanpad(s))) {
        const WgradGeom g = wgrad_geom_chanpad(s);
        note_form(ip, FORM_CHANPAD);
        void *xp = xws.take((size_t)s.N * s.H * s.W * g.pix * 2);
        float *partial = (float *)ws.take(wgrad_workspace(g));
        if (dry) return MXC_OK;
        if (pack) jobs[nj++] = relay_pad(x, xp, (long long)s.N * s.H * s.W, s.C, g.pix);
        MXC_TRY(relayout(jobs, nj, st));
        const int rc = wgrad(g, xp, dy, dw, dw_bf16, kcrs, partial, st, &v, resum);
        set_variant("bwd_weight", (std::string("chanpad+") + v).c_str());
        return rc;
    }
    if (f32_in_place(s, dtype)) {
        float *partial = (float *)ws.take(f32_wgrad_workspace(s));
        if (dry) return MXC_OK;
        const int rc = f32_wgrad(s, false, x, dy, dw, partial, st, &v);
        set_variant("bwd_weight", v);
        return rc;
    }
    const int splits = direct_bwd_weight_splits(s);
    float *partial = (float *)ws.take((size_t)splits * s.K * s.R * s.S * s.C * sizeof(float));
    if (dry) return MXC_OK;
    set_variant("bwd_weight", "direct_splitk");
    return direct_bwd_weight(s, dtype, x, dy, dw, dw_bf16, partial, splits, st);
}

// ---- fp32, either layout: the matrix-core kernels of fp32.hip read the caller's tensors in place -----------------
// ... or NHWC copies of NCHW operands, where that is faster (f32_copies); the result goes to its planes by itself.  The scratch
// for NCHW is the same either way and of the size that a converting path needs for every operand: the size query has always
// answered so.  A prepared filter stays as it lies, so its copy takes the place of dx in the scratch and has to fit there.

int run_f32(int pass, const ConvShape &s, int layout, const void *a, const void *b, void *out, const PostOp &post, Carver &fws,
            Carver &ws, hipStream_t st, bool dry, FilterMode mode)
{
    const bool nchw = layout == MXC_NCHW;
    const int RS = s.R * s.S;
    const size_t nx = (size_t)s.N * s.C * s.H * s.W * 4, nw = (size_t)s.K * s.C * s.R * s.S * 4, ny = (size_t)s.N * s.K * s.P * s.Q * 4;
    const char *v = "";
    if (pass == MXC_FWD) {
        void *x2 = nchw ? ws.take(nx) : nullptr, *w2 = nchw ? ws.take(nw) : nullptr;
        if (nchw) ws.take(ny);
        if (dry) return MXC_OK;
        const int copies = nchw ? f32_copies(s, false, false) : -1;
        if (copies >= 0) {
            const RelayJob jobs[] = {relay_to_nhwc(a, x2, s.N, s.C, s.H * s.W, s.C), relay_to_nhwc(b, w2, s.K, s.C, RS, s.C)};
            MXC_TRY(relayout4(jobs, RS == 1 ? 1 : 2, st));
            a = x2;
            if (RS > 1) b = w2;
        }
        const int rc = f32_fwd(s, nchw, copies, a, b, out, st, &v, post);
        set_variant("fwd", v);
        return rc;
    }
    if (pass == MXC_BWD_DATA) {
        // the kernel reads the filter as it lies: its prepared form is a copy
        const bool run = mode != FILTER_PREPARE_ONLY;
        void *wc = (nchw || mode != FILTER_RAW) ? fws.take(nw) : nullptr;
        void *dy2 = nullptr, *w2 = wc;
        if (nchw && run) {
            dy2 = ws.take(ny);
            void *dx2 = ws.take(nx);
            if (mode == FILTER_PREPARED) w2 = dx2;
            if (post.mask != nullptr || post.relu) ws.take(nx);
        }
        if (dry) return MXC_OK;
        if (!run) return launch_copy(b, wc, nw, st);
        PostOp post2 = post;
        post2.relu = 0;
        if (mode == FILTER_PREPARED) b = wc;
        const int copies = nchw && (RS == 1 || nw <= nx) ? f32_copies(s, true, post2.mask != nullptr) : -1;
        if (copies >= 0) {
            const RelayJob jobs[] = {relay_to_nhwc(a, dy2, s.N, s.K, s.P * s.Q, s.K), relay_to_nhwc(b, w2, s.K, s.C, RS, s.C)};
            MXC_TRY(relayout4(jobs, RS == 1 ? 1 : 2, st));
            a = dy2;
            if (RS > 1) b = w2;
        }
        const int rc = f32_bwd_data(s, nchw, copies, a, b, out, st, &v, post2);
        set_variant("bwd_data", v);
        return rc;
    }
    if (nchw) { ws.take(nx); ws.take(ny); ws.take(nw); }
    float *partial = (float *)ws.take(f32_wgrad_workspace(s));
    if (dry) return MXC_OK;
    const int rc = f32_wgrad(s, nchw, a, b, out, partial, st, &v);
    set_variant("bwd_weight", v);
    return rc;
}

// ---- one driver per pass: handles the caller's layout ---------------------------

// bf16 NCHW on the matrix cores.  The converted copies have their channels padded to whole 16-byte chunks (s carries the
// padded and the problem's own counts), all conversions before the kernel share one launch, the filter goes straight
// into the form backward-data reads, and dw leaves the split reduction in KCRS order.
int run_bf16_nchw(int pass, const ConvShape &s, const void *a, const void *b, void *out, const PostOp &post, Carver &fws, Carver &ws,
                  hipStream_t st, bool dry, FilterMode mode)
{
    const int C = real_c(s), K = real_k(s), RS = s.R * s.S;
    const bool first = s.C <= 4;           // first layers: few channels, converted by the kernels made for them
    const size_t nx = (size_t)s.N * s.C * s.H * s.W * 2, ny = (size_t)s.N * s.K * s.P * s.Q * 2, nw = (size_t)K * s.C * RS * 2;
    RelayJob jobs[MAX_RELAY_JOBS];
    int nj = 0;
    auto convert_x = [&](const void *src, void *dst) -> int {
        if (first) return launch_transpose(src, dst, s.N, C, s.H * s.W, 2, st);
        jobs[nj++] = relay_to_nhwc(src, dst, s.N, C, s.H * s.W, s.C);
        return MXC_OK;
    };
    if (pass == MXC_FWD) {
        void *x2 = ws.take(nx), *w2 = ws.take(nw), *y2 = ws.take(ny);
        if (!dry) {
            MXC_TRY(convert_x(a, x2));
            jobs[nj++] = relay_to_nhwc(b, w2, K, C, RS, s.C);
            MXC_TRY(relayout(jobs, nj, st));
        }
        PlaneOut direct{out, nullptr, K, false};
        PostOp post2 = post;
        post2.planes = &direct;
        post2.copied = true;
        MXC_TRY(fwd_nhwc(s, MXC_BF16, x2, w2, y2, post2, ws, st, dry));
        if (dry || direct.stored) return MXC_OK;
        jobs[0] = relay_to_nchw(y2, out, s.N, K, s.P * s.Q, s.K);
        return relayout(jobs, 1, st);
    }
    if (pass == MXC_BWD_DATA) {
        const bool prep = mode != FILTER_PREPARED, run = mode != FILTER_PREPARE_ONLY;
        const bool plain = mfma_bwd_data_plain(s);     // the filter form is made here, together with the conversions
        const bool resum = padded_k_resums_dx(s);
        const size_t wbytes = (size_t)K * C * RS * 2;
        void *wc = resum && mode != FILTER_RAW ? fws.take(wbytes) : nullptr;
        if (wc != nullptr && mode == FILTER_PREPARE_ONLY && !dry) MXC_TRY(launch_copy(b, wc, wbytes, st));
        void *w2 = first ? fws.take(nw) : nullptr;     // first layers: their packings start from KRSC
        void *dy2 = run ? ws.take(ny) : nullptr, *dx2 = run ? ws.take(nx) : nullptr;
        void *mask2 = run && (post.mask != nullptr || post.relu) ? ws.take(nx) : nullptr;   // see run_pass
        PostOp post2 = post;
        post2.relu = 0;
        post2.copied = true;
        FilterMode inner = mode;
        PlaneOut direct{out, post.mask, C, false};
        if (run && plain && !first && !resum && igemm_bwd_data_planes(s, post.mask != nullptr)) post2.planes = &direct;
        if (!dry) {
            if (run) jobs[nj++] = relay_to_nhwc(a, dy2, s.N, K, s.P * s.Q, s.K);
            if (run && post.mask != nullptr && post2.planes == nullptr) {
                MXC_TRY(convert_x(post.mask, mask2));
                post2.mask = mask2;
            }
            if (prep && first) jobs[nj++] = relay_to_nhwc(b, w2, K, C, RS, C);
            if (prep && plain && run) {
                Carver peek = fws;
                jobs[nj++] = relay_bwd_filter(s, b, peek.take(igemm_bwd_data_workspace(s)), true);
                inner = FILTER_PREPARED;
            }
            MXC_TRY(relayout(jobs, nj, st));
        }
        MXC_TRY(bwd_data_nhwc(s, MXC_BF16, dy2, first ? w2 : b, dx2, post2, fws, ws, st, dry, inner, !first));
        if (dry || !run || direct.stored) return MXC_OK;
        if (post2.planes != nullptr) return MXC_ERR_LAUNCH;      // the mask was left in the planes' layout for that store alone
        const Resum rs{without_padding(s), true, (const bf16_t *)a, (const bf16_t *)(mode == FILTER_PREPARED ? wc : b)};
        if (first) {
            MXC_TRY(launch_transpose(dx2, out, s.N, s.H * s.W, C, 2, st));
            return resum ? resum_dx(rs, out, st) : MXC_OK;
        }
        jobs[0] = relay_to_nchw(dx2, out, s.N, C, s.H * s.W, s.C);
        return relayout(jobs, 1, st, resum ? &rs : nullptr);
    }
    void *x2 = ws.take(nx), *dy2 = ws.take(ny);
    if (!dry) {
        MXC_TRY(convert_x(a, x2));
        jobs[nj++] = relay_to_nhwc(b, dy2, s.N, K, s.P * s.Q, s.K);
        MXC_TRY(relayout(jobs, nj, st));
    }
    const Resum rs{without_padding(s), true, (const bf16_t *)a, (const bf16_t *)b};
    return bwd_weight_nhwc(s, MXC_BF16, x2, dy2, out, pass == MXC_BWD_WEIGHT_BF16, ws, st, dry, InputPrep(), true,
                           padded_k_resums_dw(s) ? &rs : nullptr);
}

// fws / mode: see FilterMode (backward-data only; fws == ws and FILTER_RAW otherwise)
int run_pass(int pass, const ConvShape &s, int dtype, int layout, const void *a, const void *b, void *out, const PostOp &post,
             Carver &ws, hipStream_t st, bool dry, Carver *fws_opt = nullptr, FilterMode mode = FILTER_RAW)
{
    Carver &fws = fws_opt ? *fws_opt : ws;
    if (f32_in_place(s, dtype)) return run_f32(pass, s, layout, a, b, out, post, fws, ws, st, dry, mode);
    const int eb = (int)elem_size(dtype);
    const size_t nx = (size_t)s.N * s.C * s.H * s.W, nw = (size_t)s.K * s.C * s.R * s.S,
                 ny = (size_t)s.N * s.K * s.P * s.Q;
    if (layout == MXC_NHWC) {
        switch (pass) {
        case MXC_FWD: return fwd_nhwc(s, dtype, a, b, out, post, ws, st, dry);
        case MXC_BWD_DATA: return bwd_data_nhwc(s, dtype, a, b, out, post, fws, ws, st, dry, mode);
        default: return bwd_weight_nhwc(s, dtype, a, b, out, pass == MXC_BWD_WEIGHT_BF16, ws, st, dry);
        }
    }
    if (dtype == MXC_BF16 && !g_lean) {
        const ConvShape s8 = with_padded_channels(s);
        const bool ok = pass == MXC_FWD ? mfma_fwd_supported(s8) : pass == MXC_BWD_DATA ? mfma_bwd_data_supported(s8) : mfma_wgrad_supported(s8);
        if (ok) return run_bf16_nchw(pass, s8, a, b, out, post, fws, ws, st, dry, mode);
    }
    // NCHW at the boundary: convert operands into the workspace, compute, convert the result back.
    if (pass == MXC_FWD) {
        void *x2 = ws.take(nx * eb), *w2 = ws.take(nw * eb), *y2 = ws.take(ny * eb);
        if (!dry) {
            MXC_TRY(launch_transpose(a, x2, s.N, s.C, s.H * s.W, eb, st));
            MXC_TRY(launch_transpose(b, w2, s.K, s.C, s.R * s.S, eb, st));
        }
        MXC_TRY(fwd_nhwc(s, dtype, x2, w2, y2, post, ws, st, dry));
        if (!dry) MXC_TRY(launch_transpose(y2, out, s.N, s.P * s.Q, s.K, eb, st));
        return MXC_OK;
    }
    if (pass == MXC_BWD_DATA) {
        const bool prep = mode != FILTER_PREPARED, run = mode != FILTER_PREPARE_ONLY;
        void *w2 = fws.take(nw * eb);      // the KRSC filter is the first of the prepared forms
        void *dy2 = run ? ws.take(ny * eb) : nullptr, *dx2 = run ? ws.take(nx * eb) : nullptr;
        // with_mask (not the pointer) decides the carve-out, so that the size query and the call agree
        void *mask2 = run && (post.mask != nullptr || post.relu) ? ws.take(nx * eb) : nullptr;
        PostOp post2 = post;
        post2.relu = 0;
        if (!dry) {
            if (run) MXC_TRY(launch_transpose(a, dy2, s.N, s.K, s.P * s.Q, eb, st));
            if (prep) MXC_TRY(launch_transpose(b, w2, s.K, s.C, s.R * s.S, eb, st));
            if (run && post.mask != nullptr) {
                MXC_TRY(launch_transpose(post.mask, mask2, s.N, s.C, s.H * s.W, eb, st));
                post2.mask = mask2;
            }
        }
        MXC_TRY(bwd_data_nhwc(s, dtype, dy2, w2, dx2, post2, fws, ws, st, dry, mode));
        if (!dry && run) MXC_TRY(launch_transpose(dx2, out, s.N, s.H * s.W, s.C, eb, st));
        return MXC_OK;
    }
    const bool dw_bf16 = pass == MXC_BWD_WEIGHT_BF16;
    const int dwb = dw_bf16 ? 2 : 4;
    void *x2 = ws.take(nx * eb), *dy2 = ws.take(ny * eb);
    void *dw2 = ws.take(nw * dwb);
    if (!dry) {
        MXC_TRY(launch_transpose(a, x2, s.N, s.C, s.H * s.W, eb, st));
        MXC_TRY(launch_transpose(b, dy2, s.N, s.K, s.P * s.Q, eb, st));
    }
    MXC_TRY(bwd_weight_nhwc(s, dtype, x2, dy2, dw2, dw_bf16, ws, st, dry));
    if (!dry) MXC_TRY(launch_transpose(dw2, out, s.K, s.R * s.S, s.C, dwb, st));
    return MXC_OK;
}

// `post.relu` doubles, for backward-data in dry runs, as "a mask will be given" (the mask pointer is
// not known to the size query).
int entry(int pass, int N, int C, int H, int W, int K, int R, int S, int stride, int pad, int dtype, int layout,
          const void *a, const void *b, void *out, const PostOp &post, void *workspace, size_t workspace_bytes,
          void *hip_stream)
{
    ConvShape s;
    MXC_TRY(validate_shape(N, C, H, W, K, R, S, stride, pad, dtype, layout, &s));
    if (!a || !b || !out) return MXC_ERR_NULL;
    if (misaligned(a) || misaligned(b) || misaligned(out) || misaligned(workspace) || misaligned(post.mask)) return MXC_ERR_ALIGN;
    Carver need(nullptr);
    PostOp dry_post;
    dry_post.relu = (post.mask != nullptr || post.relu) ? 1 : 0;
    MXC_TRY(run_pass(pass, s, dtype, layout, nullptr, nullptr, nullptr, dry_post, need, nullptr, true));
    if (need.used > 0 && (!workspace || workspace_bytes < need.used)) return MXC_ERR_WORKSPACE;
    Carver ws(workspace);
    return run_pass(pass, s, dtype, layout, a, b, out, post, ws, (hipStream_t)hip_stream, false);
}

}  // namespace
}  // namespace mxc

// ---- scratch of the entry point that allocates nothing ------------------------------------------
// One array per GPU, part of the loaded code object: it exists on every device the library runs on
// from the first use of the library there until the process ends.  In host code the name below is
// only a handle for hipGetSymbolAddress; kernels and copies get the device address it returns.
#define MXC_STATIC_SCRATCH_BYTES (64u << 20)
static __device__ __align__(256) unsigned char scratch[MXC_STATIC_SCRATCH_BYTES];

namespace mxc {
namespace {

constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[MAX_DEVICES] = {};

// Device address of `scratch` on the current device (looked up once per device, with that device current).
int static_scratch(void **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) return MXC_ERR_LAUNCH;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return MXC_ERR_LAUNCH;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return MXC_OK;
}

}  // namespace
}  // namespace mxc

using namespace mxc;

extern "C" {

int mxc_conv2d_fwd(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, int dtype, int layout,
                   const void *x, const void *w, void *y, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return entry(MXC_FWD, N, C, H, W, K, R, S, stride, pad, dtype, layout, x, w, y, PostOp(), workspace, workspace_bytes,
                 hip_stream);
}

int mxc_conv2d_bwd_data(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, int dtype, int layout,
                        const void *dy, const void *w, void *dx, void *workspace, size_t workspace_bytes,
                        void *hip_stream)
{
    return entry(MXC_BWD_DATA, N, C, H, W, K, R, S, stride, pad, dtype, layout, dy, w, dx, PostOp(), workspace, workspace_bytes,
                 hip_stream);
}

int mxc_conv2d_bwd_weight(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, int dtype, int layout,
                          const void *x, const void *dy, void *dw, void *workspace, size_t workspace_bytes,
                          void *hip_stream)
{
    return entry(MXC_BWD_WEIGHT, N, C, H, W, K, R, S, stride, pad, dtype, layout, x, dy, dw, PostOp(), workspace,
                 workspace_bytes, hip_stream);
}

int mxc_conv2d_bwd_weight_bf16(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, int dtype, int layout,
                               const void *x, const void *dy, void *dw, void *workspace, size_t workspace_bytes,
                               void *hip_stream)
{
    if (dtype != MXC_BF16) return MXC_ERR_UNSUPPORTED;
    return entry(MXC_BWD_WEIGHT_BF16, N, C, H, W, K, R, S, stride, pad, dtype, layout, x, dy, dw, PostOp(), workspace,
                 workspace_bytes, hip_stream);
}

int mxc_conv2d_bwd_weight_static(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, int dtype, int layout,
                                 const void *x, const void *dy, void *dw, void *hip_stream)
{
    // argument errors first, as the other entry points report them; then the size against the array
    ConvShape s;
    MXC_TRY(validate_shape(N, C, H, W, K, R, S, stride, pad, dtype, layout, &s));
    if (!x || !dy || !dw) return MXC_ERR_NULL;
    if (misaligned(x) || misaligned(dy) || misaligned(dw)) return MXC_ERR_ALIGN;
    Carver need(nullptr);
    MXC_TRY(run_pass(MXC_BWD_WEIGHT, s, dtype, layout, nullptr, nullptr, nullptr, PostOp(), need, nullptr, true));
    // the faster kernels may want more scratch than the array holds; the ones that need the least come second
    const bool lean = need.used > MXC_STATIC_SCRATCH_BYTES;
    LeanScope scope(lean);
    if (lean) {
        Carver least(nullptr);
        MXC_TRY(run_pass(MXC_BWD_WEIGHT, s, dtype, layout, nullptr, nullptr, nullptr, PostOp(), least, nullptr, true));
        if (least.used > MXC_STATIC_SCRATCH_BYTES) return MXC_ERR_WORKSPACE;
    }
    void *ws = nullptr;
    MXC_TRY(static_scratch(&ws));
    // every kernel of this pass writes the part of the scratch it later reads: nothing needs clearing
    return entry(MXC_BWD_WEIGHT, N, C, H, W, K, R, S, stride, pad, dtype, layout, x, dy, dw, PostOp(), ws, MXC_STATIC_SCRATCH_BYTES,
                 hip_stream);
}

int mxc_conv2d_fwd_bias_act(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, int dtype, int layout,
                            const void *x, const void *w, const float *bias, int relu, void *y, void *workspace,
                            size_t workspace_bytes, void *hip_stream)
{
    if (relu != 0 && relu != 1) return MXC_ERR_UNSUPPORTED;
    if (bias != nullptr && ((uintptr_t)bias & 3u)) return MXC_ERR_ALIGN;
    PostOp post;
    post.bias = bias;
    post.relu = relu;
    // the forward pass's workspace does not depend on the grouped operations: query it as MXC_FWD
    ConvShape s;
    MXC_TRY(validate_shape(N, C, H, W, K, R, S, stride, pad, dtype, layout, &s));
    if (!x || !w || !y) return MXC_ERR_NULL;
    if (misaligned(x) || misaligned(w) || misaligned(y) || misaligned(workspace)) return MXC_ERR_ALIGN;
    Carver need(nullptr);
    MXC_TRY(run_pass(MXC_FWD, s, dtype, layout, nullptr, nullptr, nullptr, PostOp(), need, nullptr, true));
    if (need.used > 0 && (!workspace || workspace_bytes < need.used)) return MXC_ERR_WORKSPACE;
    Carver ws(workspace);
    return run_pass(MXC_FWD, s, dtype, layout, x, w, y, post, ws, (hipStream_t)hip_stream, false);
}

int mxc_conv2d_bwd_data_relu(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, int dtype, int layout,
                             const void *dy, const void *w, const void *x, void *dx, void *workspace, size_t workspace_bytes,
                             void *hip_stream)
{
    if (!x) return MXC_ERR_NULL;
    PostOp post;
    post.mask = x;
    return entry(MXC_BWD_DATA, N, C, H, W, K, R, S, stride, pad, dtype, layout, dy, w, dx, post, workspace, workspace_bytes,
                 hip_stream);
}

int mxc_conv2d_bwd_data_prepare_filter(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, int dtype, int layout,
                                       const void *w, void *w_prepared, size_t prepared_bytes, void *hip_stream)
{
    ConvShape s;
    MXC_TRY(validate_shape(N, C, H, W, K, R, S, stride, pad, dtype, layout, &s));
    if (!w || !w_prepared) return MXC_ERR_NULL;
    if (misaligned(w) || misaligned(w_prepared)) return MXC_ERR_ALIGN;
    Carver need(nullptr), none(nullptr);
    MXC_TRY(run_pass(MXC_BWD_DATA, s, dtype, layout, nullptr, nullptr, nullptr, PostOp(), none, nullptr, true, &need, FILTER_PREPARE_ONLY));
    if (prepared_bytes < need.used) return MXC_ERR_WORKSPACE;
    Carver fws(w_prepared);
    return run_pass(MXC_BWD_DATA, s, dtype, layout, nullptr, w, nullptr, PostOp(), none, (hipStream_t)hip_stream, false, &fws,
                    FILTER_PREPARE_ONLY);
}

int mxc_conv2d_bwd_data_prepared(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, int dtype, int layout,
                                 const void *dy, const void *w_prepared, size_t prepared_bytes, const void *x_mask, void *dx,
                                 void *workspace, size_t workspace_bytes, void *hip_stream)
{
    ConvShape s;
    MXC_TRY(validate_shape(N, C, H, W, K, R, S, stride, pad, dtype, layout, &s));
    if (!dy || !w_prepared || !dx) return MXC_ERR_NULL;
    if (misaligned(dy) || misaligned(w_prepared) || misaligned(dx) || misaligned(workspace) || misaligned(x_mask)) return MXC_ERR_ALIGN;
    PostOp post, dry_post;
    post.mask = x_mask;
    dry_post.relu = x_mask != nullptr ? 1 : 0;
    Carver needf(nullptr), need(nullptr);
    MXC_TRY(run_pass(MXC_BWD_DATA, s, dtype, layout, nullptr, nullptr, nullptr, dry_post, need, nullptr, true, &needf, FILTER_PREPARED));
    if (prepared_bytes < needf.used) return MXC_ERR_WORKSPACE;
    if (need.used > 0 && (!workspace || workspace_bytes < need.used)) return MXC_ERR_WORKSPACE;
    Carver fws(const_cast<void *>(w_prepared)), ws(workspace);
    return run_pass(MXC_BWD_DATA, s, dtype, layout, dy, nullptr, dx, post, ws, (hipStream_t)hip_stream, false, &fws, FILTER_PREPARED);
}

namespace mxc {
namespace {

// Size and kind of the prepared input of a layer.  Forward and backward-weight must read the same form to share
// a buffer; for a shape where they would not (one of them falls back to another kernel family) the prepared
// form is empty, like that of a layer that reads x as it is, and each pass packs for itself as usual.
int prepared_input_plan(const ConvShape &s, int dtype, size_t *bytes, int *form)
{
    Carver none(nullptr), xf(nullptr), xw(nullptr);
    int form_f = FORM_AS_IS, form_w = FORM_AS_IS;
    InputPrep ipf, ipw;
    ipf.xws = &xf; ipf.mode = INPUT_PREPARE_ONLY; ipf.form = &form_f;
    ipw.xws = &xw; ipw.mode = INPUT_PREPARED; ipw.form = &form_w;
    MXC_TRY(fwd_nhwc(s, dtype, nullptr, nullptr, nullptr, PostOp(), none, nullptr, true, ipf));
    MXC_TRY(bwd_weight_nhwc(s, dtype, nullptr, nullptr, nullptr, false, none, nullptr, true, ipw));
    // (a bf16 layer whose K is no multiple of 8 keeps the empty form that its callers' buffers are sized for)
    const bool shared = form_f == form_w && xf.used == xw.used && s.K % 8 == 0;
    *bytes = shared ? xf.used : 0;
    *form = shared ? form_f : FORM_AS_IS;
    return MXC_OK;
}

}  // namespace
}  // namespace mxc

int mxc_conv2d_prepare_input(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, int dtype, int layout,
                             const void *x, void *x_prepared, size_t prepared_bytes, void *hip_stream)
{
    ConvShape s;
    MXC_TRY(validate_shape(N, C, H, W, K, R, S, stride, pad, dtype, layout, &s));
    if (layout != MXC_NHWC) return MXC_ERR_UNSUPPORTED;
    if (!x) return MXC_ERR_NULL;
    if (misaligned(x) || misaligned(x_prepared)) return MXC_ERR_ALIGN;
    size_t need = 0;
    int form = FORM_AS_IS;
    MXC_TRY(prepared_input_plan(s, dtype, &need, &form));
    if (need == 0) return MXC_OK;          // the layer reads x as it is
    if (!x_prepared) return MXC_ERR_NULL;
    if (prepared_bytes < need) return MXC_ERR_WORKSPACE;
    Carver none(nullptr), xws(x_prepared);
    InputPrep ip;
    ip.xws = &xws; ip.mode = INPUT_PREPARE_ONLY;
    return fwd_nhwc(s, dtype, x, nullptr, nullptr, PostOp(), none, (hipStream_t)hip_stream, false, ip);
}

int mxc_conv2d_fwd_prepared_input(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, int dtype, int layout,
                                  const void *x_prepared, size_t prepared_bytes, const void *w, const float *bias, int relu,
                                  void *y, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    ConvShape s;
    MXC_TRY(validate_shape(N, C, H, W, K, R, S, stride, pad, dtype, layout, &s));
    if (layout != MXC_NHWC || (relu != 0 && relu != 1)) return MXC_ERR_UNSUPPORTED;
    if (!x_prepared || !w || !y) return MXC_ERR_NULL;
    if (misaligned(x_prepared) || misaligned(w) || misaligned(y) || misaligned(workspace) || ((uintptr_t)bias & 3u)) return MXC_ERR_ALIGN;
    size_t needx = 0;
    int form = FORM_AS_IS;
    MXC_TRY(prepared_input_plan(s, dtype, &needx, &form));
    if (prepared_bytes < needx) return MXC_ERR_WORKSPACE;
    PostOp post;
    post.bias = bias;
    post.relu = relu;
    InputPrep ip;
    Carver need(nullptr), nx(nullptr);
    if (needx) { ip.xws = &nx; ip.mode = INPUT_PREPARED; }
    MXC_TRY(fwd_nhwc(s, dtype, nullptr, nullptr, nullptr, PostOp(), need, nullptr, true, ip));
    if (need.used > 0 && (!workspace || workspace_bytes < need.used)) return MXC_ERR_WORKSPACE;
    Carver ws(workspace), xws(const_cast<void *>(x_prepared));
    if (needx) ip.xws = &xws;
    // an empty prepared form: x_prepared is x itself
    return fwd_nhwc(s, dtype, needx ? nullptr : x_prepared, w, y, post, ws, (hipStream_t)hip_stream, false, ip);
}

int mxc_conv2d_bwd_weight_prepared_input(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, int dtype,
                                         int layout, const void *x_prepared, size_t prepared_bytes, const void *dy, void *dw,
                                         int dw_dtype, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    ConvShape s;
    MXC_TRY(validate_shape(N, C, H, W, K, R, S, stride, pad, dtype, layout, &s));
    if (layout != MXC_NHWC || (dw_dtype != MXC_F32 && dw_dtype != MXC_BF16) || (dw_dtype == MXC_BF16 && dtype != MXC_BF16))
        return MXC_ERR_UNSUPPORTED;
    if (!x_prepared || !dy || !dw) return MXC_ERR_NULL;
    if (misaligned(x_prepared) || misaligned(dy) || misaligned(dw) || misaligned(workspace)) return MXC_ERR_ALIGN;
    size_t needx = 0;
    int form = FORM_AS_IS;
    MXC_TRY(prepared_input_plan(s, dtype, &needx, &form));
    if (prepared_bytes < needx) return MXC_ERR_WORKSPACE;
    InputPrep ip;
    Carver need(nullptr), nx(nullptr);
    if (needx) { ip.xws = &nx; ip.mode = INPUT_PREPARED; }
    MXC_TRY(bwd_weight_nhwc(s, dtype, nullptr, nullptr, nullptr, dw_dtype == MXC_BF16, need, nullptr, true, ip));
    if (need.used > 0 && (!workspace || workspace_bytes < need.used)) return MXC_ERR_WORKSPACE;
    Carver ws(workspace), xws(const_cast<void *>(x_prepared));
    if (needx) ip.xws = &xws;
    return bwd_weight_nhwc(s, dtype, needx ? nullptr : x_prepared, dy, dw, dw_dtype == MXC_BF16, ws, (hipStream_t)hip_stream, false, ip);
}

int mxc_conv2d_fwd_transform(int N, int C, int H, int W, int K, int R, int S, int stride, int pad, int dtype, int layout,
                             const void *x, const void *w, const float *bias, int relu, void *y, void *workspace,
                             size_t workspace_bytes, void *hip_stream)
{
    ConvShape s;
    MXC_TRY(validate_shape(N, C, H, W, K, R, S, stride, pad, dtype, layout, &s));
    if (dtype != MXC_BF16 || layout != MXC_NHWC || (relu != 0 && relu != 1) || !winograd_supported(s)) return MXC_ERR_UNSUPPORTED;
    if (!x || !w || !y) return MXC_ERR_NULL;
    if (misaligned(x) || misaligned(w) || misaligned(y) || misaligned(workspace) || ((uintptr_t)bias & 3u)) return MXC_ERR_ALIGN;
    size_t ub, vb, mb;
    winograd_workspace(s, &ub, &vb, &mb);
    Carver need(nullptr);
    need.take(ub); need.take(vb); need.take(mb);
    if (!workspace || workspace_bytes < need.used) return MXC_ERR_WORKSPACE;
    Carver ws(workspace);
    void *u = ws.take(ub), *v = ws.take(vb), *m = ws.take(mb);
    PostOp post;
    post.bias = bias;
    post.relu = relu;
    const char *vname = "";
    const int rc = winograd_fwd(s, x, w, y, u, v, m, (hipStream_t)hip_stream, &vname, post);
    if (rc == MXC_OK) set_variant("fwd", vname);
    return rc;
}

int mxc_bias_grad(int N, int K, int P, int Q, int dtype, int layout, const void *dy, float *db, void *workspace,
                  size_t workspace_bytes, void *hip_stream)
{
    if (N <= 0 || K <= 0 || P <= 0 || Q <= 0) return MXC_ERR_SHAPE;
    if ((long double)N * K * P * Q >= 1099511627776.0L) return MXC_ERR_SHAPE;
    if (dtype != MXC_F32 && dtype != MXC_BF16) return MXC_ERR_UNSUPPORTED;
    if (layout != MXC_NCHW && layout != MXC_NHWC) return MXC_ERR_UNSUPPORTED;
    if (!dy || !db) return MXC_ERR_NULL;
    if (misaligned(dy) || misaligned(db) || misaligned(workspace)) return MXC_ERR_ALIGN;
    const size_t need = bias_grad_scratch(N, K, (long long)P * Q, dtype, layout);
    if (!workspace || workspace_bytes < need) return MXC_ERR_WORKSPACE;
    return bias_grad(N, K, (long long)P * Q, dtype, layout, dy, db, (float *)workspace, (hipStream_t)hip_stream);
}

int mxc_fc_fwd(int N, int C, int K, int dtype, const void *x, const void *w, const float *bias, int relu, void *y,
               void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return mxc_conv2d_fwd_bias_act(N, C, 1, 1, K, 1, 1, 1, 0, dtype, MXC_NHWC, x, w, bias, relu, y, workspace, workspace_bytes,
                                   hip_stream);
}

int mxc_fc_bwd_data(int N, int C, int K, int dtype, const void *dy, const void *w, const void *x_mask, void *dx,
                    void *workspace, size_t workspace_bytes, void *hip_stream)
{
    PostOp post;
    post.mask = x_mask;
    return entry(MXC_BWD_DATA, N, C, 1, 1, K, 1, 1, 1, 0, dtype, MXC_NHWC, dy, w, dx, post, workspace, workspace_bytes, hip_stream);
}

int mxc_fc_bwd_weight(int N, int C, int K, int dtype, const void *x, const void *dy, void *dw,
                      void *workspace, size_t workspace_bytes, void *hip_stream)
{
    return mxc_conv2d_bwd_weight(N, C, 1, 1, K, 1, 1, 1, 0, dtype, MXC_NHWC, x, dy, dw, workspace, workspace_bytes, hip_stream);
}

int mxc_softmax_fwd(int N, int K, int dtype, const void *z, void *p, void *hip_stream)
{
    if (N <= 0 || K <= 0) return MXC_ERR_SHAPE;
    if (dtype != MXC_F32 && dtype != MXC_BF16) return MXC_ERR_UNSUPPORTED;
    if (!z || !p) return MXC_ERR_NULL;
    if (misaligned(z) || misaligned(p)) return MXC_ERR_ALIGN;
    return softmax_fwd(N, K, dtype, z, p, (hipStream_t)hip_stream);
}

int mxc_softmax_xent_bwd(int N, int K, int dtype, const void *p, const int *labels, float scale, void *dz, void *hip_stream)
{
    if (N <= 0 || K <= 0) return MXC_ERR_SHAPE;
    if (dtype != MXC_F32 && dtype != MXC_BF16) return MXC_ERR_UNSUPPORTED;
    if (!p || !labels || !dz) return MXC_ERR_NULL;
    if (misaligned(p) || misaligned(dz) || ((uintptr_t)labels & 3u)) return MXC_ERR_ALIGN;
    return softmax_xent_bwd(N, K, dtype, p, labels, dz, scale, (hipStream_t)hip_stream);
}

int mxc_sgd_update(size_t n, float *w, const float *g, float *v, void *w_bf16, float lr, float momentum, float wd, void *hip_stream)
{
    if (n == 0) return MXC_ERR_SHAPE;
    if (!w || !g) return MXC_ERR_NULL;
    if (!v && momentum != 0.f) return MXC_ERR_NULL;
    if (misaligned(w) || misaligned(g) || misaligned(v) || misaligned(w_bf16)) return MXC_ERR_ALIGN;
    return sgd_update(n, w, g, v, w_bf16, lr, momentum, wd, (hipStream_t)hip_stream);
}

int mxc_conv2d_workspace_bytes(int pass, int N, int C, int H, int W, int K, int R, int S, int stride, int pad,
                               int dtype, int layout, size_t *out_bytes)
{
    if (!out_bytes) return MXC_ERR_NULL;
    if (pass < MXC_FWD || pass > MXC_FWD_TRANSFORM) return MXC_ERR_UNSUPPORTED;
    if (pass == MXC_BWD_WEIGHT_BF16 && dtype != MXC_BF16) return MXC_ERR_UNSUPPORTED;
    ConvShape s;
    const int rc = validate_shape(N, C, H, W, K, R, S, stride, pad, dtype, layout, &s);
    if (rc != MXC_OK) return rc;
    if (pass == MXC_BIAS_GRAD) {
        *out_bytes = align_up(bias_grad_scratch(s.N, s.K, (long long)s.P * s.Q, dtype, layout), 256);
        return MXC_OK;
    }
    if (pass == MXC_FWD_TRANSFORM) {
        if (dtype != MXC_BF16 || layout != MXC_NHWC || !winograd_supported(s)) return MXC_ERR_UNSUPPORTED;
        size_t ub, vb, mb;
        winograd_workspace(s, &ub, &vb, &mb);
        Carver need(nullptr);
        need.take(ub); need.take(vb); need.take(mb);
        *out_bytes = need.used;
        return MXC_OK;
    }
    if (pass >= MXC_INPUT_PREPARED) {
        if (layout != MXC_NHWC || (pass == MXC_BWD_WEIGHT_PREPARED_INPUT_BF16 && dtype != MXC_BF16)) return MXC_ERR_UNSUPPORTED;
        size_t needx = 0;
        int form = FORM_AS_IS;
        MXC_TRY(prepared_input_plan(s, dtype, &needx, &form));
        if (pass == MXC_INPUT_PREPARED) { *out_bytes = needx; return MXC_OK; }
        InputPrep ip;
        Carver needw(nullptr), nx(nullptr);
        if (needx) { ip.xws = &nx; ip.mode = INPUT_PREPARED; }
        if (pass == MXC_FWD_PREPARED_INPUT) MXC_TRY(fwd_nhwc(s, dtype, nullptr, nullptr, nullptr, PostOp(), needw, nullptr, true, ip));
        else MXC_TRY(bwd_weight_nhwc(s, dtype, nullptr, nullptr, nullptr, pass == MXC_BWD_WEIGHT_PREPARED_INPUT_BF16, needw, nullptr, true, ip));
        *out_bytes = needw.used;
        return MXC_OK;
    }
    Carver need(nullptr), needf(nullptr);
    PostOp dry_post;
    dry_post.relu = pass == MXC_BWD_DATA_RELU || pass == MXC_BWD_DATA_PREPARED_RELU;
    if (pass == MXC_BWD_DATA_FILTER || pass == MXC_BWD_DATA_PREPARED || pass == MXC_BWD_DATA_PREPARED_RELU) {
        const FilterMode mode = pass == MXC_BWD_DATA_FILTER ? FILTER_PREPARE_ONLY : FILTER_PREPARED;
        const int rc3 = run_pass(MXC_BWD_DATA, s, dtype, layout, nullptr, nullptr, nullptr, dry_post, need, nullptr, true, &needf, mode);
        if (rc3 != MXC_OK) return rc3;
        *out_bytes = pass == MXC_BWD_DATA_FILTER ? needf.used : need.used;
        return MXC_OK;
    }
    const int rc2 = run_pass(pass == MXC_BWD_DATA_RELU ? MXC_BWD_DATA : pass, s, dtype, layout, nullptr, nullptr, nullptr, dry_post,
                             need, nullptr, true);
    if (rc2 != MXC_OK) return rc2;
    *out_bytes = need.used;
    return MXC_OK;
}

int mxc_layout_convert(int n, int c, int h, int w, int dtype, int src_layout, int dst_layout, const void *src,
                       void *dst, void *hip_stream)
{
    if (n <= 0 || c <= 0 || h <= 0 || w <= 0) return MXC_ERR_SHAPE;
    if ((long double)n * c * h * w >= 1099511627776.0L || !transpose_launchable(n, c, (long long)h * w) ||
        !transpose_launchable(n, (long long)h * w, c))
        return MXC_ERR_SHAPE;
    if (dtype != MXC_F32 && dtype != MXC_BF16) return MXC_ERR_UNSUPPORTED;
    if ((src_layout != MXC_NCHW && src_layout != MXC_NHWC) || (dst_layout != MXC_NCHW && dst_layout != MXC_NHWC))
        return MXC_ERR_UNSUPPORTED;
    if (!src || !dst) return MXC_ERR_NULL;
    if (misaligned(src) || misaligned(dst)) return MXC_ERR_ALIGN;
    const int eb = (int)elem_size(dtype);
    hipStream_t st = (hipStream_t)hip_stream;
    if (src_layout == dst_layout) return launch_copy(src, dst, (size_t)n * c * h * w * eb, st);
    if (src_layout == MXC_NCHW) return launch_transpose(src, dst, n, c, h * w, eb, st);
    return launch_transpose(src, dst, n, h * w, c, eb, st);
}

const char *mxc_status_string(int status)
{
    switch (status) {
    case MXC_OK: return "ok";
    case MXC_ERR_NULL: return "a required pointer is NULL";
    case MXC_ERR_SHAPE: return "invalid shape: non-positive dimension or stride, negative pad, or empty output";
    case MXC_ERR_UNSUPPORTED: return "unsupported dtype, layout or pass";
    case MXC_ERR_WORKSPACE: return "workspace missing or too small (see mxc_conv2d_workspace_bytes)";
    case MXC_ERR_ALIGN: return "a device pointer is not 16-byte aligned";
    case MXC_ERR_LAUNCH: return "the HIP runtime rejected a kernel launch";
    default: return "unknown status";
    }
}

const char *mxc_last_variant(void) { return g_variant; }

void mxc_last_plan_key(long long *M, int *Co, int *Kd)
{
    long long m = 0;
    int co = 0, kd = 0;
    igemm_last_plan_key(&m, &co, &kd);
    if (M) *M = m;
    if (Co) *Co = co;
    if (Kd) *Kd = kd;
}

long long mxc_plan_searches(void) { return g_plan_searches; }

int mxc_version(void) { return 400; }

const char *mxc_tile_name(int family, int index)
{
    return family == 0 ? igemm_tile_name(index) : family == 1 ? wgrad_tile_name(index) : family == 2 ? igemm_stream_name(index)
           : family == 3 ? f32_tile_name(index) : family == 4 ? wave_name(index) : family == 5 ? wave_dw_name(index)
           : family == 6 ? f32_wave_name(index) : family == 7 ? (index == 0 ? taps_dx_name() : nullptr) : family == 8 ? run_name(index)
           : family == 9 ? run_dw_name(index) : nullptr;
}

int mxc_probe_mfma(int workgroups, int iters, void *out, size_t out_bytes, double *flops, void *hip_stream)
{
    if (!out || !flops) return MXC_ERR_NULL;
    if (workgroups <= 0 || iters <= 0) return MXC_ERR_SHAPE;
    if (out_bytes < (size_t)workgroups * 256 * sizeof(float)) return MXC_ERR_WORKSPACE;
    if (misaligned(out)) return MXC_ERR_ALIGN;
    return probe_mfma(workgroups, iters, (float *)out, flops, (hipStream_t)hip_stream);
}

}  // extern "C"
