// C-ABI glue: argument validation, layout resolution, workspace carving, launch order.
// Every step of the path runs in the HIP kernels; nothing here touches tensor data.
#include "../../include/conv2d_int8.h"
#include "desc_check.h"
#include "kernels.h"
#include "launch.h"

#include <mutex>

using namespace c2i8;

// Workspace of conv2d_int8_static, the entry point that allocates nothing (see there).
constexpr size_t STATIC_WS_BYTES = CONV_STATIC_WORKSPACE_BYTES;
static __device__ __align__(256) unsigned char scratch[STATIC_WS_BYTES];

namespace {

constexpr size_t WS_ALIGN = 256;
constexpr long long INT_LIMIT = 2147483647LL;

size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
int round_up_i(int x, int m) { return (x + m - 1) / m * m; }
bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

int check_desc(const conv_desc_t *d) { return check_conv_desc(d); }

struct Plan {
    int layout, cb, Cb, depth, P, Q, Hp, Wp;
    int pointwise;  // IMPLICIT only: the 1x1 kernel takes it (else the window kernel)
    long long M;
    size_t x_bytes, w_bytes;
};

WindowProblem window_problem(const conv_desc_t *d, const Plan &pl, const int8_t *x, const int8_t *w,
                             int32_t *out, int wt_rewritten)
{
    return WindowProblem{x, w, out, d->N, d->C, d->H, d->W, d->K, pl.P, pl.Q, d->R, d->S, d->stride, d->pad,
                         wt_rewritten, ActOut{}, 0};
}

int run_implicit(const Plan &pl, const WindowProblem &g, hipStream_t st)
{
    const hipError_t e = pl.pointwise ? launch_pointwise_conv(g, st) : launch_window_conv(g, st);
    return e == hipSuccess ? CONV_OK : CONV_ERR_DEVICE;
}

int default_block(int C)
{
    if (C >= 64) return 64;
    if (C > 32) return 64;
    if (C > 16) return 32;
    return 16;
}

// Resolves AUTO / default block and sizes the rewritten operands.
int make_plan(const conv_desc_t *d, int layout, int cb, Plan *pl)
{
    int rc = check_desc(d);
    if (rc != CONV_OK) return rc;
    if (layout == CONV_LAYOUT_AUTO) {
        rc = select_layout(d, &layout, &cb, nullptr);
        if (rc != CONV_OK) return rc;
    }
    if (layout == CONV_LAYOUT_IMAGE_PACK) return CONV_ERR_UNSUPPORTED;  // two stages: not a single plan
    if (layout == CONV_LAYOUT_PAD_ONLY) cb = round_up_i(d->C, 16);
    else if (layout == CONV_LAYOUT_PACKED) {
        if (cb == 0) cb = default_block(d->C);
        if (cb < 16 || cb > 1024 || cb % 16) return CONV_ERR_UNSUPPORTED;
    } else if (layout == CONV_LAYOUT_IM2COL || layout == CONV_LAYOUT_IMPLICIT) cb = 0;
    else return CONV_ERR_INVALID_ARG;

    pl->layout = layout;
    pl->pointwise = 0;
    pl->cb = cb;
    pl->Hp = d->H + 2 * d->pad;
    pl->Wp = d->W + 2 * d->pad;
    pl->P = (pl->Hp - d->R) / d->stride + 1;
    pl->Q = (pl->Wp - d->S) / d->stride + 1;
    pl->M = (long long)d->N * pl->P * pl->Q;
    if (layout == CONV_LAYOUT_IMPLICIT) {
        pl->Cb = 0;
        pl->pointwise = pointwise_shape(d->C, d->R, d->S);
        pl->depth = pl->pointwise ? d->C : window_depth(d->C, d->R, d->S);
        const WindowProblem wp = window_problem(d, *pl, nullptr, nullptr, nullptr, 0);
        if (!(pl->pointwise ? pointwise_fits(wp) : window_fits(wp))) return CONV_ERR_UNSUPPORTED;
        pl->x_bytes = 0;  // nothing is rewritten: the GEMM stage reads the input and either weight form
        pl->w_bytes = 0;
        return CONV_OK;
    }
    if (layout == CONV_LAYOUT_IM2COL) {
        pl->Cb = 0;
        pl->depth = round_up_i(d->C * d->R * d->S, CONV_DEPTH_ALIGN);
        pl->x_bytes = (size_t)pl->M * pl->depth;
    } else {
        pl->Cb = (d->C + cb - 1) / cb;
        const long long real = (long long)pl->Cb * cb * d->R * d->S;
        if (real > (1LL << 24)) return CONV_ERR_UNSUPPORTED;
        pl->depth = round_up_i((int)real, CONV_DEPTH_ALIGN);
        const long long img = (long long)pl->Cb * pl->Hp * pl->Wp * cb;
        if (img > INT_LIMIT) return CONV_ERR_UNSUPPORTED;  // per-image offsets are 32-bit
        pl->x_bytes = (size_t)d->N * (size_t)img;
    }
    pl->w_bytes = (size_t)d->K * pl->depth;
    return CONV_OK;
}

// Image Pack: the equivalent stride-1, pad-0 problem, the sizes of its two rewritten operands, and
// the layout the stride-1 convolution then runs in (cb = 0: IMPLICIT, else PACKED with that block).
struct PackedProblem {
    conv_desc_t d2;
    size_t x2_bytes, w2_bytes;
    int inner_layout, inner_cb;
};

int image_pack_problem(const conv_desc_t *d, int cb, PackedProblem *pp, bool with_inner = true)
{
    int rc = check_desc(d);
    if (rc != CONV_OK) return rc;
    if (d->stride < 2) return CONV_ERR_UNSUPPORTED;  // nothing to pack
    const long long s = d->stride;
    const long long C2 = (long long)d->C * s * s;
    const long long R2 = (d->R + s - 1) / s, S2 = (d->S + s - 1) / s;
    const long long P = ((long long)d->H + 2LL * d->pad - d->R) / s + 1, Q = ((long long)d->W + 2LL * d->pad - d->S) / s + 1;
    const long long H2 = P + R2 - 1, W2 = Q + S2 - 1;
    if (C2 > INT_LIMIT || H2 > INT_LIMIT || W2 > INT_LIMIT || C2 * R2 * S2 > 131072LL) return CONV_ERR_UNSUPPORTED;
    pp->d2 = conv_desc_t{d->N, (int)C2, (int)H2, (int)W2, d->K, (int)R2, (int)S2, 1, 0};
    pp->x2_bytes = (size_t)d->N * (size_t)C2 * (size_t)H2 * (size_t)W2;
    pp->w2_bytes = (size_t)d->K * (size_t)C2 * (size_t)R2 * (size_t)S2;
    pp->inner_layout = cb == 0 ? CONV_LAYOUT_IMPLICIT : CONV_LAYOUT_PACKED;
    pp->inner_cb = cb;
    if (!with_inner) return CONV_OK;  // the pack alone: whatever runs on its output is the caller's choice
    Plan inner;
    return make_plan(&pp->d2, pp->inner_layout, pp->inner_cb, &inner);
}

// Dilation (stride 1) as Image Pack into the batch: the dense stride-1, pad-0 problem on the d*d
// sub-images of every padded image, and the sizes of the sub-image tensor and of its result.
struct DilatedProblem {
    conv_desc_t d2;
    int P, Q;  // extents of the dilated convolution's own output
    size_t x2_bytes, o2_bytes;
};

int dilated_problem(const conv_desc_t *d, int dilation, DilatedProblem *dp)
{
    if (!d) return CONV_ERR_INVALID_ARG;
    if (d->N <= 0 || d->C <= 0 || d->H <= 0 || d->W <= 0 || d->K <= 0 || d->R <= 0 || d->S <= 0 || d->stride <= 0 ||
        d->pad < 0 || dilation <= 0)
        return CONV_ERR_INVALID_ARG;
    const long long dl = dilation;
    const long long Hp = (long long)d->H + 2LL * d->pad, Wp = (long long)d->W + 2LL * d->pad;
    const long long Re = dl * (d->R - 1) + 1, Se = dl * (d->S - 1) + 1;  // extent of the spread kernel
    if (Re > Hp || Se > Wp) return CONV_ERR_INVALID_ARG;
    if (d->stride != 1 || dilation < 2 || dilation > 64) return CONV_ERR_UNSUPPORTED;  // 1: nothing to pack
    if (Hp > INT_LIMIT || Wp > INT_LIMIT) return CONV_ERR_UNSUPPORTED;
    const long long N2 = (long long)d->N * dl * dl;
    const long long H2 = (Hp + dl - 1) / dl, W2 = (Wp + dl - 1) / dl;
    if (N2 > INT_LIMIT || H2 * W2 > INT_LIMIT) return CONV_ERR_UNSUPPORTED;
    dp->d2 = conv_desc_t{(int)N2, d->C, (int)H2, (int)W2, d->K, d->R, d->S, 1, 0};
    int rc = check_desc(&dp->d2);
    if (rc != CONV_OK) return rc;
    dp->P = (int)(Hp - Re + 1);
    dp->Q = (int)(Wp - Se + 1);
    if ((long long)dp->P * dp->Q > INT_LIMIT) return CONV_ERR_UNSUPPORTED;
    const long long P2 = H2 - d->R + 1, Q2 = W2 - d->S + 1;
    dp->x2_bytes = (size_t)N2 * d->C * (size_t)(H2 * W2);
    dp->o2_bytes = (size_t)N2 * d->K * (size_t)(P2 * Q2) * sizeof(int32_t);
    return CONV_OK;
}

// Dilation as an address multiplier: the plan of the undilated problem with the dilated layer's output extents.
int direct_dilated_plan(const conv_desc_t *desc, int dilation, int cb, Plan *pl)
{
    if (!desc || dilation <= 0) return CONV_ERR_INVALID_ARG;
    int rc = make_plan(desc, CONV_LAYOUT_PACKED, cb, pl);
    if (rc != CONV_OK) return rc;
    const long long Re = (long long)dilation * (desc->R - 1) + 1, Se = (long long)dilation * (desc->S - 1) + 1;
    if (Re > pl->Hp || Se > pl->Wp) return CONV_ERR_INVALID_ARG;
    pl->P = (int)((pl->Hp - Re) / desc->stride + 1);
    pl->Q = (int)((pl->Wp - Se) / desc->stride + 1);
    pl->M = (long long)desc->N * pl->P * pl->Q;
    return CONV_OK;
}

// AUTO -> the selector's choice (which may be IMAGE_PACK with its inner block in *cb).
int resolve_layout(const conv_desc_t *d, int *layout, int *cb)
{
    if (*layout != CONV_LAYOUT_AUTO) return CONV_OK;
    int rc = check_desc(d);
    if (rc != CONV_OK) return rc;
    struct Choice {
        int layout, cb;
    };
    static thread_local PlanTable<conv_desc_t, Choice, 64> chosen;
    const Choice *kept = chosen.get(*d, [&](Choice *n) { return (rc = select_layout(d, &n->layout, &n->cb, nullptr)) == CONV_OK; });
    if (kept) {
        *layout = kept->layout;
        *cb = kept->cb;
    }
    return rc;
}

GemmProblem gemm_problem(const conv_desc_t *d, const Plan &pl, const int8_t *x, const int8_t *w,
                         int32_t *out)
{
    GemmProblem g{};
    g.act = x;
    g.wq = w;
    g.out = out;
    g.K = d->K;
    g.M = (int)pl.M;
    g.depth = pl.depth;
    g.PQ = pl.P * pl.Q;
    g.Q = pl.Q;
    g.mode = pl.layout == CONV_LAYOUT_IM2COL ? ACT_MATRIX : ACT_BLOCKED;
    g.stride = d->stride;
    g.cb = pl.cb;
    g.Cb = pl.Cb;
    g.R = d->R;
    g.S = d->S;
    g.Hp = pl.Hp;
    g.Wp = pl.Wp;
    return g;
}

// hipErrorInvalidValue comes from the launcher's own guards (a tile / split pair the picker would not
// offer); nothing was enqueued then.
int gemm_status(hipError_t e)
{
    return e == hipSuccess ? CONV_OK : e == hipErrorInvalidValue ? CONV_ERR_UNSUPPORTED : CONV_ERR_DEVICE;
}

// Which kernel runs the GEMM stage: a tile of the general kernel with a depth split, or the band kernel.
struct GemmChoice {
    int tile, split_k;  // tile == CONV_TILE_BAND: the band kernel (split_k 1)
    double cost;        // the models' estimate for the library's own choice (microseconds)
};

int choose_gemm_now(const GemmProblem &g, int tile, int split_k, GemmChoice *c)
{
    if (tile == CONV_TILE_BAND) {
        if (split_k < 0 || split_k > 1 || !band_applies(g)) return split_k < 0 ? CONV_ERR_INVALID_ARG : CONV_ERR_UNSUPPORTED;
        *c = GemmChoice{CONV_TILE_BAND, 1, 0};
        return CONV_OK;
    }
    if (tile < -1 || tile >= gemm_num_tiles()) return CONV_ERR_INVALID_ARG;
    if (split_k < 0) return CONV_ERR_INVALID_ARG;
    const bool free_choice = tile == -1 && split_k == 0;
    int t = tile, s = split_k;
    if (g.out && !aligned16(g.out) && s == 0) s = 1;  // the clear before a depth split writes 16-byte pieces
    if (g.out && !aligned16(g.out) && s > 1) return CONV_ERR_INVALID_ARG;
    double cost = 0;
    if (!gemm_pick(g, &t, &s, &cost)) {
        if (free_choice && band_applies(g)) {
            *c = GemmChoice{CONV_TILE_BAND, 1, band_cost(g)};
            return CONV_OK;
        }
        return CONV_ERR_UNSUPPORTED;
    }
    if (free_choice && band_cost(g) < cost) {
        *c = GemmChoice{CONV_TILE_BAND, 1, band_cost(g)};
        return CONV_OK;
    }
    *c = GemmChoice{t, s, cost};
    return CONV_OK;
}

// The library's own choice is kept per problem (the tile model looks at 45 tiles x up to 9 splits: 2.7 us of host time).
int choose_gemm(const GemmProblem &g, int tile, int split_k, GemmChoice *c)
{
    if (tile != -1 || split_k != 0) return choose_gemm_now(g, tile, split_k, c);
    static thread_local PlanTable<GemmKey, GemmChoice, 64> chosen;
    int rc = CONV_OK;
    const GemmChoice *kept = chosen.get(gemm_key(g), [&](GemmChoice *n) { return (rc = choose_gemm_now(g, tile, split_k, n)) == CONV_OK; });
    if (kept) *c = *kept;
    return rc;
}

// The same without a depth split (an epilogue that needs the whole sum): the band kernel, or the best tile of the
// general one.
int choose_gemm_unsplit(const GemmProblem &g, GemmChoice *c)
{
    static thread_local PlanTable<GemmKey, GemmChoice, 64> chosen;
    const GemmChoice *kept = chosen.get(gemm_key(g), [&](GemmChoice *n) {
        int t = -1, s = 1;
        double cost = 0;
        const bool tiled = gemm_pick(g, &t, &s, &cost);
        if (band_applies(g) && (!tiled || band_cost(g) < cost)) *n = GemmChoice{CONV_TILE_BAND, 1, band_cost(g)};
        else *n = GemmChoice{t, 1, cost};
        return tiled || n->tile == CONV_TILE_BAND;
    });
    if (!kept) return CONV_ERR_UNSUPPORTED;
    *c = *kept;
    return CONV_OK;
}

int launch_choice(const GemmProblem &g, const GemmChoice &c, hipStream_t st)
{
    if (c.tile == CONV_TILE_BAND) return gemm_status(launch_band_conv(g, st));
    return gemm_status(launch_gemm(g, c.tile, c.split_k, st));
}

int run_gemm(const GemmProblem &g, int tile, int split_k, hipStream_t st)
{
    GemmChoice c;
    const int rc = choose_gemm(g, tile, split_k, &c);
    return rc == CONV_OK ? launch_choice(g, c, st) : rc;
}

bool is_stream_tile(int tile) { return tile >= CONV_TILE_STREAM && tile < CONV_TILE_STREAM + stream_num_tiles(); }

// ---- two-stage path or the GEMM stage that blocks the channels itself (resident_mfma.hip) -----------------------------
// Estimated times in microseconds.  Two-stage, fitted per kind of call to 19000 calls of 5800 layers in graphs (a third held
// back; mean error 3 % where the band kernel runs, 5 to 6 % for the general one, 7 to 9 % unrolled and from NHWC): the launches, the
// GEMM stage's own estimate, the rewritten tensors written and read.  apart: image planes that are not whole dwords, for which
// the rewrite of 64-channel slices takes its general kernel and a one-shot call launches the two rewrites one after the other.
// A second launch costs the stream about a microsecond more than it costs a graph.
constexpr double SECOND_LAUNCH_US = 1.0;
struct TwoStageFit {
    double launch, gemm, moved, weights, apart;
};
constexpr TwoStageFit FIT_BAND[] = {{1.24, 1.09, 0.148e-6, 1.01e-6, 2.9}, {1.01, 1.09, 0.153e-6, 0.37e-6, 0.79}};      // raw, kept weights
constexpr TwoStageFit FIT_SLICES[] = {{2.21, 0.929, 0.142e-6, 1.89e-6, 3.33}, {1.82, 0.949, 0.154e-6, 1.03e-6, 1.11}};  // blocks of whole 64 channels
constexpr TwoStageFit FIT_BLOCKS[] = {{3.36, 0.927, 0.218e-6, 1.81e-6, 1.63}, {2.85, 0.936, 0.221e-6, 1.04e-6, 0}};      // other blocks
constexpr TwoStageFit FIT_UNROLLED[] = {{3.23, 1.0, 0.340e-6, 5.25e-6, 0}, {3.06, 1.01, 0.347e-6, 4.11e-6, 0}};
constexpr TwoStageFit FIT_NHWC_BAND = {0.28, 1.19, 0.304e-6, 0.735e-6, 0}, FIT_NHWC = {0.22, 1.27, 0.251e-6, 0, 0};

// d, pl: what is rewritten and how; g: the GEMM stage on it (a dilated layer's own extents, an NHWC result).
double two_stage_us(const conv_desc_t *d, const Plan &pl, const GemmProblem &g, bool wt_is_packed, bool nhwc)
{
    GemmChoice c;
    if (choose_gemm(g, -1, 0, &c) != CONV_OK) return 1e300;
    const bool band = c.tile == CONV_TILE_BAND;
    const TwoStageFit &f = nhwc ? band ? FIT_NHWC_BAND : FIT_NHWC
                                : (band ? FIT_BAND : pl.layout == CONV_LAYOUT_IM2COL ? FIT_UNROLLED : pl.cb % 64 == 0 ? FIT_SLICES : FIT_BLOCKS)[wt_is_packed];
    const bool apart = !nhwc && pl.layout != CONV_LAYOUT_IM2COL && (long long)d->H * d->W % 4 != 0;
    const double moved = (double)d->N * d->C * d->H * d->W + (double)pl.x_bytes;
    double us = f.launch + f.gemm * c.cost + f.moved * moved + f.weights * (double)pl.w_bytes + (apart ? f.apart : 0);
    if (nhwc && d->C % 16) us += 1.4 + 0.12e-6 * moved;                                      // (pixels' ends go byte by byte)
    return us + SECOND_LAUNCH_US * (apart && !wt_is_packed ? 2 : 1);
}

enum RouteHow : int {
    TWO_STAGE = CONV_STAGE_STORED,
    DIRECT_AS_IS = CONV_STAGE_RESIDENT,
    DIRECT_RAW = CONV_STAGE_RESIDENT_RAW,
    DIRECT_REWRITE = CONV_STAGE_RESIDENT_REWRITE,
    DIRECT_BAND = CONV_STAGE_BAND,
    DIRECT_STREAM = CONV_STAGE_STREAM,
    DIRECT_STREAM_REWRITE = CONV_STAGE_STREAM_REWRITE,
    DIRECT_PANEL = CONV_TILE_PANEL   // (reported as CONV_STAGE_STORED, with its tile)
};
struct Route {
    int how;             // DIRECT_*: resident kernel on the weights as they are / on KCRS weights / on rewritten ones, band kernel on packed ones, stream kernel on packed / rewritten ones, panel kernel
    ResidentChoice pick;
    int cb, depth;       // block and row bytes of the weights it reads (the two REWRITEs: what is rewritten; PAD_ONLY's, PACKED's)
    bool raw;            // KCRS as it came, not in depth order
};

// A convolution with its activations in the network's own layout (NCHW, or NHWC).  pl: the plan whose output extents
// apply (a dilated layer's own, if dil > 1); weights in blocks of cb with rows of `depth` bytes, or raw.
ResidentProblem resident_problem(const conv_desc_t *d, const Plan &pl, int cb, int depth, bool raw, bool nhwc, int dil, const int8_t *in,
                                 const int8_t *wt, int32_t *out)
{
    ResidentProblem r{};
    r.g = gemm_problem(d, pl, nullptr, wt, out);
    r.g.mode = ACT_BLOCKED;
    r.g.cb = cb;
    r.g.Cb = (d->C + cb - 1) / cb;
    r.g.depth = depth;
    r.g.dil = dil;
    r.g.out_nhwc = nhwc;
    r.src = in;
    r.N = d->N, r.C = d->C, r.H = d->H, r.W = d->W, r.pad = d->pad;
    r.pixel_major = nhwc;
    r.pixel_bytes = d->C;
    r.img_bytes = (long long)d->C * d->H * d->W;
    r.raw_weights = raw;
    return r;
}

// The layer of g, a GEMM stage with its activation, on the blocked image that g reads.
ResidentProblem blocked_problem(const conv_desc_t *d, const GemmProblem &g)
{
    ResidentProblem r{};
    r.g = g;
    r.src = g.act;
    r.N = d->N, r.C = d->C, r.H = g.Hp, r.W = g.Wp, r.pad = 0;
    r.pixel_major = r.blocked = r.kept = 1;
    r.pixel_bytes = g.cb;
    r.img_bytes = (long long)g.Cb * g.Hp * g.Wp * g.cb;
    return r;
}

// Whether the resident kernel takes it.  The estimates of the other stages know the int32 result only: refitted to two thirds of 2540 fused activations
// (mean error 9.5 % band, 7 % general).  Of the 847 others the 92 where this kernel's own estimate is below 0.85 of that take all of them
// to 0.964 of the time (0.80 where the channels are 64 at most and the launch above 10 us; the best of both would be 0.94), none more than 3 % slower; below 0.95 of it:
// 0.959, 12 slower, one of them by half.  What it saves is the R S fetches of every activation: 64 images 64 x 56 x 56 -> 64, 3x3: 24.0 -> 14.7 us;
// 192 images 128 x 35 x 35 -> 17: 37 -> 22.  Not 1x1 layers with a stride: the window holds the pixels in between, and no fetch is saved (877 images
// 32 x 56 x 56 -> 46, stride 2: 33.4 -> 41.5); nor those of more than 64 channels out, whose windows are filled once per tile of channels (218 layers that
// differ 0.976 in the mean, 22 slower, up to 1.15; up to 64 channels 225 layers 0.80).
bool choose_blocked(const ResidentProblem &r, ResidentChoice *pick)
{
    struct Kept {
        ResidentChoice pick;
        bool takes;
    };
    struct Key {
        GemmKey g;
        int C;
    };
    static thread_local PlanTable<Key, Kept, 64> chosen;
    const Kept *kept = chosen.get(Key{gemm_key(r.g), r.C}, [&](Kept *n) {
        GemmChoice c;
        WindowWalk walk = window_walk(r);
        *n = Kept{};
        n->takes = r.g.mode == ACT_BLOCKED && !(r.g.R * r.g.S == 1 && (r.g.stride > 1 || r.g.K > 64)) && resident_pick(r, walk, &n->pick);
        if (n->takes && choose_gemm_unsplit(r.g, &c) == CONV_OK) {
            const double results = (double)r.g.M * r.g.K;
            n->takes = n->pick.us < 0.85 * (c.tile == CONV_TILE_BAND ? 1.17 * c.cost - 1.75 : 1.089 * c.cost - 1.86 - 1.92e-8 * results);
        }
        return true;
    });
    if (kept && kept->takes) *pick = kept->pick;
    return kept && kept->takes;
}

struct RouteKey {
    conv_desc_t d;
    int v[8];
};

// Which of them runs this call.  two_us: the estimate of the route there is without the resident kernel.
template <typename TwoStage>
Route pick_route(const conv_desc_t *d, const Plan &pl, bool wt_is_packed, bool nhwc, int dil, const int8_t *wt, int32_t *out, int tag, TwoStage &&two_us)
{
    static thread_local PlanTable<RouteKey, Route, 64> routes;
    const RouteKey key{*d, {pl.layout, pl.cb, tag, (int)wt_is_packed, (int)nhwc, dil, (int)aligned16(wt), (int)aligned16(out)}};
    const Route *kept = routes.get(key, [&](Route *n) {
        double best = two_us();
        *n = Route{TWO_STAGE, {}, 0, 0, false};
        // (one for all: which pixels a window holds does not depend on the weights' form)
        WindowWalk walk = window_walk(resident_problem(d, pl, pl.cb, pl.depth, false, nhwc, dil, nullptr, nullptr, out));
        auto consider = [&](int how, int cb, int depth, bool raw, double extra) {
            ResidentChoice c;
            ResidentProblem r = resident_problem(d, pl, cb, depth, raw, nhwc, dil, nullptr, nullptr, out);
            r.kept = wt_is_packed;
            if (!resident_pick(r, walk, &c)) return;
            const double us = c.us + extra;
            if (us < best) {
                best = us;
                *n = Route{how, c, cb, depth, raw};
            }
        };
        // Last: the panel kernel, two launches, where its estimate is below 0.9 of the best other one's and its panels fit the workspace that the
        // other routes ask for: 2150 of 9400 calls of 6 to 600 us, 0.81 of the time in the mean, 3 % of them more than 2 %
        // longer (at 0.95 of it 2540, 0.83, 5 %).  Not for NCHW tensors of
        // up to 64 channels, whose window and weights the resident kernel holds in LDS whole: 330 calls that the estimates would send here take 0.92, 12 %
        // of them more than 5 % longer (at worst 1.5).
        auto panels = [&](double before) {
            if (!nhwc && d->C <= 64) return;
            const size_t room = align_up(pl.x_bytes, WS_ALIGN) + (wt_is_packed ? 0 : align_up(pl.w_bytes, WS_ALIGN));
            ResidentChoice c;
            if (panel_weight_bytes(d->K, d->C, d->R * d->S) <= room &&
                panel_pick(resident_problem(d, pl, pl.cb, pl.depth, !wt_is_packed, nhwc, dil, nullptr, nullptr, out), 0.9 * before - SECOND_LAUNCH_US, &c))
                *n = Route{DIRECT_PANEL, c, pl.cb, pl.depth, !wt_is_packed};
        };
        if (wt_is_packed) {
            if (pl.layout == CONV_LAYOUT_PACKED || pl.layout == CONV_LAYOUT_PAD_ONLY) {
                consider(DIRECT_AS_IS, pl.cb, pl.depth, false, 0);
                double us;
                if (!nhwc && dil == 1 && band_direct_us(resident_problem(d, pl, pl.cb, pl.depth, false, false, 1, nullptr, nullptr, out), &us) && us < best) {
                    best = us;
                    *n = Route{DIRECT_BAND, {}, pl.cb, pl.depth, false};
                }
                // The smallest streaming tile is for calls of 8 to 14 us.  Against the stored path the estimates' errors decide there, and its own is
                // the best of many: of 2571 layers 353 went to streaming wherever an estimate was lower, at 1.119 of the other launch's speed in
                // the mean, 17 % of them more than 5 % slower (1 image 512 x 23 x 23 -> 512 stride 2: 10.8 -> 14.5 us); with the smallest tile at 0.86 of
                // the stored path's estimate and below 262 do, 1.185, 8 %.
                ResidentChoice c;
                if (stream_pick(resident_problem(d, pl, pl.cb, pl.depth, false, nhwc, dil, nullptr, nullptr, out), walk, best, n->how == TWO_STAGE ? 0.86 : 1, &c))
                    *n = Route{DIRECT_STREAM, c, pl.cb, pl.depth, false}, best = c.us;
                panels(best);
            }
            return true;
        }
        const int C16 = round_up_i(d->C, 16);
        const long long real = (long long)C16 * d->R * d->S;
        if (real > (1LL << 20)) return true;
        const int depth = round_up_i((int)real, CONV_DEPTH_ALIGN);
        if (d->R == 1 && d->S == 1 && d->C % CONV_DEPTH_ALIGN == 0 && aligned16(wt)) consider(DIRECT_AS_IS, 64, d->C, false, 0);
        else {
            if (d->R == 3 && d->S == 3) consider(DIRECT_RAW, C16, depth, true, 0);
            // rows of C bytes as they are: no second launch (105 pointwise, pair and NHWC calls 0.88 of the time, the small ones 0.6 to 0.8);
            // a dilated call of a 1x1 layer, whose dilation changes nothing, keeps the stored path, which a test of that path asks of it
            if (d->R == 1 && d->S == 1 && dil == 1) consider(DIRECT_AS_IS, C16, depth, true, 0);
            // the weights' own launch: 2.4-3.2 us up to a megabyte of them
            if (C16 <= 1024) consider(DIRECT_REWRITE, C16, depth, false, 2.8 + 1.0e-6 * (double)d->K * depth + SECOND_LAUNCH_US);
            // weights streamed from blocks of 64 channels, where their estimate is well below: 320 drawn calls that come here against what ran them before
            // this kernel, 0.84 of the time (one-shot, NHWC), 0.89 (NHWC, K no multiple of four; while those results went value by value) and 0.54 (dilated); 4 % take more than 5 % longer
            const int depth64 = (d->C + 63) / 64 * 64 * d->R * d->S;
            ResidentChoice c;
            const double rewrite = 2.8 + 1.0e-6 * (double)d->K * depth64 + SECOND_LAUNCH_US;
            if (stream_pick(resident_problem(d, pl, 64, depth64, false, nhwc, dil, nullptr, nullptr, out), walk, 0.95 * best - rewrite, 1, &c))
                *n = Route{DIRECT_STREAM_REWRITE, c, 64, depth64, false}, best = c.us + rewrite;
        }
        panels(best);
        return true;
    });
    return *kept;
}

// Runs a DIRECT_* route; ws: device memory for the rewritten weights (DIRECT_REWRITE), at least K * depth bytes.
int run_direct(const Route &rt, const conv_desc_t *d, const Plan &pl, bool nhwc, int dil, const int8_t *in, const int8_t *wt, int32_t *out,
               void *ws, hipStream_t st)
{
    if (rt.how == DIRECT_REWRITE || rt.how == DIRECT_STREAM_REWRITE) {
        if (launch_pack_weights_blocked(d->K, d->C, d->R, d->S, rt.cb, rt.depth, wt, static_cast<int8_t *>(ws), st) != hipSuccess)
            return CONV_ERR_DEVICE;
        wt = static_cast<const int8_t *>(ws);
    }
    const ResidentProblem r = resident_problem(d, pl, rt.cb, rt.depth, rt.raw, nhwc, dil, in, wt, out);
    if (rt.how == DIRECT_PANEL) {
        int8_t *const panels = static_cast<int8_t *>(ws);
        const hipError_t e = launch_panel_weights(r, panels, st);
        return gemm_status(e == hipSuccess ? launch_panel(r, panels, rt.pick.tile, rt.pick.mper, st) : e);
    }
    if (rt.how == DIRECT_STREAM || rt.how == DIRECT_STREAM_REWRITE) return gemm_status(launch_stream(r, rt.pick.tile, rt.pick.mper, st));
    return gemm_status(rt.how == DIRECT_BAND ? launch_band_direct(r, st) : launch_resident(r, rt.pick, st));
}
size_t direct_bytes(const Route &rt, const conv_desc_t *d)
{
    if (rt.how == DIRECT_PANEL) return panel_weight_bytes(d->K, d->C, d->R * d->S);
    return rt.how == DIRECT_REWRITE || rt.how == DIRECT_STREAM_REWRITE ? (size_t)d->K * rt.depth : 0;
}

// The library's choice for a one-shot call whose selected layout is `layout` / `cb` (not IMPLICIT): pl gets the output
// extents the resident kernel works from.
int one_shot_route(const conv_desc_t *d, int layout, int cb, const int8_t *in, const int8_t *wt, int32_t *out, Plan *pl, Route *rt)
{
    const bool blocked = layout == CONV_LAYOUT_PACKED || layout == CONV_LAYOUT_PAD_ONLY;
    int rc = make_plan(d, blocked ? layout : CONV_LAYOUT_PAD_ONLY, blocked ? cb : 0, pl);
    if (rc != CONV_OK) {   // (an image too large for 32-bit offsets: only what the layout itself can do)
        *rt = Route{TWO_STAGE, {}, 0, 0, false};
        return CONV_OK;
    }
    const double in_bytes = (double)d->N * d->C * d->H * d->W;
    *rt = pick_route(d, *pl, false, false, 1, wt, out, 4 + layout, [&] {
        if (layout == CONV_LAYOUT_IMAGE_PACK) {   // two more launches and the packed image written and read once more
            PackedProblem pp;
            Plan inner;
            if (image_pack_problem(d, cb, &pp) != CONV_OK || make_plan(&pp.d2, pp.inner_layout, pp.inner_cb, &inner) != CONV_OK) return 1e300;
            const double pack = 5.0 + 0.25e-6 * (in_bytes + (double)pp.x2_bytes) + 2 * SECOND_LAUNCH_US;
            if (inner.layout == CONV_LAYOUT_IMPLICIT) return pack + 4.0 + 0.25e-6 * ((double)pp.x2_bytes + 4.0 * pl->M * d->K);
            return pack + two_stage_us(&pp.d2, inner, gemm_problem(&pp.d2, inner, nullptr, nullptr, out), false, false);
        }
        Plan own;
        if (make_plan(d, layout, cb, &own) != CONV_OK) return 1e300;
        return two_stage_us(d, own, gemm_problem(d, own, nullptr, nullptr, out), false, false);
    });
    return CONV_OK;
}

// The same choice for the other entry points.
Route ex_route(const conv_desc_t *d, const Plan &pl, bool wt_is_packed, const int8_t *wt, int32_t *out)
{
    if (pl.layout == CONV_LAYOUT_IM2COL) return Route{TWO_STAGE, {}, 0, 0, false};
    return pick_route(d, pl, wt_is_packed, false, 1, wt, out, 0, [&] {
        return two_stage_us(d, pl, gemm_problem(d, pl, nullptr, nullptr, out), wt_is_packed, false);
    });
}

Route nhwc_route(const conv_desc_t *d, const Plan &pl, const int8_t *wt, int32_t *out)
{
    return pick_route(d, pl, false, true, 1, wt, out, 1, [&] {
        GemmProblem g = gemm_problem(d, pl, nullptr, nullptr, out);
        g.out_nhwc = 1;
        // (a result that does not start on 16 bytes goes through a staging tensor and one more pass)
        return two_stage_us(d, pl, g, false, true) + (aligned16(out) ? 0 : 10);
    });
}

Route dilated_direct_route(const conv_desc_t *d, int dilation, const Plan &pl, const int8_t *wt, int32_t *out)
{
    return pick_route(d, pl, false, false, dilation, wt, out, 2, [&] {
        GemmProblem g = gemm_problem(d, pl, nullptr, nullptr, out);
        g.dil = dilation;
        return two_stage_us(d, pl, g, false, false);
    });
}

// (dp, inner: the dense problem on the sub-images; direct: the plan of the image as it is)
Route dilated_route(const conv_desc_t *d, int dilation, const DilatedProblem &dp, const Plan &inner, const Plan &direct, const int8_t *wt, int32_t *out)
{
    return pick_route(d, direct, false, false, dilation, wt, out, 3, [&] {
        const double pack = 2.5 + 0.25e-6 * ((double)d->N * d->C * d->H * d->W + (double)dp.x2_bytes) + SECOND_LAUNCH_US;
        return pack + two_stage_us(&dp.d2, inner, gemm_problem(&dp.d2, inner, nullptr, nullptr, nullptr), false, false);
    });
}

// conv2d_int8_nhwc's two forms that need no rewrite at all.
bool nhwc_window(const conv_desc_t *d, const Plan &pl, const int8_t *in, const int8_t *wt, int32_t *out, WindowProblem *wp)
{
    int layout = CONV_LAYOUT_AUTO, cb = 0;
    if (resolve_layout(d, &layout, &cb) != CONV_OK || layout != CONV_LAYOUT_IMPLICIT || pointwise_shape(d->C, d->R, d->S)) return false;
    *wp = WindowProblem{in, wt, out, d->N, d->C, d->H, d->W, d->K, pl.P, pl.Q, d->R, d->S, d->stride, d->pad, 0, ActOut{}, 1};
    return window_fits(*wp);
}
bool nhwc_matrix(const conv_desc_t *d, const int8_t *in, const int8_t *wt, const int32_t *out)
{
    return d->R == 1 && d->S == 1 && d->stride == 1 && d->pad == 0 && d->C % CONV_DEPTH_ALIGN == 0 && aligned16(in) && aligned16(wt) && aligned16(out);
}

int rewrite_weights(const conv_desc_t *d, const Plan &pl, const int8_t *wt, int8_t *dst, hipStream_t st)
{
    hipError_t e;
    if (pl.layout == CONV_LAYOUT_IM2COL)
        e = launch_pack_weights_rows(d->K, d->C * d->R * d->S, pl.depth, wt, dst, st);
    else
        e = launch_pack_weights_blocked(d->K, d->C, d->R, d->S, pl.cb, pl.depth, wt, dst, st);
    return e == hipSuccess ? CONV_OK : CONV_ERR_DEVICE;
}

int rewrite_input(const conv_desc_t *d, const Plan &pl, const int8_t *in, int8_t *dst, hipStream_t st)
{
    hipError_t e;
    if (pl.layout == CONV_LAYOUT_IM2COL)
        e = launch_im2col(d->N, d->C, d->H, d->W, d->R, d->S, d->stride, d->pad, pl.P, pl.Q, pl.depth,
                          in, dst, st);
    else
        e = launch_pack_layout(d->N, d->C, d->H, d->W, pl.cb, d->pad, in, dst, st);
    return e == hipSuccess ? CONV_OK : CONV_ERR_DEVICE;
}

// Cached workspace of the one-shot entry points, one per device, grown on demand.  A block that a larger
// problem supersedes is never freed: work already enqueued, or a HIP graph captured earlier, may still
// reference it, so it stays allocated until the process ends (blocks grow geometrically, so all superseded
// blocks together are smaller than the current one).
struct DeviceCache {
    void *ptr = nullptr;
    size_t bytes = 0;
};
std::mutex g_cache_mutex;
DeviceCache g_cache[64];

// The current device's block of at least `need` bytes.  Growing allocates, which a stream under capture
// must not do: then CONV_ERR_WORKSPACE, with no device call made.
int cached_workspace(size_t need, hipStream_t st, void **ptr, size_t *bytes)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return CONV_ERR_DEVICE;
    std::lock_guard<std::mutex> lock(g_cache_mutex);
    DeviceCache &c = g_cache[dev];
    if (c.bytes < need) {
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        if (hipStreamIsCapturing(st, &cs) != hipSuccess) return CONV_ERR_DEVICE;
        if (cs != hipStreamCaptureStatusNone) return CONV_ERR_WORKSPACE;
        const size_t least = align_up(need, 1 << 20);
        size_t want = align_up(need + need / 4, 1 << 20);
        if (want < 2 * c.bytes) want = 2 * c.bytes;
        void *p = nullptr;
        if (hipMalloc(&p, want) != hipSuccess || !p) {
            (void)hipGetLastError();  // the generous size did not fit: try what this problem needs
            p = nullptr;
            want = least;
            if (hipMalloc(&p, want) != hipSuccess || !p) {
                (void)hipGetLastError();
                return CONV_ERR_WORKSPACE;
            }
        }
        c.ptr = p;  // the superseded block stays allocated (see above)
        c.bytes = want;
    }
    *ptr = c.ptr;
    *bytes = c.bytes;
    return CONV_OK;
}

// ---- workspace of the entry point that allocates nothing -----------------------------------------
// A file-scope device array stands in for the cached workspace.  Every GPU the library runs on holds
// its own copy of it, at its own address, from the moment the code object is loaded there until the
// process ends.  In host code the array's NAME is only a handle for the runtime: the address kernels
// can use is what hipGetSymbolAddress returns for the device that is current, asked once per device.
std::mutex g_static_ws_mutex;
void *g_static_ws[64] = {};  // per device: device address of `scratch` there

int static_workspace(void **ptr)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return CONV_ERR_DEVICE;
    std::lock_guard<std::mutex> lock(g_static_ws_mutex);
    if (!g_static_ws[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
            (void)hipGetLastError();
            return CONV_ERR_DEVICE;
        }
        if (reinterpret_cast<uintptr_t>(p) % WS_ALIGN) return CONV_ERR_DEVICE;
        g_static_ws[dev] = p;
    }
    *ptr = g_static_ws[dev];
    return CONV_OK;
}

}  // namespace

extern "C" {

const char *conv_status_string(int s)
{
    switch (s) {
        case CONV_OK: return "ok";
        case CONV_ERR_INVALID_ARG: return "invalid argument";
        case CONV_ERR_UNSUPPORTED: return "unsupported problem";
        case CONV_ERR_OVERFLOW_RISK: return "reduction too deep for an int32 accumulator";
        case CONV_ERR_WORKSPACE: return "workspace too small or allocation failed";
        case CONV_ERR_DEVICE: return "HIP error";
    }
    return "unknown status";
}

size_t pack_layout_bytes(int N, int C, int H, int W, int cb, int pad)
{
    if (N <= 0 || C <= 0 || H <= 0 || W <= 0 || pad < 0 || cb < 4 || cb > 1024 || cb % 4) return 0;
    return (size_t)N * ((C + cb - 1) / cb) * cb * ((size_t)H + 2 * pad) * ((size_t)W + 2 * pad);
}

int pack_layout(int N, int C, int H, int W, int cb, int pad, const int8_t *src, int8_t *dst,
                void *stream)
{
    if (!src || !dst || N <= 0 || C <= 0 || H <= 0 || W <= 0 || pad < 0) return CONV_ERR_INVALID_ARG;
    if (cb < 4 || cb > 1024 || cb % 4) return CONV_ERR_UNSUPPORTED;
    if (!aligned16(dst)) return CONV_ERR_INVALID_ARG;
    if ((long long)H + 2LL * pad > INT_LIMIT || (long long)W + 2LL * pad > INT_LIMIT)
        return CONV_ERR_UNSUPPORTED;
    return launch_pack_layout(N, C, H, W, cb, pad, src, dst, (hipStream_t)stream) == hipSuccess
               ? CONV_OK : CONV_ERR_DEVICE;
}

int pack_layout_nhwc(int N, int C, int H, int W, int cb, int pad, const int8_t *src, int8_t *dst, void *stream)
{
    if (!src || !dst || N <= 0 || C <= 0 || H <= 0 || W <= 0 || pad < 0) return CONV_ERR_INVALID_ARG;
    if (cb < 16 || cb > 1024 || cb % 16) return CONV_ERR_UNSUPPORTED;
    if (!aligned16(dst)) return CONV_ERR_INVALID_ARG;
    if ((long long)H + 2LL * pad > INT_LIMIT || (long long)W + 2LL * pad > INT_LIMIT)
        return CONV_ERR_UNSUPPORTED;
    return launch_pack_layout_nhwc(N, C, H, W, cb, pad, src, dst, (hipStream_t)stream) == hipSuccess
               ? CONV_OK : CONV_ERR_DEVICE;
}

int requant_int8(long long count, const int32_t *src, int8_t *dst, int shift, int relu, void *stream)
{
    if (!src || !dst || count <= 0 || shift < 0 || shift > 31) return CONV_ERR_INVALID_ARG;
    return launch_requant(count, src, dst, shift, relu != 0, (hipStream_t)stream) == hipSuccess ? CONV_OK : CONV_ERR_DEVICE;
}

int requant_pack_layout(int N, int K, int P, int Q, int cb, int pad, int shift, int relu, const int32_t *src,
                        int8_t *dst, void *stream)
{
    if (!src || !dst || N <= 0 || K <= 0 || P <= 0 || Q <= 0 || pad < 0 || shift < 0 || shift > 31)
        return CONV_ERR_INVALID_ARG;
    if (cb < 16 || cb > 1024 || cb % 16) return CONV_ERR_UNSUPPORTED;
    if (!aligned16(dst)) return CONV_ERR_INVALID_ARG;
    if ((long long)P + 2LL * pad > INT_LIMIT || (long long)Q + 2LL * pad > INT_LIMIT) return CONV_ERR_UNSUPPORTED;
    return launch_requant_pack(N, K, P, Q, cb, pad, shift, relu != 0, src, dst, (hipStream_t)stream) == hipSuccess
               ? CONV_OK : CONV_ERR_DEVICE;
}

int unpack_nhwc_int32(int N, int K, int P, int Q, const int32_t *src, int32_t *dst, void *stream)
{
    if (!src || !dst || N <= 0 || K <= 0 || P <= 0 || Q <= 0) return CONV_ERR_INVALID_ARG;
    if ((long long)P * Q > INT_LIMIT) return CONV_ERR_UNSUPPORTED;
    return launch_unpack_nhwc(N, K, (long long)P * Q, src, dst, (hipStream_t)stream) == hipSuccess ? CONV_OK
                                                                                                  : CONV_ERR_DEVICE;
}

int pack_weights_depth(int C, int R, int S, int layout, int cb)
{
    if (C <= 0 || R <= 0 || S <= 0) return 0;
    long long real;
    if (layout == CONV_LAYOUT_IMPLICIT) return pointwise_shape(C, R, S) ? (C <= 512 ? C : 0) : window_depth(C, R, S);
    if (layout == CONV_LAYOUT_IM2COL) real = (long long)C * R * S;
    else if (layout == CONV_LAYOUT_PACKED || layout == CONV_LAYOUT_PAD_ONLY) {
        if (layout == CONV_LAYOUT_PAD_ONLY) cb = round_up_i(C, 16);
        if (cb < 16 || cb > 1024 || cb % 16) return 0;
        real = (long long)((C + cb - 1) / cb) * cb * R * S;
    } else return 0;
    if (real > (1LL << 24)) return 0;
    return round_up_i((int)real, CONV_DEPTH_ALIGN);
}

size_t pack_weights_bytes(int K, int C, int R, int S, int layout, int cb)
{
    if (K <= 0) return 0;
    return (size_t)K * (size_t)pack_weights_depth(C, R, S, layout, cb);
}

int pack_weights(int K, int C, int R, int S, int layout, int cb, const int8_t *src, int8_t *dst,
                 void *stream)
{
    if (!src || !dst || K <= 0 || C <= 0 || R <= 0 || S <= 0) return CONV_ERR_INVALID_ARG;
    if (layout != CONV_LAYOUT_IM2COL && layout != CONV_LAYOUT_PACKED && layout != CONV_LAYOUT_PAD_ONLY &&
        layout != CONV_LAYOUT_IMPLICIT)
        return CONV_ERR_INVALID_ARG;
    if (!aligned16(dst)) return CONV_ERR_INVALID_ARG;
    if (layout == CONV_LAYOUT_PAD_ONLY) cb = round_up_i(C, 16);
    const int depth = pack_weights_depth(C, R, S, layout, cb);
    if (depth == 0) return CONV_ERR_UNSUPPORTED;
    hipError_t e;
    if (layout == CONV_LAYOUT_IMPLICIT && pointwise_shape(C, R, S))
        e = launch_pack_weights_rows(K, C, depth, src, dst, (hipStream_t)stream);  // [K][C] as it is
    else if (layout == CONV_LAYOUT_IMPLICIT)
        e = launch_pack_weights_window(K, C, R, S, src, dst, (hipStream_t)stream);
    else if (layout == CONV_LAYOUT_IM2COL)
        e = launch_pack_weights_rows(K, C * R * S, depth, src, dst, (hipStream_t)stream);
    else
        e = launch_pack_weights_blocked(K, C, R, S, cb, depth, src, dst, (hipStream_t)stream);
    return e == hipSuccess ? CONV_OK : CONV_ERR_DEVICE;
}

size_t im2col_bytes(int N, int C, int H, int W, int R, int S, int stride, int pad, int kg_pad)
{
    conv_desc_t d{N, C, H, W, 1, R, S, stride, pad};
    if (check_desc(&d) != CONV_OK || kg_pad < C * R * S || kg_pad % 16) return 0;
    const long long P = (H + 2LL * pad - R) / stride + 1, Q = (W + 2LL * pad - S) / stride + 1;
    return (size_t)N * P * Q * kg_pad;
}

int im2col_int8(int N, int C, int H, int W, int R, int S, int stride, int pad, int kg_pad,
                const int8_t *src, int8_t *dst, void *stream)
{
    conv_desc_t d{N, C, H, W, 1, R, S, stride, pad};
    int rc = check_desc(&d);
    if (rc != CONV_OK) return rc;
    if (!src || !dst || !aligned16(dst)) return CONV_ERR_INVALID_ARG;
    if (kg_pad < C * R * S || kg_pad % 16) return CONV_ERR_INVALID_ARG;
    const int P = (H + 2 * pad - R) / stride + 1, Q = (W + 2 * pad - S) / stride + 1;
    return launch_im2col(N, C, H, W, R, S, stride, pad, P, Q, kg_pad, src, dst, (hipStream_t)stream) ==
                   hipSuccess ? CONV_OK : CONV_ERR_DEVICE;
}

int im2col_nhwc_int8(int N, int C, int H, int W, int R, int S, int stride, int pad, int kg_pad,
                     const int8_t *src, int8_t *dst, void *stream)
{
    conv_desc_t d{N, C, H, W, 1, R, S, stride, pad};
    int rc = check_desc(&d);
    if (rc != CONV_OK) return rc;
    if (!src || !dst || !aligned16(dst)) return CONV_ERR_INVALID_ARG;
    if (C % 16 == 0 && !aligned16(src)) return CONV_ERR_INVALID_ARG;  // 16-byte loads of a tap's channels
    if (kg_pad < C * R * S || kg_pad % 16) return CONV_ERR_INVALID_ARG;
    const int P = (H + 2 * pad - R) / stride + 1, Q = (W + 2 * pad - S) / stride + 1;
    return launch_im2col_nhwc(N, C, H, W, R, S, stride, pad, P, Q, kg_pad, src, dst, (hipStream_t)stream) == hipSuccess
               ? CONV_OK : CONV_ERR_DEVICE;
}

int pack_weights_rsc(int K, int C, int R, int S, const int8_t *src, int8_t *dst, void *stream)
{
    if (K <= 0 || C <= 0 || R <= 0 || S <= 0 || !src || !dst) return CONV_ERR_INVALID_ARG;
    if ((long long)C * R * S > 131072LL) return CONV_ERR_OVERFLOW_RISK;
    const int depth = round_up_i(C * R * S, CONV_DEPTH_ALIGN);
    return launch_pack_weights_rsc(K, C, R, S, depth, src, dst, (hipStream_t)stream) == hipSuccess ? CONV_OK
                                                                                                  : CONV_ERR_DEVICE;
}

int image_pack_desc(const conv_desc_t *desc, conv_desc_t *packed)
{
    if (!packed) return CONV_ERR_INVALID_ARG;
    PackedProblem pp;
    int rc = image_pack_problem(desc, 16, &pp, false);
    if (rc != CONV_OK) return rc;
    *packed = pp.d2;
    return CONV_OK;
}

size_t image_pack_bytes(const conv_desc_t *desc)
{
    PackedProblem pp;
    return image_pack_problem(desc, 16, &pp, false) == CONV_OK ? pp.x2_bytes : 0;
}

size_t image_pack_weights_bytes(const conv_desc_t *desc)
{
    PackedProblem pp;
    return image_pack_problem(desc, 16, &pp, false) == CONV_OK ? pp.w2_bytes : 0;
}

int image_pack_int8(const conv_desc_t *desc, const int8_t *src, int8_t *dst, void *stream)
{
    PackedProblem pp;
    int rc = image_pack_problem(desc, 16, &pp, false);
    if (rc != CONV_OK) return rc;
    if (!src || !dst || (reinterpret_cast<uintptr_t>(dst) & 3)) return CONV_ERR_INVALID_ARG;
    return launch_image_pack(desc->N, desc->C, desc->H, desc->W, desc->stride, desc->pad, pp.d2.H, pp.d2.W, src, dst,
                             (hipStream_t)stream) == hipSuccess ? CONV_OK : CONV_ERR_DEVICE;
}

int image_pack_weights(const conv_desc_t *desc, const int8_t *src, int8_t *dst, void *stream)
{
    PackedProblem pp;
    int rc = image_pack_problem(desc, 16, &pp, false);
    if (rc != CONV_OK) return rc;
    if (!src || !dst) return CONV_ERR_INVALID_ARG;
    return launch_image_pack_weights(desc->K, desc->C, desc->R, desc->S, desc->stride, src, dst,
                                     (hipStream_t)stream) == hipSuccess ? CONV_OK : CONV_ERR_DEVICE;
}

int dilated_desc(const conv_desc_t *desc, int dilation, conv_desc_t *inner)
{
    if (!inner) return CONV_ERR_INVALID_ARG;
    DilatedProblem dp;
    int rc = dilated_problem(desc, dilation, &dp);
    if (rc != CONV_OK) return rc;
    *inner = dp.d2;
    return CONV_OK;
}

size_t dilation_pack_bytes(const conv_desc_t *desc, int dilation)
{
    DilatedProblem dp;
    return dilated_problem(desc, dilation, &dp) == CONV_OK ? dp.x2_bytes : 0;
}

int dilation_pack_int8(const conv_desc_t *desc, int dilation, const int8_t *src, int8_t *dst, void *stream)
{
    DilatedProblem dp;
    int rc = dilated_problem(desc, dilation, &dp);
    if (rc != CONV_OK) return rc;
    if (!src || !dst) return CONV_ERR_INVALID_ARG;
    const hipError_t e = launch_dilation_pack(desc->N, desc->C, desc->H, desc->W, desc->pad, dilation, dp.d2.H, dp.d2.W,
                                              src, dst, (hipStream_t)stream);
    return e == hipSuccess ? CONV_OK : e == hipErrorInvalidValue ? CONV_ERR_UNSUPPORTED : CONV_ERR_DEVICE;
}

int dilation_unpack_int32(const conv_desc_t *desc, int dilation, const int32_t *src, int32_t *dst, void *stream)
{
    DilatedProblem dp;
    int rc = dilated_problem(desc, dilation, &dp);
    if (rc != CONV_OK) return rc;
    if (!src || !dst) return CONV_ERR_INVALID_ARG;
    const hipError_t e = launch_dilation_unpack(desc->N, desc->K, dp.P, dp.Q, dilation, dp.d2.H - desc->R + 1,
                                                dp.d2.W - desc->S + 1, src, dst, (hipStream_t)stream);
    return e == hipSuccess ? CONV_OK : e == hipErrorInvalidValue ? CONV_ERR_UNSUPPORTED : CONV_ERR_DEVICE;
}

size_t conv2d_int8_dilated_workspace_bytes(const conv_desc_t *desc, int dilation, int layout, int cb)
{
    DilatedProblem dp;
    if (dilated_problem(desc, dilation, &dp) != CONV_OK) return 0;
    if (resolve_layout(&dp.d2, &layout, &cb) != CONV_OK) return 0;
    Plan pl;
    if (make_plan(&dp.d2, layout, cb, &pl) != CONV_OK) return 0;
    const size_t inner = conv2d_int8_workspace_bytes(&dp.d2, layout, cb, 0);
    // the GEMM stage interleaves in its epilogue; only IMPLICIT stores the sub-images' results
    const size_t ob = pl.layout == CONV_LAYOUT_IMPLICIT ? align_up(dp.o2_bytes, WS_ALIGN) : 0;
    return align_up(dp.x2_bytes, WS_ALIGN) + ob + inner;
}

int conv2d_int8_dilated(const conv_desc_t *desc, int dilation, int layout, int cb, const int8_t *in, const int8_t *wt,
                        int32_t *out, void *workspace, size_t workspace_bytes, void *stream)
{
    DilatedProblem dp;
    int rc = dilated_problem(desc, dilation, &dp);
    if (rc != CONV_OK) return rc;
    const bool library_chooses = layout == CONV_LAYOUT_AUTO;
    rc = resolve_layout(&dp.d2, &layout, &cb);
    if (rc != CONV_OK) return rc;
    if (!in || !wt || !out || !workspace || (reinterpret_cast<uintptr_t>(workspace) & (WS_ALIGN - 1)))
        return CONV_ERR_INVALID_ARG;
    Plan pl;
    rc = make_plan(&dp.d2, layout, cb, &pl);  // the dense problem runs in one single-stage layout
    if (rc != CONV_OK) return rc;
    const size_t inner = conv2d_int8_workspace_bytes(&dp.d2, layout, cb, 0);
    const bool stored = pl.layout == CONV_LAYOUT_IMPLICIT;  // else the GEMM stage's epilogue interleaves
    const size_t xb = align_up(dp.x2_bytes, WS_ALIGN), ob = stored ? align_up(dp.o2_bytes, WS_ALIGN) : 0;
    if (workspace_bytes < xb + ob + inner) return CONV_ERR_WORKSPACE;
    Plan direct;
    if (library_chooses && direct_dilated_plan(desc, dilation, 0, &direct) == CONV_OK) {
        // the library's choice may also be the kernel that reads its taps `dilation` pixels apart from the image as it is
        const Route rt = dilated_route(desc, dilation, dp, pl, direct, wt, out);
        if (rt.how != TWO_STAGE && direct_bytes(rt, desc) <= workspace_bytes)
            return run_direct(rt, desc, direct, false, dilation, in, wt, out, workspace, (hipStream_t)stream);
    }
    int8_t *x2 = static_cast<int8_t *>(workspace);
    void *ws = inner ? static_cast<void *>(x2 + xb + ob) : nullptr;
    rc = dilation_pack_int8(desc, dilation, in, x2, stream);
    if (rc != CONV_OK) return rc;
    if (stored) {
        int32_t *o2 = reinterpret_cast<int32_t *>(x2 + xb);
        rc = conv2d_int8_ex(&dp.d2, layout, cb, x2, wt, 0, o2, ws, inner, stream);
        if (rc != CONV_OK) return rc;
        return dilation_unpack_int32(desc, dilation, o2, out, stream);
    }
    // both rewrites of the dense problem, then its GEMM stage writing the dilated layer's own output
    hipStream_t st = (hipStream_t)stream;
    int8_t *xq = static_cast<int8_t *>(ws), *wq = xq + align_up(pl.x_bytes, WS_ALIGN);
    const conv_desc_t &e2 = dp.d2;
    const hipError_t e = launch_rewrite_fused(pl.layout == CONV_LAYOUT_IM2COL, e2.N, e2.C, e2.H, e2.W, e2.K, e2.R, e2.S,
                                              e2.stride, e2.pad, pl.P, pl.Q, pl.cb, pl.depth, x2, xq, wt, wq, st);
    if (e == hipErrorNotSupported) {
        rc = rewrite_weights(&dp.d2, pl, wt, wq, st);
        if (rc != CONV_OK) return rc;
        rc = rewrite_input(&dp.d2, pl, x2, xq, st);
        if (rc != CONV_OK) return rc;
    } else if (e != hipSuccess) return CONV_ERR_DEVICE;
    GemmProblem g = gemm_problem(&dp.d2, pl, xq, wq, out);
    g.il_d = dilation;
    g.il_P = dp.P;
    g.il_Q = dp.Q;
    GemmChoice c;
    rc = choose_gemm_unsplit(g, &c);
    return rc == CONV_OK ? launch_choice(g, c, st) : rc;
}

size_t conv2d_int8_dilated_direct_workspace_bytes(const conv_desc_t *desc, int dilation, int cb)
{
    Plan pl;
    if (direct_dilated_plan(desc, dilation, cb, &pl) != CONV_OK) return 0;
    return align_up(pl.x_bytes, WS_ALIGN) + align_up(pl.w_bytes, WS_ALIGN);
}

int conv2d_int8_dilated_direct(const conv_desc_t *desc, int dilation, int cb, const int8_t *in, const int8_t *wt,
                               int32_t *out, void *workspace, size_t workspace_bytes, void *stream)
{
    Plan pl;
    int rc = direct_dilated_plan(desc, dilation, cb, &pl);
    if (rc != CONV_OK) return rc;
    if (!in || !wt || !out || !workspace || (reinterpret_cast<uintptr_t>(workspace) & (WS_ALIGN - 1)))
        return CONV_ERR_INVALID_ARG;
    const size_t xb = align_up(pl.x_bytes, WS_ALIGN);
    if (workspace_bytes < xb + align_up(pl.w_bytes, WS_ALIGN)) return CONV_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    const Route rt = dilated_direct_route(desc, dilation, pl, wt, out);
    if (rt.how != TWO_STAGE && direct_bytes(rt, desc) <= workspace_bytes) return run_direct(rt, desc, pl, false, dilation, in, wt, out, workspace, st);
    int8_t *xq = static_cast<int8_t *>(workspace), *wq = xq + xb;
    const hipError_t e = launch_rewrite_fused(false, desc->N, desc->C, desc->H, desc->W, desc->K, desc->R, desc->S,
                                              desc->stride, desc->pad, pl.P, pl.Q, pl.cb, pl.depth, in, xq, wt, wq, st);
    if (e == hipErrorNotSupported) {
        rc = rewrite_weights(desc, pl, wt, wq, st);
        if (rc != CONV_OK) return rc;
        rc = rewrite_input(desc, pl, in, xq, st);
        if (rc != CONV_OK) return rc;
    } else if (e != hipSuccess) return CONV_ERR_DEVICE;
    GemmProblem g = gemm_problem(desc, pl, xq, wq, out);
    g.dil = dilation;
    return run_gemm(g, -1, 0, st);
}

int mfma_probe_int8(int blocks, int iters, int32_t *out, void *stream)
{
    if (blocks <= 0 || blocks > (1 << 20) || iters <= 0 || !out) return CONV_ERR_INVALID_ARG;
    return launch_mfma_probe(blocks, iters, out, (hipStream_t)stream) == hipSuccess ? CONV_OK : CONV_ERR_DEVICE;
}

int gemm_int8_nt(int X, int Y, int Z, const int8_t *A, const int8_t *B, int32_t *Cout, void *stream)
{
    if (X <= 0 || Y <= 0 || Z <= 0 || !A || !B || !Cout) return CONV_ERR_INVALID_ARG;
    if (Z % CONV_DEPTH_ALIGN) return CONV_ERR_UNSUPPORTED;
    if (Z > 131072) return CONV_ERR_OVERFLOW_RISK;
    if (!aligned16(A) || !aligned16(B)) return CONV_ERR_INVALID_ARG;
    GemmProblem g{};
    g.act = B;
    g.wq = A;
    g.out = Cout;
    g.K = X;
    g.M = Y;
    g.depth = Z;
    g.PQ = Y;
    g.Q = Y;
    g.mode = ACT_MATRIX;
    return run_gemm(g, -1, 0, (hipStream_t)stream);
}

int conv2d_int8_num_tiles(void) { return gemm_num_tiles(); }

int conv2d_int8_tile_info(int tile, int *rows, int *cols, int *threads, int *steps)
{
    if (tile < 0 || tile >= gemm_num_tiles()) return CONV_ERR_INVALID_ARG;
    TileInfo t = gemm_tile_info(tile);
    if (rows) *rows = t.rows;
    if (cols) *cols = t.cols;
    if (threads) *threads = t.threads;
    if (steps) *steps = t.steps;
    return CONV_OK;
}

int conv2d_int8_packed(const conv_desc_t *desc, int layout, int cb, const int8_t *in_packed,
                       const int8_t *wt_packed, int32_t *out, int tile, int split_k, void *stream)
{
    if (layout == CONV_LAYOUT_AUTO) return CONV_ERR_INVALID_ARG;
    Plan pl;
    int rc = make_plan(desc, layout, cb, &pl);
    if (rc != CONV_OK) return rc;
    if (pl.layout == CONV_LAYOUT_IMPLICIT) {
        if (!in_packed || !wt_packed || !out) return CONV_ERR_INVALID_ARG;
        if (tile != -1 || (split_k != 0 && split_k != 1)) return CONV_ERR_UNSUPPORTED;
        return run_implicit(pl, window_problem(desc, pl, in_packed, wt_packed, out, 1), (hipStream_t)stream);
    }
    if (!in_packed || !wt_packed || !out || !aligned16(in_packed) || !aligned16(wt_packed))
        return CONV_ERR_INVALID_ARG;
    return run_gemm(gemm_problem(desc, pl, in_packed, wt_packed, out), tile, split_k,
                    (hipStream_t)stream);
}

int conv2d_int8_packed_nhwc(const conv_desc_t *desc, int layout, int cb, const int8_t *in_packed,
                            const int8_t *wt_packed, int32_t *out_nhwc, int tile, int split_k, void *stream)
{
    if (layout == CONV_LAYOUT_AUTO) return CONV_ERR_INVALID_ARG;
    Plan pl;
    int rc = make_plan(desc, layout, cb, &pl);
    if (rc != CONV_OK) return rc;
    if (pl.layout == CONV_LAYOUT_IMPLICIT) return CONV_ERR_UNSUPPORTED;  // those kernels write NKPQ
    if (!in_packed || !wt_packed || !out_nhwc || !aligned16(in_packed) || !aligned16(wt_packed) || !aligned16(out_nhwc))
        return CONV_ERR_INVALID_ARG;
    GemmProblem g = gemm_problem(desc, pl, in_packed, wt_packed, out_nhwc);
    g.out_nhwc = 1;
    return run_gemm(g, tile, split_k, (hipStream_t)stream);
}

// how: REQUANT_CHOOSE, REQUANT_STORED (the GEMM stages of conv2d_int8_packed), or a tile of the resident kernel with its pixels.
enum : int { REQUANT_STORED = -1, REQUANT_CHOOSE = -2 };
static int packed_requant(const conv_desc_t *desc, int layout, int cb, const int8_t *in_packed, const int8_t *wt_packed, int8_t *out_blocked, int out_cb,
                          int out_pad, int shift, int relu, int how, int pixels, void *stream)
{
    if (layout == CONV_LAYOUT_AUTO) return CONV_ERR_INVALID_ARG;
    Plan pl;
    int rc = make_plan(desc, layout, cb, &pl);
    if (rc != CONV_OK) return rc;
    if (!in_packed || !wt_packed || !out_blocked || out_pad < 0 || shift < 0 || shift > 31) return CONV_ERR_INVALID_ARG;
    const bool implicit = pl.layout == CONV_LAYOUT_IMPLICIT;  // reads the NCHW input and either weight form as they are
    if ((!implicit && (!aligned16(in_packed) || !aligned16(wt_packed))) || !aligned16(out_blocked)) return CONV_ERR_INVALID_ARG;
    if (out_cb != 16 && out_cb != 32 && out_cb != 64) return CONV_ERR_UNSUPPORTED;
    const long long Hq = (long long)pl.P + 2LL * out_pad, Wq = (long long)pl.Q + 2LL * out_pad;
    const long long Cbq = (desc->K + out_cb - 1) / out_cb;
    if (Hq > INT_LIMIT || Wq > INT_LIMIT) return CONV_ERR_UNSUPPORTED;
    hipStream_t st = (hipStream_t)stream;
    // The kernels write the interior pixels, with zeros for the channels that the last block lacks; only a border is left to a clear.
    // (One before every ragged last block took 1.5 to 7 us: 727 images 128 x 7 x 7 -> 254.)
    auto clear = [&] { return out_pad ? launch_fill_zero(out_blocked, (size_t)desc->N * (size_t)Cbq * (size_t)Hq * (size_t)Wq * (size_t)out_cb, st) : hipSuccess; };
    if (implicit) {
        if (how >= 0) return CONV_ERR_UNSUPPORTED;
        if (clear() != hipSuccess) return CONV_ERR_DEVICE;
        WindowProblem wp = window_problem(desc, pl, in_packed, wt_packed, nullptr, 1);
        int lg = 0;
        while ((1 << lg) < out_cb) ++lg;
        wp.act = ActOut{out_blocked, shift, relu != 0, lg, out_pad, (int)Hq, (int)Wq, (int)Cbq};
        return run_implicit(pl, wp, st);
    }
    GemmProblem g = gemm_problem(desc, pl, in_packed, wt_packed, nullptr);
    g.act_out = out_blocked;
    g.act_shift = shift;
    g.act_relu = relu != 0;
    g.o_cb = out_cb;
    g.o_pad = out_pad;
    if (how != REQUANT_STORED) {
        const ResidentProblem r = blocked_problem(desc, g);
        ResidentChoice pick{how, pixels, 0};
        if (how >= 0 && !resident_applies(r, how, pixels)) return CONV_ERR_UNSUPPORTED;
        if (how >= 0 || choose_blocked(r, &pick)) {
            if (clear() != hipSuccess) return CONV_ERR_DEVICE;
            return gemm_status(how >= 0 ? launch_resident_forced(r, pick.tile, pick.mper, st) : launch_resident(r, pick, st));
        }
    }
    GemmChoice c;
    rc = choose_gemm_unsplit(g, &c);
    if (rc != CONV_OK) return rc;
    if (clear() != hipSuccess) return CONV_ERR_DEVICE;
    return launch_choice(g, c, st);
}

int conv2d_int8_packed_requant(const conv_desc_t *desc, int layout, int cb, const int8_t *in_packed, const int8_t *wt_packed, int8_t *out_blocked,
                               int out_cb, int out_pad, int shift, int relu, void *stream)
{
    return packed_requant(desc, layout, cb, in_packed, wt_packed, out_blocked, out_cb, out_pad, shift, relu, REQUANT_CHOOSE, 0, stream);
}

int conv2d_int8_resident_requant(const conv_desc_t *desc, int layout, int cb, const int8_t *in_packed, const int8_t *wt_packed, int8_t *out_blocked,
                                 int out_cb, int out_pad, int shift, int relu, int tile, int pixels, void *stream)
{
    if (tile == -1 ? pixels != 0 : tile < 0 || tile >= resident_num_tiles() || pixels < 32 || pixels > 1024 || pixels % 32) return CONV_ERR_INVALID_ARG;
    return packed_requant(desc, layout, cb, in_packed, wt_packed, out_blocked, out_cb, out_pad, shift, relu, tile, pixels, stream);
}

int conv2d_int8_query_tiling(const conv_desc_t *desc, int layout, int cb, int *tile, int *split_k)
{
    if (layout == CONV_LAYOUT_AUTO || !tile || !split_k) return CONV_ERR_INVALID_ARG;
    Plan pl;
    int rc = make_plan(desc, layout, cb, &pl);
    if (rc != CONV_OK) return rc;
    *tile = -1;
    *split_k = 1;
    if (pl.layout == CONV_LAYOUT_IMPLICIT) return CONV_OK;
    GemmChoice c;
    rc = choose_gemm(gemm_problem(desc, pl, nullptr, nullptr, nullptr), -1, 0, &c);
    if (rc != CONV_OK) return rc;
    *tile = c.tile;
    *split_k = c.split_k;
    return CONV_OK;
}

int conv2d_int8_query_stage(const conv_desc_t *desc, int entry, int layout, int cb, int wt_is_packed, int dilation, int *stage, int *tile,
                            int *pixels)
{
    if (!stage || !tile || !pixels) return CONV_ERR_INVALID_ARG;
    Plan pl;
    Route rt{TWO_STAGE, {}, 0, 0};
    bool as_is = false;
    int rc = CONV_OK;
    if (entry == CONV_ENTRY_DILATED) {
        DilatedProblem dp;
        Plan inner;
        const bool library_chooses = layout == CONV_LAYOUT_AUTO;
        if ((rc = dilated_problem(desc, dilation, &dp)) != CONV_OK || (rc = resolve_layout(&dp.d2, &layout, &cb)) != CONV_OK ||
            (rc = make_plan(&dp.d2, layout, cb, &inner)) != CONV_OK)
            return rc;
        if (library_chooses && direct_dilated_plan(desc, dilation, 0, &pl) == CONV_OK)
            rt = dilated_route(desc, dilation, dp, inner, pl, nullptr, nullptr);
    } else if (entry == CONV_ENTRY_DILATED_DIRECT) {
        if ((rc = direct_dilated_plan(desc, dilation, cb, &pl)) != CONV_OK) return rc;
        rt = dilated_direct_route(desc, dilation, pl, nullptr, nullptr);
    } else if (entry == CONV_ENTRY_NHWC) {
        if ((rc = make_plan(desc, CONV_LAYOUT_PACKED, 0, &pl)) != CONV_OK) return rc;
        WindowProblem wp;
        as_is = nhwc_window(desc, pl, nullptr, nullptr, nullptr, &wp) || nhwc_matrix(desc, nullptr, nullptr, nullptr);
        if (!as_is) rt = nhwc_route(desc, pl, nullptr, nullptr);
    } else if (entry == CONV_ENTRY_ONE_SHOT || entry == CONV_ENTRY_EX) {
        if (entry == CONV_ENTRY_ONE_SHOT) layout = CONV_LAYOUT_AUTO, cb = 0, wt_is_packed = 0;
        if ((rc = resolve_layout(desc, &layout, &cb)) != CONV_OK) return rc;
        as_is = layout == CONV_LAYOUT_IMPLICIT;
        if (layout != CONV_LAYOUT_IMAGE_PACK && (rc = make_plan(desc, layout, cb, &pl)) != CONV_OK) return rc;
        if (entry == CONV_ENTRY_ONE_SHOT && !as_is) rc = one_shot_route(desc, layout, cb, nullptr, nullptr, nullptr, &pl, &rt);
        if (rc == CONV_OK && rt.how == TWO_STAGE && !as_is && layout != CONV_LAYOUT_IMAGE_PACK) {   // (what conv2d_int8_ex makes of it)
            if ((rc = make_plan(desc, layout, cb, &pl)) == CONV_OK) rt = ex_route(desc, pl, wt_is_packed != 0, nullptr, nullptr);
        }
        if (rc != CONV_OK) return rc;
    } else return CONV_ERR_INVALID_ARG;
    const bool panel = !as_is && rt.how == DIRECT_PANEL;
    *stage = as_is ? CONV_STAGE_AS_IS : panel ? CONV_STAGE_STORED : rt.how;
    const bool stream = rt.how == DIRECT_STREAM || rt.how == DIRECT_STREAM_REWRITE, given = rt.how == DIRECT_BAND || rt.how == TWO_STAGE;
    *tile = given ? -1 : rt.pick.tile + (stream ? CONV_TILE_STREAM : panel ? CONV_TILE_PANEL : 0);
    *pixels = given ? 0 : rt.pick.mper;
    return CONV_OK;
}

// ---- the resident kernel on its own --------------------------------------------------------------------------------
static int resident_forced(const conv_desc_t *desc, int dilation, int nhwc, int wt_cb, int tile, int pixels, const int8_t *in, const int8_t *wt,
                           int32_t *out, ResidentProblem *r)
{
    const bool band = tile == CONV_TILE_BAND, stream = is_stream_tile(tile);
    if (stream && (wt_cb <= 0 || pixels < 1 || pixels > stream_tile_info(tile - CONV_TILE_STREAM).cols)) return CONV_ERR_INVALID_ARG;
    if (wt_cb < 0 || (stream ? false : band ? pixels != 0 : tile < 0 || tile >= resident_num_tiles() || pixels < 32 || pixels > 1024 || pixels % 32)) return CONV_ERR_INVALID_ARG;
    Plan pl;
    const int rc = direct_dilated_plan(desc, dilation, wt_cb ? wt_cb : 16, &pl);
    if (rc != CONV_OK) return rc;
    if (!wt_cb && desc->R != 3) return CONV_ERR_UNSUPPORTED;   // (raw 1x1 weights: only the library's own choice)
    *r = resident_problem(desc, pl, wt_cb ? pl.cb : round_up_i(desc->C, 16), pl.depth, wt_cb == 0, nhwc != 0, dilation, in, wt, out);
    return (stream ? stream_applies(*r, tile - CONV_TILE_STREAM, pixels) : band ? band_direct_applies(*r) : resident_applies(*r, tile, pixels)) ? CONV_OK : CONV_ERR_UNSUPPORTED;
}

int conv2d_int8_resident_tile_info(int tile, int *rows, int *cols, int *threads)
{
    if ((tile < 0 || tile >= resident_num_tiles()) && !is_stream_tile(tile)) return CONV_ERR_INVALID_ARG;
    const TileInfo t = is_stream_tile(tile) ? stream_tile_info(tile - CONV_TILE_STREAM) : resident_tile_info(tile);
    if (rows) *rows = t.rows;
    if (cols) *cols = t.cols;
    if (threads) *threads = t.threads;
    return CONV_OK;
}

int conv2d_int8_resident_applies(const conv_desc_t *desc, int dilation, int nhwc, int wt_cb, int tile, int pixels)
{
    ResidentProblem r;
    return resident_forced(desc, dilation, nhwc, wt_cb, tile, pixels, nullptr, nullptr, nullptr, &r);
}

int conv2d_int8_resident(const conv_desc_t *desc, int dilation, int nhwc, const int8_t *in, const int8_t *wt, int wt_cb, int32_t *out, int tile,
                         int pixels, void *stream)
{
    ResidentProblem r;
    const int rc = resident_forced(desc, dilation, nhwc, wt_cb, tile, pixels, in, wt, out, &r);
    if (rc != CONV_OK) return rc;
    if (!in || !wt || !out || (wt_cb && !aligned16(wt))) return CONV_ERR_INVALID_ARG;
    if (is_stream_tile(tile)) return gemm_status(launch_stream_forced(r, tile - CONV_TILE_STREAM, pixels, (hipStream_t)stream));
    return gemm_status(tile == CONV_TILE_BAND ? launch_band_direct(r, (hipStream_t)stream) : launch_resident_forced(r, tile, pixels, (hipStream_t)stream));
}

// ---- the panel kernel on its own -------------------------------------------------------------------------------------
static int panel_forced(const conv_desc_t *desc, int dilation, int nhwc, int wt_cb, int tile, int pixels, const int8_t *in, const int8_t *wt, int32_t *out,
                        ResidentProblem *r)
{
    if (wt_cb < 0 || tile < 0 || tile >= panel_num_tiles() || pixels < 1 || pixels > panel_tile_info(tile).cols) return CONV_ERR_INVALID_ARG;
    Plan pl;
    const int rc = direct_dilated_plan(desc, dilation, wt_cb ? wt_cb : 16, &pl);
    if (rc != CONV_OK) return rc;
    *r = resident_problem(desc, pl, pl.cb, pl.depth, wt_cb == 0, nhwc != 0, dilation, in, wt, out);
    return panel_applies(*r, tile, pixels) ? CONV_OK : CONV_ERR_UNSUPPORTED;
}

int conv2d_int8_panel_tile_info(int tile, int *rows, int *cols)
{
    if (tile < 0 || tile >= panel_num_tiles()) return CONV_ERR_INVALID_ARG;
    const TileInfo t = panel_tile_info(tile);
    if (rows) *rows = t.rows;
    if (cols) *cols = t.cols;
    return CONV_OK;
}

size_t conv2d_int8_panel_workspace_bytes(const conv_desc_t *desc, int dilation, int nhwc, int wt_cb, int tile, int pixels)
{
    ResidentProblem r;
    return panel_forced(desc, dilation, nhwc, wt_cb, tile, pixels, nullptr, nullptr, nullptr, &r) == CONV_OK
               ? panel_weight_bytes(desc->K, desc->C, desc->R * desc->S)
               : 0;
}

int conv2d_int8_panel(const conv_desc_t *desc, int dilation, int nhwc, const int8_t *in, const int8_t *wt, int wt_cb, int32_t *out, int tile,
                      int pixels, void *workspace, size_t workspace_bytes, void *stream)
{
    ResidentProblem r;
    const int rc = panel_forced(desc, dilation, nhwc, wt_cb, tile, pixels, in, wt, out, &r);
    if (rc != CONV_OK) return rc;
    if (!in || !wt || !out || !workspace || (wt_cb && !aligned16(wt)) || !aligned16(workspace)) return CONV_ERR_INVALID_ARG;
    if (workspace_bytes < panel_weight_bytes(desc->K, desc->C, desc->R * desc->S)) return CONV_ERR_WORKSPACE;
    int8_t *const panels = static_cast<int8_t *>(workspace);
    const hipError_t e = launch_panel_weights(r, panels, (hipStream_t)stream);
    return gemm_status(e == hipSuccess ? launch_panel(r, panels, tile, pixels, (hipStream_t)stream) : e);
}

int conv2d_int8_tile_applies(const conv_desc_t *desc, int layout, int cb, int tile, int split_k)
{
    if (layout == CONV_LAYOUT_AUTO || (tile < 0 && tile != CONV_TILE_BAND) || tile >= gemm_num_tiles() || split_k < 1)
        return CONV_ERR_INVALID_ARG;
    Plan pl;
    int rc = make_plan(desc, layout, cb, &pl);
    if (rc != CONV_OK) return rc;
    if (pl.layout == CONV_LAYOUT_IMPLICIT) return CONV_ERR_UNSUPPORTED;
    GemmChoice c;
    return choose_gemm(gemm_problem(desc, pl, nullptr, nullptr, nullptr), tile, split_k, &c);
}

size_t conv2d_int8_tile_lds_bytes(const conv_desc_t *desc, int layout, int cb, int tile, int split_k)
{
    if (conv2d_int8_tile_applies(desc, layout, cb, tile, split_k) != CONV_OK) return 0;
    Plan pl;
    if (make_plan(desc, layout, cb, &pl) != CONV_OK) return 0;
    const GemmProblem g = gemm_problem(desc, pl, nullptr, nullptr, nullptr);
    return tile == CONV_TILE_BAND ? band_lds_bytes(g) : gemm_tile_lds_bytes(g, tile, split_k);
}

size_t conv2d_int8_workspace_bytes(const conv_desc_t *desc, int layout, int cb, int wt_is_packed)
{
    if (resolve_layout(desc, &layout, &cb) != CONV_OK) return 0;
    if (layout == CONV_LAYOUT_IMAGE_PACK) {
        PackedProblem pp;
        if (wt_is_packed || image_pack_problem(desc, cb, &pp) != CONV_OK) return 0;
        return align_up(pp.x2_bytes, WS_ALIGN) + align_up(pp.w2_bytes, WS_ALIGN) +
               conv2d_int8_workspace_bytes(&pp.d2, pp.inner_layout, pp.inner_cb, 0);
    }
    Plan pl;
    if (make_plan(desc, layout, cb, &pl) != CONV_OK) return 0;
    return align_up(pl.x_bytes, WS_ALIGN) + (wt_is_packed ? 0 : align_up(pl.w_bytes, WS_ALIGN));
}

// conv2d_int8_ex and conv2d_int8_stored.  stored: whatever a layout rewrites goes through the workspace.
static int run_explicit(const conv_desc_t *desc, int layout, int cb, const int8_t *in, const int8_t *wt, int wt_is_packed, int32_t *out,
                        void *workspace, size_t workspace_bytes, void *stream, bool stored)
{
    int rc = resolve_layout(desc, &layout, &cb);
    if (rc != CONV_OK) return rc;
    if (layout == CONV_LAYOUT_IMAGE_PACK) {
        // rewrite both operands into the stride-1 problem, then run that problem in its inner layout
        PackedProblem pp;
        rc = image_pack_problem(desc, cb, &pp);
        if (rc != CONV_OK) return rc;
        if (wt_is_packed) return CONV_ERR_UNSUPPORTED;
        if (!in || !wt || !out || !workspace) return CONV_ERR_INVALID_ARG;
        if (reinterpret_cast<uintptr_t>(workspace) % WS_ALIGN) return CONV_ERR_INVALID_ARG;
        const size_t xb = align_up(pp.x2_bytes, WS_ALIGN), wb = align_up(pp.w2_bytes, WS_ALIGN);
        const size_t inner = conv2d_int8_workspace_bytes(&pp.d2, pp.inner_layout, pp.inner_cb, 0);
        if (workspace_bytes < xb + wb + inner) return CONV_ERR_WORKSPACE;
        int8_t *x2 = static_cast<int8_t *>(workspace), *w2 = x2 + xb;
        hipStream_t st = (hipStream_t)stream;
        if (launch_image_pack(desc->N, desc->C, desc->H, desc->W, desc->stride, desc->pad, pp.d2.H, pp.d2.W, in, x2,
                              st) != hipSuccess ||
            launch_image_pack_weights(desc->K, desc->C, desc->R, desc->S, desc->stride, wt, w2, st) != hipSuccess)
            return CONV_ERR_DEVICE;
        return run_explicit(&pp.d2, pp.inner_layout, pp.inner_cb, x2, w2, 0, out, inner ? w2 + wb : nullptr, inner, stream, stored);
    }
    Plan pl;
    rc = make_plan(desc, layout, cb, &pl);
    if (rc != CONV_OK) return rc;
    if (!in || !wt || !out) return CONV_ERR_INVALID_ARG;
    if (pl.layout == CONV_LAYOUT_IMPLICIT)
        return run_implicit(pl, window_problem(desc, pl, in, wt, out, wt_is_packed ? 1 : 0), (hipStream_t)stream);
    if (!workspace) return CONV_ERR_INVALID_ARG;
    if (reinterpret_cast<uintptr_t>(workspace) % WS_ALIGN) return CONV_ERR_INVALID_ARG;
    if (wt_is_packed && !aligned16(wt)) return CONV_ERR_INVALID_ARG;
    const size_t xb = align_up(pl.x_bytes, WS_ALIGN);
    const size_t need = xb + (wt_is_packed ? 0 : align_up(pl.w_bytes, WS_ALIGN));
    if (workspace_bytes < need) return CONV_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    const Route rt = stored ? Route{TWO_STAGE, {}, 0, 0} : ex_route(desc, pl, wt_is_packed != 0, wt, out);
    if (rt.how != TWO_STAGE && direct_bytes(rt, desc) <= workspace_bytes) return run_direct(rt, desc, pl, false, 1, in, wt, out, workspace, st);
    int8_t *xq = static_cast<int8_t *>(workspace);
    const int8_t *wq = wt;
    bool rewritten = false;
    if (!wt_is_packed) {
        int8_t *wdst = xq + xb;
        wq = wdst;
        // both rewrites in one launch when the tiled input kernels apply
        hipError_t e = launch_rewrite_fused(pl.layout == CONV_LAYOUT_IM2COL, desc->N, desc->C, desc->H,
                                            desc->W, desc->K, desc->R, desc->S, desc->stride, desc->pad,
                                            pl.P, pl.Q, pl.cb, pl.depth, in, xq, wt, wdst, st);
        if (e == hipSuccess) rewritten = true;
        else if (e != hipErrorNotSupported) return CONV_ERR_DEVICE;
        else {
            rc = rewrite_weights(desc, pl, wt, wdst, st);
            if (rc != CONV_OK) return rc;
        }
    }
    if (!rewritten) {
        rc = rewrite_input(desc, pl, in, xq, st);
        if (rc != CONV_OK) return rc;
    }
    return run_gemm(gemm_problem(desc, pl, xq, wq, out), -1, 0, st);
}

int conv2d_int8_ex(const conv_desc_t *desc, int layout, int cb, const int8_t *in, const int8_t *wt,
                   int wt_is_packed, int32_t *out, void *workspace, size_t workspace_bytes,
                   void *stream)
{
    return run_explicit(desc, layout, cb, in, wt, wt_is_packed, out, workspace, workspace_bytes, stream, false);
}

int conv2d_int8_stored(const conv_desc_t *desc, int layout, int cb, const int8_t *in, const int8_t *wt,
                       int wt_is_packed, int32_t *out, void *workspace, size_t workspace_bytes,
                       void *stream)
{
    return run_explicit(desc, layout, cb, in, wt, wt_is_packed, out, workspace, workspace_bytes, stream, true);
}

int conv2d_int8(int N, int C, int H, int W, int K, int R, int S, int stride, int pad,
                const int8_t *in, const int8_t *wt, int32_t *out, void *stream)
{
    conv_desc_t d{N, C, H, W, K, R, S, stride, pad};
    int layout = CONV_LAYOUT_AUTO, cb = 0;
    int rc = resolve_layout(&d, &layout, &cb);
    if (rc != CONV_OK) return rc;
    if (!in || !wt || !out) return CONV_ERR_INVALID_ARG;
    const size_t need = conv2d_int8_workspace_bytes(&d, layout, cb, 0);
    if (need == 0) {  // IMPLICIT: nothing to stage (any other layout reports its problem here)
        if (layout != CONV_LAYOUT_IMPLICIT) return CONV_ERR_UNSUPPORTED;
        // Large batches: every workgroup of the stencil-unrolling kernel brings the tile's weight rows into the
        // padded depth order on its way into LDS, dword by dword; rows rewritten once by a small kernel are copied
        // in 16-byte pieces instead (a tenth of a workgroup's instructions).  Worth its launch from a few thousand
        // workgroups on (C3 at N=512: 495 -> 405 us); below that the single launch stays.
        const int depth = pack_weights_depth(C, R, S, CONV_LAYOUT_IMPLICIT, 0);
        const long long P = ((long long)H + 2 * pad - R) / stride + 1, Q = ((long long)W + 2 * pad - S) / stride + 1;
        if (!pointwise_shape(C, R, S) && depth > 0 && (long long)N * P * Q >= (1LL << 21)) {
            void *ws = nullptr;
            size_t ws_bytes = 0;
            if (cached_workspace(align_up((size_t)K * depth, WS_ALIGN), (hipStream_t)stream, &ws, &ws_bytes) == CONV_OK &&
                launch_pack_weights_window(K, C, R, S, wt, static_cast<int8_t *>(ws), (hipStream_t)stream) == hipSuccess)
                return conv2d_int8_ex(&d, layout, 0, in, static_cast<const int8_t *>(ws), 1, out, nullptr, 0, stream);
        }
        return conv2d_int8_ex(&d, layout, 0, in, wt, 0, out, nullptr, 0, stream);
    }
    // (the workspace rule is a property of the problem, whichever kernel the library then takes)
    void *ws = nullptr;
    size_t ws_bytes = 0;
    rc = cached_workspace(need, (hipStream_t)stream, &ws, &ws_bytes);
    if (rc != CONV_OK) return rc;
    Route rt;
    Plan pl;
    rc = one_shot_route(&d, layout, cb, in, wt, out, &pl, &rt);
    if (rc != CONV_OK) return rc;
    if (rt.how != TWO_STAGE && direct_bytes(rt, &d) <= ws_bytes)
        return run_direct(rt, &d, pl, false, 1, in, wt, out, ws, (hipStream_t)stream);
    return conv2d_int8_ex(&d, layout, cb, in, wt, 0, out, ws, ws_bytes, stream);
}

int conv2d_int8_static(int N, int C, int H, int W, int K, int R, int S, int stride, int pad,
                       const int8_t *in, const int8_t *wt, int32_t *out, void *stream)
{
    conv_desc_t d{N, C, H, W, K, R, S, stride, pad};
    int layout = CONV_LAYOUT_AUTO, cb = 0;
    int rc = resolve_layout(&d, &layout, &cb);
    if (rc != CONV_OK) return rc;
    if (!in || !wt || !out) return CONV_ERR_INVALID_ARG;
    const size_t need = conv2d_int8_workspace_bytes(&d, layout, cb, 0);
    if (need == 0) {  // IMPLICIT: nothing to stage (any other layout reports its problem here)
        if (layout != CONV_LAYOUT_IMPLICIT) return CONV_ERR_UNSUPPORTED;
        return conv2d_int8_ex(&d, layout, 0, in, wt, 0, out, nullptr, 0, stream);
    }
    if (need > STATIC_WS_BYTES) return CONV_ERR_WORKSPACE;  // the rewritten operands do not fit the fixed array
    void *ws = nullptr;
    rc = static_workspace(&ws);
    if (rc != CONV_OK) return rc;
    // Both rewrites write every byte of what the GEMM stage reads (zero borders and padding included), and a
    // depth split clears `out` with a kernel of its own: nothing is assumed about what the last call left.
    return conv2d_int8_ex(&d, layout, cb, in, wt, 0, out, ws, STATIC_WS_BYTES, stream);
}

int conv2d_int8_nhwc(int N, int C, int H, int W, int K, int R, int S, int stride, int pad,
                     const int8_t *in, const int8_t *wt, int32_t *out, void *stream)
{
    // The window kernel or a matrix product on the tensors as they are, the resident kernel, or channel blocking straight
    // from the NHWC source and a GEMM stage that writes NHWC.
    conv_desc_t d{N, C, H, W, K, R, S, stride, pad};
    Plan pl;
    int rc = make_plan(&d, CONV_LAYOUT_PACKED, 0, &pl);
    if (rc != CONV_OK) return rc;
    if (!in || !wt || !out) return CONV_ERR_INVALID_ARG;
    {   // the selector's choice is the kernel that unrolls the stencil itself, and its NHWC form takes the shape: one launch
        WindowProblem wp;
        if (nhwc_window(&d, pl, in, wt, out, &wp)) return launch_window_conv(wp, (hipStream_t)stream) == hipSuccess ? CONV_OK : CONV_ERR_DEVICE;
    }
    if (nhwc_matrix(&d, in, wt, out)) {
        // A 1x1 layer on NHWC tensors is a plain matrix product of operands that are depth-contiguous as they are:
        // pixels x channels times the weight rows, into pixels x output channels.  No rewrite, one launch.
        if (pointwise_nhwc_split_fits(pl.M, C, K))   // a grid that leaves most of the chip idle: the depth split over a workgroup's waves
            return launch_pointwise_nhwc_split(in, wt, out, pl.M, C, K, (hipStream_t)stream) == hipSuccess ? CONV_OK : CONV_ERR_DEVICE;
        GemmProblem g{};
        g.act = in;
        g.wq = wt;
        g.out = out;
        g.K = K;
        g.M = (int)pl.M;
        g.depth = C;
        g.PQ = pl.P * pl.Q;
        g.Q = pl.Q;
        g.mode = ACT_MATRIX;
        g.out_nhwc = 1;
        return run_gemm(g, -1, 0, (hipStream_t)stream);
    }
    // The GEMM stage's epilogue writes NHWC itself (a lane's four values are four consecutive channels of a
    // pixel); only a result that does not start on 16 bytes goes through an NKPQ staging tensor and a pass.
    const bool direct = aligned16(out);
    const size_t xb = align_up(pl.x_bytes, WS_ALIGN), wb = align_up(pl.w_bytes, WS_ALIGN);
    const size_t ob = direct ? 0 : align_up((size_t)pl.M * d.K * sizeof(int32_t), WS_ALIGN);
    const size_t need = xb + wb + ob;
    void *ws = nullptr;
    size_t ws_bytes = 0;
    hipStream_t st = (hipStream_t)stream;
    const Route rt = nhwc_route(&d, pl, wt, out);
    rc = cached_workspace(need, st, &ws, &ws_bytes);
    if (rc != CONV_OK) return rc;
    if (rt.how != TWO_STAGE && direct_bytes(rt, &d) <= ws_bytes) return run_direct(rt, &d, pl, true, 1, in, wt, out, ws, st);
    int8_t *xq = static_cast<int8_t *>(ws), *wq = xq + xb;
    int32_t *nkpq = reinterpret_cast<int32_t *>(wq + wb);
    const hipError_t e = launch_rewrite_fused_nhwc(N, C, H, W, K, R, S, pad, pl.cb, pl.depth, in, xq, wt, wq, st);
    if (e == hipErrorNotSupported) {
        if (launch_pack_layout_nhwc(N, C, H, W, pl.cb, pad, in, xq, st) != hipSuccess) return CONV_ERR_DEVICE;
        rc = rewrite_weights(&d, pl, wt, wq, st);
        if (rc != CONV_OK) return rc;
    } else if (e != hipSuccess) return CONV_ERR_DEVICE;
    if (direct) {
        GemmProblem g = gemm_problem(&d, pl, xq, wq, out);
        g.out_nhwc = 1;
        return run_gemm(g, -1, 0, st);
    }
    rc = run_gemm(gemm_problem(&d, pl, xq, wq, nkpq), -1, 0, st);
    if (rc != CONV_OK) return rc;
    return launch_unpack_nhwc(N, K, (long long)pl.P * pl.Q, nkpq, out, st) == hipSuccess ? CONV_OK : CONV_ERR_DEVICE;
}

}  // extern "C"
