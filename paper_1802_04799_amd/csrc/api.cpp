// C ABI of libtvg: argument validation (host only, before any device call),
// planning and dispatch to the kernel launchers.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <initializer_list>
#include <utility>
#include <mutex>
#include <unordered_map>
#include <vector>
#include "tvg_internal.h"

namespace {

using tvg::ConvProblem;

const int64_t kMaxElems = (int64_t)1 << 31;

// Product of positive extents, saturating at kMaxElems (every factor is below 2^31, so a
// partial product below 2^31 times the next factor stays inside 64 bits).
int64_t count_elems(std::initializer_list<int64_t> extents)
{
    int64_t n = 1;
    for (int64_t e : extents) {
        n *= e;
        if (n >= kMaxElems) return kMaxElems;
    }
    return n;
}

tvg_status make_problem(const tvg_conv_desc *d, bool depthwise, ConvProblem *out)
{
    if (!d) return TVG_ERR_NULL;
    if (d->n < 1 || d->c < 1 || d->h < 1 || d->w < 1 || d->k < 1 || d->r < 1 || d->s < 1)
        return TVG_ERR_BAD_SHAPE;
    if (d->stride_h < 1 || d->stride_w < 1 || d->stride_h > 8 || d->stride_w > 8)
        return TVG_ERR_BAD_SHAPE;
    // The filter extent is bounded before anything is computed from the padding: with r, s <= 16
    // and pad < r every sum below stays far inside the int range (h, w < 2^31 - 32 is implied by
    // the element-count limit, checked in 64 bits).
    if (d->r > 16 || d->s > 16) return TVG_ERR_UNSUPPORTED;
    if (d->pad_h < 0 || d->pad_w < 0 || d->pad_h >= d->r || d->pad_w >= d->s)
        return TVG_ERR_BAD_SHAPE;
    if ((int64_t)d->h + 2 * d->pad_h < d->r || (int64_t)d->w + 2 * d->pad_w < d->s)
        return TVG_ERR_BAD_SHAPE;
    if (d->dtype != TVG_F32 && d->dtype != TVG_BF16) return TVG_ERR_UNSUPPORTED;
    if (d->flags & ~(uint32_t)(TVG_RELU | TVG_STREAM_OUT)) return TVG_ERR_UNSUPPORTED;
    if (count_elems({d->n, d->c, d->h, d->w}) >= kMaxElems) return TVG_ERR_UNSUPPORTED;
    if (depthwise) {
        if (d->k != d->c) return TVG_ERR_BAD_SHAPE;
        if (d->r != 3 || d->s != 3) return TVG_ERR_UNSUPPORTED;
        if (d->stride_h != d->stride_w || d->stride_h > 2) return TVG_ERR_UNSUPPORTED;
        if (d->pad_h != 1 || d->pad_w != 1) return TVG_ERR_UNSUPPORTED;
        // one band of input rows (4 output rows) of one plane must fit 64 KB of LDS as fp32
        if ((int64_t)(3 * d->stride_h + 3) * ((int64_t)d->w + 2) > tvg::kDwBandFloats)
            return TVG_ERR_UNSUPPORTED;
    }
    ConvProblem p;
    p.N = d->n; p.IC = d->c; p.H = d->h; p.W = d->w; p.OC = d->k; p.R = d->r; p.S = d->s;
    p.sh = d->stride_h; p.sw = d->stride_w; p.ph = d->pad_h; p.pw = d->pad_w;
    const int64_t oh = ((int64_t)d->h + 2 * d->pad_h - d->r) / d->stride_h + 1;
    const int64_t ow = ((int64_t)d->w + 2 * d->pad_w - d->s) / d->stride_w + 1;
    if (oh >= kMaxElems || ow >= kMaxElems) return TVG_ERR_UNSUPPORTED;
    p.OH = (int)oh;
    p.OW = (int)ow;
    const int64_t ny = count_elems({d->n, d->k, p.OH, p.OW});
    const int64_t nw = count_elems({d->k, depthwise ? 1 : d->c, d->r, d->s});
    if (ny >= kMaxElems || nw >= kMaxElems) return TVG_ERR_UNSUPPORTED;
    p.K = (depthwise ? 1 : d->c) * d->r * d->s;
    p.npix = d->n * p.OH * p.OW;
    p.dtype = d->dtype;
    p.relu = (d->flags & TVG_RELU) ? 1 : 0;
    p.stream_out = (d->flags & TVG_STREAM_OUT) ? 1 : 0;
    *out = p;
    return TVG_OK;
}

// Problems whose tile shape a caller has fixed (tvg_conv2d_set_tile): a short list under a
// mutex - planning reads it on every call, a tuner writes it a few times per shape.
struct TileEntry {
    int key[12];
    tvg::Knobs knobs;
};
std::mutex g_tile_mutex;
std::vector<TileEntry> g_tiles;
constexpr size_t kMaxTileEntries = 1024;

void tile_key(const ConvProblem &p, int (&key)[12])
{
    const int k[12] = {p.N, p.IC, p.H, p.W, p.OC, p.R, p.S, p.sh, p.sw, p.ph, p.pw, p.dtype};
    memcpy(key, k, sizeof(k));
}

// Everything planning derives from a problem, computed once per distinct problem: which
// kernel takes it and with what launch shape.  The descriptor's flags do not enter (no plan
// depends on them).  A hash table under a mutex; tvg_conv2d_set_tile empties it, and so does the
// 257th distinct problem.  The launch-bound batch-1 layers spend 1-5 us per call in planning
// otherwise.
struct Dispatch {
    bool rows_shape, patch_shape, stem_shape, pw_shape, pwr_shape, pwd_shape, f32_shape, any_shape, tiled_shape, pw32_shape, strips_shape;
    tvg::RowsPlan rows;             // few tiles: in front of the 3x3 and 1x1 kernels
    tvg::StripsPlan strips;         // in front of the 3x3 kernels
    tvg::Patch3x3Plan patch;
    tvg::StemPlan stem;
    tvg::Pw1x1Plan pw, pwr;         // pwr: in front of pw
    tvg::PwDeepPlan pwd;            // the deep-reduction 1x1 kernel, where its rule (or a knob) picks it
    tvg::F32SmallPlan f32;
    tvg::ConvAnyPlan any;
    tvg::F32TiledPlan tiled;
    tvg::F32PwPlan pw32;            // fp32 1x1: in front of the three kernels that follow
    tvg::ConvPlan generic;          // the generic kernel's plan, reduction split allowed
    tvg::ConvPlan generic_single;   // the same in a single pass (no workspace)
};
struct ProblemKey {
    int v[12];
    bool operator==(const ProblemKey &o) const { return memcmp(v, o.v, sizeof(v)) == 0; }
};
struct ProblemHash {
    size_t operator()(const ProblemKey &k) const
    {
        uint64_t h = 0x9E3779B97F4A7C15ull;
        for (int e : k.v) h = (h ^ (uint32_t)e) * 0xFF51AFD7ED558CCDull, h ^= h >> 29;
        return (size_t)h;
    }
};
std::mutex g_dispatch_mutex;
std::unordered_map<ProblemKey, Dispatch, ProblemHash> g_dispatch;
constexpr size_t kMaxDispatchEntries = 256;

Dispatch dispatch_for(const ConvProblem &p)
{
    ProblemKey key;
    tile_key(p, key.v);
    {
        std::lock_guard<std::mutex> lock(g_dispatch_mutex);
        const auto it = g_dispatch.find(key);
        if (it != g_dispatch.end()) return it->second;
    }
    Dispatch d{};
    d.patch_shape = tvg::plan_conv3x3_patch(p, &d.patch);
    d.stem_shape = !d.patch_shape && tvg::plan_conv7x7s2_stem(p, &d.stem);
    d.pw_shape = !d.patch_shape && !d.stem_shape && tvg::plan_conv1x1(p, &d.pw);
    d.pwr_shape = d.pw_shape && tvg::plan_conv1x1_rows(p, &d.pwr);
    d.rows_shape = (d.patch_shape || d.pw_shape) && tvg::plan_conv_rows(p, &d.rows);
    d.strips_shape = d.patch_shape && !d.rows_shape && tvg::plan_conv3x3_strips(p, d.patch, &d.strips);
    {
        // stages knob of a 1x1 problem: 2 = the deep-reduction kernel.  No rule picks it: measured at
        // batch 32 / 64 over thirteen MobileNet and ResNet-50 pointwise shapes it takes 1.15-1.5 times
        // as long as the general kernel (512 -> 512 at 14x14: 15.7 against 12.5 us).
        const int want = tvg::forced_knobs(p).stages;
        d.pwd_shape = d.pw_shape && want == 2 && tvg::plan_conv1x1_deep(p, &d.pwd);
    }
    d.any_shape = !d.patch_shape && !d.stem_shape && !d.pw_shape && tvg::plan_conv_bf16_any(p, &d.any);
    d.tiled_shape = tvg::plan_conv_f32_tiled(p, &d.tiled);
    d.f32_shape = !d.tiled_shape && tvg::plan_conv_f32_small(p, &d.f32);
    // fp32 1x1 by what it takes the place of: tiles as the throughput kernel cuts them, narrow ones where the
    // launch-bound kernel would run or the gather kernel's 128 x 128 tiles are fewer than CUs, its own where there are more
    d.pw32_shape = tvg::plan_conv_f32_pw(p, d.f32_shape, d.tiled_shape ? d.tiled.nt : 0, &d.pw32);
    d.generic = tvg::plan_conv(p, true);
    d.generic_single = tvg::plan_conv(p, false);
    std::lock_guard<std::mutex> lock(g_dispatch_mutex);
    if (g_dispatch.size() >= kMaxDispatchEntries) g_dispatch.clear();
    g_dispatch.emplace(key, d);
    return d;
}

void forget_dispatch()
{
    std::lock_guard<std::mutex> lock(g_dispatch_mutex);
    g_dispatch.clear();
}

// Bytes of workspace that the dispatch's kernels want.
size_t dense_workspace(const Dispatch &d)
{
    if (d.patch_shape || d.stem_shape || d.pw_shape || d.tiled_shape || d.pw32_shape) return 0;
    return d.any_shape ? d.any.workspace_bytes : d.f32_shape ? d.f32.workspace_bytes : d.generic.workspace_bytes;
}

// One dense convolution through whichever kernel takes it (ptr.workspace: workspace_bytes of scratch).
tvg_status run_dense(const ConvProblem &p, const Dispatch &d, const tvg::ConvPointers &ptr, size_t workspace_bytes,
                     hipStream_t stream)
{
    if (d.rows_shape && tvg::conv_rows_pointers_ok(ptr)) return tvg::launch_conv_rows(p, d.rows, ptr, stream);
    if (d.strips_shape && tvg::conv3x3_strips_pointers_ok(ptr)) return tvg::launch_conv3x3_strips(p, d.strips, ptr, stream);
    if (d.patch_shape && tvg::conv3x3_patch_pointers_ok(ptr))
        return tvg::launch_conv3x3_patch(p, d.patch, ptr, stream);
    if (d.stem_shape && tvg::conv7x7s2_stem_pointers_ok(ptr))
        return tvg::launch_conv7x7s2_stem(p, d.stem, ptr, stream);
    if (d.pwd_shape && tvg::conv1x1_deep_pointers_ok(ptr)) return tvg::launch_conv1x1_deep(p, d.pwd, ptr, stream);
    if (d.pwr_shape && tvg::conv1x1_rows_pointers_ok(ptr)) return tvg::launch_conv1x1_rows(p, d.pwr, ptr, stream);
    if (d.pw_shape && tvg::conv1x1_pointers_ok(ptr)) return tvg::launch_conv1x1(p, d.pw, ptr, stream);
    const auto workspace_short = [&](size_t need) {
        return need > 0 && (!ptr.workspace || workspace_bytes < need ||
                            reinterpret_cast<uintptr_t>(ptr.workspace) % 256 != 0);
    };
    // A caller with less memory than the query reported gets the gather kernel, if that has enough: such
    // problems ran there, within its smaller workspace, before their weights were packed.
    const bool any_short = d.any_shape && workspace_short(d.any.workspace_bytes);
    if (d.any_shape && !any_short && tvg::conv_bf16_any_pointers_ok(ptr))
        return tvg::launch_conv_bf16_any(p, d.any, ptr, stream);
    if (d.pw32_shape && tvg::conv_f32_pw_pointers_ok(ptr)) return tvg::launch_conv_f32_pw(p, d.pw32, ptr, stream);
    if (d.tiled_shape && tvg::conv_f32_tiled_pointers_ok(ptr))
        return tvg::launch_conv_f32_tiled(p, d.tiled, ptr, stream);
    if (d.f32_shape && tvg::conv_f32_small_pointers_ok(ptr) && !(d.pw32_shape && workspace_short(d.f32.workspace_bytes))) {
        if (workspace_short(d.f32.workspace_bytes)) return TVG_ERR_WORKSPACE;
        return tvg::launch_conv_f32_small(p, d.f32, ptr, stream);
    }
    // A problem shaped for a specialised kernel reported a zero workspace; if its pointers
    // rule that kernel out, the generic kernel runs it in a single pass over the reduction.
    // (an fp32 problem whose x is not 16-byte aligned, a bf16 one at an odd address: the generic
    // kernel, within the workspace that the query reported if that is all the caller has)
    const tvg::ConvPlan &plan =
        (d.patch_shape || d.stem_shape || d.pw_shape || d.tiled_shape || d.pw32_shape ||
         ((d.f32_shape || (d.any_shape && !any_short)) && workspace_short(d.generic.workspace_bytes)))
            ? d.generic_single : d.generic;
    if (workspace_short(plan.workspace_bytes)) return TVG_ERR_WORKSPACE;
    return tvg::launch_conv_igemm(p, plan, ptr, stream);
}

// Scratch memory of tvg_conv2d_fused_static: the split-reduction partials of the generic kernel
// live in this array instead of a caller's workspace.  Every GPU that loads the library holds
// its own copy at its own address until the process ends.  In host code the array's name is
// only a handle for hipGetSymbolAddress; kernels are given the resolved device address.
constexpr size_t kStaticScratchBytes = (size_t)16 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices];      // device address of `scratch` per device, once resolved

// The current device's copy of `scratch`; resolved on the first call per device.
tvg_status static_scratch(void **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return TVG_ERR_LAUNCH;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return TVG_ERR_LAUNCH;
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return TVG_OK;
}

}  // namespace

namespace tvg {

Knobs forced_knobs(const ConvProblem &p)
{
    int key[12];
    tile_key(p, key);
    std::lock_guard<std::mutex> lock(g_tile_mutex);
    for (const TileEntry &e : g_tiles)
        if (memcmp(e.key, key, sizeof(key)) == 0) return e.knobs;
    return Knobs{0, 0, 0, 0, 0, 0};
}

}  // namespace tvg

extern "C" {

// Stores, replaces or (knobs all zero) forgets the problem's entry in the knob table.
static tvg_status store_knobs(const ConvProblem &p, const tvg::Knobs &k)
{
    const bool clear = !k.mt && !k.nt && !k.stages && !k.split_k && !k.lds_pitch && !k.row_loads;
    int key[12];
    tile_key(p, key);
    forget_dispatch();                     // plans made under the old table are stale
    std::lock_guard<std::mutex> lock(g_tile_mutex);
    for (size_t i = 0; i < g_tiles.size(); ++i)
        if (memcmp(g_tiles[i].key, key, sizeof(key)) == 0) {
            if (clear) g_tiles.erase(g_tiles.begin() + (long)i);
            else g_tiles[i].knobs = k;
            return TVG_OK;
        }
    if (clear) return TVG_OK;
    if (g_tiles.size() >= kMaxTileEntries) return TVG_ERR_UNSUPPORTED;
    TileEntry e;
    memcpy(e.key, key, sizeof(key));
    e.knobs = k;
    g_tiles.push_back(e);
    return TVG_OK;
}

static bool known_tile(int mt, int nt)
{
    return (mt == 64 && (nt == 512 || nt == 256 || nt == 128 || nt == 64)) || (mt == 128 && (nt == 256 || nt == 128 || nt == 64));
}

tvg_status tvg_conv2d_set_tile(const tvg_conv_desc *desc, int32_t mt, int32_t nt)
{
    ConvProblem p;
    tvg_status st = make_problem(desc, false, &p);
    if (st != TVG_OK) return st;
    if (!(mt == 0 && nt == 0) && !known_tile(mt, nt)) return TVG_ERR_UNSUPPORTED;
    tvg::Knobs k = tvg::forced_knobs(p);      // the other knobs stay as they are
    k.mt = mt;
    k.nt = nt;
    return store_knobs(p, k);
}

tvg_status tvg_conv2d_set_knobs(const tvg_conv_desc *desc, const tvg_conv_knobs *knobs)
{
    ConvProblem p;
    tvg_status st = make_problem(desc, false, &p);
    if (st != TVG_OK) return st;
    if (!knobs) return store_knobs(p, tvg::Knobs{0, 0, 0, 0, 0, 0});
    if (!((knobs->mt == 0 && knobs->nt == 0) || known_tile(knobs->mt, knobs->nt))) return TVG_ERR_UNSUPPORTED;
    if (knobs->stages < 0 || knobs->stages > 2 || knobs->split_k < 0 || knobs->split_k > 32 ||
        knobs->lds_pitch < 0 || knobs->lds_pitch > 2 || knobs->row_loads < 0 || knobs->row_loads > 2)
        return TVG_ERR_UNSUPPORTED;
    return store_knobs(p, tvg::Knobs{knobs->mt, knobs->nt, knobs->stages, knobs->split_k,
                                     knobs->lds_pitch, knobs->row_loads});
}

tvg_status tvg_conv2d_get_knobs(const tvg_conv_desc *desc, tvg_conv_knobs *knobs)
{
    if (!knobs) return TVG_ERR_NULL;
    ConvProblem p;
    tvg_status st = make_problem(desc, false, &p);
    if (st != TVG_OK) return st;
    const Dispatch d = dispatch_for(p);
    tvg_conv_knobs k = {0, 0, 0, 0, 0, 0};
    if (d.rows_shape) {
        // no knobs: fixing one selects the 3x3 or 1x1 kernel behind it
    } else if (d.strips_shape) {
        k.stages = 1;
        k.split_k = d.strips.kg;
        k.row_loads = 2;
    } else if (d.patch_shape) {
        k.mt = d.patch.mt;
        k.nt = d.patch.nt;
        k.stages = d.patch.dbuf ? 2 : 1;
        if (d.patch.dbuf) {
            k.split_k = d.patch.kg == 2 ? 2 : 1;       // (kg 3 names the channel split: mt = 128)
            if (p.sh == 1) k.lds_pitch = d.patch.pws == p.W + 2 ? 1 : 2;
            if (p.W % 2 != 0 && p.W <= 7 && p.sh == 1) k.row_loads = d.patch.px == 8 ? 2 : 1;
        }
    } else if (d.stem_shape) {
        k.mt = d.stem.mt;
        k.nt = d.stem.nt;
        k.stages = 1;
    } else if (d.pwd_shape) {
        k.mt = 64;
        k.nt = 128;
        k.stages = 2;
    } else if (d.pwr_shape) {
        k.mt = d.pwr.mt;
        k.nt = d.pwr.nt;
        k.stages = 1;
        k.row_loads = 2;
    } else if (d.pw_shape) {
        k.mt = d.pw.mt;
        k.nt = d.pw.nt;
        k.stages = 1;
    } else if (d.pw32_shape) {
        // none either
    } else if (d.f32_shape) {
        k.stages = 1;
        k.split_k = d.f32.nw * d.f32.ksplit;     // waves of a workgroup x slices across workgroups
    } else if (!d.any_shape && !d.tiled_shape) {     // (those two have no knobs: fixing one selects the gather kernel)
        k.mt = d.generic.mt;
        k.nt = d.generic.nt;
        k.stages = 2;
        k.split_k = d.generic.splits;
    }
    *knobs = k;
    return TVG_OK;
}

tvg_status tvg_conv2d_get_plan(const tvg_conv_desc *desc, int32_t *kernel, int32_t *mt, int32_t *nt)
{
    if (!kernel || !mt || !nt) return TVG_ERR_NULL;
    ConvProblem p;
    tvg_status st = make_problem(desc, false, &p);
    if (st != TVG_OK) return st;
    const Dispatch d = dispatch_for(p);
    if (d.rows_shape) {
        *kernel = d.patch_shape ? TVG_KERNEL_3X3 : TVG_KERNEL_1X1;
        *mt = 16;
        *nt = 16 * d.rows.nj;
    } else if (d.strips_shape) {
        *kernel = TVG_KERNEL_3X3_STRIPS;
        *mt = d.strips.kg == 4 ? 32 : 64;
        *nt = d.strips.sr * d.strips.t8 * d.strips.b * 8 / p.sh;
    } else if (d.patch_shape) {
        *kernel = d.patch.dbuf ? TVG_KERNEL_3X3_PIPELINED : TVG_KERNEL_3X3;
        *mt = d.patch.mt;
        *nt = d.patch.nt;
    } else if (d.stem_shape) {
        *kernel = TVG_KERNEL_STEM;
        *mt = d.stem.mt;
        *nt = d.stem.nt;
    } else if (d.pwd_shape) {
        *kernel = TVG_KERNEL_1X1_DEEP;
        *mt = 64;
        *nt = 128;
    } else if (d.pwr_shape) {
        *kernel = TVG_KERNEL_1X1;
        *mt = d.pwr.mt;
        *nt = d.pwr.nt;
    } else if (d.pw_shape) {
        *kernel = TVG_KERNEL_1X1;
        *mt = d.pw.mt;
        *nt = d.pw.nt;
    } else if (d.pw32_shape) {
        *kernel = d.f32_shape ? TVG_KERNEL_F32_SMALL : TVG_KERNEL_GENERIC;
        *mt = d.pw32.mt;
        *nt = d.pw32.nt;
    } else if (d.f32_shape) {
        *kernel = TVG_KERNEL_F32_SMALL;
        *mt = d.f32.stem ? 32 : d.f32.tile;
        *nt = d.f32.stem ? 64 : d.f32.tile;
    } else {
        *kernel = TVG_KERNEL_GENERIC;
        *mt = d.tiled_shape ? 64 : d.any_shape ? d.any.mt : d.generic.mt;
        *nt = d.tiled_shape ? d.tiled.nt : d.any_shape ? d.any.nt : d.generic.nt;
    }
    return TVG_OK;
}


tvg_status tvg_conv2d_workspace_size(const tvg_conv_desc *desc, size_t *bytes)
{
    if (!bytes) return TVG_ERR_NULL;
    ConvProblem p;
    tvg_status st = make_problem(desc, false, &p);
    if (st != TVG_OK) return st;
    *bytes = dense_workspace(dispatch_for(p));
    return TVG_OK;
}

tvg_status tvg_dwconv2d_workspace_size(const tvg_conv_desc *desc, size_t *bytes)
{
    if (!bytes) return TVG_ERR_NULL;
    ConvProblem p;
    tvg_status st = make_problem(desc, true, &p);
    if (st != TVG_OK) return st;
    *bytes = 0;
    return TVG_OK;
}

tvg_status tvg_conv2d_fused(const tvg_conv_desc *desc, const void *x, const void *w,
                            const float *scale, const float *shift, const float *bias,
                            const void *residual, void *y, void *workspace,
                            size_t workspace_bytes, void *hip_stream)
{
    ConvProblem p;
    tvg_status st = make_problem(desc, false, &p);
    if (st != TVG_OK) return st;
    if (!x || !w || !scale || !shift || !y) return TVG_ERR_NULL;
    const tvg::ConvPointers ptr{x, w, scale, shift, bias, residual, y, static_cast<float *>(workspace)};
    return run_dense(p, dispatch_for(p), ptr, workspace_bytes, static_cast<hipStream_t>(hip_stream));
}

tvg_status tvg_conv2d_fused_dual(const tvg_conv_desc *desc, int32_t k1, uint32_t flags2,
                                 const void *x, const void *w, const float *scale,
                                 const float *shift, const float *bias, const void *residual1,
                                 void *y1, void *y2, void *hip_stream)
{
    ConvProblem p;
    tvg_status st = make_problem(desc, false, &p);
    if (st != TVG_OK) return st;
    if (k1 < 1 || k1 >= p.OC) return TVG_ERR_BAD_SHAPE;
    if (flags2 & ~(uint32_t)(TVG_RELU | TVG_STREAM_OUT | TVG_CENTRE_TAP_ONLY)) return TVG_ERR_UNSUPPORTED;
    if (!x || !w || !scale || !shift || !y1 || !y2) return TVG_ERR_NULL;
    tvg::Patch3x3Plan plan;
    if (!tvg::plan_conv3x3_patch(p, &plan, k1)) return TVG_ERR_UNSUPPORTED;
    const tvg::ConvPointers ptr{x, w, scale, shift, bias, residual1, y1, nullptr};
    if (!tvg::conv3x3_patch_pointers_ok(ptr)) return TVG_ERR_UNSUPPORTED;
    const bool centre = (flags2 & TVG_CENTRE_TAP_ONLY) != 0;
    const int relu2 = (flags2 & TVG_RELU ? 1 : 0) | (flags2 & TVG_STREAM_OUT ? 2 : 0);
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    // Each head has the bits of a call of its own, so the kernel for few tiles, whose waves split the reduction, takes
    // exactly the heads that it would take then: both in one launch where their split is the same, or each in one.  So does
    // the kernel of strips, which has no two-head launches.
    ConvProblem h1 = p, h2 = p;
    h1.OC = k1;
    h2.OC = p.OC - k1;
    h2.relu = relu2 & 1;
    h2.stream_out = relu2 >> 1;
    const ConvProblem h2_3x3 = h2;
    if (centre) {
        h2.R = h2.S = 1;
        h2.ph = h2.pw = 0;
        h2.K = h2.IC;
    }
    const Dispatch d1 = dispatch_for(h1), d2 = dispatch_for(h2);
    const tvg::ConvPointers ptr2{x, static_cast<const char *>(w) + (size_t)k1 * p.IC * 18, scale + k1, shift + k1,
                                 bias ? bias + k1 : nullptr, nullptr, y2, nullptr};
    const bool rows1 = d1.rows_shape && tvg::conv_rows_pointers_ok(ptr), rows2 = d2.rows_shape && tvg::conv_rows_pointers_ok(ptr2);
    const bool strips1 = !rows1 && d1.strips_shape && tvg::conv3x3_strips_pointers_ok(ptr);
    const bool strips2 = !rows2 && d2.strips_shape && tvg::conv3x3_strips_pointers_ok(ptr2);
    const tvg::DualHead dual{k1, relu2, centre ? 1 : 0, y2};
    if (!rows1 && !rows2 && !strips1 && !strips2) return tvg::launch_conv3x3_patch(p, plan, ptr, stream, &dual);
    tvg::RowsPlan rows;
    if (rows1 && rows2 && tvg::plan_conv_rows_dual(p, d1.rows, d2.rows, centre, &rows))
        return tvg::launch_conv_rows(p, rows, ptr, stream, &dual);
    // One launch each, in the tiles of the head's own call; a 1x1 head's weights lie in 3x3 filters and want instances
    // that read those.  (The single-stage plan of a head exists where that of both does.)
    tvg::Patch3x3Plan plan1 = d1.patch, plan2 = d2.patch;
    if (!d1.patch_shape && !tvg::plan_conv3x3_patch(h1, &plan1, k1)) return TVG_ERR_UNSUPPORTED;
    if ((centre || !d2.patch_shape) && !tvg::plan_conv3x3_patch(h2_3x3, &plan2, k1)) return TVG_ERR_UNSUPPORTED;
    if (rows2 && centre && !tvg::plan_conv_rows_centre(h2, &rows)) return TVG_ERR_UNSUPPORTED;
    st = rows1 ? tvg::launch_conv_rows(h1, d1.rows, ptr, stream)
               : strips1 ? tvg::launch_conv3x3_strips(h1, d1.strips, ptr, stream) : tvg::launch_conv3x3_patch(h1, plan1, ptr, stream);
    if (st != TVG_OK) return st;
    if (strips2) return tvg::launch_conv3x3_strips(h2, d2.strips, ptr2, stream);
    if (rows2) return tvg::launch_conv_rows(h2, centre ? rows : d2.rows, ptr2, stream, nullptr, centre);
    if (!centre) return tvg::launch_conv3x3_patch(h2, plan2, ptr2, stream);
    const tvg::DualHead alone{0, relu2, 1, y2};
    return tvg::launch_conv3x3_patch(h2_3x3, plan2, ptr2, stream, &alone);
}

tvg_status tvg_conv2d_fused_static(const tvg_conv_desc *desc, const void *x, const void *w,
                                   const float *scale, const float *shift, const float *bias,
                                   const void *residual, void *y, void *hip_stream)
{
    size_t need = 0;
    tvg_status st = tvg_conv2d_workspace_size(desc, &need);       // validates the descriptor
    if (st != TVG_OK) return st;
    if (need > kStaticScratchBytes) {      // packed weights that do not fit: what the gather kernel needs
        ConvProblem p;
        make_problem(desc, false, &p);
        const Dispatch d = dispatch_for(p);
        if (d.any_shape) need = d.generic.workspace_bytes;
    }
    if (!x || !w || !scale || !shift || !y) return TVG_ERR_NULL;
    if (need > kStaticScratchBytes) return TVG_ERR_WORKSPACE;     // before any device call
    void *ws = nullptr;
    if (need > 0) {
        st = static_scratch(&ws);
        if (st != TVG_OK) return st;
    }
    return tvg_conv2d_fused(desc, x, w, scale, shift, bias, residual, y, ws, need, hip_stream);
}

size_t tvg_static_scratch_bytes(void) { return kStaticScratchBytes; }

tvg_status tvg_conv2d_prepack_size(const tvg_conv_desc *desc, size_t *packed_bytes, size_t *workspace_bytes)
{
    if (!packed_bytes || !workspace_bytes) return TVG_ERR_NULL;
    ConvProblem p;
    tvg_status st = make_problem(desc, false, &p);
    if (st != TVG_OK) return st;
    tvg::WinoPlan plan;
    if (!tvg::plan_conv3x3_winograd(p, &plan)) return TVG_ERR_UNSUPPORTED;
    *packed_bytes = plan.u_bytes;
    *workspace_bytes = plan.v_bytes;
    return TVG_OK;
}

tvg_status tvg_conv2d_prepack(const tvg_conv_desc *desc, const void *w, void *packed,
                              size_t packed_bytes, void *hip_stream)
{
    ConvProblem p;
    tvg_status st = make_problem(desc, false, &p);
    if (st != TVG_OK) return st;
    tvg::WinoPlan plan;
    if (!tvg::plan_conv3x3_winograd(p, &plan)) return TVG_ERR_UNSUPPORTED;
    if (!w || !packed) return TVG_ERR_NULL;
    if (packed_bytes < plan.u_bytes || reinterpret_cast<uintptr_t>(packed) % 16 != 0) return TVG_ERR_WORKSPACE;
    if (reinterpret_cast<uintptr_t>(w) % 16 != 0) return TVG_ERR_UNSUPPORTED;
    return tvg::launch_winograd_prepack(p, w, packed, static_cast<hipStream_t>(hip_stream));
}

tvg_status tvg_conv2d_fused_prepacked(const tvg_conv_desc *desc, const void *x, const void *packed,
                                      const float *scale, const float *shift, const float *bias,
                                      const void *residual, void *y, void *workspace,
                                      size_t workspace_bytes, void *hip_stream)
{
    ConvProblem p;
    tvg_status st = make_problem(desc, false, &p);
    if (st != TVG_OK) return st;
    tvg::WinoPlan plan;
    if (!tvg::plan_conv3x3_winograd(p, &plan)) return TVG_ERR_UNSUPPORTED;
    if (!x || !packed || !scale || !shift || !y) return TVG_ERR_NULL;
    if (!workspace || workspace_bytes < plan.v_bytes || reinterpret_cast<uintptr_t>(workspace) % 256 != 0)
        return TVG_ERR_WORKSPACE;
    if (reinterpret_cast<uintptr_t>(packed) % 16 != 0 || reinterpret_cast<uintptr_t>(x) % 2 != 0 ||
        reinterpret_cast<uintptr_t>(y) % 2 != 0 || reinterpret_cast<uintptr_t>(residual) % 2 != 0)
        return TVG_ERR_UNSUPPORTED;
    const tvg::ConvPointers ptr{x, nullptr, scale, shift, bias, residual, y, static_cast<float *>(workspace)};
    return tvg::launch_conv3x3_winograd(p, plan, packed, ptr, static_cast<hipStream_t>(hip_stream));
}

tvg_status tvg_dwconv2d_fused(const tvg_conv_desc *desc, const void *x, const void *w,
                              const float *scale, const float *shift, const float *bias,
                              const void *residual, void *y, void *workspace,
                              size_t workspace_bytes, void *hip_stream)
{
    (void)workspace;
    (void)workspace_bytes;
    ConvProblem p;
    tvg_status st = make_problem(desc, true, &p);
    if (st != TVG_OK) return st;
    if (!x || !w || !scale || !shift || !y) return TVG_ERR_NULL;
    tvg::ConvPointers ptr{x, w, scale, shift, bias, residual, y, nullptr};
    return tvg::launch_dwconv3x3(p, ptr, static_cast<hipStream_t>(hip_stream));
}

// The 1x1 stage of the block as a problem of its own: reads the depthwise stage's output.
static tvg_status make_pw_problem(const tvg_conv_desc *dw_desc, const ConvProblem &dw, int32_t pw_k,
                                  uint32_t pw_flags, ConvProblem *pw)
{
    if (pw_k < 1) return TVG_ERR_BAD_SHAPE;
    tvg_conv_desc d = *dw_desc;
    d.h = dw.OH; d.w = dw.OW; d.k = pw_k; d.r = d.s = 1;
    d.stride_h = d.stride_w = 1; d.pad_h = d.pad_w = 0;
    d.flags = pw_flags;
    return make_problem(&d, false, pw);
}

// Bytes of the block's intermediate tensor t at the start of the workspace.
static size_t dwpw_t_bytes(const ConvProblem &dw)
{
    const size_t elem = dw.dtype == TVG_BF16 ? 2 : 4;
    return ((size_t)dw.N * dw.IC * dw.OH * dw.OW * elem + 255) & ~(size_t)255;
}

tvg_status tvg_dwpw_workspace_size(const tvg_conv_desc *dw_desc, int32_t pw_k, size_t *bytes)
{
    if (!bytes) return TVG_ERR_NULL;
    ConvProblem dw, pw;
    tvg_status st = make_problem(dw_desc, true, &dw);
    if (st != TVG_OK) return st;
    st = make_pw_problem(dw_desc, dw, pw_k, 0, &pw);
    if (st != TVG_OK) return st;
    *bytes = dwpw_t_bytes(dw) + dense_workspace(dispatch_for(pw));      // + packed weights, partial sums
    return TVG_OK;
}

tvg_status tvg_dwpw_one_kernel(const tvg_conv_desc *dw_desc, int32_t pw_k, int32_t *available)
{
    if (!available) return TVG_ERR_NULL;
    ConvProblem dw, pw;
    tvg_status st = make_problem(dw_desc, true, &dw);
    if (st != TVG_OK) return st;
    st = make_pw_problem(dw_desc, dw, pw_k, 0, &pw);
    if (st != TVG_OK) return st;
    tvg::DwPwPlan plan;
    *available = tvg::plan_dwpw(dw, pw.OC, &plan) ? 1 : 0;
    return TVG_OK;
}

tvg_status tvg_dwpw_fused(const tvg_conv_desc *dw_desc, int32_t pw_k, uint32_t pw_flags,
                          const void *x, const void *w_dw, const float *scale_dw,
                          const float *shift_dw, const void *w_pw, const float *scale_pw,
                          const float *shift_pw, const float *bias_pw, const void *residual,
                          void *y, void *workspace, size_t workspace_bytes, void *hip_stream)
{
    ConvProblem dw, pw;
    tvg_status st = make_problem(dw_desc, true, &dw);
    if (st != TVG_OK) return st;
    st = make_pw_problem(dw_desc, dw, pw_k, pw_flags, &pw);
    if (st != TVG_OK) return st;
    if (!x || !w_dw || !scale_dw || !shift_dw || !w_pw || !scale_pw || !shift_pw || !y)
        return TVG_ERR_NULL;
    for (const void *q : {x, w_pw, residual, (const void *)y})
        if (reinterpret_cast<uintptr_t>(q) % 16 != 0) return TVG_ERR_UNSUPPORTED;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    tvg::DwPwPlan plan;
    if (!workspace && workspace_bytes == 0) {          // the caller asks for the one-kernel form
        if (!tvg::plan_dwpw(dw, pw.OC, &plan)) return TVG_ERR_WORKSPACE;
        const tvg::DwPwPointers ptr{x, w_dw, scale_dw, shift_dw, w_pw, scale_pw, shift_pw, bias_pw,
                                    residual, y};
        return tvg::launch_dwpw(dw, pw.OC, pw.relu, pw.stream_out, plan, ptr, stream);
    }
    // Less than the query reports will do where it holds t and the gather kernel's partial sums, which run
    // the 1x1 stage then.
    const size_t t_bytes = dwpw_t_bytes(dw);
    const Dispatch d = dispatch_for(pw);
    const bool whole = workspace_bytes >= t_bytes + dense_workspace(d);
    if (!workspace || reinterpret_cast<uintptr_t>(workspace) % 256 != 0 ||
        (!whole && workspace_bytes < t_bytes + d.generic.workspace_bytes))
        return TVG_ERR_WORKSPACE;
    dw.stream_out = 0;                       // t is read by the next launch
    const tvg::ConvPointers dptr{x, w_dw, scale_dw, shift_dw, nullptr, nullptr, workspace, nullptr};
    st = tvg::launch_dwconv3x3(dw, dptr, stream);
    if (st != TVG_OK) return st;
    const tvg::ConvPointers pptr{workspace, w_pw, scale_pw, shift_pw, bias_pw, residual, y,
                                 reinterpret_cast<float *>(static_cast<char *>(workspace) + t_bytes)};
    return whole ? run_dense(pw, d, pptr, workspace_bytes - t_bytes, stream)
                 : tvg::launch_conv_igemm(pw, d.generic, pptr, stream);
}

tvg_status tvg_plan_arena(const tvg_tensor_life *tensors, int32_t count, uint64_t *offsets,
                          uint64_t *arena_bytes)
{
    if (!tensors || !offsets || !arena_bytes) return TVG_ERR_NULL;
    if (count < 1 || count > 4096) return TVG_ERR_BAD_SHAPE;
    for (int32_t i = 0; i < count; ++i)
        if (tensors[i].bytes < 1 || tensors[i].bytes > ((uint64_t)1 << 48) ||
            tensors[i].first_step < 0 || tensors[i].last_step < tensors[i].first_step)
            return TVG_ERR_BAD_SHAPE;
    const uint64_t kAlign = 256;
    std::vector<int32_t> order(count);
    for (int32_t i = 0; i < count; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
        return tensors[a].bytes > tensors[b].bytes;          // ties keep their index order
    });
    std::vector<char> placed(count, 0);
    std::vector<std::pair<uint64_t, uint64_t>> busy;          // [begin, end) of conflicting tensors
    uint64_t arena = 0;
    for (int32_t oi = 0; oi < count; ++oi) {
        const int32_t t = order[oi];
        const uint64_t size = (tensors[t].bytes + kAlign - 1) / kAlign * kAlign;
        busy.clear();
        for (int32_t j = 0; j < count; ++j)
            if (placed[j] && tensors[j].first_step <= tensors[t].last_step &&
                tensors[t].first_step <= tensors[j].last_step) {
                const uint64_t sz = (tensors[j].bytes + kAlign - 1) / kAlign * kAlign;
                busy.emplace_back(offsets[j], offsets[j] + sz);
            }
        std::sort(busy.begin(), busy.end());
        uint64_t at = 0;                                      // lowest gap that holds `size`
        for (const auto &b : busy) {
            if (b.first >= at + size) break;
            if (b.second > at) at = b.second;
        }
        offsets[t] = at;
        placed[t] = 1;
        if (at + size > arena) arena = at + size;
    }
    *arena_bytes = arena;
    return TVG_OK;
}

tvg_status tvg_maxpool2d_3x3s2(int32_t n, int32_t c, int32_t h, int32_t w, int32_t dtype,
                               const void *x, void *y, void *hip_stream)
{
    if (n < 1 || c < 1 || h < 1 || w < 1) return TVG_ERR_BAD_SHAPE;
    if (dtype != TVG_F32 && dtype != TVG_BF16) return TVG_ERR_UNSUPPORTED;
    if (count_elems({n, c, h, w}) >= kMaxElems) return TVG_ERR_UNSUPPORTED;
    if (!x || !y) return TVG_ERR_NULL;
    return tvg::launch_maxpool3x3s2(n, c, h, w, dtype, x, y, static_cast<hipStream_t>(hip_stream));
}

const char *tvg_status_string(tvg_status status)
{
    switch (status) {
    case TVG_OK: return "ok";
    case TVG_ERR_NULL: return "a required pointer is NULL";
    case TVG_ERR_BAD_SHAPE: return "bad shape, stride or padding";
    case TVG_ERR_UNSUPPORTED: return "unsupported dtype, flag, size or kernel extent";
    case TVG_ERR_WORKSPACE: return "workspace missing or too small";
    case TVG_ERR_LAUNCH: return "HIP launch failed";
    }
    return "unknown status";
}

int tvg_version(void) { return 100; }

}  // extern "C"
