// fp32 fused conv2d at throughput size: 1x1, 3x3, 5x5 and 7x7 filters, any channel counts, equal
// strides, any padding below the filter (none for 1x1).  One launch, nothing but y written.
//
// v_mfma_f32_32x32x2_f32 takes one k value per lane and 64 cycles for 4096 operations, so that the LDS
// (three 256-byte reads per two MFMAs) is far from its limit and the fp32 input is an operand as it
// stands: the rows a tile needs lie in LDS as [channel][row][column] with a zero border, and 32
// consecutive pixels are 32 consecutive words for every tap.  What has to stay out of the loop is
// address arithmetic: the gather kernel divides and tests bounds for every element of every
// (pixel, k) pair, that is R*S times for each input element, where a tile's rows are fetched once.
//   - A workgroup of four waves owns 64 output channels x 64 NJ consecutive pixels of one image; a
//     wave 32 x 32 NJ.  Which input element a thread copies is worked out once; per chunk
//     of CIC channels the addresses advance by a constant.
//   - Weights: a channel's run of CIC*R*R floats of a chunk is contiguous in OIHW (16-byte loads),
//     and the LDS pitch is odd, so that the 32 lanes of an operand read 32 banks.
//   - Chunks are double-buffered: registers receive the next one while the matrix cores work, one
//     barrier per chunk.
//   - MFMAs start from zero again after a filter row (5x5: 20 products, 7x7: 28), a chunk (3x3: 72) or a part of
//     one (1x1: 8 to 32), and their sums are added to the totals in plain adds.
//
// What bounds it: per chunk, the wait for LDS operands at each filter row and the barrier, and rounds of tiles
// that do not fill the CUs; the matrix pipe is busy for 47 to 48 % of the time in the first three of these.
// 32 x 128 -> 128, 3x3 at 28x28: 127 us by the 32 x 32 tiles of the launch-bound kernel, 99 here
// (75 TFLOP/s); 32 x 64 -> 64 at 56x56: 146 by the gather kernel, 101; 1x1, 32 x 512 -> 512 at 14x14: 128, 59;
// 16 x 64 -> 128, 1x1 stride 2 at 56x56: 36, 12.
// Error against 64 bits over the 54 smaller of 85 such shapes, relative to the kernels that ran them before:
// 0.83 in the geometric mean, 0.36 to 1.00.  (With whole chunks as chains: 1.00, 0.36 to 1.59.)
#include <algorithm>

#include "tvg_device.h"
#include "tvg_internal.h"

namespace tvg {

namespace {

constexpr int kRsrcFlags = 0x00020000;
constexpr uint32_t kOutOfRange = 0x80000000u;      // and everything above: tensors stay below 2 GiB
constexpr int kMT = 64;
constexpr size_t kMaxLds = 160 * 1024;

struct TiledArgs {
    const float *x, *w, *scale, *shift, *bias, *residual;
    float *y;
    int IC, OC, OH, OW, OHW;
    int H, W, HW;                         // the map as the patch sees it (see `flat`), elements per channel
    int stride, ph, pw;
    int vsh, csw;                         // patch rows and columns from one output row / column to the next
    int pitch, plane;                     // patch floats per row and per channel
    int mtiles, tpi, nchunks, relu, vmode, buf_floats;
    uint32_t x_bytes, w_bytes;
    Divider by_mtiles, by_tpi, by_ow, by_plane, by_pitch;
};

__device__ __forceinline__ float load_f32(__amdgpu_buffer_rsrc_t r, uint32_t off)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}

// CHAINS: how a 1x1 chunk's 16 MFMAs are summed - one chain, 2: two of eight, 4: four of four, added in pairs
template <int R, int CIC, int NJ, int PT, int CHAINS>
__global__ __launch_bounds__(256, 2) void conv_f32_tiled_kernel(const TiledArgs a)
{
    constexpr int RS = R * R, CPH = CIC / 2, NT = 64 * NJ;
    constexpr int RUN = CIC * RS, WP = RUN | 1;            // a channel's run of a chunk, its LDS pitch
    static_assert(RUN % 4 == 0 && CIC % 2 == 0, "runs are whole 16-byte pieces");
    constexpr int PIECES = RUN / 4, WSLOTS = (kMT * PIECES + 255) / 256;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    float *ss = smem, *bufs = smem + 2 * kMT;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave & 1, wn = wave >> 1;
    const int lrow = lane & 31, lhalf = lane >> 5;
    int mt, pt, ow0;
    const int n = divide(divide(xcd_remap(blockIdx.x, gridDim.x), a.by_mtiles, &mt), a.by_tpi, &pt);
    const int m0 = mt * kMT, p0 = pt * NT;
    const int npx = min(NT, a.OHW - p0);
    const int oh0 = divide(p0, a.by_ow, &ow0);
    const int nrows = (divide(p0 + npx - 1, a.by_ow, &ow0) - oh0) * a.vsh + R;

    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.x), 0, a.x_bytes, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.w), 0, a.w_bytes, kRsrcFlags);

    // ---- copy tasks: element e of the chunk's patch, piece q of its weight runs -----------------
    uint32_t xoff[PT];
#pragma unroll
    for (int k = 0; k < PT; ++k) {
        const int e = tid + k * 256;
        int v, col;
        const int ch = divide(e, a.by_plane, &v), row = divide(v, a.by_pitch, &col);
        const int ih = R == 1 ? (oh0 + row) * a.stride : oh0 * a.stride + row - a.ph;
        const int iw = R == 1 ? col * a.stride : col - a.pw;
        const bool ok = ch < CIC && row < nrows && (unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W;
        xoff[k] = ok ? 4u * ((uint32_t)(n * a.IC + ch) * (uint32_t)a.HW + (uint32_t)(ih * a.W + iw)) : kOutOfRange;
    }
    uint32_t woff[WSLOTS];
#pragma unroll
    for (int k = 0; k < WSLOTS; ++k) {
        const int q = tid + k * 256, row = q / PIECES;
        woff[k] = row < kMT && m0 + row < a.OC
                      ? 4u * (uint32_t)((m0 + row) * a.IC * RS + (q - row * PIECES) * 4) : kOutOfRange;
    }

    float xreg[PT];
    uint4v wreg[WSLOTS];
    auto load_chunk = [&](int c) __attribute__((always_inline)) {
        const int left = min(CIC, a.IC - c * CIC);         // channels of this chunk; the others read as zero
        const uint32_t xc = 4u * (uint32_t)(c * CIC * a.HW), wc = 4u * (uint32_t)(c * RUN);
        const int xend = left * a.plane;
#pragma unroll
        for (int k = 0; k < PT; ++k)
            xreg[k] = load_f32(xrsrc, tid + k * 256 < xend && xoff[k] != kOutOfRange ? xoff[k] + xc : kOutOfRange);
        if (left == CIC) {
#pragma unroll
            for (int k = 0; k < WSLOTS; ++k)
                wreg[k] = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(
                    wrsrc, woff[k] != kOutOfRange ? woff[k] + wc : kOutOfRange, 0, 0));
        } else {
#pragma unroll
            for (int k = 0; k < WSLOTS; ++k) {
                const int q = tid + k * 256, at = (q % PIECES) * 4;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const bool ok = at + e < left * RS && woff[k] != kOutOfRange;
                    wreg[k][e] = __builtin_amdgcn_raw_buffer_load_b32(wrsrc, ok ? woff[k] + wc + 4u * e : kOutOfRange, 0, 0);
                }
            }
        }
    };
    auto store_chunk = [&](int buf) __attribute__((always_inline)) {
        float *wl = bufs + buf * a.buf_floats, *pl = wl + kMT * WP;
#pragma unroll
        for (int k = 0; k < WSLOTS; ++k) {
            const int q = tid + k * 256, row = q / PIECES;
            if (row < kMT) {
                float *d = wl + row * WP + (q - row * PIECES) * 4;
#pragma unroll
                for (int e = 0; e < 4; ++e) d[e] = __uint_as_float(wreg[k][e]);
            }
        }
#pragma unroll
        for (int k = 0; k < PT; ++k)
            if (tid + k * 256 < CIC * a.plane) pl[tid + k * 256] = xreg[k];
    };

    // ---- operand addresses -------------------------------------------------------------------
    const int abase = (wm * 32 + lrow) * WP + lhalf * CPH * RS;
    int bbase[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int pl = wn * 32 * NJ + j * 32 + lrow;
        const int p = p0 + (pl < npx ? pl : 0);            // (lanes past the end shadow pixel 0; dropped)
        int ow;
        const int oh = divide(p, a.by_ow, &ow);
        bbase[j] = kMT * WP + lhalf * CPH * a.plane + (oh - oh0) * a.vsh * a.pitch + ow * a.csw;
    }

    float16v acc[1][NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[0][j][v] = 0.0f;

    stage_scale_shift(ss, m0, kMT, a.scale, a.shift, a.bias, a.OC, tid, 256);
    load_chunk(0);
    store_chunk(0);
    __syncthreads();
    for (int c = 0; c < a.nchunks; ++c) {
        const float *buf = bufs + (c & 1) * a.buf_floats;
        if (c + 1 < a.nchunks) load_chunk(c + 1);
        // pixel operand first: the accumulator tile is D[pixel][channel]
        if constexpr (CHAINS > 1) {
            // Eight channels (per half-wave) of one pixel group at a time; their sums are added while the next
            // ones are under way.
            float16v pa, pb;
            auto add = [&](int j) __attribute__((always_inline)) {
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[0][j][v] += CHAINS == 4 ? pa[v] + pb[v] : pb[v];
                // (nothing is emitted here: it keeps the compiler from putting off all sums of the chunk to its
                // end, which holds 16 registers each and costs a workgroup per CU: 13.9 us against 15.5 at
                // 8 x 64 -> 128, 56x56)
                asm volatile("" : "+v"(acc[0][j]));
            };
#pragma unroll
            for (int t = 0; t < CPH / 8 * NJ; ++t) {
                const int j = t % NJ, ch = t / NJ * 8;
                float16v qa, qb;
#pragma unroll
                for (int v = 0; v < 16; ++v) qa[v] = qb[v] = 0.0f;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    qa = __builtin_amdgcn_mfma_f32_32x32x2f32(buf[bbase[j] + (ch + e) * a.plane], buf[abase + ch + e], qa, 0, 0, 0);
                if (CHAINS == 4 && t > 0) add((t - 1) % NJ);
                if (CHAINS == 2) qb = qa;
#pragma unroll
                for (int e = 4; e < 8; ++e)
                    qb = __builtin_amdgcn_mfma_f32_32x32x2f32(buf[bbase[j] + (ch + e) * a.plane], buf[abase + ch + e], qb, 0, 0, 0);
                if (CHAINS == 2 && t > 0) add((t - 1) % NJ);       // (in mid-chain: 65.7 us against 59.9 at 32 x 512 -> 512, 14x14)
                pa = qa;
                pb = qb;
            }
            add(NJ - 1);
        } else {
            float16v part[NJ];
            auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) part[j][v] = 0.0f;
            };
            auto add = [&]() __attribute__((always_inline)) {
#pragma unroll
                for (int j = 0; j < NJ; ++j)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[0][j][v] += part[j][v];
            };
            if constexpr (R <= 3) clear();
#pragma unroll 1                        // (3x3 rows unrolled: 104 us against 99 at 32 x 128 -> 128, 28x28)
            for (int r = 0; r < R; ++r) {
                if constexpr (R > 3) clear();
#pragma unroll
                for (int ch = 0; ch < CPH; ++ch)
#pragma unroll
                    for (int s = 0; s < R; ++s) {
                        const float wv = buf[abase + r * R + ch * RS + s];
#pragma unroll
                        for (int j = 0; j < NJ; ++j) {
                            const float xv = buf[bbase[j] + r * a.pitch + ch * a.plane + s];
                            part[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(xv, wv, part[j], 0, 0, 0);
                        }
                    }
                if constexpr (R > 3) add();
            }
            if constexpr (R <= 3) add();
        }
        if (c + 1 < a.nchunks) store_chunk((c + 1) & 1);
        __syncthreads();
    }

    // (the loop ended on a barrier: the buffers are free to stage the tail)
    unsigned char *stage = reinterpret_cast<unsigned char *>(bufs) + wave * kStageBytes;
    const int img = n * a.OHW;
    const TailArgs tail{a.scale, a.shift, a.bias, a.residual, a.y, a.OC, a.OHW, img + a.OHW, a.relu};
    store_acc_tiles<float, 1, NJ>(acc, stage, lane, m0 + wm * 32, img + p0 + wn * 32 * NJ, tail, a.vmode, ss, wm * 32);
}

template <int R, int CIC, int NJ, int PT, int CHAINS>
tvg_status launch_one(const TiledArgs &a, long tiles, size_t lds, hipStream_t stream)
{
    static const bool ok = hipFuncSetAttribute(reinterpret_cast<const void *>(conv_f32_tiled_kernel<R, CIC, NJ, PT, CHAINS>),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)kMaxLds) == hipSuccess;
    if (!ok) return TVG_ERR_LAUNCH;
    hipLaunchKernelGGL((conv_f32_tiled_kernel<R, CIC, NJ, PT, CHAINS>), dim3((unsigned)tiles), dim3(256), lds, stream, a);
    return hipGetLastError() == hipSuccess ? TVG_OK : TVG_ERR_LAUNCH;
}

template <int R, int CIC, int CHAINS = 1>
tvg_status launch_filter(const TiledArgs &a, const F32TiledPlan &t, hipStream_t stream)
{
#define TVG_TILED_ONE(NJ_, PT_) launch_one<R, CIC, NJ_, PT_, CHAINS>(a, t.tiles, t.lds_bytes, stream)
    // (1x1 without a stride: a tile is one row of the map as the patch sees it)
    if constexpr (R == 1 && CHAINS < 4) return t.nt == 128 ? TVG_TILED_ONE(2, 16) : TVG_TILED_ONE(1, 8);
    if (t.nt == 128) return t.pt == 8 ? TVG_TILED_ONE(2, 8) : t.pt == 16 ? TVG_TILED_ONE(2, 16) : TVG_TILED_ONE(2, 32);
    return t.pt == 8 ? TVG_TILED_ONE(1, 8) : t.pt == 16 ? TVG_TILED_ONE(1, 16) : TVG_TILED_ONE(1, 32);
#undef TVG_TILED_ONE
}

int ceil_div(int a, int b) { return (a + b - 1) / b; }

int chunk_channels(int R) { return R == 1 ? 32 : R == 3 ? 8 : 4; }

// The map as the patch sees it.  A 1x1 filter of stride 1 has no rows: the map is cut into rows of one tile.
void map_view(const ConvProblem &p, int nt, int *W, int *OH, int *OW)
{
    const bool flat = p.R == 1 && p.sh == 1;
    *W = flat ? nt : p.W;
    *OW = flat ? nt : p.OW;
    *OH = flat ? ceil_div(p.OH * p.OW, nt) : p.OH;
}

bool fit_tile(const ConvProblem &p, int nt, F32TiledPlan *t)
{
    const int cic = chunk_channels(p.R), run = cic * p.R * p.R;
    int W, OH, OW;
    map_view(p, nt, &W, &OH, &OW);
    const int orows = std::min(OH, (nt + OW - 2) / OW + (p.R == 1 && p.sh == 1 ? 0 : 1));   // output rows a tile touches
    const int rows = p.R == 1 ? orows : (orows - 1) * p.sh + p.R;
    t->nt = nt;
    t->pitch = p.R == 1 ? OW : W + 2 * p.pw;
    const long plane = (long)rows * t->pitch;
    if (plane * cic > 32 * 256) return false;
    t->plane = (int)plane;
    t->pt = plane * cic <= 8 * 256 ? 8 : plane * cic <= 16 * 256 ? 16 : 32;
    t->nchunks = ceil_div(p.IC, cic);
    t->buf_floats = (kMT * (run | 1) + cic * t->plane + 3) / 4 * 4;
    t->lds_bytes = (size_t)2 * kMT * 4 +
                   std::max((size_t)(t->nchunks > 1 ? 2 : 1) * t->buf_floats * 4, (size_t)4 * kStageBytes);
    t->tpi = ceil_div(p.OH * p.OW, nt);
    t->tiles = (long)p.N * t->tpi * ceil_div(p.OC, kMT);
    return t->lds_bytes <= kMaxLds && t->tiles < (1L << 31);
}

}  // namespace

bool plan_conv_f32_tiled(const ConvProblem &p, F32TiledPlan *plan)
{
    if (p.dtype != TVG_F32 || p.R != p.S || p.sh != p.sw) return false;
    if (p.R != 1 && p.R != 3 && p.R != 5 && p.R != 7) return false;
    if (p.R == 1 ? p.ph || p.pw : p.sh > p.R) return false;
    if ((size_t)p.N * p.IC * p.H * p.W >= ((size_t)1 << 29) || (size_t)p.OC * p.K >= ((size_t)1 << 29))
        return false;                                        // 32-bit byte offsets, the sign bit marks "outside"
    const Knobs knobs = forced_knobs(p);
    if (knobs.mt || knobs.nt || knobs.split_k) return false;     // a caller who shapes the gather kernel
    // Where the gather kernel has 128 x 128 tiles for every CU and aligned weight rows, it is the better one
    // for 1x1 filters (nothing to share between taps): 32 x 256 -> 256 at 28x28 50 us against 60, this kernel
    // 0.58 to 1.27 times as fast on 42 such shapes, 0.89 in the geometric mean.
    const long gtiles = (long)ceil_div(p.OC, 128) * ceil_div(p.npix, 128);
    if (p.R == 1 && gtiles >= kComputeUnits && p.IC % 4 == 0) return false;
    if (p.R == 7 && gtiles >= kComputeUnits) return false;       // (40 x 12 -> 128 at 40x40: 127 us against 135)
    F32TiledPlan t;
    bool found = false;
    for (int nt : {128, 64}) {
        if (!fit_tile(p, nt, &t)) continue;
        if (found && plan->tiles >= 2 * kComputeUnits && 8 * t.tiles >= 14 * plan->tiles) continue;
        *plan = t;
        found = true;
    }
    if (!found) return false;
    // One workgroup per CU hides no latency; with a deep reduction the waves that split it in the launch-bound
    // kernel do (32 x 512 -> 512, 3x3 at 7x7: 119 us against 127; 4 x 64 -> 64 at 56x56: 29 against 24).
    if (p.R > 1 && plan->tiles <= kComputeUnits && plan->nchunks > 16) return false;
    // The share of the matrix cores' turns that is not padding: channels filled up to tiles and chunks, pixels to
    // tiles, tiles to whole rounds of the CUs.  Timed against the kernels below on 580 shapes (420 drawn at random,
    // the ResNet-18 and MobileNet layers at ten batches): the 85 that this rule takes run 0.93 to 3.3 times as
    // fast, one of them below 1 (1x1 2.1 times in the geometric mean, 3x3 1.34, 5x5 1.85, 7x7 1.43).  Below the line
    // it is no longer a safe choice: 3x3 from 0.6 to 0.75 0.75 to 1.31 times, from 0.5 to 0.6 0.67 to 1.51; 1x1 from
    // 0.5 to 0.6 0.67 to 2.12, and 0.3 to 1 where the share is small.  (5x5 would gain down to 0.25: 0.93 to 2.6 times.)
    const double rounds = (double)((plan->tiles + kComputeUnits - 1) / kComputeUnits);
    const double useful = (double)p.npix * p.OC * p.IC /
                          (rounds * kComputeUnits * kMT * plan->nt * plan->nchunks * chunk_channels(p.R));
    return useful >= (p.R == 1 && p.IC % 8 == 0 ? 0.6 : 0.75);
}

bool conv_f32_tiled_pointers_ok(const ConvPointers &ptr)
{
    return reinterpret_cast<uintptr_t>(ptr.x) % 4 == 0 && reinterpret_cast<uintptr_t>(ptr.w) % 4 == 0;
}

tvg_status launch_conv_f32_tiled(const ConvProblem &p, const F32TiledPlan &t, const ConvPointers &ptr, hipStream_t stream)
{
    TiledArgs a;
    a.x = static_cast<const float *>(ptr.x);
    a.w = static_cast<const float *>(ptr.w);
    a.scale = ptr.scale; a.shift = ptr.shift; a.bias = ptr.bias;
    a.residual = static_cast<const float *>(ptr.residual);
    a.y = static_cast<float *>(ptr.y);
    a.IC = p.IC; a.OC = p.OC; a.OHW = p.OH * p.OW;
    map_view(p, t.nt, &a.W, &a.OH, &a.OW);
    a.H = p.R == 1 && p.sh == 1 ? a.OH : p.H;
    a.HW = p.H * p.W;
    a.stride = p.sh; a.ph = p.ph; a.pw = p.pw;
    a.vsh = p.R == 1 ? 1 : p.sh;
    a.csw = p.R == 1 ? 1 : p.sw;
    a.pitch = t.pitch; a.plane = t.plane;
    a.mtiles = ceil_div(p.OC, kMT); a.tpi = t.tpi; a.nchunks = t.nchunks;
    a.relu = p.relu | (p.stream_out << 1);
    a.vmode = pick_store_vmode(p.dtype, a.OHW, ptr.y, ptr.residual);
    a.buf_floats = t.buf_floats;
    a.by_mtiles = make_divider(a.mtiles); a.by_tpi = make_divider(a.tpi); a.by_ow = make_divider(a.OW);
    a.by_plane = make_divider(a.plane); a.by_pitch = make_divider(a.pitch);
    a.x_bytes = (uint32_t)((size_t)p.N * p.IC * a.HW * 4);
    a.w_bytes = (uint32_t)((size_t)p.OC * p.K * 4);
    // 1x1: the fewest chains whose error is not above that of the kernels that ran these problems before (the
    // launch-bound kernel's waves split the reduction).  Relative to it, by channels, with one / two / four chains:
    // 32: 1.52 1.17 0.98, 64: 1.38 1.09 0.94, 128: 1.19 1.00 0.89, 256: 1.00 0.91 0.84.  Two chains cost 0 to 2 % of
    // the time, four 1 to 3 % at few channels and 4 to 9 % at many; under a stride four are as fast as one.
    if (p.R == 1) {
        if (t.nchunks <= 2 || p.sh > 1) return launch_filter<1, 32, 4>(a, t, stream);
        return t.nchunks < 8 ? launch_filter<1, 32, 2>(a, t, stream) : launch_filter<1, 32>(a, t, stream);
    }
    if (p.R == 3) return launch_filter<3, 8>(a, t, stream);
    if (p.R == 5) return launch_filter<5, 4>(a, t, stream);
    return launch_filter<7, 4>(a, t, stream);
}

}  // namespace tvg
