// bf16 fused conv2d for any filter, stride, padding and channel count: what the specialised kernels
// (3x3 with 16 n channels, 1x1 with 8 n, the stems) do not take.  Two launches: a small one that
// lays the weights out as MFMA operands in the workspace, and the convolution.
//
// The matrix core wants eight consecutive k per lane, and here k runs over input channels with the
// filter tap fixed, so that the pixel operand of every tap is the same LDS patch at a shifted
// address (the patch holds 16-byte words of eight channels of one input position).
//   - Weights.  In OIHW eight channels of one tap lie R*S elements apart and rows start anywhere
//     (2-byte aligned for odd IC*R*S).  Transposing them in every workgroup costs R*S*8 scalar
//     reads per row and octet and is repeated for every pixel tile; the pack launch does it once,
//     coalesced both ways through LDS, and pads channels to whole octets and rows to whole tiles
//     with zeros.  A step's weights are then 512 consecutive bytes per half-wave, which every wave
//     loads straight into its operand registers, a turn of the loop ahead; they never touch LDS.
//     (The first version copied them to LDS a block of steps ahead, one barrier per block:
//     15.0 us against 13.4 on the example below.)
//   - Input.  A tile is NT consecutive output pixels of an image, or, for small maps, of the flattened
//     (n, oh, ow) order; images then own (OH-1)*sh + R "virtual rows" of the patch each.  A thread
//     fetches PX horizontally adjacent pixels of eight channels with one load per channel - rows of
//     any width: the last group of a row is moved back to end at the row's end, loads are 2-byte
//     aligned - and writes PX words.  Columns are stored by phase modulo the stride, so that the
//     pixels of an operand are adjacent words for every stride.
//   - Reduction.  Units (tap, octet) of a chunk of CO octets are numbered in a row and an MFMA step
//     takes two of them, one per half-wave; their patch offsets come from a small LDS table.  CO is
//     chosen so that little of the last turn is padding, whatever R, S and IC are.
// The patch is double-buffered (one chunk ahead, in registers), one barrier per chunk.
//
// What bounds it: latency.  At 6 x 83 x 45 x 37 -> 139, 3x3 (486 workgroups of 64 x 64 with one chunk each, about two
// per CU) the pack launch takes 4 us and this kernel 12, a tenth of them on the matrix pipe.  The gather kernel
// with its split reduction took 62 + 8 us.  Larger problems: 9 x 24 x 99 x 99 -> 200, 5x5, 256 us before, 58 now
// (366 TFLOP/s, matrix pipe 20 %); 27 x 168 x 10 x 76 -> 312, 3x3, 132 before, 33 now (583, 28 %), both beside 5 us of
// packing.  About half of the LDS cycles are bank conflicts.
#include <type_traits>

#include "tvg_device.h"
#include "tvg_internal.h"

namespace tvg {

namespace {

constexpr int kWord = 16;                 // bytes: eight channels of one position
constexpr int kRsrcFlags = 0x00020000;
constexpr uint32_t kOutOfRange = 0x80000000u;      // and everything above: tensors stay below 2 GiB
constexpr size_t kMaxLds = 160 * 1024;
constexpr int kNoTap = 1 << 24;           // patch offset of a unit without a tap: past the LDS

struct AnyArgs {
    const bf16_t *x, *packed;
    const float *scale, *shift, *bias;
    const bf16_t *residual;
    bf16_t *y;
    float *ws;                            // partial sums [splits][N][OC][OH][OW] when splits > 1
    int N, IC, H, W, OC, OH, OW, sh, sw, ph, pw, R, S, npix, relu, vmode;
    int co, nchunks, chunks_per_split;    // octets per chunk, chunks in all and per workgroup
    int steps;                            // MFMA steps per chunk
    int rows, pws, cp;                    // patch rows (bound), row pitch in words, words per column phase
    int vh, vsh;                          // virtual rows per image and per output row
    int groups;                           // loads per patch row
    int mtiles, splits, tpi;              // tpi: pixel tiles per image, 0 = tiles cross images
    int border;                           // zero columns per patch row
    uint32_t x_bytes, packed_bytes;
    int tab_bytes, patch_bytes, zero_at;  // LDS: unit table, one patch, offset of the word of zeros
    Divider by_ohw, by_ow, by_vh, by_r, by_groups, by_mtiles, by_co, by_s, by_sw, by_tpi, by_border;
};

__device__ __forceinline__ uint32_t pack_halves(uint32_t a, uint32_t b, int half)
{
    return __builtin_amdgcn_perm(b, a, half ? 0x07060302u : 0x05040100u);
}

template <int PX> struct RawPixels { uint32_t d[PX >= 2 ? PX / 2 : 1]; };

// MFMA steps per turn of the loop; a chunk's steps are a multiple of it.  It is also how far ahead
// the weights are requested: a step is MI*NJ MFMAs of 32 cycles, and a packed weight word that no
// workgroup of the XCD has read yet comes from the memory-side cache (500 cycles and more).
constexpr int ring_of(int mi) { return mi == 1 ? 8 : 4; }

// WM x (4 / WM) waves of (32 MI) channels x (32 NJ) pixels; PX pixels per load, PT load tasks per thread.
template <int WM, int MI, int NJ, int PX, int PT>
__global__ __launch_bounds__(256, 2) void conv_bf16_any_kernel(const AnyArgs a)
{
    constexpr int RING = ring_of(MI);
    constexpr int WN = 4 / WM, WTM = 32 * MI, WTN = 32 * NJ, MT = WM * WTM, NT = WN * WTN;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const int lrow = lane & 31, lhalf = lane >> 5;
    int mt;
    const int ntile = divide(xcd_remap(blockIdx.x, gridDim.x), a.by_mtiles, &mt);
    const int m0 = mt * MT;
    int n0 = ntile * NT, n_end = a.npix;
    if (a.tpi) {                                       // tiles that stay within an image
        const int n = divide(ntile, a.by_tpi, &n0);
        n_end = (n + 1) * (a.OH * a.OW);
        n0 = n * (a.OH * a.OW) + n0 * NT;
    }
    const int H = a.H, W = a.W, HW = H * W, OHW = a.OH * a.OW;
    const int c_beg = blockIdx.y * a.chunks_per_split;
    const int c_end = min(a.nchunks, c_beg + a.chunks_per_split);

    int *tab = reinterpret_cast<int *>(smem);
    float *ss = reinterpret_cast<float *>(smem + a.tab_bytes);
    unsigned char *patch = smem + a.tab_bytes + 2 * MT * 4;
    const int plane = a.rows * a.pws * kWord;          // one octet of the patch

    // ---- weights: RING steps ahead, in registers ------------------------------------------------
    // (this wave's 32 MI channels of a step: two half-waves of 512 MI consecutive bytes)
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t *>(a.packed), 0, a.packed_bytes, kRsrcFlags);
    const uint32_t wlane = (lhalf * MT + wm * WTM + lrow) * kWord;
    // Chunk after chunk, in the same order for every tile, so that equal images of a batch get equal results.
    // (Beginning each pixel tile at another chunk, to spread the requests of tiles that keep pace over more
    // lines, took 0.98 to 1.12 times as long over 23 shapes.)
    uint32_t wat = (uint32_t)(mt * a.nchunks + c_beg) * (uint32_t)(a.steps * 2 * MT * kWord);
    uint4v wreg[RING][MI];
    auto load_weights = [&](int slot) __attribute__((always_inline)) {      // (past the end: zeros or a neighbour, unused)
#pragma unroll
        for (int i = 0; i < MI; ++i)
            wreg[slot][i] = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, wlane + i * 512, wat, 0));
        wat += 2 * MT * kWord;
    };

    // ---- tile geometry (uniform) -----------------------------------------------------------
    int rem, ow_;
    const int p_last = min(n0 + NT, n_end) - 1;
    const int na = divide(n0, a.by_ohw, &rem), oha = divide(rem, a.by_ow, &ow_);
    const int nb = divide(p_last, a.by_ohw, &rem), ohb = divide(rem, a.by_ow, &ow_);
    const int vr0 = na * a.vh + oha * a.vsh;
    const int nrows = nb * a.vh + ohb * a.vsh + a.R - vr0;     // <= a.rows

    // ---- patch load tasks: (virtual row, octet, pixel group) ---------------------------------
    uint32_t goff[PT];        // byte offset of the task's pixels in channel 8*octet of x
    int ldst[PT];             // byte offset of the row in its octet plane, -1 = no task
    int lq[PT], lph[PT];      // word and phase of the first pixel
    int loct[PT];
#pragma unroll
    for (int k = 0; k < PT; ++k) {
        int g, v;
        int row = divide(tid + k * 256, a.by_groups, &g);
        row = divide(row, a.by_co, &loct[k]);
        const int n = divide(vr0 + row, a.by_vh, &v);
        int ih = v - a.ph;
        if (a.vsh < a.sh) {                           // fewer filter rows than the stride: no overlap, rows skipped
            int r;
            const int oh = divide(v, a.by_r, &r);
            ih = oh * a.sh + r - a.ph;
        }
        const int c0 = min(g * PX, W - PX);
        ldst[k] = -1;
        goff[k] = kOutOfRange;
        lq[k] = divide(c0 + a.pw, a.by_sw, &lph[k]);
        if (row < nrows) {
            // (rows outside the image are written too, with the zeros an out-of-range load returns)
            ldst[k] = loct[k] * plane + row * a.pws * kWord;
            if (ih >= 0 && ih < H && n < a.N)
                goff[k] = 2u * (uint32_t)((n * a.IC + loct[k] * 8) * HW + ih * W + c0);
        }
    }

    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t *>(a.x), 0, a.x_bytes, kRsrcFlags);

    RawPixels<PX> raw[PT][8];
    auto load_patch = [&](int c) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < PT; ++k) {
            const int left = a.IC - 1 - (c * a.co + loct[k]) * 8;      // channels past the last: sign bit, out of range
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                const uint32_t off = (goff[k] + 2u * (uint32_t)((c * a.co * 8 + q) * HW)) |
                                     ((uint32_t)(left - q) & kOutOfRange);
                if constexpr (PX == 8) {
                    const uint4v v = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(xrsrc, off, 0, 0));
#pragma unroll
                    for (int d = 0; d < 4; ++d) raw[k][q].d[d] = v[d];
                } else if constexpr (PX == 4) {
                    const uint2v v = __builtin_bit_cast(uint2v, __builtin_amdgcn_raw_buffer_load_b64(xrsrc, off, 0, 0));
                    raw[k][q].d[0] = v[0];
                    raw[k][q].d[1] = v[1];
                } else {
                    raw[k][q].d[0] = __builtin_amdgcn_raw_buffer_load_b16(xrsrc, off, 0, 0);
                }
            }
        }
    };
    auto store_patch = [&](unsigned char *dst) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < PT; ++k) {
            if (ldst[k] < 0) continue;
            int q = lq[k], f = lph[k];
#pragma unroll
            for (int e = 0; e < PX; ++e) {
                uint32_t o[4];
#pragma unroll
                for (int d = 0; d < 4; ++d)
                    o[d] = pack_halves(raw[k][2 * d].d[e >> 1], raw[k][2 * d + 1].d[e >> 1], e & 1);
                *reinterpret_cast<uint4v *>(dst + ldst[k] + (f * a.cp + q) * kWord) = uint4v{o[0], o[1], o[2], o[3]};
                if (++f == a.sw) { f = 0; ++q; }
            }
        }
    };

    // (the tail's parameters first: memory answers in order, and they are needed before the patch is)
    float sc = 0.0f, sf = 0.0f;
    if (a.splits == 1 && tid < MT && m0 + tid < a.OC) {
        sc = a.scale[m0 + tid];
        sf = a.shift[m0 + tid];
        if (a.bias) sf = fmaf(a.bias[m0 + tid], sc, sf);
    }
    load_patch(c_beg);
#pragma unroll
    for (int d = 0; d < RING; ++d) {
        load_weights(d);
        __builtin_amdgcn_sched_barrier(0);
    }

    // patch offsets of the units, [half-wave][step]; a few steps past the end are read ahead, never used
    const int tpitch = a.steps + RING;
    for (int u = tid; u < 2 * tpitch; u += 256) {
        int o, s, f;
        int t = divide(u, a.by_co, &o);
        const int r = divide(t, a.by_s, &s), q = divide(s, a.by_sw, &f);
        tab[(u & 1) * tpitch + (u >> 1)] = t < a.R * a.S ? o * plane + (r * a.pws + f * a.cp + q) * kWord : kNoTap;
    }
    if (tid == 0) *reinterpret_cast<uint4v *>(smem + a.zero_at) = uint4v{0u, 0u, 0u, 0u};
    // zero columns left and right of the image: no load task writes them
    for (int i = tid; i < (c_end - c_beg > 1 ? 2 : 1) * a.co * a.rows * a.border; i += 256) {
        int e, f;
        const int row = divide(i, a.by_border, &e);             // (buffer, octet, row)
        const int q = divide(e < a.pw ? e : e + W, a.by_sw, &f);
        *reinterpret_cast<uint4v *>(patch + (row * a.pws + f * a.cp + q) * kWord) = uint4v{0u, 0u, 0u, 0u};
    }
    if (tid < MT) {
        ss[2 * tid] = sc;
        ss[2 * tid + 1] = sf;
    }

    int pb[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int p = n0 + wn * WTN + j * 32 + lrow;
        pb[j] = 0;                                  // pixels past the end shadow the first word
        if (p < n_end) {
            int r, ow;
            const int n = divide(p, a.by_ohw, &r), oh = divide(r, a.by_ow, &ow);
            pb[j] = ((n * a.vh + oh * a.vsh - vr0) * a.pws + ow) * kWord;
        }
    }

    float16v acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    store_patch(patch);
    __syncthreads();

    // One turn = RING steps.  A step's pixels are requested two steps ahead, their table entries a
    // turn ahead, its weights RING steps ahead: a lone wave per SIMD sees neither latency.
    typedef int int4v __attribute__((ext_vector_type(4)));
    struct Offsets { int4v v[RING / 4]; };
    const Offsets *tb = reinterpret_cast<const Offsets *>(tab + lhalf * tpitch);
    const int turns = a.steps / RING, patch_at = a.tab_bytes + 2 * MT * 4;
    for (int c = c_beg; c < c_end; ++c) {
        const int P = patch_at + ((c - c_beg) & 1) * a.patch_bytes;
        if (c + 1 < c_end) load_patch(c + 1);
        uint4v bf[4][NJ];
        // A unit without a tap multiplies zeros by zeros: its weights against pixels of the image would turn an
        // infinity there into a NaN.  Its offset is past everything and the word of zeros lies last, so that one
        // minimum per address selects it; only a chunk's last turn has such units.  (A minimum in every turn:
        // 0 to 2 % slower; a compare and select: 1 to 4 %; branches around the MFMAs of such steps: 2 to 18 %.)
        auto fetch = [&](int off, int slot, bool surplus) __attribute__((always_inline)) {
#pragma unroll
            for (int j = 0; j < NJ; ++j)
                bf[slot][j] = *reinterpret_cast<const uint4v *>(smem + (surplus ? min(P + pb[j] + off, a.zero_at) : P + pb[j] + off));
        };
        Offsets cur = tb[0];
        fetch(cur.v[0][0], 0, true);
        fetch(cur.v[0][1], 1, true);
        auto turn = [&](int t, auto last) __attribute__((always_inline)) {
            const Offsets nxt = tb[t + 1];
#pragma unroll
            for (int d = 0; d < RING; ++d) {
                fetch(d + 2 < RING ? cur.v[(d + 2) / 4][(d + 2) & 3] : nxt.v[0][d + 2 - RING], (d + 2) & 3, last || d + 2 >= RING);
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int j = 0; j < NJ; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            __builtin_bit_cast(bf16x8v, bf[d & 3][j]), __builtin_bit_cast(bf16x8v, wreg[d][i]), acc[i][j], 0, 0, 0);
                load_weights(d);
                __builtin_amdgcn_sched_barrier(0);
            }
            cur = nxt;
        };
        for (int t = 0; t + 1 < turns; ++t) turn(t, std::false_type{});
        turn(turns - 1, std::true_type{});
        if (c + 1 < c_end) store_patch(patch + ((c + 1 - c_beg) & 1) * a.patch_bytes);
        __syncthreads();
    }

    if (a.splits == 1) {                            // the patches are free to stage the tail
        unsigned char *stage = patch + wave * (MI * NJ * kStageBytes);
        const TailArgs tail{a.scale, a.shift, a.bias, a.residual, a.y, a.OC, OHW, n_end, a.relu};
        store_acc_tiles_batched<MI, NJ>(acc, stage, lane, m0 + wm * WTM, n0 + wn * WTN, tail, a.vmode, ss, wm * WTM);
        return;
    }
    // raw sums of this slice: value v of a lane is pixel 8*(v/4) + 4*lhalf + v%4 of channel lrow
    float *wsp = a.ws + (size_t)blockIdx.y * ((size_t)a.npix * a.OC);
    const bool vec = OHW % 4 == 0;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        const int p0t = n0 + wn * WTN + j * 32;
        const int nt0 = p0t / OHW, remt = p0t - nt0 * OHW;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int oc = m0 + wm * WTM + i * 32 + lrow;
            if (oc >= a.OC) continue;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int pl = 8 * g + 4 * lhalf;
                int n = nt0, rm = remt + pl;
                while (rm >= OHW) { rm -= OHW; ++n; }
                if (vec) {
                    if (p0t + pl < n_end)
                        *reinterpret_cast<float4v *>(wsp + (size_t)(n * a.OC + oc) * OHW + rm) =
                            float4v{acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
                } else {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        if (p0t + pl + q < n_end) wsp[(size_t)(n * a.OC + oc) * OHW + rm] = acc[i][j][4 * g + q];
                        if (++rm >= OHW) { rm -= OHW; ++n; }
                    }
                }
            }
        }
    }
}

// ---- the pack launch: 16 output channels x one chunk per workgroup -----------------------------
// Packed order: [channel tile][chunk][unit = (tap, octet)][channel of the tile], 16-byte words of
// eight input channels, zeros past OC, IC and the last unit.
struct PackArgs {
    const bf16_t *w;
    bf16_t *packed;
    int IC, OC, T, co, nchunks, octets, steps, mt;
    int row_pitch;                        // elements per staged row (an odd number of dwords: 16 rows, distinct banks)
    Divider by_octets, by_t4;             // octets in all (chunks are filled up with zeros), 4-element pieces per row
};

// One workgroup: 16 output channels x one octet.  Their 8 T elements are contiguous in every row.
__global__ __launch_bounds__(256) void pack_weights_kernel(const PackArgs a)
{
    extern __shared__ __attribute__((aligned(16))) bf16_t rows[];
    const int tid = threadIdx.x;
    int oct;
    const int og = divide(blockIdx.x, a.by_octets, &oct);
    const int oc0 = og * 16, ic0 = oct * 8, n8 = 8 * a.T;
    const int n_el = max(0, min(a.IC - ic0, 8)) * a.T;
    // pieces of four elements, 2-byte aligned in memory; whole pieces are one load each, all in flight
    constexpr int U = 4;
    for (int i0 = tid; i0 < 16 * (n8 / 4); i0 += 256 * U) {
        uint2v v[U];
        int at[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            int piece;
            const int r = divide(i0 + k * 256, a.by_t4, &piece);
            const int e = piece * 4, oc = oc0 + r;
            at[k] = r < 16 ? r * a.row_pitch + e : -1;
            v[k] = uint2v{0u, 0u};
            if (r < 16 && oc < a.OC) {
                const bf16_t *src = a.w + ((size_t)oc * a.IC + ic0) * a.T + e;
                if (e + 4 <= n_el) {
                    __builtin_memcpy(&v[k], src, 8);
                } else {
#pragma unroll
                    for (int q = 0; q < 3; ++q)
                        if (e + q < n_el) v[k][q >> 1] |= (uint32_t)src[q] << (16 * (q & 1));
                }
            }
        }
#pragma unroll
        for (int k = 0; k < U; ++k)
            if (at[k] >= 0) {
                uint32_t *d = reinterpret_cast<uint32_t *>(rows + at[k]);
                d[0] = v[k][0];
                d[1] = v[k][1];
            }
    }
    __syncthreads();
    const int tile = oc0 / a.mt, ocl = oc0 - tile * a.mt;
    const int c = oct / a.co, o = oct - c * a.co;
    uint4v *dst = reinterpret_cast<uint4v *>(a.packed) + (size_t)(tile * a.nchunks + c) * (a.steps * 2 * a.mt) + ocl;
    // units of this octet: (tap, octet); the last octet of a chunk also clears the chunk's surplus units
    const int units = a.T + (o == a.co - 1 ? 2 * a.steps - a.T * a.co : 0);
    for (int i = tid; i < units * 16; i += 256) {
        const int r = i & 15, t = i >> 4;
        uint4v v = {0u, 0u, 0u, 0u};
        if (t < a.T) {
            const bf16_t *e = rows + r * a.row_pitch + t;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                v[q] = (uint32_t)e[2 * q * a.T] | ((uint32_t)e[(2 * q + 1) * a.T] << 16);
        }
        dst[(size_t)(t < a.T ? t * a.co + o : a.T * (a.co - 1) + t) * a.mt + r] = v;
    }
}

template <typename K>
bool allow_lds(K kernel)
{
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)kMaxLds) == hipSuccess;
}

template <int WM, int MI, int NJ, int PX, int PT>
tvg_status launch_one(const AnyArgs &a, dim3 grid, size_t lds, hipStream_t stream)
{
    static const bool ok = allow_lds(conv_bf16_any_kernel<WM, MI, NJ, PX, PT>);
    if (!ok) return TVG_ERR_LAUNCH;
    hipLaunchKernelGGL((conv_bf16_any_kernel<WM, MI, NJ, PX, PT>), grid, dim3(256), lds, stream, a);
    return hipGetLastError() == hipSuccess ? TVG_OK : TVG_ERR_LAUNCH;
}

template <int WM, int MI, int NJ>
tvg_status launch_tile(const AnyArgs &a, int px, int pt, dim3 grid, size_t lds, hipStream_t stream)
{
    if (px == 8) return pt == 1 ? launch_one<WM, MI, NJ, 8, 1>(a, grid, lds, stream) : launch_one<WM, MI, NJ, 8, 2>(a, grid, lds, stream);
    if (px == 4) return pt == 1 ? launch_one<WM, MI, NJ, 4, 1>(a, grid, lds, stream) : launch_one<WM, MI, NJ, 4, 2>(a, grid, lds, stream);
    return pt == 1 ? launch_one<WM, MI, NJ, 1, 1>(a, grid, lds, stream) : launch_one<WM, MI, NJ, 1, 2>(a, grid, lds, stream);
}

int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Fits a tile shape to the problem: octets per chunk, LDS.  False if it has no room.
bool fit_tile(const ConvProblem &p, int mt, int nt, size_t lds_limit, ConvAnyPlan *plan)
{
    const int T = p.R * p.S, octets = ceil_div(p.IC, 8);
    plan->mt = mt;
    plan->nt = nt;
    plan->px = p.W >= 8 ? 8 : p.W >= 4 ? 4 : 1;
    plan->groups = ceil_div(p.W, plan->px);
    plan->vsh = p.R < p.sh ? p.R : p.sh;
    plan->vh = (p.OH - 1) * plan->vsh + p.R;
    // Tiles stay within an image where that wastes at most a sixteenth of their pixels (and the filter
    // has rows to share): a tile that crosses images stages R rows twice.
    const int ohw = p.OH * p.OW, tpi = ceil_div(ohw, nt);
    plan->tpi = p.R > 1 && 16 * ((long)tpi * nt - ohw) <= ohw ? tpi : 0;
    plan->ntiles = plan->tpi ? (long)p.N * tpi : ceil_div(p.npix, nt);
    // patch rows of the tallest tile (of all, or of a full cycle of them)
    int rows = 0;
    for (long i = 0; i < plan->ntiles && i < (plan->tpi ? tpi : 65536); ++i) {
        const int lo = (int)i * nt, hi = (plan->tpi && lo + nt > ohw ? ohw : lo + nt > p.npix ? p.npix : lo + nt) - 1;
        const int r = (hi / ohw) * plan->vh + hi % ohw / p.OW * plan->vsh + p.R - ((lo / ohw) * plan->vh + lo % ohw / p.OW * plan->vsh);
        rows = r > rows ? r : rows;
    }
    if (!plan->tpi && plan->ntiles > 65536)          // (a bound: ceil((NT-1)/OW) + 1 output rows, R rows apart at a new image)
        rows = ceil_div(nt - 1, p.OW) * plan->vsh + p.R + ceil_div(nt - 1, ohw) * (p.R - plan->vsh);
    plan->rows = rows;
    const int need = (p.OW - 1) * p.sw + p.S, have = p.W + p.pw;
    plan->cp = ceil_div(need > have ? need : have, p.sw);
    plan->pws = plan->cp * p.sw;
    const size_t plane = (size_t)rows * plan->pws * kWord;
    const size_t stage = (size_t)(mt / 32) * (nt / 32) * kStageBytes;
    // Octets per chunk: the fewest MFMA steps in all (a chunk's steps are rounded up to whole turns),
    // then the fewest chunks.
    const int ring = ring_of(mt == 64 && nt == 256 ? 2 : 1);
    long best = -1;
    for (int co = octets < 16 ? octets : 16; co >= 1; --co) {
        const int nchunks = ceil_div(octets, co), steps = ceil_div(ceil_div(co * T, 2), ring) * ring;
        const long tasks = (long)rows * plan->groups * co;
        if (tasks > 512 || co * 8 * T > 2040) continue;      // (the pack launch stages 16 rows of an octet in 64 KB)
        const int tab_bytes = (2 * (steps + ring) * 4 + 15) / 16 * 16;
        const size_t body = (nchunks > 1 ? 2 : 1) * plane * co;
        const size_t lds_bytes = tab_bytes + 2 * mt * 4 + (body + kWord > stage ? body + kWord : stage);
        if (lds_bytes > lds_limit || (best >= 0 && (long)nchunks * (steps + 3) >= best)) continue;   // (a chunk change costs about 3 steps)
        best = (long)nchunks * (steps + 3);
        plan->co = co;
        plan->pt = tasks > 256 ? 2 : 1;
        plan->nchunks = nchunks;
        plan->steps = steps;
        plan->tab_bytes = tab_bytes;
        plan->patch_bytes = (int)(plane * co);
        plan->lds_bytes = lds_bytes;
    }
    return best >= 0;
}

}  // namespace

bool plan_conv_bf16_any(const ConvProblem &p, ConvAnyPlan *plan)
{
    if (p.dtype != TVG_BF16) return false;
    const Knobs knobs = forced_knobs(p);
    if (knobs.mt || knobs.nt || knobs.split_k) return false;     // a caller who fixes the gather kernel's tile or split
    if ((size_t)p.N * p.IC * p.H * p.W * 2 >= (size_t)kOutOfRange) return false;
    if ((int64_t)p.N * ((int64_t)(p.OH - 1) * p.sh + p.R) >= ((int64_t)1 << 30)) return false;
    // Tile: 64 channels unless the last 32 would be padding; the widest pixel tile that still
    // gives every CU a workgroup, else the one with the most workgroups.
    const int mt = p.OC % 64 != 0 && p.OC % 64 <= 32 && p.OC <= 96 ? 32 : 64;
    bool found = false;
    for (int nt : {256, 128, 64}) {
        if (mt == 32 && nt == 64) continue;
        ConvAnyPlan t;
        if (!fit_tile(p, mt, nt, 80 * 1024, &t) && !fit_tile(p, mt, nt, kMaxLds, &t)) continue;
        *plan = t;
        found = true;
        if ((long)ceil_div(p.OC, mt) * t.ntiles >= kComputeUnits) break;
    }
    if (!found) return false;
    const size_t packed = (size_t)ceil_div(p.OC, mt) * plan->nchunks * plan->steps * 2 * mt * kWord;
    if (packed >= ((size_t)1 << 31)) return false;
    plan->packed_bytes = (packed + 255) / 256 * 256;
    const long tiles = ceil_div(p.OC, mt) * plan->ntiles;
    if (tiles > 0x7FFFFFFF) return false;
    // Fewer tiles than three quarters of the CUs: slices of at least two chunks on workgroups of their
    // own, and a third launch adds them, where that saves more steps (about 0.08 us each for a lone
    // workgroup) than the launch and the partial sums cost (about 6 us).
    int splits = 1;
    if (4 * tiles <= 3 * kComputeUnits) {
        splits = (int)(2 * kComputeUnits / tiles);
        if (splits > plan->nchunks / 2) splits = plan->nchunks / 2;
        if (splits > 16) splits = 16;
        if (splits < 1 || (long)plan->nchunks * plan->steps * (splits - 1) < 80L * splits) splits = 1;
    }
    plan->chunks_per_split = ceil_div(plan->nchunks, splits);
    plan->splits = ceil_div(plan->nchunks, plan->chunks_per_split);
    plan->tiles = tiles;
    plan->workspace_bytes = plan->packed_bytes +
                            (plan->splits > 1 ? (size_t)plan->splits * p.npix * p.OC * sizeof(float) : 0);
    return true;
}

bool conv_bf16_any_pointers_ok(const ConvPointers &ptr)
{
    return reinterpret_cast<uintptr_t>(ptr.x) % 2 == 0 && reinterpret_cast<uintptr_t>(ptr.w) % 2 == 0 &&
           reinterpret_cast<uintptr_t>(ptr.y) % 2 == 0 && reinterpret_cast<uintptr_t>(ptr.residual) % 2 == 0;
}

tvg_status launch_conv_bf16_any(const ConvProblem &p, const ConvAnyPlan &plan, const ConvPointers &ptr, hipStream_t stream)
{
    const int T = p.R * p.S, mtiles = ceil_div(p.OC, plan.mt);
    PackArgs k;
    k.w = static_cast<const bf16_t *>(ptr.w);
    k.packed = reinterpret_cast<bf16_t *>(ptr.workspace);
    k.IC = p.IC; k.OC = p.OC; k.T = T; k.co = plan.co; k.nchunks = plan.nchunks; k.steps = plan.steps; k.mt = plan.mt;
    k.octets = plan.co * plan.nchunks;
    k.row_pitch = (8 * T + 2) | 2;
    k.by_octets = make_divider(k.octets);
    k.by_t4 = make_divider(2 * T);
    hipLaunchKernelGGL(pack_weights_kernel, dim3((unsigned)(mtiles * (plan.mt / 16) * k.octets)), dim3(256),
                       (size_t)16 * k.row_pitch * 2, stream, k);
    if (hipGetLastError() != hipSuccess) return TVG_ERR_LAUNCH;

    AnyArgs a;
    a.x = static_cast<const bf16_t *>(ptr.x);
    a.packed = k.packed;
    a.scale = ptr.scale; a.shift = ptr.shift; a.bias = ptr.bias;
    a.residual = static_cast<const bf16_t *>(ptr.residual);
    a.y = static_cast<bf16_t *>(ptr.y);
    a.ws = reinterpret_cast<float *>(reinterpret_cast<char *>(ptr.workspace) + plan.packed_bytes);
    a.N = p.N; a.IC = p.IC; a.H = p.H; a.W = p.W; a.OC = p.OC; a.OH = p.OH; a.OW = p.OW;
    a.sh = p.sh; a.sw = p.sw; a.ph = p.ph; a.pw = p.pw; a.R = p.R; a.S = p.S; a.npix = p.npix;
    a.relu = p.relu | (p.stream_out << 1);
    a.vmode = pick_store_vmode(p.dtype, p.OH * p.OW, ptr.y, ptr.residual);
    a.co = plan.co; a.nchunks = plan.nchunks; a.chunks_per_split = plan.chunks_per_split;
    a.steps = plan.steps;
    a.rows = plan.rows; a.pws = plan.pws; a.cp = plan.cp; a.vh = plan.vh; a.vsh = plan.vsh; a.groups = plan.groups;
    a.mtiles = mtiles; a.splits = plan.splits;
    a.x_bytes = (uint32_t)((size_t)p.N * p.IC * p.H * p.W * 2);
    a.packed_bytes = (uint32_t)plan.packed_bytes;
    a.tab_bytes = plan.tab_bytes; a.patch_bytes = plan.patch_bytes;
    a.zero_at = plan.tab_bytes + 2 * plan.mt * 4 + (plan.nchunks > 1 ? 2 : 1) * plan.patch_bytes;
    a.by_ohw = make_divider(p.OH * p.OW); a.by_ow = make_divider(p.OW); a.by_vh = make_divider(plan.vh);
    a.by_r = make_divider(p.R); a.by_groups = make_divider(plan.groups); a.by_mtiles = make_divider(mtiles);
    a.by_co = make_divider(plan.co); a.by_s = make_divider(p.S); a.by_sw = make_divider(p.sw);
    a.tpi = plan.tpi;
    a.by_tpi = make_divider(plan.tpi ? plan.tpi : 1);
    a.border = p.pw + ((p.OW - 1) * p.sw + p.S > p.W + p.pw ? (p.OW - 1) * p.sw + p.S - p.W - p.pw : 0);
    a.by_border = make_divider(a.border ? a.border : 1);
    const dim3 grid((unsigned)plan.tiles, (unsigned)plan.splits);
    tvg_status st;
#define TVG_ANY_TILE(WM_, MI_, NJ_) launch_tile<WM_, MI_, NJ_>(a, plan.px, plan.pt, grid, plan.lds_bytes, stream)
    if (plan.mt == 32) st = plan.nt == 256 ? TVG_ANY_TILE(1, 1, 2) : TVG_ANY_TILE(1, 1, 1);
    else if (plan.nt == 256) st = TVG_ANY_TILE(1, 2, 2);
    else if (plan.nt == 128) st = TVG_ANY_TILE(2, 1, 2);
    else st = TVG_ANY_TILE(2, 1, 1);
#undef TVG_ANY_TILE
    if (st != TVG_OK || plan.splits == 1) return st;
    ConvPointers rp = ptr;
    rp.workspace = a.ws;
    return launch_splitk_reduce(p, plan.splits, rp, stream);
}

}  // namespace tvg
