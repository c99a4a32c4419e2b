// bf16 3x3 (pad 1) and 1x1 convolutions, stride 1 or 2, of problems with few tiles: small batches, deep layers.
//
// Such a layer is one round of workgroups or less, so its time is that of one workgroup from its first instruction
// to its last store.  The 64 x 64 tiles of the other kernels walk the whole reduction in one chain (512 -> 512 at 7x7,
// batch 1: 8 workgroups of 32 steps, 36 us).  Here a workgroup owns 16 channels x 16 NJ pixels, its waves take 32
// input channels each and add their sums through LDS at the end, and no step of a wave waits for another wave.
//   - Input rows lie in LDS as they lie in memory, [channel][row][column], copied with 16-byte loads; gfx950's
//     transposing LDS read turns four pixels of four channels into operand order, so nothing is packed.
//   - Column taps.  Such a read wants 8-byte aligned pixels, a column tap shifts them by two bytes.  So the three
//     column taps of a row multiply the SAME operand into three accumulators, D_s, and the shift happens once, on the
//     sums: y[p] = D_0[p - 1] + D_1[p] + D_2[p + 1], masked at the row's ends.  That also reads a third of the
//     operands.  Stride 2: even and odd columns are staged apart, taps 1 and 2 share an accumulator.
//   - 3x3 weights: 16-byte pieces with adjacent lanes on adjacent pieces, through LDS into 144-byte runs per lane,
//     transposed by byte permutes.  (Loaded straight into the runs, one lane per output channel, every lane of a load
//     is on a line of its own: 9.6 us against 6.6 on the layer above.)
//   - Few chunks (64 channels): a wave takes one filter row of a chunk, three times the waves (64 -> 64 at 56x56,
//     batch 1, 6.6 -> 5.5 us; 64 -> 128 stride 2 5.6 -> 4.8).
//   - Divisions by what the host knows are a high multiply and a shift, on the scalar unit where they are uniform:
//     0.5 us of every layer against the float reciprocal, which has no scalar form.
// Sums do not depend on tile, batch or output channels, only on the input channels (and the split into filter rows).
// Measured, us, batch 1 (4): 64 -> 64 56x56 7.3 -> 5.5; 64 -> 128 s2 7.7 -> 4.8; 128 -> 128 28x28 9.0 -> 5.1 (9.3 -> 6.7);
// 128 -> 256 s2 11.1 -> 4.9 (11.4 -> 6.7); 256 -> 256 14x14 13.3 -> 5.4 (13.6 -> 7.4); 256 -> 512 s2 21.0 -> 5.5 (19.4 ->
// 7.1); 512 -> 512 7x7 35.8 -> 6.3 (20.1 -> 7.4); 1x1: 512 -> 512 14x14 7.6 -> 4.3 (7.9 -> 6.4), 1024 -> 1024 7x7 13.7 ->
// 5.9 (13.8 -> 7.2).  The ResNet-18 body at batch 1: 282 -> 114 us.  About 3 us of each is launch and first loads.
#include <algorithm>
#include <type_traits>

#include "tvg_device.h"
#include "tvg_internal.h"

namespace tvg {

namespace {

constexpr int kRsrcFlags = 0x00020000;
constexpr uint32_t kOutOfRange = 0x80000000u;      // and everything above: tensors stay below 2 GiB
constexpr int kChunk = 32;                         // input channels per turn: the depth of one MFMA
constexpr int kWeightRow = 592;                    // 576 bytes of a 3x3 chunk's weights per output channel, and a gap: distinct banks
constexpr int kOctetGap = 128;                     // between channel octets of the staged rows: distinct banks
constexpr int kMaxWaves = 8;

typedef short short4v __attribute__((ext_vector_type(4)));
typedef short short8v __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) short4v *lds_short4;

struct RowsArgs {
    const bf16_t *x, *w;
    const float *scale, *shift, *bias;
    const bf16_t *residual;
    bf16_t *y, *y2;                    // y2: output of the channels from k1 on (two-head launches)
    int N, IC, H, W, OC, OH, OW, relu, relu2, k1, centre2, vec;
    int tr, groups, cblocks, t8;       // a tile: output rows, 4-pixel groups per row, tiles across a row; 8-pixel loads per staged row
    int vh, rows, images;              // staged ("virtual") rows per image and per tile, images a tile may touch
    int dg, drow, dch;                 // 64 load tasks further: pieces of a row, rows, channels
    int row_bytes, plane, region;      // LDS bytes per staged row, per channel and per wave
    int ptiles, nch;                   // pixel tiles, chunks
    uint32_t x_bytes, w_bytes;
    Divider by_ptiles, by_oh, by_vh, by_t8, by_rows, by_groups, by_cblocks;
};

// A wave's LDS operations execute in order; this keeps the compiler from reordering them.
__device__ __forceinline__ void wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// R x R filter, stride ST; UNAL: rows of an odd number of pixels; 16 output channels x 16 NJ pixel slots per
// workgroup, PT load tasks per lane and chunk.
// RS: a wave takes one filter row of a chunk (waves = 3 x chunks, the rows outermost).  DUAL: two heads.
// CENTRE (R = 1): the weights are the centre taps of 3x3 filters (a two-head call's second head on its own).
template <int R, int ST, bool UNAL, int NJ, int PT, bool RS, bool DUAL, bool CENTRE = false>
__global__ __launch_bounds__(64 * kMaxWaves) void conv_rows_kernel(const RowsArgs a)
{
    constexpr int NT = 16 * NJ, QT = 4 * NJ;
    constexpr int NS = R == 1 ? 1 : ST == 1 ? 3 : 2;        // accumulator sets: column taps that share a shift
    constexpr int MID = NS > 1 ? 1 : 0;                     // the set without a shift
    constexpr int VR = R == 1 ? 1 : ST;                     // staged rows per output row
    constexpr int PITCH = NT + 4;                           // floats per channel of the partial sums
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nwaves = blockDim.x >> 6;
    const int l16 = lane & 15, quad = lane >> 4;
    int pt, cb, oh0;
    const int m0 = 16 * divide(xcd_remap(blockIdx.x, gridDim.x), a.by_ptiles, &pt);
    const int row0 = divide(pt, a.by_cblocks, &cb) * a.tr, HW = a.H * a.W;
    const int n0 = divide(row0, a.by_oh, &oh0), col0 = cb * a.groups * 4;
    const int vrow = oh0 * VR, vr0 = n0 * a.vh + vrow;
    const bool head2 = DUAL && m0 >= a.k1, centre = head2 && a.centre2;
    const int c0 = RS ? wave % a.nch : wave, r0 = RS ? wave / a.nch : 0;        // first chunk, first filter row

    float *ss = reinterpret_cast<float *>(smem);
    unsigned char *body = smem + 2 * 16 * 4;
    unsigned char *mine = body + wave * a.region;          // this wave's: a chunk's 3x3 weights first, then its input rows

    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(a.x), 0, a.x_bytes, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(a.w), 0, a.w_bytes, kRsrcFlags);

    // ---- weights.  1x1: a lane's eight channels, straight into the operand.  3x3: 36 pieces of 16 bytes per output
    // channel and chunk, adjacent lanes adjacent pieces (channels past the last are out of range: zeros)
    constexpr int WL = R == 3 ? 9 : 1;
    uint32_t woff[WL];
    int wdst[WL];
    if constexpr (R == 3) {
#pragma unroll
        for (int k = 0; k < WL; ++k) {
            const int id = lane + 64 * k, oc = id / 36, piece = id % 36;
            woff[k] = __umul24(__umul24(m0 + oc, a.IC), 18u) + piece * 16;
            wdst[k] = oc * kWeightRow + piece * 16;
        }
    } else {
        woff[0] = CENTRE ? __umul24(__umul24(m0 + l16, a.IC) + 8 * quad, 18u) + 8 : 2u * (__umul24(m0 + l16, a.IC) + 8 * quad);
    }
    uint4v wraw[WL];
    auto load_weights = [&](int c) __attribute__((always_inline)) {
        if constexpr (CENTRE) {
            uint32_t tap[8];
#pragma unroll
            for (int e = 0; e < 8; ++e)
                tap[e] = __builtin_amdgcn_raw_buffer_load_b16(wrsrc, woff[0] + 18 * e, c * (2 * kChunk * 9), 0);
#pragma unroll
            for (int d = 0; d < 4; ++d) wraw[0][d] = tap[2 * d] | (tap[2 * d + 1] << 16);
            return;
        }
#pragma unroll
        for (int k = 0; k < WL; ++k)
            wraw[k] = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, woff[k], c * (2 * kChunk * R * R), 0));
    };
    load_weights(c0);

    // ---- input load tasks: eight pixels of a staged row of one channel ------------------------
    uint32_t goff[PT];
    int dst[PT], odd[PT];
    {
        int g8, row;
        int ch = divide(lane, a.by_t8, &g8);
        ch = divide(ch, a.by_rows, &row);
#pragma unroll
        for (int k = 0; k < PT; ++k) {
            int n = n0, v = row + r0 + vrow;
            if (a.images > 1) n = divide(vr0 + row + r0, a.by_vh, &v);
            const int ih = R == 3 ? v - 1 : v * ST;
            goff[k] = kOutOfRange;
            dst[k] = -1;
            odd[k] = 0;
            if (ch < kChunk) {
                dst[k] = __umul24(ch, a.plane) + (ch >> 3) * kOctetGap + __umul24(row, a.row_bytes) + g8 * (ST == 1 ? 16 : 8);
                if (ih >= 0 && ih < a.H && n < a.N) {
                    const uint32_t at = __umul24(__umul24(n, a.IC) + ch, HW) + __umul24(ih, a.W) + col0 + g8 * 8;
                    goff[k] = 2u * (UNAL ? at & ~1u : at);
                    odd[k] = (int)(at & 1) | (g8 << 1);
                }
            }
            g8 += a.dg;
            row += a.drow;
            ch += a.dch;
            if (g8 >= a.t8) { g8 -= a.t8; ++row; }
            if (row >= a.rows) { row -= a.rows; ++ch; }
        }
    }
    uint32_t raw[PT][UNAL ? 5 : 4];
    auto load_rows = [&](int c) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < PT; ++k) {
            const uint4v v = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(xrsrc, goff[k], c * 2 * kChunk * HW, 0));
#pragma unroll
            for (int d = 0; d < 4; ++d) raw[k][d] = v[d];
            if constexpr (UNAL) raw[k][4] = __builtin_amdgcn_raw_buffer_load_b32(xrsrc, goff[k] + 16, c * 2 * kChunk * HW, 0);
        }
    };
    load_rows(c0);

    // ---- pixel operand addresses.  A transposing read takes 4 pixels of 4 channels from each of 4 lanes: lane =
    // (channel octet of the chunk, channel, group of four pixels)
    int pb[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        int cg, oh;
        const int row = divide(4 * j + (lane & 3), a.by_groups, &cg);
        int at = row * VR;                         // staged row of filter row 0
        bool in = row < a.tr;
        if (a.images > 1) {
            const int n = divide(row0 + row, a.by_oh, &oh);
            at = __umul24(n, a.vh) + oh * VR - vr0;
            in = in && n < a.N;
        }
        pb[j] = in ? __umul24(at, a.row_bytes) + cg * 8 : 0;
        pb[j] += (8 * quad + ((lane >> 2) & 3)) * a.plane + quad * kOctetGap;
    }

    float4v acc[NS][NJ];
#pragma unroll
    for (int s = 0; s < NS; ++s)
#pragma unroll
        for (int j = 0; j < NJ; ++j) acc[s][j] = float4v{0.0f, 0.0f, 0.0f, 0.0f};

    if (tid < 16) {
        float sc = 0.0f, sf = 0.0f;
        if (m0 + tid < a.OC) {
            sc = a.scale[m0 + tid];
            sf = a.shift[m0 + tid];
            if (a.bias) sf = fmaf(a.bias[m0 + tid], sc, sf);
        }
        ss[2 * tid] = sc;
        ss[2 * tid + 1] = sf;
    }

    for (int c = c0; c < a.nch; c += nwaves) {
        uint32_t wr[4 * WL];                       // channels 8 quad .. + 7 of the lane's output channel, taps innermost
        if constexpr (R == 3) {
#pragma unroll
            for (int k = 0; k < WL; ++k) *reinterpret_cast<uint4v *>(mine + wdst[k]) = wraw[k];
            wave_fence();
#pragma unroll
            for (int k = 0; k < WL; ++k) {
                const uint4v v = *reinterpret_cast<const uint4v *>(mine + l16 * kWeightRow + quad * 144 + k * 16);
#pragma unroll
                for (int d = 0; d < 4; ++d) wr[4 * k + d] = v[d];
            }
            wave_fence();
        } else {
#pragma unroll
            for (int d = 0; d < 4; ++d) wr[d] = wraw[0][d];
        }
#pragma unroll
        for (int k = 0; k < PT; ++k) {
            if (dst[k] < 0) continue;
            uint32_t v[4];
#pragma unroll
            for (int d = 0; d < 4; ++d) v[d] = raw[k][d];
            if constexpr (UNAL) {
#pragma unroll
                for (int d = 0; d < 4; ++d) v[d] = __builtin_amdgcn_alignbit(raw[k][d + 1], raw[k][d], (odd[k] & 1) * 16);
                if constexpr (R == 3 && ST == 2) {           // the column right of an odd row is padding
                    const int last = (a.W - 8 * (odd[k] >> 1)) >> 1;
#pragma unroll
                    for (int d = 0; d < 4; ++d) v[d] = d == last ? v[d] & 0xFFFFu : v[d];
                }
            }
            if constexpr (ST == 1) {
                *reinterpret_cast<uint4v *>(mine + dst[k]) = uint4v{v[0], v[1], v[2], v[3]};
            } else {                               // even columns, then odd ones
                *reinterpret_cast<uint2v *>(mine + dst[k]) =
                    uint2v{__builtin_amdgcn_perm(v[1], v[0], 0x05040100u), __builtin_amdgcn_perm(v[3], v[2], 0x05040100u)};
                if constexpr (R == 3)
                    *reinterpret_cast<uint2v *>(mine + dst[k] + a.t8 * 8) =
                        uint2v{__builtin_amdgcn_perm(v[1], v[0], 0x07060302u), __builtin_amdgcn_perm(v[3], v[2], 0x07060302u)};
            }
        }
        wave_fence();
        if (c + nwaves < a.nch) {                  // (every raw register is free again)
            load_weights(c + nwaves);
            load_rows(c + nwaves);
        }
        // one filter row: its weights from the lane's run, its operand read once for the three column taps
        auto filter_row = [&](auto rc, auto middle) __attribute__((always_inline)) {
            constexpr int r = rc;
            uint4v wop[R];
#pragma unroll
            for (int s = 0; s < R; ++s)
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    if constexpr (R == 1) {
                        wop[s][d] = wr[d];
                    } else {
                        const int e0 = 18 * d + 3 * r + s, e1 = e0 + 9;
                        const uint32_t sel = ((e0 & 1) ? 0x0302u : 0x0100u) | ((e1 & 1) ? 0x07060000u : 0x05040000u);
                        wop[s][d] = __builtin_amdgcn_perm(wr[e1 >> 1], wr[e0 >> 1], sel);
                    }
                }
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
#pragma unroll
                for (int f = 0; f < (R == 3 && ST == 2 && !middle ? 2 : 1); ++f) {
                    const unsigned char *p = mine + pb[j] + (RS ? 0 : r * a.row_bytes) + f * a.t8 * 8;
                    const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4)(p));
                    const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4)(p + 4 * a.plane));
                    const bf16x8v px = __builtin_bit_cast(bf16x8v, short8v{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
#pragma unroll
                    for (int s = 0; s < R; ++s) {
                        if (R == 3 && ST == 2 && (s == 1) != (f == 0)) continue;
                        if (middle && s != 1) continue;
                        const int set = R == 1 ? 0 : ST == 1 ? s : s == 0 ? 0 : 1;
                        acc[set][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(px, __builtin_bit_cast(bf16x8v, wop[s]), acc[set][j], 0, 0, 0);
                    }
                }
            }
        };
        typedef std::false_type all_taps;
        if constexpr (R == 1) {
            filter_row(std::integral_constant<int, 0>{}, all_taps{});
        } else if (DUAL && centre) {
            if (!RS || r0 == 1) filter_row(std::integral_constant<int, 1>{}, std::true_type{});
        } else if constexpr (RS) {
            if (r0 == 0) filter_row(std::integral_constant<int, 0>{}, all_taps{});
            else if (r0 == 1) filter_row(std::integral_constant<int, 1>{}, all_taps{});
            else filter_row(std::integral_constant<int, 2>{}, all_taps{});
        } else {
            filter_row(std::integral_constant<int, 0>{}, all_taps{});
            filter_row(std::integral_constant<int, 1>{}, all_taps{});
            filter_row(std::integral_constant<int, 2>{}, all_taps{});
        }
        wave_fence();
    }

    // ---- the column taps' sums meet: pixel p takes D0[p - 1] + D1[p] + D2[p + 1] (a lane holds four adjacent
    // pixels, group 4 j + quad, of one channel) --------------------------------------------------
    __syncthreads();
    float *part = reinterpret_cast<float *>(body) + (wave * 16 + l16) * PITCH;
    float before[NJ], after[NJ];
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        if (NS > 1) before[j] = __uint_as_float(__builtin_amdgcn_ds_bpermute(((lane + 48) & 63) * 4, __float_as_uint(acc[0][j][3])));
        if (NS > 2) after[j] = __uint_as_float(__builtin_amdgcn_ds_bpermute(((lane + 16) & 63) * 4, __float_as_uint(acc[NS - 1][j][0])));
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
        float4v o = acc[MID][j];
        int cg = 0;
        if constexpr (NS > 1) {
            divide(4 * j + quad, a.by_groups, &cg);
            const float b = quad > 0 ? before[j] : j > 0 ? before[j > 0 ? j - 1 : 0] : 0.0f;
            o[0] += cg > 0 ? b : 0.0f;
#pragma unroll
            for (int q = 1; q < 4; ++q) o[q] += acc[0][j][q - 1];
        }
        if constexpr (NS > 2) {
            const float f = quad < 3 ? after[j] : j + 1 < NJ ? after[j + 1 < NJ ? j + 1 : j] : 0.0f;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float v = q < 3 ? acc[NS - 1][j][q < 3 ? q + 1 : 3] : f;
                o[q] += 4 * cg + q + 1 < a.OW ? v : 0.0f;
            }
        }
        *reinterpret_cast<float4v *>(part + 16 * j + 4 * quad) = o;
    }
    __syncthreads();

    // ---- sum over the waves, tail, stores: four pixels of one channel per item.  Plain ones under the store hint too, as
    // all 8-byte stores are: with it eleven layers of a network take 48.8 us against 47.1 at batch 1, 69.1 against 68.3 at 4.
    const float *sum = reinterpret_cast<const float *>(body);
    const float floor_v = relu_floor((head2 ? a.relu2 : a.relu) & 1);
    bf16_t *y = head2 ? a.y2 : a.y;
    const bf16_t *residual = head2 ? nullptr : a.residual;
    const int k0 = head2 ? a.k1 : 0, kn = head2 ? a.OC - a.k1 : a.k1;           // (k1 = OC without a second head)
    for (int item = tid; item < 16 * QT; item += nwaves * 64) {
        const int ocl = item / QT, q = item % QT;
        int cg, oh;
        const int row = divide(q, a.by_groups, &cg);
        const int col = col0 + 4 * cg;
        int n = n0;
        oh = oh0 + row;
        if (a.images > 1) n = divide(row0 + row, a.by_oh, &oh);
        if (row >= a.tr || n >= a.N || oh >= a.OH || m0 + ocl >= a.OC || col >= a.OW) continue;
        const int idx = __umul24(__umul24(n, kn) + m0 + ocl - k0, a.OH * a.OW) + __umul24(oh, a.OW) + col;
        float4v o = *reinterpret_cast<const float4v *>(sum + ocl * PITCH + 4 * q);
        for (int w = 1; w < nwaves; ++w) o += *reinterpret_cast<const float4v *>(sum + (w * 16 + ocl) * PITCH + 4 * q);
        const float sc = ss[2 * ocl], sf = ss[2 * ocl + 1];
        float f[4], r[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (a.vec) {
            if (residual) Group4<bf16_t>::unpack(*reinterpret_cast<const uint2v *>(residual + idx), r);
#pragma unroll
            for (int e = 0; e < 4; ++e) f[e] = fmaxf(fmaf(o[e], sc, sf) + r[e], floor_v);
            *reinterpret_cast<uint2v *>(y + idx) = Group4<bf16_t>::pack(f);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (col + e < a.OW) {
                    const float rr = residual ? bf16_to_f32(residual[idx + e]) : 0.0f;
                    y[idx + e] = f32_to_bf16(fmaxf(fmaf(o[e], sc, sf) + rr, floor_v));
                }
        }
    }
}

// Geometry of a launch for NJ blocks of 16 pixel slots and at most most_rows output rows; false where a tile does
// not fit.
bool set_geometry(const ConvProblem &p, int nj, bool rs, RowsPlan *g, int most_rows = 64)
{
    // a 1x1 layer without a stride has no rows: an image is one row, tiled across (rows of 4n pixels)
    const bool flat = p.R == 1 && p.sh == 1 && (p.H * p.W) % 4 == 0;
    const int OH = flat ? 1 : p.OH, OW = flat ? p.H * p.W : p.OW, W = flat ? p.H * p.W : p.W;
    g->flat = flat;
    g->nj = nj;
    const int slots = 4 * nj, all = (OW + 3) / 4;
    if (flat) {
        g->groups = slots;
        g->cblocks = (all + slots - 1) / slots;
        g->tr = 1;
        g->t8 = slots / 2;
    } else {
        if (all > slots) return false;
        g->groups = all;
        g->cblocks = 1;
        g->tr = std::min({slots / all, p.N * OH, most_rows});
        g->t8 = (W + 7) / 8;
    }
    const int vs = p.R == 1 ? 1 : p.sh, halo = p.R == 1 ? 0 : 3 - p.sh;       // staged rows per output row, more per image
    g->vh = (OH - 1) * vs + (p.R == 1 ? 1 : 3);
    g->images = p.N == 1 || OH % g->tr == 0 ? 1 : g->tr % OH == 0 ? g->tr / OH : (g->tr + OH - 2) / OH + 1;
    g->rs = rs;
    g->rows = g->tr * vs + halo * g->images - (g->rs ? 2 : 0);
    g->pt = (kChunk * g->rows * g->t8 + 63) / 64;
    // (the instances that hold more loads run out of registers)
    if (g->pt > 12 - 4 * (int)rs - 4 * (int)(nj == 4 && W % 2 != 0) || (nj == 4 && p.R == 3 && p.sh == 2)) return false;
    const int row_bytes = g->t8 * 16;
    g->plane = (g->rows * row_bytes + 31) / 64 * 64 + 32;                      // an odd number of 32 bytes: distinct banks
    g->region = std::max(p.R == 3 ? 16 * kWeightRow : 0, kChunk * g->plane + 4 * kOctetGap);
    g->nw = std::min(kMaxWaves, p.IC / kChunk) * (g->rs ? 3 : 1);
    g->lds_bytes = 16 * 8 + (size_t)g->nw * std::max(g->region, 16 * (16 * nj + 4) * 4);
    if (g->lds_bytes > 160 * 1024) return false;
    g->ptiles = (long)((p.N * OH + g->tr - 1) / g->tr) * g->cblocks;
    g->tiles = g->ptiles * ((p.OC + 15) / 16);
    return true;
}

template <int R, int ST, bool UNAL, int NJ, int PT, bool RS, bool DUAL, bool CENTRE = false>
tvg_status launch(const RowsArgs &args, const RowsPlan &plan, hipStream_t stream)
{
    const auto kernel = conv_rows_kernel<R, ST, UNAL, NJ, PT, RS, DUAL, CENTRE>;
    static bool configured = false;                // opt in to > 64 KB of dynamic LDS once per instance
    if (!configured && plan.lds_bytes > 64 * 1024) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
            return TVG_ERR_LAUNCH;
        configured = true;
    }
    kernel<<<dim3((unsigned)plan.tiles), dim3(64 * plan.nw), plan.lds_bytes, stream>>>(args);
    return hipGetLastError() == hipSuccess ? TVG_OK : TVG_ERR_LAUNCH;
}

template <int R, int ST, bool UNAL, int NJ, int PT>
tvg_status launch_rs(const RowsArgs &args, const RowsPlan &plan, hipStream_t stream)
{
    if constexpr (R == 3) {
        const bool dual = args.k1 < args.OC;
        if (plan.rs) {
            if constexpr (PT <= 8 && !(PT == 8 && UNAL && NJ == 4)) {
                if constexpr (ST == 2)
                    if (dual) return launch<R, ST, UNAL, NJ, PT, true, true>(args, plan, stream);
                return launch<R, ST, UNAL, NJ, PT, true, false>(args, plan, stream);
            }
            return TVG_ERR_UNSUPPORTED;
        }
        if constexpr (ST == 2)
            if (dual) return launch<R, ST, UNAL, NJ, PT, false, true>(args, plan, stream);
    }
    return launch<R, ST, UNAL, NJ, PT, false, false>(args, plan, stream);
}

template <int R, int ST, bool UNAL, int NJ>
tvg_status launch_pt(const RowsArgs &args, const RowsPlan &plan, hipStream_t stream)
{
    if (plan.pt <= 4) return launch_rs<R, ST, UNAL, NJ, 4>(args, plan, stream);
    if (plan.pt <= 8) return launch_rs<R, ST, UNAL, NJ, 8>(args, plan, stream);
    if constexpr (UNAL && NJ == 4) return TVG_ERR_UNSUPPORTED;
    else return launch_rs<R, ST, UNAL, NJ, 12>(args, plan, stream);
}

template <int R, int ST, bool UNAL>
tvg_status launch_nj(const RowsArgs &args, const RowsPlan &plan, hipStream_t stream)
{
    if (plan.nj == 1) return launch_pt<R, ST, UNAL, 1>(args, plan, stream);
    if (plan.nj == 2) return launch_pt<R, ST, UNAL, 2>(args, plan, stream);
    if constexpr (R == 3 && ST == 2) return TVG_ERR_UNSUPPORTED;
    else return launch_pt<R, ST, UNAL, 4>(args, plan, stream);
}

}  // namespace

bool plan_conv_rows(const ConvProblem &p, RowsPlan *plan)
{
    if (p.dtype != TVG_BF16 || p.R != p.S || (p.R != 1 && p.R != 3)) return false;
    if (p.ph != p.R / 2 || p.pw != p.R / 2 || p.sh != p.sw || p.sh > 2 || p.IC % kChunk != 0) return false;
    if ((int64_t)p.N * p.IC * p.H * p.W >= (1 << 30) || (int64_t)p.OC * p.IC * p.R * p.R >= (1 << 30)) return false;
    if ((int64_t)p.N * p.IC >= (1 << 22) || (int64_t)p.OC * p.IC >= (1 << 22) || (int64_t)p.N * (p.H + 2) >= (1 << 22) ||
        (int64_t)p.H * p.W >= (1 << 22) || p.npix >= (1 << 22))
        return false;                                          // 24-bit products
    const Knobs k = forced_knobs(p);
    if (k.mt || k.nt || k.stages || k.split_k || k.lds_pitch || k.row_loads) return false;
    const int nch = p.IC / kChunk;
    // What fits one round: at most 2048 waves, eight per CU, in the narrowest tile that keeps to it.  Beyond it the other
    // kernels' larger tiles win (256 -> 256 14x14: 13.8 us there against 13.1 at batch 6 and 2688 waves; 128 -> 128
    // 28x28 at batch 16, 7168 waves, 12.3 against 19.7), except where those have few tiles and a long chain: 3x3, deep
    // and strided layers up to 3584 waves (512 -> 512 7x7, batch 16, 20.5 against 16.7; 256 -> 512 s2, batch 8, 19.6 against
    // 12.6), deep 1x1 layers without a stride up to 4096 (512 -> 512 14x14, batch 4, 7.9 against 6.4; 8192 waves 8.0 against
    // 9.6).
    // 1x1 without a stride: reductions of 1, 2 and 4 chunks are whole in flight in the other kernel (64 -> 128 56x56 at
    // batch 1 3.1 us against 3.6).  With one they are too, and only narrow tiles gain on it, at one chunk the narrowest
    // (32 -> 192, 29 images 31x19, 64 pixels, 3.4 there and 6.3 here; 128 -> 192, 6 images 20x51, 4.4 and 5.5, 2 images 18x18,
    // 16 pixels, 4.7 and 3.4).
    // 3x3, up to three chunks: workgroups of a few waves, which wide tiles keep busy.  One chunk, in filter rows or, in
    // the narrowest tile, whole (32 -> 256, 17 images 44x11, stride 2, whole in 32-pixel tiles, 6.7 us there and 9.1
    // here): 32 pixels up to two workgroups per CU, 64 one (32 -> 192, 7 images 10x10, 420 workgroups of 32, 5.5 and 4.5, 32 ->
    // 48, 34 images 12x11, 612, 5.4 and 6.4; 32 -> 289, 10 images 12x12, 456 of 64, 5.6 and 6.3).  Two, in filter rows: one per CU,
    // each 57 KB of LDS (64 -> 128, 8 images 17x17, stride 2, 288 workgroups, 9.3 and 12.3), and none whole at stride 1
    // (7.3, 7.4).  Three: two per CU of 64 pixels, or 32 under a stride (96 -> 500, 2 images 31x31, 512 workgroups, 11.1 and
    // 8.3, 96 -> 192, 20 images 35x7, 540, 9.9 and 12.3).
    const auto most_waves = [&](int nj, bool rs) {
        if (p.R == 1 && p.sh == 2) return nch <= 4 && nj > (nch == 1 ? 1 : 2) ? 0 : 2048;
        if (p.R == 1) {
            if (nch == 3 && nj == 4) return 1200;              // (96 -> 96, 9 images 26x26, 1782 waves, 4.4 and 4.7)
            // (maps of an odd number of pixels are tiled by rows: 96 -> 160, 5 images 19x19, 4.7 us there against 5.7)
            if (p.H * p.W % 4 != 0 && nch < 16) return 512;
            return nch < 16 ? 2048 : 4096;
        }
        if (nch == 1) return nj == 1 ? (rs || p.sh == 2 ? 2048 : 0) : !rs ? 0 : 3 * kComputeUnits * (nj == 2 ? 2 : 1);
        if (nch == 2) return rs ? 6 * kComputeUnits : p.sh == 1 ? 0 : 2048;
        if (nch == 3 && nj * p.sh >= 4) return 3 * kComputeUnits * 2;
        return nch >= 16 || (nch >= 8 && p.sh == 2) ? 3584 : 2048;
    };
    if (p.R == 1 && p.sh == 1 && (nch == 1 || nch == 2 || nch == 4)) return false;
    for (int round : {2048, 4096})
        for (int rs = p.R == 3 && nch <= 2 ? 1 : 0; rs >= 0; --rs)
            for (int nj : {1, 2, 4})
                if (set_geometry(p, nj, rs != 0, plan) && plan->tiles * plan->nw <= std::min(round, most_waves(nj, rs != 0))) return true;
    return false;
}

bool plan_conv_rows_dual(const ConvProblem &p, const RowsPlan &head1, const RowsPlan &head2, bool centre, RowsPlan *plan)
{
    // (two heads in one launch are built for stride 2; the same split of the sums has the same bits)
    if (p.sh != 2 || (!centre && head1.rs != head2.rs)) return false;
    return set_geometry(p, head1.nj, head1.rs != 0, plan);
}

bool plan_conv_rows_centre(const ConvProblem &p, RowsPlan *plan)
{
    // One instance per stride and row alignment: the widest tile, of as many rows as its loads hold (one always is).
    for (int rows = 16; rows >= 1; --rows)
        if (set_geometry(p, 4, false, plan, rows) && plan->pt <= 4 * p.sh) return true;
    return false;
}

bool conv_rows_pointers_ok(const ConvPointers &ptr)
{
    return reinterpret_cast<uintptr_t>(ptr.x) % 16 == 0 && reinterpret_cast<uintptr_t>(ptr.w) % 16 == 0 &&
           reinterpret_cast<uintptr_t>(ptr.y) % 2 == 0 && reinterpret_cast<uintptr_t>(ptr.residual) % 2 == 0;
}

tvg_status launch_conv_rows(const ConvProblem &p, const RowsPlan &plan, const ConvPointers &ptr, hipStream_t stream,
                            const DualHead *dual, bool centre)
{
    RowsArgs a{};
    a.x = static_cast<const bf16_t *>(ptr.x);
    a.w = static_cast<const bf16_t *>(ptr.w);
    a.scale = ptr.scale; a.shift = ptr.shift; a.bias = ptr.bias;
    a.residual = static_cast<const bf16_t *>(ptr.residual);
    a.y = static_cast<bf16_t *>(ptr.y);
    a.N = p.N; a.IC = p.IC; a.OC = p.OC;
    a.H = plan.flat ? 1 : p.H;
    a.W = plan.flat ? p.H * p.W : p.W;
    a.OH = plan.flat ? 1 : p.OH;
    a.OW = plan.flat ? p.H * p.W : p.OW;
    a.relu = p.relu;
    a.k1 = dual ? dual->oc1 : p.OC;
    a.y2 = dual ? static_cast<bf16_t *>(dual->y2) : nullptr;
    a.relu2 = dual ? dual->relu2 : 0;
    a.centre2 = dual ? dual->centre2 : 0;
    a.vec = a.OW % 4 == 0 && (reinterpret_cast<uintptr_t>(ptr.y) | reinterpret_cast<uintptr_t>(ptr.residual) |
                              reinterpret_cast<uintptr_t>(a.y2)) % 8 == 0;
    a.tr = plan.tr; a.groups = plan.groups; a.cblocks = plan.cblocks; a.t8 = plan.t8;
    a.vh = plan.vh; a.rows = plan.rows; a.images = plan.images;
    a.dg = 64 % plan.t8;
    a.drow = 64 / plan.t8 % plan.rows;
    a.dch = 64 / plan.t8 / plan.rows;
    a.row_bytes = plan.t8 * 16; a.plane = plan.plane; a.region = plan.region;
    a.ptiles = (int)plan.ptiles;
    a.nch = p.IC / kChunk;
    a.x_bytes = ((uint32_t)((int64_t)p.N * p.IC * p.H * p.W) * 2 + 3) & ~3u;   // (up to the end of the last pixel's word)
    a.w_bytes = (uint32_t)(p.OC * p.IC * (centre ? 9 : p.R * p.S)) * 2;
    a.by_ptiles = make_divider(a.ptiles); a.by_oh = make_divider(a.OH); a.by_vh = make_divider(a.vh);
    a.by_t8 = make_divider(a.t8); a.by_rows = make_divider(a.rows); a.by_groups = make_divider(a.groups);
    a.by_cblocks = make_divider(a.cblocks);
    const bool odd = a.W % 2 != 0;
    if (centre) {
        if (p.sh == 1) return odd ? launch<1, 1, true, 4, 4, false, false, true>(a, plan, stream) : launch<1, 1, false, 4, 4, false, false, true>(a, plan, stream);
        return odd ? launch<1, 2, true, 4, 8, false, false, true>(a, plan, stream) : launch<1, 2, false, 4, 8, false, false, true>(a, plan, stream);
    }
    if (p.R == 1) {
        if (p.sh == 1) return odd ? launch_nj<1, 1, true>(a, plan, stream) : launch_nj<1, 1, false>(a, plan, stream);
        return odd ? launch_nj<1, 2, true>(a, plan, stream) : launch_nj<1, 2, false>(a, plan, stream);
    }
    if (p.sh == 1) return odd ? launch_nj<3, 1, true>(a, plan, stream) : launch_nj<3, 1, false>(a, plan, stream);
    return odd ? launch_nj<3, 2, true>(a, plan, stream) : launch_nj<3, 2, false>(a, plan, stream);
}

}  // namespace tvg
