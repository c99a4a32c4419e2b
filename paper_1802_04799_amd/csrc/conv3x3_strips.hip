// bf16 3x3 convolutions (pad 1, stride 1 or 2) at throughput size.
//
// Bound: no single unit.  At batch 64 the matrix pipes are busy 37 to 40 % of the time without a stride (128 -> 128 at 28x28, 256 ->
// 256 at 14x14, 512 -> 512 at 7x7, at about 1.9 GHz) and 20 to 23 % under one, the LDS 13 to 22 %; the rest is the in-order stream of one or two
// waves on a SIMD: a tile's set-up and tail around a loop of 2 to 16 chunks.  The 64 x 256 tiles of the pipelined kernel
// read 1 KB of LDS per 32x32x16 MFMA, as much as the LDS delivers, and spend a third of their loop on making channel words
// of NCHW rows.  Here:
//   - A wave owns 16 output channels of four strips of B rows x 8 pixels (4 to 8 rows).  Strip and column pair are the pixel
//     rows of an MFMA, so the operand of a strip's input row serves three output rows, and the chunk's weights of all nine
//     taps stay in registers: 0.2 KB of LDS per 16x16x32 MFMA instead of 0.5.
//   - Input rows lie in LDS as in memory but for even and odd columns being apart; gfx950's transposing read makes operands
//     of them.  A column tap that would shift the operand by a pixel multiplies it unshifted into sums of its own (se, so),
//     and the shift is made once, on the sums: even column i = ae[i] + se[i - 1], odd column i = ao[i] + so[i + 1].
//     (Three columns of sums, as without the halves, would be 168 registers instead of 112 at seven rows.)
//   - A wave's weights are its own: 16-byte pieces straight from memory into LDS, read back as a lane's 144-byte run of
//     eight channels and transposed by byte permutes.  Only the rows are shared and need barriers.
//   - Each access is placed between MFMAs (nine weight pieces and five row loads in a burst stop a wave for 0.3 us), nothing
//     but barriers waits for other waves, both barriers are amid MFMAs, and a workgroup goes on to its next tile without one.
//   - What a tile's set-up and tail need is read anew there (kernel arguments, lane numbers), not kept through the loop.
// Rows of an odd number of pixels take funnel shifts to lay down, and with few tiles two groups of waves split the reduction.
// With fewer still four groups of two waves do, on 32 output channels: twice the workgroups, a quarter of the chain of chunks.
// Rows of more than 32 pixels are cut into windows of four strips that overlap by one.
// Under a stride the two halves are what a filter's columns take anyway: two sums (ae, se), each pixel of them fed by every
// other row, so that an operand serves half as many MFMAs: 0.76 KB of LDS per MFMA, and 7 to 10 instructions instead of 4 to 6.
// us, warm, in the kernels behind and here, without and with a residual: 128 -> 128 at 28x28, batch 32 15.1 / 16.7 -> 13.9 /
// 13.7, batch 128 39.6 / 44.4 -> 34.6 / 35.9 (850 TFLOP/s without); 256 -> 256 at 14x14, batch 128 37.4 / 41.7 -> 34.9 / 35.6; 512 ->
// 512 at 7x7, batch 128 38.1 / 55.9 -> 37.0 / 38.6; 192 -> 192 at 56x56, batch 16 53.2 / 55.7 -> 37.0 / 39.8; stride 2, 256 -> 512 at
// 14x14, batch 128 36.1 / 44.5 -> 30.7 / 32.7, 512 -> 512 at 28x28, batch 16 36.1 / 38.1 -> 28.3 / 28.6.  Four groups (behind,
// one group, two, with buffers in turn -> four): 256 -> 256 at 14x14, batch 16 13.4, 13.9 -> 11.7; 512 -> 512 at 14x14, batch 8 23.7, 22.6 ->
// 15.7, at 7x7, batch 32 20.8, 25.2, 21.1 -> 18.0.
#include <algorithm>
#include <type_traits>

#include "tvg_device.h"
#include "tvg_internal.h"

namespace tvg {

namespace {

constexpr int kRsrcFlags = 0x00020000;
constexpr uint32_t kOutOfRange = 0x80000000u;      // and everything above: tensors stay below 2 GiB
constexpr int kChunk = 32;                         // input channels per step: the depth of one MFMA
constexpr int kWeightBytes = 16 * kChunk * 9 * 2;  // a wave's weights of a chunk
constexpr int kOctetGap = 128;                     // between channel octets of the staged rows: distinct banks

typedef short short4v __attribute__((ext_vector_type(4)));
typedef short short8v __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) short4v *lds_short4;
// (pieces of rows of an odd number of pixels start at any element)
typedef uint32_t uint4e __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t uint2e __attribute__((ext_vector_type(2), aligned(2)));
typedef uint32_t uint1e __attribute__((aligned(2)));

struct StripsArgs {
    const bf16_t *x, *w;
    const float *scale, *shift, *bias;
    const bf16_t *residual;
    bf16_t *y;
    int N, IC, H, W, OC, OH, OW, relu, nt;
    int t8, spi, sr, rows;             // strips per row, strip rows per image and per tile, staged rows per tile
    int windows;                       // parts of a row (strip rows of their own) where it has more than four strips
    int dg, drow, dch;                 // 256 load tasks further: pieces, rows, channels
    int row_bytes, strip_bytes, half, plane;       // LDS: a staged row's even columns, a strip row, the odd columns, a channel
    int rows_bytes;                    // the staged rows of a group and stage
    int ptiles, nch;
    uint32_t dump;                     // LDS: 256 bytes that nothing reads
    int pixels_first;                  // order of tiles: the pixel tiles of a channel tile follow each other, or the reverse
    int tiles_per, tiles_more;         // tiles per workgroup, workgroups with one more
    uint32_t x_bytes, w_bytes, y_bytes;
    Divider by_inner, by_spi, by_t8, by_rows, by_windows;
};

// 16 bytes per lane from a buffer straight into LDS at `lds` + 16 lane.  In assembly because the compiler waits for all
// loads in flight before any LDS read that follows its own form; whoever reads the bytes waits with wait_loads.  (M0 is an
// output, so that the compiler knows that it has changed.)  An SGPR that a vector instruction wrote has to be five wait states
// old when a memory instruction reads it, and the compiler keeps no distance to what is inside.  FAR keeps it: for instances
// that keep SGPRs in lanes of vector registers and read them back where they are wanted.  The others' operands come from scalar
// instructions, which a test reads from the machine code, and five wait states are longer than an MFMA hides: 32 images
// 128 -> 128 at 28x28 14.2 us instead of 13.9, ResNet-18 body at batch 32 313.8 us instead of 307.3.
template <bool FAR> __device__ __forceinline__ void load_to_lds(uint32_t lds, uint32_t offset, const uint4v &rsrc, uint32_t uniform_offset)
{
    uint32_t m0;
    asm volatile("s_mov_b32 m0, %1\n\ts_nop %5\n\tbuffer_load_dwordx4 %2, %3, %4 offen lds"
                 : "={m0}"(m0) : "s"(lds), "v"(offset), "s"(rsrc), "s"(uniform_offset), "n"(FAR ? 3 : 0) : "memory");
}

// The kernel's arguments read anew, and a value that looks new: what a tile's set-up and tail derive from them would
// otherwise be kept in registers through the tile's loop, which has none to spare.
typedef const __attribute__((address_space(4))) StripsArgs *ArgsPtr;
__device__ __forceinline__ ArgsPtr fresh_args()
{
    ArgsPtr p = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
}
__device__ __forceinline__ int fresh(int v)
{
    asm volatile("" : "+v"(v));
    return v;
}
__device__ __forceinline__ int fresh_uniform(int v)
{
    asm volatile("" : "+s"(v));
    return v;
}
__device__ __forceinline__ int divide(int n, const __attribute__((address_space(4))) Divider &v, int *rem)
{
    const Divider d{v.d, v.m, v.s};
    return divide(n, d, rem);
}

// until at most N younger memory operations are in flight
template <int N> __device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" :: "n"(N) : "memory"); }

// Windows of a row of more than four strips: four strips each, which overlap by one, since the sums of a window's first
// column (and without a stride those of its last) miss the column beside it.
constexpr int kWindowStep = 24;                    // columns of the input

// The channel tile of a tile, and in *pt its pixel tile.
template <class A> __device__ __forceinline__ int split_tile(A &a, int t, int *pt)
{
    int inner;
    const int outer = divide(t, a.by_inner, &inner);
    *pt = a.pixels_first ? inner : outer;
    return a.pixels_first ? outer : inner;
}

// Whether a workgroup may go on to further tiles.  Not with odd rows: store_row takes the parity of a row's start from goff,
// which next_rows has overwritten for the next tile by then.  Nor where groups split the reduction: what they exchange lies over
// the weights and rows of the next step.  Planning gives these a workgroup per tile, and launch refuses anything else.
constexpr bool walks_tiles(bool odd_rows, int groups) { return !odd_rows && groups == 1; }

// WM waves along the output channels, 16 each, in each of KG groups that split the reduction.
// ANY: output rows start at any element, by their length or by the addresses of y and the residual.  (An instance of its own: a
// branch for it makes the others' code a fifth longer, which costs 0.1 to 0.4 us where it is fetched anew between layers.)
template <int B, int ST, bool UNAL, int KG, int WM, bool ANY>
__global__ __launch_bounds__(64 * WM * KG, 2) void conv3x3_strips_kernel(const StripsArgs a)
{
    constexpr int kIn = ST == 1 ? B + 2 : 2 * B + 1;      // input rows of a strip
    constexpr int kWaves = WM;
    constexpr int PT = (2 * kIn + WM - 1) / WM;           // load tasks per thread: 32 channels of as many rows of 4 strips
    constexpr int kStages = ST == 1 && KG <= 2 ? 2 : 1;   // of staged rows
    constexpr int BO = ST == 1 ? B : 1;                   // (sums of odd columns: without a stride)
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, quad = lane >> 4;
    const int kg = wave / kWaves, wave_m = wave % kWaves;
    const int HW = a.H * a.W;
    // this workgroup's tiles: adjacent ones, so that they share weights and rows in the L2 of their XCD, whose first
    // workgroups (one to a CU before any CU has two) take one more each
    int tile, tiles;
    {
        const int xcd = blockIdx.x & 7, local = blockIdx.x >> 3, q = gridDim.x >> 3, more = a.tiles_more >> 3;
        const int before = xcd * q + min(xcd, (int)(gridDim.x & 7)), longer = more + (xcd < (a.tiles_more & 7) ? 1 : 0);
        tile = (before + local) * a.tiles_per + xcd * more + min(xcd, a.tiles_more & 7) + min(local, longer);
        tiles = a.tiles_per + (local < longer ? 1 : 0);
    }

    const int weights_at = wave * kWeightBytes;
    unsigned char *weights = smem + weights_at;
    unsigned char *staged = smem + KG * kWaves * kWeightBytes + kg * kStages * a.rows_bytes;
    int to_other = kStages == 2 ? a.rows_bytes : 0;       // (from the stage read to the one written)

    // ---- weights: 36 pieces of 16 bytes per output channel and chunk, four lanes on adjacent pieces; a piece's place
    // among its four changes with the channel (distinct banks for the reads below).  Channels past the last: zeros.
    const uint32_t lds_weights = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)weights;
    uint32_t woff;
    auto load_weights = [&](int k, uint32_t bytes, int c) __attribute__((always_inline)) {
        load_to_lds<UNAL>(lds_weights + 1024 * k, woff, raw_buffer(a.w, bytes), c * (2 * kChunk * 9) + 64 * k);
    };
    // a lane's run: channels 8 quad .. + 7 of output channel l16, pieces 9 quad .. + 8
    int wrun[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int t = quad + j;
        wrun[j] = weights_at + (2 * quad + (t >> 2)) * 1024 + l16 * 64 + (((t & 3) ^ ((l16 >> 1) & 3)) << 4);
    }

    // ---- input load tasks: eight pixels of a staged row of one channel
    uint32_t goff[PT];
    int dst[PT];
    auto set_weights = [&](int t) __attribute__((always_inline)) {
        const auto &a = *fresh_args();
        const int lane = fresh(tid & 63), wm = fresh_uniform(wave_m);
        int pt;
        const int cb = split_tile(a, t, &pt);
        woff = __umul24(__umul24((cb * kWaves + wm) * 16 + (lane >> 2), a.IC), 18u) + (((lane & 3) ^ ((lane >> 3) & 3)) << 4);
    };
    // offsets of a tile's tasks (and, the first time, their places in LDS)
    auto set_tile = [&](int t, bool first) __attribute__((always_inline)) {
        const auto &a = *fresh_args();
        const int id = fresh(tid & (64 * kWaves - 1)), HW = a.H * a.W;
        int pt, g8, row;
        split_tile(a, t, &pt);
        int ch = divide(id, a.by_t8, &g8);
        ch = divide(ch, a.by_rows, &row);
#pragma unroll
        for (int k = 0; k < PT; ++k) {
            int rb, window;
            ch &= kChunk - 1;                                    // tasks beyond the last repeat the first ones
            const int s = row / kIn, rho = row - s * kIn;
            const int n = divide(pt * a.sr + s, a.by_spi, &rb);
            rb = divide(rb, a.by_windows, &window);
            const int ih = rb * B * ST + rho - 1;
            goff[k] = kOutOfRange;
            if (ih >= 0 && ih < a.H && n < a.N)
                goff[k] = 2u * (__umul24(__umul24(n, a.IC) + ch, HW) + __umul24(ih, a.W) + window * kWindowStep + g8 * 8);
            if (first) {
                dst[k] = __umul24(ch, a.plane) + (ch >> 3) * kOctetGap + __umul24(s, a.strip_bytes) + __umul24(rho, a.row_bytes) + g8 * 8;
                if constexpr (UNAL) dst[k] = dst[k] * 16 + g8;     // (t8 <= 16)
            }
            g8 += a.dg;
            row += a.drow;
            ch += a.dch;
            if (g8 >= a.t8) { g8 -= a.t8; ++row; }
            if (row >= a.rows) { row -= a.rows; ++ch; }
        }
    };
    uint32_t raw[PT][UNAL ? 5 : 4];
    auto load_row = [&](int k, const __amdgpu_buffer_rsrc_t &rsrc, int c) __attribute__((always_inline)) {
        const uint32_t at = UNAL ? goff[k] & ~3u : goff[k];
        const uint4v v = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(rsrc, at, c * 2 * kChunk * HW, 0));
#pragma unroll
        for (int d = 0; d < 4; ++d) raw[k][d] = v[d];
        if constexpr (UNAL) raw[k][4] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, at + 16, c * 2 * kChunk * HW, 0);
    };
    auto store_row = [&](int k, unsigned char *to) __attribute__((always_inline)) {
        uint32_t v[4];
#pragma unroll
        for (int d = 0; d < 4; ++d) v[d] = raw[k][d];
        int at = dst[k];
        if constexpr (UNAL) {
            const int last = (a.W - 8 * (at & 15)) >> 1;                          // the column right of an odd row is padding
            at >>= 4;
#pragma unroll
            for (int d = 0; d < 4; ++d) {
                v[d] = __builtin_amdgcn_alignbit(raw[k][d + 1], raw[k][d], (goff[k] & 2) * 8);
                v[d] = d == last ? v[d] & 0xFFFFu : v[d];
            }
        }
        *reinterpret_cast<uint2v *>(to + at) =
            uint2v{__builtin_amdgcn_perm(v[1], v[0], 0x05040100u), __builtin_amdgcn_perm(v[3], v[2], 0x05040100u)};
        *reinterpret_cast<uint2v *>(to + at + a.half) =
            uint2v{__builtin_amdgcn_perm(v[1], v[0], 0x07060302u), __builtin_amdgcn_perm(v[3], v[2], 0x07060302u)};
    };

    // ---- pixel operand address: lane = (channel octet of the chunk, channel, strip), four columns of one parity
    int px;
    {
        int g8;
        int s = divide(lane & 3, a.by_t8, &g8);
        if (s >= a.sr) s = 0, g8 = 0;
        px = (8 * quad + ((lane >> 2) & 3)) * a.plane + quad * kOctetGap + s * a.strip_bytes + g8 * 8;
    }

    // Steps: chunk after chunk, tile after tile.  A step's weights are requested in the first rows of the step before, its
    // rows in the last rows of the step but one before; they are laid down in LDS, one by one as the requests of the step
    // after take their registers, in the last rows of the step before.  The two barriers around that are the only points
    // where waves wait for each other, and both are amid MFMAs: what a wave does between two steps and at a tile's end
    // the other wave of its SIMD covers.  Requests beyond the last step go to a buffer of no bytes.
    const int end = tile + tiles;
    int rows_tile = tile, rows_c = kg, weights_tile = tile, weights_c = kg;        // what to request next
    auto rows_rsrc = [&]() __attribute__((always_inline)) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(a.x), 0, rows_tile < end ? a.x_bytes : 0, kRsrcFlags);
    };
    auto next_rows = [&]() __attribute__((always_inline)) {
        rows_c += KG;
        if (rows_c >= a.nch) {
            rows_c = kg;
            if (++rows_tile < end) set_tile(rows_tile, false);
        }
    };
    auto next_weights = [&]() __attribute__((always_inline)) {
        weights_c += KG;
        if (weights_c >= a.nch) {
            weights_c = kg;
            if (++weights_tile < end) set_weights(weights_tile);
        }
    };
    set_weights(tile);
#pragma unroll
    for (int k = 0; k < 9; ++k) load_weights(k, a.w_bytes, kg);
    next_weights();
    set_tile(tile, true);
#pragma unroll
    for (int k = 0; k < PT; ++k) load_row(k, rows_rsrc(), kg);
    next_rows();
    // The weights of the later steps are on their way from memory into the XCD's L2 meanwhile: its workgroups, which walk the
    // same ones, touch a share of their lines each.  (Weights that the call before has not left there cost a memory
    // latency per step otherwise: ResNet-18 body at batch 32 346 -> 327 us, at batch 128 767 -> 760.)
    if (a.nch > 2 * KG) {
        int pt;
        const int cb = split_tile(a, tile, &pt), shares = gridDim.x < 32 ? 1 : gridDim.x < 128 || !a.pixels_first ? 4 : 16;
        const uint4v rsrc = raw_buffer(a.w, a.w_bytes);
        const uint32_t first = cb * (16 * kWaves * 18) * a.IC;                 // 9 lines of 128 bytes per input channel
        for (int at = ((a.pixels_first ? blockIdx.x >> 3 : pt) & (shares - 1)) * (64 * kWaves * KG) + tid; at < 9 * a.IC * kWaves / 4; at += shares * 64 * kWaves * KG)
            touch_line(a.dump, first + 128 * at, rsrc);
    }
    wait_loads<0>();
#pragma unroll
    for (int k = 0; k < PT; ++k) store_row(k, staged);
#pragma unroll
    for (int k = 0; k < PT; ++k) load_row(k, rows_rsrc(), rows_c);
    next_rows();
    __syncthreads();

    for (; tile < end; ++tile) {
        float4v ae[B], se[B], ao[BO], so[BO];
#pragma unroll
        for (int b = 0; b < B; ++b) ae[b] = se[b] = ao[b < BO ? b : 0] = so[b < BO ? b : 0] = float4v{0.0f, 0.0f, 0.0f, 0.0f};

        float sc = 0.0f, sf = 0.0f, bias = 0.0f;
        int rem;
        for (int c = kg; c < a.nch; c += KG) {
            uint32_t wr[36];
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                const uint4v v = *reinterpret_cast<const uint4v *>(smem + wrun[k & 3] + 1024 * (k >> 2));
#pragma unroll
                for (int d = 0; d < 4; ++d) wr[4 * k + d] = v[d];
            }
            auto read = [&](const unsigned char *p) __attribute__((always_inline)) {
                const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4)(p));
                const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4)(p + 4 * a.plane));
                return __builtin_bit_cast(bf16x8v, short8v{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
            };
            const unsigned char *p = staged + px;
            bf16x8v even = read(p), odd = read(p + a.half);
            uint4v wop[9];
#pragma unroll
            for (int t = 0; t < 9; ++t)
#pragma unroll
                for (int d = 0; d < 4; ++d) {
                    const int e0 = 18 * d + t, e1 = e0 + 9;
                    const uint32_t sel = ((e0 & 1) ? 0x0302u : 0x0100u) | ((e1 & 1) ? 0x07060000u : 0x05040000u);
                    wop[t][d] = __builtin_amdgcn_perm(wr[e1 >> 1], wr[e0 >> 1], sel);
                }
            unsigned char *other = staged + to_other;
            to_other = -to_other;
            if (c + KG >= a.nch) {                       // the tile's scales and shifts, which its tail wants
                const int cb = split_tile(*fresh_args(), tile, &rem);
                const int oc = min((cb * kWaves + wave_m) * 16 + l16, a.OC - 1);
                sc = a.scale[oc];
                sf = a.shift[oc];
                if (a.bias) bias = a.bias[oc];
            }
            const auto tap = [&](int t) __attribute__((always_inline)) { return __builtin_bit_cast(bf16x8v, wop[t]); };
#pragma unroll
            for (int rho = 0; rho < kIn; ++rho) {
                const bf16x8v e = even, o = odd;
                p += a.row_bytes;
                if (rho + 1 < kIn) {
                    even = read(p);
                    odd = read(p + a.half);
                }
                // (filter row r of output row b; under a stride odd input rows are the middle rows of filters)
#pragma unroll
                for (int r = 0; r < 3; ++r) {
                    const int b = (rho - r) / ST;
                    if (rho < r || b >= B || (rho - r) % ST != 0) continue;
                    if constexpr (ST == 1) ao[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(e, tap(3 * r), ao[b], 0, 0, 0);
                    ae[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(e, tap(3 * r + 1), ae[b], 0, 0, 0);
                    if constexpr (ST == 1) so[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(e, tap(3 * r + 2), so[b], 0, 0, 0);
                }
#pragma unroll
                for (int r = 0; r < 3; ++r) {
                    const int b = (rho - r) / ST;
                    if (rho < r || b >= B || (rho - r) % ST != 0) continue;
                    se[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(o, tap(3 * r), se[b], 0, 0, 0);
                    if constexpr (ST == 1) ao[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(o, tap(3 * r + 1), ao[b], 0, 0, 0);
                    ae[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(o, tap(3 * r + 2), ae[b], 0, 0, 0);
                }
                // (from the second row on: the first one's MFMAs have the weights read in registers)
#pragma unroll
                for (int k = 0; k < 9; ++k)
                    if (rho == 1 + k * (kIn / 3) / 9) load_weights(k, weights_tile < end ? a.w_bytes : 0, weights_c);
                if (rho == kIn / 3) next_weights();
                if constexpr (kStages == 2) {
                    constexpr int kFirst = (B + 3) / 2, kRows = B + 1 - kFirst;    // the rows that lay rows down
                    if (rho == kFirst - 1) __syncthreads();
#pragma unroll
                    for (int k = 0; k < PT; ++k)
                        if (rho == kFirst + k * kRows / PT) {
                            store_row(k, other);
                            load_row(k, rows_rsrc(), rows_c);
                        }
                    if (rho == B) {
                        next_rows();
                        __syncthreads();
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (kStages == 1) {
                __syncthreads();
#pragma unroll
                for (int k = 0; k < PT; ++k) {
                    store_row(k, staged);
                    load_row(k, rows_rsrc(), rows_c);
                }
                next_rows();
                __syncthreads();
            }
            staged = other;
            wait_loads<PT * (UNAL ? 2 : 1)>();             // the next step's weights are there, the rows requested after them may not be
        }

        // ---- the strip whose sums the lane holds.  (Arguments in registers first: read where they are used, each is a
        // scalar load to wait for.)
        const auto &f = *fresh_args();
        const int lane = fresh(tid & 63), l16 = lane & 15, quad = lane >> 4;
        const int wm = fresh_uniform(wave_m);
        const int OH = f.OH, OW = f.OW, OC = f.OC, sr = f.sr, windows = f.windows;
        const bf16_t *residual = f.residual;
        bf16_t *y = f.y;
        const bool nt = f.nt != 0;
        constexpr int PX = 8 / ST;                                    // output pixels of a strip's row
        int pt, my_g8, my_rb, window;
        const int cb = split_tile(f, tile, &pt);
        const int my_s = divide(quad, f.by_t8, &my_g8);
        const int my_n = divide(pt * sr + my_s, f.by_spi, &my_rb);
        my_rb = divide(my_rb, f.by_windows, &window);
        const int oc0 = (cb * kWaves + wm) * 16, oc = oc0 + l16, col0 = window * (kWindowStep / ST) + PX * my_g8;
        const int rest = OW - col0, row0 = my_rb * B;                 // columns from the strip's first on, first row
        // pixels [from, to) of the strip's row: windows meet inside a strip without a stride, and at its end with one
        const int from = window > 0 && my_g8 == 0 ? (ST == 1 ? 4 : PX) : 0;
        const int to = min(ST == 1 && window + 1 < windows && my_g8 == 3 ? 4 : PX, rest);
        const bool mine = my_s < sr && my_n < f.N && oc < OC && from < to;
        // bytes of the strip's row b from the tensor's start; what is not there is out of range
        const uint32_t y_at = mine ? 2u * (uint32_t)(((my_n * OC + oc) * OH + row0) * OW + col0) : kOutOfRange;
        const auto row_at = [&](int b) __attribute__((always_inline)) { return row0 + b < OH ? y_at + 2 * b * OW : kOutOfRange; };
        const auto kept = [&](int b) __attribute__((always_inline)) { return KG == 1 || b % KG == kg; };

        uint4v res[B];
#pragma unroll
        for (int b = 0; b < B; ++b) res[b] = uint4v{0, 0, 0, 0};
        if (residual) {
            if constexpr (ANY) {
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    const uint32_t at = row_at(b);
                    if (!kept(b) || at >= kOutOfRange) continue;
                    const bf16_t *r = residual + at / 2;
                    if (to >= PX) {
                        if constexpr (ST == 1) {
                            res[b] = *reinterpret_cast<const uint4e *>(r);
                        } else {
                            const uint2v v = *reinterpret_cast<const uint2e *>(r);
                            res[b][0] = v[0];
                            res[b][1] = v[1];
                        }
                    } else {
                        if (to & 4) {
                            const uint2v v = *reinterpret_cast<const uint2e *>(r);
                            res[b][0] = v[0];
                            res[b][1] = v[1];
                        }
                        uint32_t last = 0, one = 0;
                        if (to & 2) last = *reinterpret_cast<const uint1e *>(r + (to & 4));
                        if (to & 1) one = r[to - 1];
                        // the pair after the first four or none, then the single pixel
                        const uint32_t w0 = to & 2 ? last : one, w1 = to & 2 ? one : 0u;
                        if (to & 4) { res[b][2] = w0; res[b][3] = w1; }
                        else { res[b][0] = w0; res[b][1] = w1; }
                    }
                }
            } else {
                const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(residual), 0, f.y_bytes, kRsrcFlags);
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    if (!kept(b)) continue;
                    if constexpr (ST == 1) {
                        res[b] = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(rsrc, row_at(b), 0, 0));
                    } else {
                        const uint2v v = __builtin_bit_cast(uint2v, __builtin_amdgcn_raw_buffer_load_b64(rsrc, row_at(b), 0, 0));
                        res[b][0] = v[0];
                        res[b][1] = v[1];
                    }
                }
            }
        }

        // ---- the shifted sums: even column i takes se[i - 1], odd column i so[i + 1] (with a stride, every column se[i - 1]);
        // those of the neighbouring strips are the lanes' 16 further on either side
        {
            const bool has_left = my_g8 > 0, has_right = rest > 8;
            const int from_left = ((lane + 48) & 63) * 4, from_right = ((lane + 16) & 63) * 4;
            float l[B], r[B];
#pragma unroll
            for (int b = 0; b < B; ++b) {
                l[b] = __uint_as_float(__builtin_amdgcn_ds_bpermute(from_left, __float_as_uint(se[b][3])));
                if constexpr (ST == 1) r[b] = __uint_as_float(__builtin_amdgcn_ds_bpermute(from_right, __float_as_uint(so[b][0])));
            }
#pragma unroll
            for (int b = 0; b < B; ++b) {
                ae[b][0] += has_left ? l[b] : 0.0f;
#pragma unroll
                for (int v = 1; v < 4; ++v) ae[b][v] += se[b][v - 1];
                if constexpr (ST == 1) {
#pragma unroll
                    for (int v = 0; v < 3; ++v) ao[b][v] += 2 * v + 2 < rest ? so[b][v + 1] : 0.0f;
                    ao[b][3] += has_right ? r[b] : 0.0f;
                }
            }
        }

        // ---- groups that split the reduction: group k keeps the rows b = k (mod groups) and adds all groups' sums in order
        if constexpr (KG > 1) {
            __syncthreads();
            float4v *all = reinterpret_cast<float4v *>(smem);
#pragma unroll
            for (int b = 0; b < B; ++b) {
                if (kept(b)) continue;
                all[((wave * B + b) * 2) * 64 + lane] = ae[b];
                all[((wave * B + b) * 2 + 1) * 64 + lane] = ao[b];
            }
            __syncthreads();
#pragma unroll
            for (int b = 0; b < B; ++b) {
                if (!kept(b)) continue;
                float4v e = float4v{0.0f, 0.0f, 0.0f, 0.0f}, o = e;
                for (int g = 0; g < KG; ++g) {
                    const int from = ((g * kWaves + wm) * B + b) * 2;
                    e += g == kg ? ae[b] : all[from * 64 + lane];
                    o += g == kg ? ao[b] : all[(from + 1) * 64 + lane];
                }
                ae[b] = e;
                ao[b] = o;
            }
        }

        // ---- tail: a lane holds PX adjacent pixels of row b of its strip, of channel oc
        sf = fmaf(bias, sc, sf);
        const float floor_v = relu_floor(f.relu & 1);
        auto finish = [&](int b) __attribute__((always_inline)) {
            uint4v out = {0, 0, 0, 0};
#pragma unroll
            for (int d = 0; d < PX / 2; ++d) {
                const float first = ST == 1 ? ae[b][d] : ae[b][(2 * d) & 3], second = ST == 1 ? ao[b < BO ? b : 0][d] : ae[b][(2 * d + 1) & 3];
                const float lo = fmaxf(fmaf(first, sc, sf) + __uint_as_float(res[b][d] << 16), floor_v);
                const float hi = fmaxf(fmaf(second, sc, sf) + __uint_as_float(res[b][d] & 0xFFFF0000u), floor_v);
                out[d] = f32x2_to_bf16x2(lo, hi);
            }
            return out;
        };
        if constexpr (ANY) {
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const uint32_t at = row_at(b);
                if (!kept(b) || at >= kOutOfRange) continue;
                const uint4v out = finish(b);
                bf16_t *p = y + at / 2;
                if (ST == 1 && !UNAL && from > 0) {                   // (a window's first strip: its last four)
                    *reinterpret_cast<uint2e *>(p + 4) = uint2v{out[2], out[3]};
                } else if (to >= PX) {
                    if constexpr (ST == 1) *reinterpret_cast<uint4e *>(p) = out;
                    else *reinterpret_cast<uint2e *>(p) = uint2v{out[0], out[1]};
                } else {
                    if (to & 4) *reinterpret_cast<uint2e *>(p) = uint2v{out[0], out[1]};
                    const uint32_t pair = to & 4 ? out[2] : out[0], after = to & 4 ? out[3] : out[1];
                    if (to & 2) *reinterpret_cast<uint1e *>(p + (to & 4)) = pair;
                    if (to & 1) p[to - 1] = (bf16_t)(to & 2 ? after : pair);
                }
            }
        } else {
            const __amdgpu_buffer_rsrc_t yrsrc = __builtin_amdgcn_make_buffer_rsrc(y, 0, f.y_bytes, kRsrcFlags);
            const bool halves = (OW & 4) != 0 || windows > 1;
            auto store = [&](auto hint) __attribute__((always_inline)) {
#pragma unroll
                for (int b = 0; b < B; ++b) {
                    if (!kept(b)) continue;
                    const uint4v out = finish(b);
                    const uint32_t at = row_at(b);
                    if constexpr (ST == 1) {
                        __builtin_amdgcn_raw_buffer_store_b128(out, yrsrc, to - from == 8 ? at : kOutOfRange, 0, hint);
                        // strips in part: four pixels, the first or the last, and a row's last two
                        if (halves) {
                            const bool upper = from > 0;
                            __builtin_amdgcn_raw_buffer_store_b64(uint2v{upper ? out[2] : out[0], upper ? out[3] : out[1]}, yrsrc,
                                                                  to - from < 8 && to - from >= 4 ? at + 2 * from : kOutOfRange, 0, 0);
                        }
                        if (OW & 2)
                            __builtin_amdgcn_raw_buffer_store_b32(to & 4 ? out[2] : out[0], yrsrc, to & 2 ? at + 2 * (to & 4) : kOutOfRange, 0, 0);
                    } else {
                        __builtin_amdgcn_raw_buffer_store_b64(uint2v{out[0], out[1]}, yrsrc, to == 4 ? at : kOutOfRange, 0, 0);
                        if (OW & 2) __builtin_amdgcn_raw_buffer_store_b32(out[0], yrsrc, to == 2 ? at : kOutOfRange, 0, 0);
                    }
                }
            };
            if (ST == 1 && nt) store(std::integral_constant<int, 2>{});
            else store(std::integral_constant<int, 0>{});
        }
    }
}

template <int B, int ST, bool UNAL, int KG, int WM, bool ANY>
tvg_status launch_instance(const StripsArgs &args, const StripsPlan &plan, hipStream_t stream)
{
    if (!walks_tiles(UNAL, KG) && plan.workgroups != plan.tiles) return TVG_ERR_LAUNCH;
    const auto kernel = conv3x3_strips_kernel<B, ST, UNAL, KG, WM, ANY>;
    static bool configured = false;                // opt in to > 64 KB of dynamic LDS once per instance
    if (!configured && plan.lds_bytes > 64 * 1024) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
            return TVG_ERR_LAUNCH;
        configured = true;
    }
    kernel<<<dim3((unsigned)plan.workgroups), dim3(64 * WM * KG), plan.lds_bytes, stream>>>(args);
    return hipGetLastError() == hipSuccess ? TVG_OK : TVG_ERR_LAUNCH;
}

template <int B, int ST, bool UNAL, int KG, int WM = 4>
tvg_status launch(const StripsArgs &args, const StripsPlan &plan, hipStream_t stream)
{
    const bool any = args.OW % 2 != 0 || (reinterpret_cast<uintptr_t>(args.y) | reinterpret_cast<uintptr_t>(args.residual)) % 4 != 0;
    if constexpr (!UNAL)
        if (!any) return launch_instance<B, ST, UNAL, KG, WM, false>(args, plan, stream);
    return launch_instance<B, ST, UNAL, KG, WM, true>(args, plan, stream);
}

template <int ST, bool UNAL, int KG>
tvg_status launch_b(const StripsArgs &args, const StripsPlan &plan, hipStream_t stream)
{
    switch (plan.b) {
    case 4: return launch<4, ST, UNAL, KG>(args, plan, stream);
    case 5: return launch<5, ST, UNAL, KG>(args, plan, stream);
    case 6: return launch<6, ST, UNAL, KG>(args, plan, stream);
    case 7: return launch<7, ST, UNAL, KG>(args, plan, stream);
    default:
        if constexpr (ST == 1) return launch<8, ST, UNAL, KG>(args, plan, stream);
        else return TVG_ERR_UNSUPPORTED;
    }
}

// Geometry of a launch with strips of b rows; false where a tile does not fit.
bool set_geometry(const ConvProblem &p, int b, int kg, StripsPlan *g)
{
    const int waves = kg == 4 ? 2 : 4;                 // along the channels
    const int strips = (p.W + 7) / 8, in = p.sh == 1 ? b + 2 : 2 * b + 1;
    g->b = b;
    g->kg = kg;
    g->t8 = std::min(strips, 4);
    if (p.IC / kChunk % kg != 0 || (kg == 2 && p.W % 2 == 0) || (kg > 1 && p.sh == 2) || (kg == 4 && b != 4)) return false;
    // (a window's first column, and without a stride its last, is its neighbour's)
    g->windows = strips <= 4 ? 1 : p.sh == 1 ? (p.W - 8 + 23) / 24 : (strips - 1 + 2) / 3;
    if (g->windows > 1 && p.W % 4 != 0) return false;
    g->spi = (p.OH + b - 1) / b * g->windows;
    g->sr = std::min(4 / g->t8, p.N * g->spi);
    g->rows = g->sr * in;
    g->row_bytes = g->t8 * 8;
    // the channels of a read are an odd number of 32 bytes apart, its four strips in a row on four eighths of 32 bytes,
    // also across strip rows: distinct banks
    // (unless that leaves no room for a second workgroup: strips of 8 rows, reads of two turns)
    const int strip = in * g->row_bytes, stages = p.sh == 1 && kg <= 2 ? 2 : 1;
    for (int pad : {((8 * g->t8 - strip) % 32 + 32) % 32, 0}) {
        g->strip_bytes = strip + pad;
        g->half = g->sr * g->strip_bytes;
        g->plane = (2 * g->half + 31) / 64 * 64 + 32;
        g->rows_bytes = kChunk * g->plane + 4 * kOctetGap;
        // two stages of rows (under a stride, where they are twice as many, one), and the weights; at the end what two groups exchange
        g->lds_bytes = kg * (waves * kWeightBytes + stages * (size_t)g->rows_bytes) + 256;
        if (g->lds_bytes <= std::min(kg, 2) * (size_t)80 * 1024) break;
    }
    if (kg > 1) g->lds_bytes = std::max(g->lds_bytes, (size_t)kg * waves * b * 2048 + 256);
    if (g->lds_bytes > 160 * 1024) return false;
    g->ptiles = ((long)p.N * g->spi + g->sr - 1) / g->sr;
    g->tiles = g->ptiles * ((p.OC + 16 * waves - 1) / (16 * waves));
    g->workgroups = walks_tiles(p.W % 2 != 0, kg) ? std::min(g->tiles, 2L * kComputeUnits) : g->tiles;
    return true;
}

// Times in us on both sides of the dispatch, fitted to calls without a residual of 31400 shapes of 64 to 512 input channels that
// were timed in every form of this kernel and in the kernel behind it (maps of 3 to 112 rows and columns, 32 to 512 output
// channels, batches of 1 to 128; the geometric mean of repeated calls and of calls over buffers of 120 MB; standard deviation
// of the fits 2 to 5 %, strided windows 7.5, the kernels behind 4.7).  A CU's tiles run in pairs, two waves on a SIMD.  row,
// short_row: per tile and row of a strip, the latter for maps of 5, 6, 7 or 14 columns; mbyte, x_mbyte: of
// y and of x.
struct Fit { float launch, tile, pair0, pair1, single0, single1, mbyte, row, short_row, x_mbyte; };
constexpr Fit kEven = {4.49f, 0.0f, 0.60f, 0.269f, 0.441f, 0.16f, 0.24f, 0.13f, 0.14f, 0.0f};            // rows of 2n pixels
constexpr Fit kWindows = {4.14f, 0.0f, 0.71f, 0.248f, 0.489f, 0.16f, 0.26f, 0.17f, 0.0f, 0.02f};         // ... of more than 32
constexpr Fit kOdd[2] = {{4.54f, 0.0f, 0.75f, 0.239f, 0.375f, 0.20f, 0.34f, 0.29f, 0.13f, 0.0f},         // one group, two
                         {2.31f, 1.49f, 0.76f, 0.278f, 0.0f, 0.0f, 0.46f, 0.55f, 0.14f, 0.0f}};
constexpr Fit kQuarters[2] = {{1.65f, 0.0f, 0.0f, 0.53f, 0.0f, 0.0f, 0.37f, 1.12f, 0.06f, 0.02f},        // four groups: even, odd rows
                              {2.16f, 0.0f, 0.0f, 0.599f, 0.0f, 0.0f, 0.64f, 1.25f, 0.07f, 0.0f}};
constexpr Fit kStride2[2] = {{4.94f, 0.0f, 0.67f, 0.203f, 0.413f, 0.14f, 0.37f, 0.13f, 0.12f, 0.005f},   // even, odd rows
                             {4.42f, 0.03f, 1.08f, 0.17f, 0.56f, 0.17f, 0.39f, 0.32f, 0.0f, 0.001f}};
constexpr Fit kStride2Windows = {3.95f, 0.0f, 0.82f, 0.184f, 0.536f, 0.129f, 0.34f, 0.20f, 0.0f, 0.06f};

float x_mbytes(const ConvProblem &p) { return 2e-6f * p.N * p.IC * p.H * p.W; }

float strips_us(const ConvProblem &p, const StripsPlan &g)
{
    const bool odd = p.W % 2 != 0, short_rows = odd ? p.W == 5 || p.W == 7 : p.W == 6 || p.W == 14;
    const Fit &f = p.sh == 2 ? (g.windows > 1 ? kStride2Windows : kStride2[odd])
                             : g.kg == 4 ? kQuarters[odd] : g.windows > 1 ? kWindows : odd ? kOdd[g.kg - 1] : kEven;
    const long q = (g.tiles + kComputeUnits - 1) / kComputeUnits;
    const bool two = g.kg == 1 && g.lds_bytes <= 80 * 1024;
    const float pairs = g.kg > 1 ? q : two ? q / 2 : 0, singles = g.kg > 1 ? 0 : two ? q % 2 : q;
    return f.launch + q * (f.tile + g.b * (f.row + (short_rows ? f.short_row : 0.0f))) +
           p.IC / kChunk / g.kg * (pairs * (f.pair0 + f.pair1 * g.b) + singles * (f.single0 + f.single1 * g.b)) +
           f.mbyte * 2e-6f * p.OC * p.npix + f.x_mbyte * x_mbytes(p);
}

// The kernels behind, by what decides their speed: stages, pixels per tile, pixels per load and load tasks per thread.  (8-pixel
// loads of rows of 8n pixels meet on banks.)  The first row that fits; pair, single: per 16 input channels and 64 output channels.
// rows: 1 of an odd number of pixels, 0 even, 8 of 8n, -1 any; px, pt: at least.
struct TiledFit { int sh, dbuf, nt, groups, rows, px, pt; float launch, tile, pair, single, mbyte, x_mbyte; };
constexpr TiledFit kTiled[] = {
    {1, 0, 64, 0, 1, 1, 1, 4.79f, 0.0f, 0.93f, 0.68f, 0.21f, 0.0f},
    {1, 0, 64, 0, 8, 1, 3, 5.14f, 0.0f, 1.40f, 0.82f, 0.0f, 0.0f}, {1, 0, 64, 0, 8, 1, 1, 4.40f, 0.0f, 0.92f, 0.64f, 0.14f, 0.015f},
    {1, 0, 64, 0, 0, 1, 3, 5.42f, 0.0f, 1.36f, 0.79f, 0.04f, 0.0f}, {1, 0, 64, 0, 0, 1, 1, 4.61f, 0.0f, 0.91f, 0.67f, 0.20f, 0.0f},
    {1, 0, 128, 0, 1, 1, 3, 5.27f, 0.0f, 1.65f, 0.78f, 0.28f, 0.0f}, {1, 0, 128, 0, 1, 1, 1, 2.50f, 0.11f, 1.61f, 0.47f, 0.42f, 0.0f},
    {1, 0, 128, 0, 8, 1, 3, 6.12f, 0.0f, 1.39f, 0.89f, 0.12f, 0.019f}, {1, 0, 128, 0, 8, 1, 1, 2.63f, 0.37f, 1.46f, 0.51f, 0.19f, 0.009f},
    {1, 0, 128, 0, 0, 1, 3, 6.05f, 0.0f, 1.39f, 0.92f, 0.18f, 0.013f}, {1, 0, 128, 0, 0, 1, 1, 3.27f, 0.09f, 1.46f, 0.53f, 0.31f, 0.0f},
    {1, 0, 256, 0, -1, 8, 1, 3.44f, 1.32f, 2.39f, 1.44f, 0.05f, 0.019f}, {1, 0, 256, 0, -1, 2, 1, 6.78f, 0.0f, 1.89f, 0.86f, 0.17f, 0.026f},
    {1, 0, 256, 0, -1, 1, 1, 5.68f, 1.16f, 2.06f, 1.82f, 0.25f, 0.0f}, {1, 0, 512, 0, -1, 8, 1, 6.41f, 2.55f, 3.40f, 1.98f, 0.0f, 0.053f},
    {1, 1, 64, 1, 1, 8, 1, 3.80f, 0.0f, 0.81f, 0.48f, 0.40f, 0.007f}, {1, 1, 64, 1, 1, 1, 1, 4.15f, 0.0f, 0.95f, 0.60f, 0.39f, 0.0f},
    {1, 1, 64, 1, 8, 8, 1, 3.11f, 0.57f, 2.28f, 1.22f, 0.12f, 0.031f}, {1, 1, 64, 1, 0, 2, 2, 4.77f, 0.0f, 1.42f, 0.79f, 0.67f, 0.0f},
    {1, 1, 64, 1, 0, 2, 1, 3.57f, 0.23f, 1.06f, 0.60f, 0.38f, 0.005f},
    {1, 1, 128, 1, 1, 8, 1, 4.23f, 0.58f, 1.02f, 0.60f, 0.23f, 0.0f}, {1, 1, 128, 1, 1, 1, 3, 0.0f, 2.67f, 1.43f, 1.12f, 0.53f, 0.007f},
    {1, 1, 128, 1, 1, 1, 1, 0.0f, 2.54f, 1.07f, 0.91f, 0.46f, 0.004f}, {1, 1, 128, 1, 8, 8, 1, 4.27f, 0.80f, 2.39f, 1.26f, 0.0f, 0.0f},
    {1, 1, 128, 1, 0, 2, 2, 5.01f, 0.12f, 1.60f, 0.88f, 0.41f, 0.012f}, {1, 1, 128, 1, 0, 2, 1, 3.37f, 0.83f, 1.19f, 0.70f, 0.38f, 0.0f},
    {1, 1, 256, 1, 1, 8, 1, 5.09f, 0.73f, 1.64f, 0.90f, 0.49f, 0.0f}, {1, 1, 256, 1, 1, 1, 1, 7.15f, 0.10f, 1.72f, 1.02f, 0.43f, 0.0f},
    {1, 1, 256, 1, 8, 8, 1, 5.87f, 0.58f, 2.55f, 1.36f, 0.09f, 0.021f}, {1, 1, 256, 1, 0, 2, 2, 5.72f, 0.40f, 1.91f, 1.06f, 0.28f, 0.023f},
    {1, 1, 256, 1, 0, 2, 1, 5.38f, 0.0f, 1.64f, 0.88f, 0.37f, 0.011f},
    // two groups of waves split the reduction: a single round of tiles
    {1, 1, 128, 2, 1, 1, 3, 5.95f, 0.0f, 0.0f, 0.79f, 0.36f, 0.014f}, {1, 1, 128, 2, 1, 1, 1, 4.52f, 0.0f, 0.0f, 0.61f, 0.59f, 0.0f},
    {1, 1, 256, 2, 1, 1, 1, 6.69f, 0.0f, 0.0f, 0.92f, 0.56f, 0.0f},
    {2, 0, 64, 0, -1, 2, 1, 4.08f, 0.0f, 1.19f, 1.03f, 0.06f, 0.012f}, {2, 0, 64, 0, -1, 1, 3, 4.82f, 0.0f, 1.44f, 1.15f, 0.08f, 0.0f},
    {2, 0, 64, 0, -1, 1, 1, 3.98f, 0.0f, 1.14f, 0.96f, 0.16f, 0.0f},
    {2, 0, 128, 0, -1, 2, 1, 3.58f, 0.0f, 1.62f, 0.85f, 0.35f, 0.031f}, {2, 0, 128, 0, -1, 1, 1, 3.30f, 1.0f, 2.27f, 1.81f, 0.40f, 0.078f},
    {2, 0, 256, 0, -1, 2, 1, 5.09f, 1.27f, 2.47f, 1.91f, 0.15f, 0.03f}, {2, 0, 256, 0, -1, 1, 1, 5.42f, 1.01f, 2.90f, 2.82f, 0.19f, 0.003f},
    {2, 1, 256, 1, -1, 2, 1, 4.50f, 0.0f, 0.0f, 1.90f, 0.40f, 0.0f},                  // (maps of a few rows or columns)
    {2, 1, 128, 1, -1, 8, 1, 4.42f, 0.0f, 0.0f, 1.05f, 0.27f, 0.002f}, {2, 1, 128, 1, -1, 2, 1, 4.57f, 0.0f, 0.0f, 0.95f, 0.51f, 0.0f},
};

// 0 where no row of the table fits
float tiled_us(const ConvProblem &p, const Patch3x3Plan &g)
{
    const int rows = p.W % 2 != 0 ? 1 : p.W % 8 == 0 ? 8 : 0;
    const long q = (((long)p.npix + g.nt - 1) / g.nt * ((p.OC + g.mt - 1) / g.mt) + kComputeUnits - 1) / kComputeUnits;
    for (const TiledFit &f : kTiled)
        if (f.sh == p.sh && f.dbuf == g.dbuf && f.nt == g.nt && (!g.dbuf || f.groups == g.kg) && (f.rows < 0 || f.rows == rows) && g.px >= f.px && g.pt >= f.pt)
            return f.launch + f.tile * q + p.IC / 16 * (g.mt == 128 ? 1.9f : 1.0f) * (q / 2 * f.pair + q % 2 * f.single) +
                   f.mbyte * 2e-6f * p.OC * p.npix + f.x_mbyte * x_mbytes(p);
    return 0.0f;
}

}  // namespace

bool plan_conv3x3_strips(const ConvProblem &p, const Patch3x3Plan &patch, StripsPlan *plan)
{
    if (p.dtype != TVG_BF16 || p.R != 3 || p.S != 3 || p.ph != 1 || p.pw != 1 || p.sh > 2 || p.sw != p.sh || p.IC % kChunk != 0) return false;
    if ((int64_t)p.N * p.IC * p.H * p.W >= (1 << 30) || (int64_t)p.OC * p.IC * 9 >= (1 << 30) ||
        (int64_t)p.N * p.OC * p.OH * p.OW >= (1 << 30)) return false;
    if ((int64_t)p.N * p.IC >= (1 << 22) || (int64_t)p.OC * p.IC >= (1 << 22) || p.H * p.W >= (1 << 22)) return false;   // 24-bit products
    const Knobs k = forced_knobs(p);
    const bool named = !k.mt && !k.nt && !k.lds_pitch && k.stages == 1 && k.row_loads == 2 && k.split_k <= 4;
    if (!named && (k.mt || k.nt || k.stages || k.split_k || k.lds_pitch || k.row_loads)) return false;
    // One chunk is not worth the set-up (306 shapes: 1.01 times as fast in the geometric mean, 99 slower).  Two groups
    // that split the reduction pay where rows are odd, whose pixels take more instructions to lay down.  Four, of half the output
    // channels, pay where the tiles of the others leave compute units idle and a workgroup's serial chain of chunks is the time.
    if (!named && p.IC < 2 * kChunk) return false;
    float best = 0.0f;
    StripsPlan g;
    for (int kg : {1, 2, 4})
        for (int b = 4; b <= (p.sh == 1 ? 8 : 7); ++b) {
            if (named && k.split_k && kg != k.split_k) continue;
            if (!set_geometry(p, b, kg, &g)) continue;
            const float us = strips_us(p, g);
            if (best == 0.0f || us < best) best = us, *plan = g;
        }
    if (best == 0.0f || named) return best > 0.0f;
    // What the fits leave open goes to the kernels behind, but for calls with a residual, which a plan serves too (three of five
    // unstrided layers of a residual network have one): they cost 1.01 to 1.13 times as much here and 1.04 to 1.8 behind, the more the
    // fewer pixels of a plane lie at aligned addresses.  Further from the line: outputs beyond 24 MB, whose store hint the
    // kernels behind make more of; two chunks in windows in a single round of tiles, which nothing else on the CU covers (16 images of
    // 64 -> 64 at 56x56 amid ResNet-18's layers 124.6 us a pass, 121.8 behind).
    // Odd rows of less than 8 pixels in one group of waves are where the fits are worst.
    // Of 14200 shapes without a residual 0.9 % are more than 5 % slower than in the kernel behind and 0.25 % more than 10 %, at worst 1.27
    // times (by the rule before, which did not know the load width of the kernels behind, 1.3 and 0.35 %); of 4100 with one 0.3 and 0.1 %
    // (0.5 and 0.2 %).  Time over the time behind in the geometric mean, without and with: rows of up to 32 even pixels 0.82 and 0.77, odd
    // 0.92 and 0.84 (0.93 and 0.88 before), longer ones 0.83 and 0.81, under a stride 0.81, of more than 32 pixels 0.86.
    const int plane = p.OH * p.OW;
    float margin = p.sh == 2 ? (plan->windows > 1 ? 1.09f : 1.04f) : plane % 8 == 0 ? 1.01f : plane % 4 == 0 ? 0.975f : plane % 2 == 0 ? 0.895f : p.W < 8 && plan->kg == 1 ? 1.06f : 0.945f;
    if (2e-6f * p.OC * p.npix > 24.0f) margin *= 1.05f;
    if (p.sh == 1 && plan->windows > 1 && p.IC == 2 * kChunk && plan->tiles <= kComputeUnits) margin *= 1.04f;
    return best * margin < tiled_us(p, patch);
}

bool conv3x3_strips_pointers_ok(const ConvPointers &ptr)
{
    // (x and w as for the kernels behind; y and the residual take accesses of the width that they allow)
    return (reinterpret_cast<uintptr_t>(ptr.x) | reinterpret_cast<uintptr_t>(ptr.w)) % 16 == 0 &&
           (reinterpret_cast<uintptr_t>(ptr.y) | reinterpret_cast<uintptr_t>(ptr.residual)) % 2 == 0;
}

tvg_status launch_conv3x3_strips(const ConvProblem &p, const StripsPlan &plan, const ConvPointers &ptr, hipStream_t stream)
{
    StripsArgs a{};
    a.x = static_cast<const bf16_t *>(ptr.x);
    a.w = static_cast<const bf16_t *>(ptr.w);
    a.scale = ptr.scale; a.shift = ptr.shift; a.bias = ptr.bias;
    a.residual = static_cast<const bf16_t *>(ptr.residual);
    a.y = static_cast<bf16_t *>(ptr.y);
    a.N = p.N; a.IC = p.IC; a.H = p.H; a.W = p.W; a.OC = p.OC; a.OH = p.OH; a.OW = p.OW;
    a.relu = p.relu;
    // (not where windows share the lines of a row: half a line that is written past the caches costs more than it saves.  16 images,
    // 192 -> 192 at 56x56 41.4 us with the hint taken, 35.3 without; 64 of 64 -> 64 at 56x56 38.9 and 25.3; 16 of 64 -> 64 at 112x112 44.6 and 30.6)
    a.nt = p.stream_out && plan.windows == 1;
    a.t8 = plan.t8; a.spi = plan.spi; a.sr = plan.sr; a.rows = plan.rows; a.windows = plan.windows;
    const int threads = plan.kg == 4 ? 128 : 256;                              // of a group
    a.dg = threads % plan.t8;
    a.drow = threads / plan.t8 % plan.rows;
    a.dch = threads / plan.t8 / plan.rows;
    a.row_bytes = plan.row_bytes; a.strip_bytes = plan.strip_bytes; a.half = plan.half; a.plane = plan.plane;
    a.rows_bytes = plan.rows_bytes;
    a.ptiles = (int)plan.ptiles;
    // An XCD walks adjacent tiles, so that with pixel tiles first x comes into the chip's eight L2s once per channel tile, and
    // with channel tiles first the weights once per XCD.  Where the first is ten times the second, channel tiles go first
    // (2391 shapes: 1.01 times as fast in the mean, 0.97 to 1.33; 32 images, 192 -> 192 at 56x56 under a stride 37.8 -> 29.8 us, 8 of
    // 192 -> 512 at 80x80 106.8 -> 92.2, 64 of 128 -> 256 at 28x28 under a stride 18.2 -> 16.6; at 6 to 10 times 0.965 to 1.1).
    const int64_t channel_tiles = plan.tiles / plan.ptiles;
    a.pixels_first = channel_tiles == 1 || channel_tiles * p.N * p.H * p.W < 10 * 8 * 9 * (int64_t)p.OC;
    a.nch = p.IC / kChunk;
    a.dump = (uint32_t)plan.lds_bytes - 256;
    a.tiles_per = (int)(plan.tiles / plan.workgroups); a.tiles_more = (int)(plan.tiles % plan.workgroups);
    a.x_bytes = ((uint32_t)((int64_t)p.N * p.IC * p.H * p.W) * 2 + 3) & ~3u;   // (up to the end of the last pixel's word)
    a.w_bytes = (uint32_t)(p.OC * p.IC * 9) * 2;
    a.y_bytes = (uint32_t)((int64_t)p.N * p.OC * p.OH * p.OW) * 2;
    a.by_inner = make_divider(a.pixels_first ? a.ptiles : (int)channel_tiles); a.by_spi = make_divider(a.spi); a.by_t8 = make_divider(a.t8);
    a.by_rows = make_divider(a.rows); a.by_windows = make_divider(a.windows);
    if (plan.kg == 4) return p.W % 2 != 0 ? launch<4, 1, true, 4, 2>(a, plan, stream) : launch<4, 1, false, 4, 2>(a, plan, stream);
    if (p.sh == 2) return p.W % 2 != 0 ? launch_b<2, true, 1>(a, plan, stream) : launch_b<2, false, 1>(a, plan, stream);
    if (p.W % 2 != 0) return plan.kg == 2 ? launch_b<1, true, 2>(a, plan, stream) : launch_b<1, true, 1>(a, plan, stream);
    return launch_b<1, false, 1>(a, plan, stream);
}

}  // namespace tvg
