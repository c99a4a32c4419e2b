// bf16 fused 1x1 convolution without a stride, input channels a multiple of 32, at throughput size.
//
// A GEMM whose weights lie k innermost and whose pixels do not.  The kernel beside it (conv1x1_kernel) fetches a pixel
// operand as eight 2-byte loads and packs it; here pixels lie in LDS as they lie in memory, [channel][pixel], from
// 16-byte loads, and gfx950's transposing LDS read (4 pixels x 4 channels from each of 16 lanes) makes the operand: an
// eighth of the load instructions and no packing.
//   - Pixels are numbered in groups of eight per image, the last one of an image partly empty (196 pixels: 25 groups, 49:
//     7), so that a load never crosses an image.  Maps of 2n pixels: 4-byte aligned loads and stores; odd maps: the
//     aligned words around a group, shifted into place, and stores of single pixels with adjacent lanes on adjacent ones.
//   - Chunks of 32 channels (64 from 1024 on), two LDS stages, one barrier per chunk, 2 or 4 chunks in flight in registers.
//   - The tail goes through LDS as fp32, so that residual and output move in 16-byte pieces of a channel row.
// What bounds it: on the layers of a network a fixed 6 us (launch, first loads, tail) and then the LDS: 224 cycles per
// chunk and tile of 64 channels x 128 pixels against 128 of the matrix pipe.  us before -> now at batch 32: 512 -> 512
// 14x14 12.2 -> 11.2, 1024 -> 1024 7x7 14.9 -> 12.1, 256 -> 256 28x28 12.6 -> 11.1; batch 8: 256 -> 256 28x28 6.8 -> 5.2; batch
// 128: 512 -> 512 37.6 -> 30; 96 -> 143, 26 images 83x26: 45.5 -> 12.8.  Of 253 shapes 179 take it (or the kernel for few
// tiles), 1.32 times as fast in the geometric mean.
#include "tvg_device.h"
#include "tvg_internal.h"

namespace tvg {

namespace {

constexpr int kRsrcFlags = 0x00020000;
constexpr uint32_t kOutOfRange = 0x80000000u;      // and everything above: tensors stay below 2 GiB

typedef uint32_t uint4u __attribute__((ext_vector_type(4), aligned(4)));      // eight pixels of a map of 2n pixels
typedef short short4v __attribute__((ext_vector_type(4)));
typedef short short8v __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) short4v *lds_short4;

struct PwRowsArgs {
    const bf16_t *x, *w;
    const float *scale, *shift, *bias;
    const bf16_t *residual;
    bf16_t *y;
    int IC, OC, HW, relu, mtiles, nchunks, vec;
    int g8, ngroups;                   // groups of eight pixels per image and in all
    uint32_t x_bytes, w_bytes;
    Divider by_mtiles, by_g8;
};

// MT output channels x NT pixel slots, 256 threads; a chunk is CH input channels; UNAL: maps of an odd number of pixels.
template <int MT, int NT, int CH, bool UNAL>
__global__ __launch_bounds__(256) void conv1x1_rows_kernel(const PwRowsArgs a)
{
    constexpr int WM = 2, WN = 2;                  // waves along channels, along pixels
    constexpr int MI = MT / WM / 32, NJ = NT / WN / 32;
    constexpr int GT = NT / 8;                     // pixel groups per tile
    constexpr int XT = CH * GT / 256, WT = MT * (CH / 8) / 256;          // load tasks per thread
    constexpr int XP = NT * 2 + 64, WP = CH * 2 + 16;                    // LDS pitches: distinct banks
    constexpr int XB = CH * XP, STAGE = XB + MT * WP;
    constexpr int AHEAD = CH == 64 ? 2 : 4;        // chunks in flight in registers
    constexpr int SP = NT + 4;                     // floats per staged channel row of the tail
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const int lrow = lane & 31, lhalf = lane >> 5;
    int mt;
    const int g0 = divide(xcd_remap(blockIdx.x, gridDim.x), a.by_mtiles, &mt) * GT;
    const int m0 = mt * MT;
    float *ss = reinterpret_cast<float *>(smem);
    unsigned char *stages = smem + MT * 8;

    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(a.x), 0, a.x_bytes, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(a.w), 0, a.w_bytes, kRsrcFlags);
    uint32_t xoff[XT], woff[WT];
    int xdst[XT], wdst[WT], odd[XT];
#pragma unroll
    for (int k = 0; k < XT; ++k) {
        const int id = tid + 256 * k, g = id % GT, ch = id / GT;
        int r;
        const int n = divide(g0 + g, a.by_g8, &r);
        const uint32_t at = (uint32_t)((n * a.IC + ch) * a.HW + 8 * r);
        odd[k] = (int)(at & 1);
        xoff[k] = g0 + g < a.ngroups ? 2u * (UNAL ? at & ~1u : at) : kOutOfRange;
        xdst[k] = ch * XP + g * 16;
    }
#pragma unroll
    for (int k = 0; k < WT; ++k) {
        const int id = tid + 256 * k, piece = id % (CH / 8), oc = id / (CH / 8);
        woff[k] = m0 + oc < a.OC ? 2u * (uint32_t)((m0 + oc) * a.IC + 8 * piece) : kOutOfRange;
        wdst[k] = XB + oc * WP + piece * 16;
    }
    uint32_t xraw[AHEAD][XT][UNAL ? 5 : 4];
    uint4v wraw[AHEAD][WT];
    auto load = [&](int slot, int c) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < XT; ++k) {
            const uint4v v = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(xrsrc, xoff[k], c * CH * a.HW * 2, 0));
#pragma unroll
            for (int d = 0; d < 4; ++d) xraw[slot][k][d] = v[d];
            if constexpr (UNAL) xraw[slot][k][4] = __builtin_amdgcn_raw_buffer_load_b32(xrsrc, xoff[k] + 16, c * CH * a.HW * 2, 0);
        }
#pragma unroll
        for (int k = 0; k < WT; ++k)
            wraw[slot][k] = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, woff[k], c * CH * 2, 0));
    };
    auto stage = [&](int slot, unsigned char *dst) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < XT; ++k) {
            uint4v v;
#pragma unroll
            for (int d = 0; d < 4; ++d)
                v[d] = UNAL ? __builtin_amdgcn_alignbit(xraw[slot][k][UNAL ? d + 1 : d], xraw[slot][k][d], odd[k] * 16) : xraw[slot][k][d];
            *reinterpret_cast<uint4v *>(dst + xdst[k]) = v;
        }
#pragma unroll
        for (int k = 0; k < WT; ++k) *reinterpret_cast<uint4v *>(dst + wdst[k]) = wraw[slot][k];
    };
#pragma unroll
    for (int d = 0; d < AHEAD; ++d) {
        load(d, min(d, a.nchunks - 1));
        __builtin_amdgcn_sched_barrier(0);
    }
    if (tid < MT) {
        float sc = 0.0f, sf = 0.0f;
        if (m0 + tid < a.OC) {
            sc = a.scale[m0 + tid];
            sf = a.shift[m0 + tid];
            if (a.bias) sf = fmaf(a.bias[m0 + tid], sc, sf);
        }
        ss[2 * tid] = sc;
        ss[2 * tid + 1] = sf;
    }

    // operand addresses: a transposing read takes 4 pixels of 4 channels from each of 16 lanes
    const int l16 = lane & 15, sub = (lane >> 4) & 1;
    const int xat = (8 * lhalf + (l16 >> 2)) * XP + (wn * NJ * 32 + sub * 16 + (l16 & 3) * 4) * 2;
    const int wat = XB + (wm * MI * 32 + lrow) * WP + lhalf * 16;

    float16v acc[MI][NJ];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;

    auto multiply = [&](const unsigned char *src) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < CH / 16; ++k) {
            bf16x8v px[NJ], wt[MI];
#pragma unroll
            for (int i = 0; i < MI; ++i) wt[i] = *reinterpret_cast<const bf16x8v *>(src + wat + i * 32 * WP + k * 32);
#pragma unroll
            for (int j = 0; j < NJ; ++j) {
                const unsigned char *p = src + xat + k * 16 * XP + j * 64;
                const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4)(p));
                const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4)(p + 4 * XP));
                px[j] = __builtin_bit_cast(bf16x8v, short8v{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
            }
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NJ; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(px[j], wt[i], acc[i][j], 0, 0, 0);
        }
    };

    stage(0, stages);
    load(0, min(AHEAD, a.nchunks - 1));
    __syncthreads();
    // chunk c: multiply its stage, then put chunk c + 1 into the other one (its readers are past the last barrier)
    int c = 0;
    for (; c + AHEAD <= a.nchunks - 1; c += AHEAD) {
#pragma unroll
        for (int d = 0; d < AHEAD; ++d) {
            multiply(stages + (d & 1) * STAGE);
            __builtin_amdgcn_sched_barrier(0);
            stage((d + 1) % AHEAD, stages + ((d + 1) & 1) * STAGE);
            load((d + 1) % AHEAD, min(c + d + 1 + AHEAD, a.nchunks - 1));
            __builtin_amdgcn_sched_barrier(0);
            __syncthreads();
        }
    }
#pragma unroll
    for (int d = 0; d < AHEAD; ++d) {
        if (c + d >= a.nchunks) break;
        multiply(stages + (d & 1) * STAGE);
        if (c + d + 1 < a.nchunks) stage((d + 1) % AHEAD, stages + ((d + 1) & 1) * STAGE);
        __syncthreads();
    }

    // ---- tail: scaled sums through LDS, then eight pixels of one channel per thread --------------
    float *out = reinterpret_cast<float *>(stages);
#pragma unroll
    for (int i = 0; i < MI; ++i) {
        const int row = (wm * MI + i) * 32 + lrow;
        const float sc = ss[2 * row], sf = ss[2 * row + 1];
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float4v o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = fmaf(acc[i][j][4 * q + e], sc, sf);
                *reinterpret_cast<float4v *>(out + row * SP + (wn * NJ + j) * 32 + 8 * q + 4 * lhalf) = o;
            }
    }
    __syncthreads();
    const float floor_v = relu_floor(a.relu & 1);
    if (UNAL || !a.vec) {                          // adjacent lanes adjacent pixels
        for (int id = tid; id < MT * NT; id += 256) {
            const int p = id % NT, row = id / NT;
            int r;
            const int n = divide(g0 + p / 8, a.by_g8, &r);
            r = 8 * r + p % 8;
            if (n * a.g8 >= a.ngroups || r >= a.HW || m0 + row >= a.OC) continue;
            const int idx = (n * a.OC + m0 + row) * a.HW + r;
            const float rr = a.residual ? bf16_to_f32(a.residual[idx]) : 0.0f;
            a.y[idx] = f32_to_bf16(fmaxf(out[row * SP + p] + rr, floor_v));
        }
        return;
    }
#pragma unroll
    for (int k = 0; k < MT * GT / 256; ++k) {
        const int id = tid + 256 * k, g = id % GT, row = id / GT;
        int r;
        const int n = divide(g0 + g, a.by_g8, &r);
        if (g0 + g >= a.ngroups || m0 + row >= a.OC) continue;
        const int idx = (n * a.OC + m0 + row) * a.HW + 8 * r, left = a.HW - 8 * r;
        const float4v o0 = *reinterpret_cast<const float4v *>(out + row * SP + 8 * g);
        const float4v o1 = *reinterpret_cast<const float4v *>(out + row * SP + 8 * g + 4);
        float f[8] = {o0[0], o0[1], o0[2], o0[3], o1[0], o1[1], o1[2], o1[3]};
        if (left >= 8) {
            if (a.residual) {
                const uint4v v = *reinterpret_cast<const uint4u *>(a.residual + idx);
#pragma unroll
                for (int e = 0; e < 8; ++e) f[e] += __uint_as_float(e & 1 ? v[e >> 1] & 0xFFFF0000u : v[e >> 1] << 16);
            }
            uint4u v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = f32x2_to_bf16x2(fmaxf(f[2 * e], floor_v), fmaxf(f[2 * e + 1], floor_v));
            if (a.relu & 2) __builtin_nontemporal_store(v, reinterpret_cast<uint4u *>(a.y + idx));
            else *reinterpret_cast<uint4u *>(a.y + idx) = v;
        } else {                                   // the last group of a map that is no multiple of eight
#pragma unroll
            for (int e = 0; e < 6; e += 2)
                if (e < left) {
                    uint32_t rr = 0;
                    if (a.residual) rr = *reinterpret_cast<const uint32_t *>(a.residual + idx + e);
                    *reinterpret_cast<uint32_t *>(a.y + idx + e) =
                        f32x2_to_bf16x2(fmaxf(f[e] + __uint_as_float(rr << 16), floor_v),
                                        fmaxf(f[e + 1] + __uint_as_float(rr & 0xFFFF0000u), floor_v));
                }
        }
    }
}

template <int MT, int NT, int CH, bool UNAL>
tvg_status launch(const PwRowsArgs &args, long tiles, hipStream_t stream)
{
    const auto kernel = conv1x1_rows_kernel<MT, NT, CH, UNAL>;
    constexpr size_t stages = 2 * (size_t)(CH * (NT * 2 + 64) + MT * (CH * 2 + 16)), tail = (size_t)MT * (NT + 4) * 4;
    constexpr size_t lds = MT * 8 + (stages > tail ? stages : tail);
    static bool configured = false;                // opt in to > 64 KB of dynamic LDS once per instance
    if (!configured && lds > 64 * 1024) {
        if (hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024) != hipSuccess)
            return TVG_ERR_LAUNCH;
        configured = true;
    }
    kernel<<<dim3((unsigned)tiles), dim3(256), lds, stream>>>(args);
    return hipGetLastError() == hipSuccess ? TVG_OK : TVG_ERR_LAUNCH;
}

template <int MT, int NT, int CH>
tvg_status launch_align(const PwRowsArgs &args, long tiles, hipStream_t stream)
{
    return args.HW % 2 ? launch<MT, NT, CH, true>(args, tiles, stream) : launch<MT, NT, CH, false>(args, tiles, stream);
}

}  // namespace

bool plan_conv1x1_rows(const ConvProblem &p, Pw1x1Plan *plan)
{
    if (p.dtype != TVG_BF16 || p.R != 1 || p.S != 1 || p.ph || p.pw || p.sh != 1 || p.sw != 1 || p.IC % 32 != 0) return false;
    if ((size_t)p.N * p.IC * p.H * p.W * 2 > (size_t)kOutOfRange || (size_t)p.OC * p.IC * 2 > (size_t)kOutOfRange) return false;
    const Knobs k = forced_knobs(p);
    const bool named = k.row_loads == 2 && k.stages != 2 && !k.split_k && !k.lds_pitch;      // 1x1: rows as they lie in memory
    if (!named && (k.mt || k.nt || k.stages || k.split_k || k.lds_pitch || k.row_loads)) return false;
    const long groups = (long)p.N * ((p.H * p.W + 7) / 8);
    const auto tiles = [&](int mt, int nt) { return (long)((p.OC + mt - 1) / mt) * ((groups + nt / 8 - 1) / (nt / 8)); };
    int mt = 64, nt = 64;
    if (k.mt) {
        mt = k.mt;
        nt = k.nt;
        if (!((mt == 64 && (nt == 64 || nt == 128)) || (mt == 128 && nt == 128))) return false;
    } else {
        // Where the kernel that packs pixels in registers stays: reductions of one or two chunks, which it has in flight as a
        // whole (64 -> 128, 8 images 56x56, 4.3 us there, 4.8 here; 41 shapes of two chunks 0.79 to 1.9 times as fast here, half of
        // them below 0.97; one chunk and a large map: 18.5 and 16.4), large odd maps (19 shapes 0.81 to 1.5, half of them below 1).
        // Not four chunks on few tiles (ten shapes 1.00 to 1.18; 128 -> 256, one image 28x28, 3.9 and 3.4).
        // Wider tiles from where they still cover the chip (128 images, 512 -> 512 14x14, 31 -> 30; 1024 -> 1024 7x7, 35.6 ->
        // 30.7; 32 images, 256 -> 512 14x14, 8.5 but 8.7).
        const bool odd = p.H * p.W % 2 != 0;
        const long t = tiles(64, 64);
        if ((odd && p.H * p.W > 1024) || p.IC == 64 || (p.IC == 32 && (odd || t < 3000))) return false;
        if (p.IC >= 1024 && t >= 1500) mt = nt = 128;
        else if (!odd && (p.IC >= 512 ? t >= 800 : p.IC >= 256 ? t >= 1500 : p.IC == 32)) nt = 128;
    }
    plan->mt = mt;
    plan->nt = nt;
    plan->tiles = tiles(mt, nt);
    return true;
}

bool conv1x1_rows_pointers_ok(const ConvPointers &ptr)
{
    return reinterpret_cast<uintptr_t>(ptr.w) % 16 == 0 && reinterpret_cast<uintptr_t>(ptr.x) % 16 == 0;
}

tvg_status launch_conv1x1_rows(const ConvProblem &p, const Pw1x1Plan &plan, const ConvPointers &ptr, hipStream_t stream)
{
    PwRowsArgs a;
    a.x = static_cast<const bf16_t *>(ptr.x);
    a.w = static_cast<const bf16_t *>(ptr.w);
    a.scale = ptr.scale; a.shift = ptr.shift; a.bias = ptr.bias;
    a.residual = static_cast<const bf16_t *>(ptr.residual);
    a.y = static_cast<bf16_t *>(ptr.y);
    a.IC = p.IC; a.OC = p.OC; a.HW = p.H * p.W;
    a.relu = p.relu | (p.stream_out << 1);
    a.vec = a.HW % 2 == 0 && (reinterpret_cast<uintptr_t>(ptr.y) | reinterpret_cast<uintptr_t>(ptr.residual)) % 4 == 0;
    a.mtiles = (p.OC + plan.mt - 1) / plan.mt;
    a.g8 = (a.HW + 7) / 8;
    a.ngroups = p.N * a.g8;
    a.x_bytes = ((uint32_t)((size_t)p.N * p.IC * a.HW) * 2 + 3) & ~3u;         // (up to the end of the last pixel's word)
    a.w_bytes = (uint32_t)((size_t)p.OC * p.IC * 2);
    a.by_mtiles = make_divider(a.mtiles);
    a.by_g8 = make_divider(a.g8);
    const bool deep = p.IC >= 1024 && p.IC % 64 == 0;
    a.nchunks = p.IC / (deep && plan.nt == 64 ? 64 : 32);
    if (plan.mt == 128) return launch_align<128, 128, 32>(a, plan.tiles, stream);
    if (plan.nt == 128) return launch_align<64, 128, 32>(a, plan.tiles, stream);
    return deep ? launch_align<64, 64, 64>(a, plan.tiles, stream) : launch_align<64, 64, 32>(a, plan.tiles, stream);
}

}  // namespace tvg
