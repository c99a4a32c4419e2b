// fp32 fused 1x1 convolution, any equal strides, input channels a multiple of 8, on few tiles and at throughput size.
//
// v_mfma_f32_32x32x2_f32 takes one k value per lane and 64 cycles, so that neither operand needs the LDS: a lane
// fetches four channels of its output channel's weights with one 16-byte load and one, two or four adjacent pixels of
// four input channels with four loads, which is PXL operand pairs per channel - k may run in any order, and the
// operand's 32 pixels may be every PXL-th one.  A step of eight channels is 4 PXL NB MFMAs (256 PXL NB cycles) and five
// loads, kAhead steps in flight, no barrier and no address arithmetic (channel offsets are scalar).
//   - Four waves: KS of them split the reduction and add their tiles through LDS, in pairs, 4 / KS lie side by side
//     along the output channels.  Few tiles: KS = 4 and the narrowest of 32, 64 or 128 pixels that stays within one
//     round of workgroups.  Throughput: KS = 2, tiles of 64 channels x 64 or 128 pixels.
//   - Consecutive workgroups take the channel tiles of one pixel tile and meet in an XCD's L2.
// What bounds it: the matrix pipe (51 % of its rate at 32 x 512 -> 512, 14x14) and the plain adds of short chains, on few
// tiles the first loads.  us before -> now:
// batch 4, 512 -> 512 14x14 19.3 -> 8.7 (the launch-bound kernel), 256 -> 256 28x28 13.5 -> 8.8 (the kernel with rows in
// LDS); batch 1, 512 -> 512 14x14 20.6 -> 5.7, stride 3 15.4 -> 6.8; batch 32, 512 -> 512 14x14 59.7 -> 42 (the gather
// kernel).  MobileNet body, batch 4: 283 -> 197.  Of 602 shapes 516 take it, 1.75 times as fast in the geometric mean, three
// of them by 0.94 to 0.97 (strides, where the kernel with rows in LDS stood); their error against 64 bits is 0.69 of the
// former kernels' in the geometric mean and 1.00 at most where there are a thousand outputs to take it from.
#include <algorithm>

#include "tvg_device.h"
#include "tvg_internal.h"

namespace tvg {

namespace {

constexpr int kRsrcFlags = 0x00020000;
constexpr uint32_t kOutOfRange = 0x80000000u;      // and everything above: tensors stay below 2 GiB
constexpr int kStep = 8;                           // input channels per step: four per half-wave
constexpr int kAhead = 4;                          // steps in flight

struct PwArgs {
    const float *x, *w, *scale, *shift, *bias, *residual;
    float *y;
    int IC, OC, HW, OHW, OW, W, npix, stride, relu, vec, mtiles, steps;
    uint32_t x_bytes, w_bytes;
    Divider by_mtiles, by_ohw, by_ow;
};

template <int PXL> struct Pixels;
template <> struct Pixels<4> { typedef float4v vec; };
template <> struct Pixels<2> { typedef float vec __attribute__((ext_vector_type(2))); };
template <> struct Pixels<1> { typedef float vec __attribute__((ext_vector_type(1))); };

// A wave: 32 MI output channels x 32 PXL NB pixels, PXL adjacent pixels per lane; KS waves split the reduction, WM
// waves lie side by side along the channels.  Chains of CHAIN steps are added to TOT totals in turn.
template <int NB, int PXL, int KS, int CHAIN, int TOT>
__global__ __launch_bounds__(256, 2) void conv_f32_pw_kernel(const PwArgs a)
{
    typedef typename Pixels<PXL>::vec pixels;
    constexpr int WM = 4 / KS, NT = 32 * PXL * NB, MT = 32 * WM;
    extern __shared__ __attribute__((aligned(16))) float smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wk = wave % KS, wm = wave / KS;
    const int lrow = lane & 31, lhalf = lane >> 5;
    int mt;
    const int p0 = divide(xcd_remap(blockIdx.x, gridDim.x), a.by_mtiles, &mt) * NT;
    const int m0 = mt * MT;

    const __amdgpu_buffer_rsrc_t xrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.x), 0, a.x_bytes, kRsrcFlags);
    const __amdgpu_buffer_rsrc_t wrsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(a.w), 0, a.w_bytes, kRsrcFlags);
    uint32_t xoff[NB];
    const int woc = m0 + wm * 32 + lrow;
    const uint32_t woff = woc < a.OC ? 4u * (uint32_t)(woc * a.IC + 4 * lhalf) : kOutOfRange;
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int p = p0 + (b * 32 + lrow) * PXL;
        int r;
        const int n = divide(p, a.by_ohw, &r);
        if (a.stride != 1) {
            int ow;
            const int oh = divide(r, a.by_ow, &ow);
            r = (oh * a.W + ow) * a.stride;
        }
        xoff[b] = p < a.npix ? 4u * (uint32_t)((n * a.IC + 4 * lhalf) * a.HW + r) : kOutOfRange;
    }
    const int s_beg = wk * a.steps / KS, s_end = (wk + 1) * a.steps / KS;

    float4v wreg[kAhead];
    pixels xreg[kAhead][NB][4];
    auto load = [&](int slot, int s) __attribute__((always_inline)) {
        const int c = s * kStep;
        wreg[slot] = __builtin_bit_cast(float4v, __builtin_amdgcn_raw_buffer_load_b128(wrsrc, woff, c * 4, 0));
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int at = (c + q) * a.HW * 4;
                if constexpr (PXL == 4) xreg[slot][b][q] = __builtin_bit_cast(pixels, __builtin_amdgcn_raw_buffer_load_b128(xrsrc, xoff[b], at, 0));
                else if constexpr (PXL == 2) xreg[slot][b][q] = __builtin_bit_cast(pixels, __builtin_amdgcn_raw_buffer_load_b64(xrsrc, xoff[b], at, 0));
                else xreg[slot][b][q][0] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(xrsrc, xoff[b], at, 0));
            }
    };
    // (steps past a wave's last are requested too, from channel rows that exist or out of range, and not used)
#pragma unroll
    for (int d = 0; d < kAhead; ++d) {
        load(d, min(s_beg + d, a.steps - 1));
        __builtin_amdgcn_sched_barrier(0);
    }

    // Chains of CHAIN steps start from zero and are added to the totals in plain adds.
    float16v acc[NB][PXL], sum[TOT][NB][PXL];
#pragma unroll
    for (int t = 0; t < TOT; ++t)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int e = 0; e < PXL; ++e)
#pragma unroll
                for (int v = 0; v < 16; ++v) sum[t][b][e][v] = 0.0f;

    auto multiply = [&](int slot, bool first, bool last) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int e = 0; e < PXL; ++e) {
                    float16v c = acc[b][e];
                    if (first && q == 0)
#pragma unroll
                        for (int v = 0; v < 16; ++v) c[v] = 0.0f;
                    acc[b][e] = __builtin_amdgcn_mfma_f32_32x32x2f32(wreg[slot][q], xreg[slot][b][q][e], c, 0, 0, 0);
                }
        if (last) {
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int e = 0; e < PXL; ++e) sum[slot / CHAIN % TOT][b][e] += acc[b][e];
        }
    };
    int s = s_beg;
    for (; s + kAhead <= s_end; s += kAhead) {
#pragma unroll
        for (int d = 0; d < kAhead; ++d) {
            multiply(d, d % CHAIN == 0, d % CHAIN == CHAIN - 1);
            load(d, min(s + kAhead + d, a.steps - 1));
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    const int left = s_end - s;                    // 0 .. 3 steps, the last one ends its chain
    if (left == 1) {
        multiply(0, true, true);
    } else if (left == 2) {
        multiply(0, true, CHAIN == 1);
        multiply(1, CHAIN == 1, true);
    } else if (left == 3) {
        multiply(0, true, CHAIN == 1);
        multiply(1, CHAIN == 1, CHAIN <= 2);
        multiply(2, CHAIN <= 2, true);
    }

#pragma unroll
    for (int d = 1; d < TOT; d *= 2)
#pragma unroll
        for (int t = 0; t + d < TOT; t += 2 * d)
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int e = 0; e < PXL; ++e) sum[t][b][e] += sum[t + d][b][e];

    // value v of a lane: channel 8 (v / 4) + 4 lhalf + v % 4, pixel PXL lrow + e
    auto finish = [&](pixels o, int oc, int p) __attribute__((always_inline)) {
        if (oc >= a.OC || p >= a.npix) return;                     // (whole groups: OH * OW is a multiple of PXL)
        int r;
        const int n = divide(p, a.by_ohw, &r);
        const size_t idx = (size_t)(n * a.OC + oc) * a.OHW + r;
        const float sc = a.scale[oc], sf = a.bias ? fmaf(a.bias[oc], sc, a.shift[oc]) : a.shift[oc];
        pixels res;
        if (a.residual) {
            if (a.vec) res = *reinterpret_cast<const pixels *>(a.residual + idx);
            else
#pragma unroll
                for (int e = 0; e < PXL; ++e) res[e] = a.residual[idx + e];
        }
#pragma unroll
        for (int e = 0; e < PXL; ++e) {
            float t = fmaf(o[e], sc, sf);
            if (a.residual) t += res[e];
            o[e] = a.relu ? fmaxf(t, 0.0f) : t;    // (without a ReLU a NaN stays one, as after a split reduction)
        }
        // (the store hint of a call changes nothing here, 202 us with and without for six layers at batch 32, and is not taken)
        if (a.vec) *reinterpret_cast<pixels *>(a.y + idx) = o;
        else
#pragma unroll
            for (int e = 0; e < PXL; ++e) a.y[idx + e] = o[e];
    };
    // [wave of the split][channel of the tile][pixel]
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        float *row = smem + (wk * MT + wm * 32 + 8 * (v >> 2) + 4 * lhalf + (v & 3)) * NT;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            pixels o;
#pragma unroll
            for (int e = 0; e < PXL; ++e) o[e] = sum[0][b][e][v];
            *reinterpret_cast<pixels *>(row + (b * 32 + lrow) * PXL) = o;
        }
    }
    __syncthreads();
    constexpr int PER = NT / PXL;
    for (int item = tid; item < MT * PER; item += 256) {
        const int row = item / PER, g = item % PER;
        pixels o[KS];
#pragma unroll
        for (int k = 0; k < KS; ++k) o[k] = *reinterpret_cast<const pixels *>(smem + (k * MT + row) * NT + g * PXL);
#pragma unroll
        for (int d = 1; d < KS; d *= 2)            // in pairs
#pragma unroll
            for (int k = 0; k + d < KS; k += 2 * d) o[k] += o[k + d];
        finish(o[0], m0 + row, p0 + g * PXL);
    }
}

template <int NB, int PXL, int KS, int CHAIN, int TOT = CHAIN == 1 && NB * PXL <= 2 ? 2 : 1>
tvg_status launch(const PwArgs &args, long tiles, hipStream_t stream)
{
    const auto kernel = conv_f32_pw_kernel<NB, PXL, KS, CHAIN, TOT>;
    constexpr size_t lds = (size_t)4 * 32 * 32 * PXL * NB * 4;      // KS partial tiles of 32 * (4 / KS) channels: 64 KB at most
    static_assert(lds <= 64 * 1024, "more wants an opt-in");
    kernel<<<dim3((unsigned)tiles), dim3(256), lds, stream>>>(args);
    return hipGetLastError() == hipSuccess ? TVG_OK : TVG_ERR_LAUNCH;
}

template <int NB, int PXL>
tvg_status launch_split(const PwArgs &args, const F32PwPlan &plan, hipStream_t stream)
{
    // Chains no longer than those of the kernels that ran these problems before: 8 channels where four waves split the
    // reduction (the sums hide behind the loads); where two do, 8 up to 127 channels, 16 up to 255, 32, and half of that under
    // a stride (256 -> 512 at 28x28, stride 2: error against 64 bits 0.97e-7 with 16, 1.14e-7 with 32, 0.98e-7 in the
    // kernel with rows in LDS).
    const int channels = args.stride > 1 ? args.IC / 2 : args.IC;
    // Two totals where the registers allow, four for long reductions (2048 channels at 7x7, 64 chains per wave: error
    // against 64 bits 1.30e-7 with two, 1.08e-7 with four, 1.22e-7 in the kernel before; 0.1 us of a launch).
    if constexpr (NB * PXL == 1)
        if (plan.ks == 4 && args.IC > 1024) return launch<NB, PXL, 4, 1, 4>(args, plan.tiles, stream);
    if (plan.ks == 4) return launch<NB, PXL, 4, 1>(args, plan.tiles, stream);
    if (channels < 128) return launch<NB, PXL, 2, 1>(args, plan.tiles, stream);
    if (channels < 256) return launch<NB, PXL, 2, 2>(args, plan.tiles, stream);
    return launch<NB, PXL, 2, 4>(args, plan.tiles, stream);
}

void set_tile(const ConvProblem &p, int ks, int nb, int pxl, F32PwPlan *plan)
{
    plan->ks = ks;
    plan->nb = nb;
    plan->pxl = pxl;
    const int mt = 32 * (4 / ks), nt = 32 * nb * pxl;
    plan->mt = mt;
    plan->nt = nt;
    plan->tiles = (long)((p.OC + mt - 1) / mt) * ((p.npix + nt - 1) / nt);
}

}  // namespace

bool plan_conv_f32_pw(const ConvProblem &p, bool few_tiles, int nt, F32PwPlan *plan)
{
    if (p.dtype != TVG_F32 || p.R != 1 || p.S != 1 || p.ph || p.pw || p.sh != p.sw || p.IC % kStep != 0) return false;
    // Problems of other kernels' few tiles: the launch-bound ones, and those of the gather kernel (strides from 3 on, long
    // rows) whose 128 x 128 tiles are fewer than CUs, where it splits the reduction.
    few_tiles = few_tiles || (nt == 0 && (long)((p.OC + 127) / 128) * ((p.npix + 127) / 128) < kComputeUnits);
    if (p.IC < (few_tiles ? 32 : 64)) return false;
    if ((size_t)p.N * p.IC * p.H * p.W >= ((size_t)1 << 29) || (size_t)p.OC * p.IC >= ((size_t)1 << 29)) return false;   // 32-bit byte offsets
    const Knobs k = forced_knobs(p);
    if (k.mt || k.nt || k.stages || k.split_k || k.lds_pitch || k.row_loads) return false;
    const int OHW = p.OH * p.OW, most = p.sh > 1 ? 1 : OHW % 4 == 0 ? 4 : OHW % 2 == 0 ? 2 : 1;
    if (few_tiles) {
        for (int w = 1; w <= 4; w *= 2) {
            set_tile(p, 4, w <= most ? 1 : w / most, std::min(w, most), plan);
            if (plan->tiles <= kComputeUnits) break;
        }
        return true;
    }
    // (64 channels under a stride: 32 images, 64 -> 128 at 56x56, 20.0 us in the kernel with rows in LDS, 23.1 here)
    if (p.sh > 1 && p.IC < 72) return false;
    if (nt == 0) {
        // In place of the gather kernel's 128 x 128 tiles: without a stride (64 images, 128 -> 128 at 56x56, stride 2, 33 us
        // there and 52 here), where the reduction is not short (64 -> 128, 16 images 56x56, 19.7 us there and 22.4 here) and
        // 64-channel tiles waste little (136 -> 104, 36 images 52x52, 47.8 and 49.8).  128 -> 512, 64 images 28x28, 89 and 83;
        // 256 -> 256, 32 images, 49.5 and 42; 1024 -> 1024, 7x7, 57 and 44.
        // Up to 255 channels tiles of 64 pixels where they come out in fewer rounds, two tiles per CU (184 -> 293, 6 images
        // 40x81, 3 rounds and 2 of 128 pixels, 32 and 37 us; 128 -> 512 above 97 and 83), and on maps that no wide loads fit.
        if (p.sh > 1 || p.IC < 128 || 6 * p.OC < 5 * ((p.OC + 63) / 64 * 64)) return false;
        const auto rounds = [&](int t) {
            set_tile(p, 2, 1, t / 32, plan);
            return (plan->tiles + 2 * kComputeUnits - 1) / (2 * kComputeUnits);
        };
        nt = p.IC >= 256 || (most == 4 && 8 * rounds(128) <= 5 * rounds(64)) ? 128 : 64;
    }
    const int pxl = std::min(most, nt / 32);
    set_tile(p, 2, nt / 32 / pxl, pxl, plan);
    // Under a stride on small maps, where 32 adjacent pixels are many short rows, against the kernel with rows in LDS: while
    // every tile has a place, two per CU (256 -> 1024 at 14x14, 32 images, 400 tiles, 22.7 us there and 20.9 here; 64
    // images, 784 tiles, 34.7 and 39.4; 256 -> 256 at 56x56, 16 images, 784 tiles, 45.6 and 42.1).
    return p.sh == 1 || p.OW >= 16 || plan->tiles <= 2 * kComputeUnits;
}

bool conv_f32_pw_pointers_ok(const ConvPointers &ptr)
{
    // (buffer loads of any width want 4 bytes: weights that are views into one parameter buffer run here too)
    return reinterpret_cast<uintptr_t>(ptr.x) % 4 == 0 && reinterpret_cast<uintptr_t>(ptr.w) % 4 == 0;
}

tvg_status launch_conv_f32_pw(const ConvProblem &p, const F32PwPlan &plan, const ConvPointers &ptr, hipStream_t stream)
{
    PwArgs a;
    a.x = static_cast<const float *>(ptr.x);
    a.w = static_cast<const float *>(ptr.w);
    a.scale = ptr.scale; a.shift = ptr.shift; a.bias = ptr.bias;
    a.residual = static_cast<const float *>(ptr.residual);
    a.y = static_cast<float *>(ptr.y);
    a.IC = p.IC; a.OC = p.OC; a.HW = p.H * p.W; a.OHW = p.OH * p.OW; a.OW = p.OW; a.W = p.W;
    a.npix = p.npix; a.stride = p.sh; a.relu = p.relu;
    a.vec = (reinterpret_cast<uintptr_t>(ptr.y) | reinterpret_cast<uintptr_t>(ptr.residual)) % (4u * plan.pxl) == 0;
    a.mtiles = (p.OC + plan.mt - 1) / plan.mt;
    a.steps = p.IC / kStep;
    a.x_bytes = (uint32_t)((size_t)p.N * p.IC * p.H * p.W * 4);
    a.w_bytes = (uint32_t)((size_t)p.OC * p.IC * 4);
    a.by_mtiles = make_divider(a.mtiles); a.by_ohw = make_divider(a.OHW); a.by_ow = make_divider(a.OW);
    if (plan.pxl == 4) return launch_split<1, 4>(a, plan, stream);
    if (plan.pxl == 2) return plan.nb == 1 ? launch_split<1, 2>(a, plan, stream) : launch_split<2, 2>(a, plan, stream);
    if (plan.nb == 1) return launch_split<1, 1>(a, plan, stream);
    return plan.nb == 2 ? launch_split<2, 1>(a, plan, stream) : launch_split<4, 1>(a, plan, stream);
}

}  // namespace tvg
