// cf_ffn.hip -- the two-launch block of cf_ffn.h: the depth-wise kernel and
// the launcher.
#include "cf_ffn.h"
#include "cf_kernels.h"

namespace cf {
namespace ffn {

// Depth-wise KS x KS conv with s0, b0: one thread makes 8 channels of TW
// neighbouring output pixels, so an input vector is loaded once per kernel
// row for up to KS outputs.  Loads go straight to global memory: the C / 8
// threads of a strip read one pixel's channels contiguously and neighbouring
// strips meet in L1.  fp32 sums; at KS >= 5 an fp16 kernel row is summed in
// packed fp16 first, its taps at a quarter (as the fused kernels do for the
// whole window).
struct DwArgs {
    const uint16_t *x, *w;
    uint16_t *d;
    const float *s0, *b0;
    int H, W, C;
    uint32_t strips;  // N * H * ceil(W / TW)
    FastDiv sw, h;    // strips per row, H
};

template <typename T, int KS, int TW>
__global__ __launch_bounds__(256) void dw_strip_kernel(DwArgs a) {
    constexpr int PAD = KS / 2, XV = TW + KS - 1;
    constexpr bool ROW16 = !T::is_bf16 && KS >= 5;
    const int c8n = a.C / 8;  // a power of two, at most 64
    const int c0 = 8 * ((int)threadIdx.x & (c8n - 1));
    const uint32_t strip = blockIdx.x * (256 / c8n) + threadIdx.x / c8n;
    if (strip >= a.strips)
        return;
    const uint32_t row = fdiv(strip, a.sw), n = fdiv(row, a.h);
    const int h = (int)(row - n * a.h.d), w0 = (int)(strip - row * a.sw.d) * TW;
    float acc[TW][8];
#pragma unroll
    for (int t = 0; t < TW; t++)
#pragma unroll
        for (int e = 0; e < 8; e++)
            acc[t][e] = 0.0f;
    const uint16_t *xn = a.x + (size_t)n * a.H * a.W * a.C + c0;
#pragma unroll 1
    for (int i = 0; i < KS; i++) {  // not unrolled: over few pixels the launch is instruction fetch
        const int hh = h + i - PAD;
        if (hh < 0 || hh >= a.H)
            continue;
        const uint16_t *xr = xn + (size_t)hh * a.W * a.C;
        u32x4 xv[XV];
#pragma unroll
        for (int j = 0; j < XV; j++) {
            const int c = w0 + j - PAD;
            const bool in = c >= 0 && c < a.W;
            xv[j] = *reinterpret_cast<const u32x4 *>(xr + (size_t)(in ? c : 0) * a.C);
#pragma unroll
            for (int d = 0; d < 4; d++)
                xv[j][d] = in ? xv[j][d] : 0u;
        }
        u32x4 tv[KS];
#pragma unroll
        for (int j = 0; j < KS; j++)
            tv[j] = *reinterpret_cast<const u32x4 *>(a.w + (size_t)(i * KS + j) * a.C + c0);
        if constexpr (ROW16) {
#pragma unroll
            for (int d = 0; d < 4; d++) {
                half2v tw[KS], xw[XV];
#pragma unroll
                for (int j = 0; j < KS; j++) {
                    const uint32_t v = tv[j][d];
                    tw[j] = __builtin_bit_cast(half2v, v) * splat2(0.25f);
                }
#pragma unroll
                for (int j = 0; j < XV; j++) {
                    const uint32_t v = xv[j][d];
                    xw[j] = __builtin_bit_cast(half2v, v);
                }
#pragma unroll
                for (int t = 0; t < TW; t++) {
                    half2v s = tw[0] * xw[t];
#pragma unroll
                    for (int j = 1; j < KS; j++)
                        s = __builtin_elementwise_fma(tw[j], xw[t + j], s);
                    acc[t][2 * d] = fmaf((float)s.x, 4.0f, acc[t][2 * d]);
                    acc[t][2 * d + 1] = fmaf((float)s.y, 4.0f, acc[t][2 * d + 1]);
                }
            }
        } else {
#pragma unroll
            for (int j = 0; j < KS; j++)
#pragma unroll
                for (int d = 0; d < 4; d++)
#pragma unroll
                    for (int t = 0; t < TW; t++) {
                        acc[t][2 * d] = fmaf(T::lo(xv[t + j][d]), T::lo(tv[j][d]), acc[t][2 * d]);
                        acc[t][2 * d + 1] = fmaf(T::hi(xv[t + j][d]), T::hi(tv[j][d]), acc[t][2 * d + 1]);
                    }
        }
    }
    float sc[8], bi[8];
#pragma unroll
    for (int e = 0; e < 8; e++) {
        sc[e] = a.s0 ? a.s0[c0 + e] : 1.0f;
        bi[e] = a.b0 ? a.b0[c0 + e] : 0.0f;
    }
    uint16_t *dr = a.d + ((size_t)row * a.W + w0) * a.C + c0;
#pragma unroll
    for (int t = 0; t < TW; t++)
        if (w0 + t < a.W) {
            u32x4 o;
#pragma unroll
            for (int d = 0; d < 4; d++)
                o[d] = T::pack2(fmaf(acc[t][2 * d], sc[2 * d], bi[2 * d]),
                                fmaf(acc[t][2 * d + 1], sc[2 * d + 1], bi[2 * d + 1]));
            *reinterpret_cast<u32x4 *>(dr + (size_t)t * a.C) = o;
        }
}

// The same over few pixels: one thread per pixel and 8 channels, every load of
// the window (KS = 7: of a row) issued before the first use, since the launch
// is one chain of latencies (addresses clamped, values outside dropped).
template <typename T, int KS>
__global__ __launch_bounds__(256) void dw_pixel_kernel(DwArgs a) {
    constexpr int PAD = KS / 2, RB = KS <= 3 ? KS : 1;  // rows per batch of loads
    const int c8n = a.C / 8;
    const int c0 = 8 * ((int)threadIdx.x & (c8n - 1));
    const uint32_t p = blockIdx.x * (256 / c8n) + threadIdx.x / c8n;
    if (p >= a.strips)
        return;
    const uint32_t row = fdiv(p, a.sw), n = fdiv(row, a.h);
    const int h = (int)(row - n * a.h.d), w = (int)(p - row * a.sw.d);
    const uint16_t *xn = a.x + (size_t)n * a.H * a.W * a.C + c0;
    float acc[8], sc[8], bi[8];
#pragma unroll
    for (int e = 0; e < 8; e++) {
        acc[e] = 0.0f;
        sc[e] = a.s0 ? a.s0[c0 + e] : 1.0f;
        bi[e] = a.b0 ? a.b0[c0 + e] : 0.0f;
    }
#pragma unroll 1
    for (int i0 = 0; i0 < KS; i0 += RB) {
        u32x4 xv[RB][KS], tv[RB][KS];
#pragma unroll
        for (int i = 0; i < RB; i++)
#pragma unroll
            for (int j = 0; j < KS; j++) {
                const int hh = min(max(h + i0 + i - PAD, 0), a.H - 1), c = min(max(w + j - PAD, 0), a.W - 1);
                xv[i][j] = *reinterpret_cast<const u32x4 *>(xn + ((size_t)hh * a.W + c) * a.C);
                tv[i][j] = *reinterpret_cast<const u32x4 *>(a.w + (size_t)((i0 + i) * KS + j) * a.C + c0);
            }
#pragma unroll
        for (int i = 0; i < RB; i++)
#pragma unroll
            for (int j = 0; j < KS; j++) {
                const int hh = h + i0 + i - PAD, c = w + j - PAD;
                const bool in = hh >= 0 && hh < a.H && c >= 0 && c < a.W;
#pragma unroll
                for (int d = 0; d < 4; d++) {
                    const uint32_t v = in ? xv[i][j][d] : 0u;
                    acc[2 * d] = fmaf(T::lo(v), T::lo(tv[i][j][d]), acc[2 * d]);
                    acc[2 * d + 1] = fmaf(T::hi(v), T::hi(tv[i][j][d]), acc[2 * d + 1]);
                }
            }
    }
    u32x4 o;
#pragma unroll
    for (int d = 0; d < 4; d++)
        o[d] = T::pack2(fmaf(acc[2 * d], sc[2 * d], bi[2 * d]), fmaf(acc[2 * d + 1], sc[2 * d + 1], bi[2 * d + 1]));
    *reinterpret_cast<u32x4 *>(a.d + (size_t)p * a.C + c0) = o;
}

constexpr int64_t FEW_PIXELS = 4096;
int64_t round_pixels() { return (int64_t)64 * device_cu_count(); }  // one 64-pixel tile for each CU

// TW = 0: one pixel per thread
template <typename T, int KS, int TW>
hipError_t dw_launch(const void *x, void *d, const BlockW &w, const Shape &s, hipStream_t st) {
    DwArgs a{};
    a.x = (const uint16_t *)x;
    a.w = (const uint16_t *)w.dw_w;
    a.d = (uint16_t *)d;
    a.s0 = w.s0;
    a.b0 = w.b0;
    a.H = s.H;
    a.W = s.W;
    a.C = s.C;
    const uint32_t sw = (uint32_t)ceil_div(s.W, TW ? TW : 1);
    a.strips = (uint32_t)s.N * s.H * sw;
    a.sw = make_fastdiv(sw);
    a.h = make_fastdiv((uint32_t)s.H);
    const uint32_t per = 256 / (s.C / 8);
    const dim3 grid((a.strips + per - 1) / per);
    if constexpr (TW == 0)
        hipLaunchKernelGGL((dw_pixel_kernel<T, KS>), grid, dim3(256), 0, st, a);
    else
        hipLaunchKernelGGL((dw_strip_kernel<T, KS, TW>), grid, dim3(256), 0, st, a);
    return hipGetLastError();
}

template <typename T>
hipError_t depthwise(const void *x, void *d, const BlockW &w, const Shape &s, bool grouped, hipStream_t st) {
    // both kernels add in the same order where a row is summed in fp32, so a
    // micro-batch gives the bits of its whole batch; a block with hidden groups
    // always sums in fp32 (as the kernels of a handful of pixels do)
    if (grouped || ((int64_t)s.N * s.H * s.W <= FEW_PIXELS && (T::is_bf16 || s.k < 5)))
        switch (s.k) {
        case 1: return dw_launch<T, 1, 0>(x, d, w, s, st);
        case 3: return dw_launch<T, 3, 0>(x, d, w, s, st);
        case 5: return dw_launch<T, 5, 0>(x, d, w, s, st);
        default: return dw_launch<T, 7, 0>(x, d, w, s, st);
        }
    // strips of 7 or 4 pixels, whichever covers a row with less overhang
    const bool seven = ceil_div(s.W, 7) * 7 <= ceil_div(s.W, 4) * 4;
    switch (s.k) {
    case 1: return dw_launch<T, 1, 4>(x, d, w, s, st);
    case 3: return seven ? dw_launch<T, 3, 7>(x, d, w, s, st) : dw_launch<T, 3, 4>(x, d, w, s, st);
    case 5: return seven ? dw_launch<T, 5, 7>(x, d, w, s, st) : dw_launch<T, 5, 4>(x, d, w, s, st);
    default: return seven ? dw_launch<T, 7, 7>(x, d, w, s, st) : dw_launch<T, 7, 4>(x, d, w, s, st);
    }
}

template <typename T, int C, int NT, int PG, int ACT>
hipError_t ffn_launch(const Args &a, int groups, hipStream_t st) {
    const void *k = (const void *)ffn_kernel<T, C, NT, PG, ACT>;
    hipError_t e = allow_full_lds(k);
    if (e != hipSuccess)
        return e;
    constexpr uint32_t PX = PG * 16 * NT;
    Args b = a;
    void *args[] = {&b};
    return hipLaunchKernel(k, dim3((a.P + PX - 1) / PX, groups), dim3(PG * shares(C) * 64), args,
                           lds_bytes(C, a.per * chunk(C)), st);
}

template <typename T, int ACT>
hipError_t ffn(const Args &a, int C, int groups, bool f32, hipStream_t st) {
    if constexpr (!T::is_bf16 && ACT == ACT_GELU)
        if (f32)
            return C == 512 ? ffn_launch<T, 512, 1, 4, ACT_GELU_F32>(a, groups, st)
                            : ffn_launch<T, 256, 1, 2, ACT_GELU_F32>(a, groups, st);
    if (C == 512)
        return ffn_launch<T, 512, 1, 4, ACT>(a, groups, st);
    if (C == 128)
        return ffn_launch<T, 128, 2, 2, ACT>(a, groups, st);
    // C = 256: the pixel tile grows with the batch, so that the weights are
    // streamed as seldom as the CUs can be kept in one round (256 CUs): 32 pixels
    // up to 8192 (30 images of 14 x 14 in bf16: 33.7 us against 36.0 and 49.9 with
    // 64 and 128), 64 up to 16384 (fp16, k = 5: 34.4 against 43.4 with 128),
    // then 128 (128 images, fp16: 51.3 against 58.9 with 64)
    if (groups > 1 || 2 * (int64_t)a.P <= round_pixels())
        return ffn_launch<T, 256, 1, 2, ACT>(a, groups, st);
    if (a.P <= round_pixels())
        return ffn_launch<T, 256, 1, 4, ACT>(a, groups, st);
    return ffn_launch<T, 256, 2, 4, ACT>(a, groups, st);
}

template <typename T>
hipError_t block(const void *x, void *y, const BlockW &w, const Shape &s, int groups, float *part, hipStream_t st) {
    hipError_t e = depthwise<T>(x, y, w, s, groups > 1, st);
    if (e != hipSuccess)
        return e;
    Args a{};
    a.x = (const uint16_t *)x;
    a.y = (uint16_t *)y;
    a.w1 = (const uint16_t *)w.w1;
    a.w2 = (const uint16_t *)w.w2;
    a.s1 = w.s1;
    a.b1 = w.b1;
    a.s2 = w.s2;
    a.b2 = w.b2;
    a.P = (uint32_t)((int64_t)s.N * s.H * s.W);
    a.EC = s.E * s.C;
    a.part = groups > 1 ? part : nullptr;
    a.per = group_chunks(a.EC / chunk(s.C), groups);
    const bool f32 = s.cfg == CFG_FFN_F32;
    return s.act == ACT_GELU   ? ffn<T, ACT_GELU>(a, s.C, groups, f32, st)
           : s.act == ACT_RELU ? ffn<T, ACT_RELU>(a, s.C, groups, f32, st)
                               : ffn<T, ACT_NONE>(a, s.C, groups, f32, st);
}

}  // namespace ffn

// Where the two launches beat one: C = 256 and 512 in both types, C = 128 in
// bf16 (N = 128, 28 x 28: 87 us against 168; in fp16 the single kernel of
// cf_wide.h does as well, 72 against 70 us, with one launch).  N = 128,
// 14 x 14, C = 256: k = 7 58.7 against 69.6 us in fp16, k = 3 57.4 against
// 295.8 in bf16; in fp16 k = 3 is even (51.3 against 52.9 on cold inputs, 57
// against 54 inside a stage), so above one round of 64-pixel tiles it keeps
// the single launch.  C = 512, 11 to 100 images of 7 x 7: 97 us against
// 160 (fp16) and 265 to 535 (bf16).  E up to 14 (7 at C = 512) by the LDS.
bool ffn_applies(const Shape &s) {
    const int64_t P = (int64_t)s.N * s.H * s.W;
    return ((s.C == 128 && s.bf16) || (s.C == 256 && (s.bf16 || s.k >= 5 || P <= ffn::round_pixels())) || s.C == 512) &&
           P < ((int64_t)1 << 31) - 4096 && ffn::dw_launchable((int64_t)s.N * s.H, s.W, s.C) &&
           ffn::lds_bytes(s.C, s.E * s.C) <= (s.C == 128 ? 80u : 160u) * 1024;
}

// Groups enough to give every CU a workgroup, with at least two chunks each at
// C = 512 (one is all prologue), and partials within 16 MiB.  Per block in a
// captured graph, groups 1 / 2 / 4 / 8 / 16 / 32: 4 images of 14 x 14 at
// C = 256 fp16 39.0 / 24.7 / 22.4 / 22.4 / 29.0 / - us; one image of 7 x 7 at
// C = 512 bf16 64.8 / 60.7 / 37.2 / 28.3 / 24.8 / 24.3 us.  C = 128 gains
// nothing (20.4 / 19.9 / 21.1 us for 4 images of 28 x 28 in bf16).  At C = 256,
// E = 1 four chunks are all prologue and reduction: k = 3 fp16, with groups /
// without (up to 64 pixels the slice kernel, in blocks of 32) 11.6 / 11.9 us for 4
// pixels, 13.3 / 12.2 for 16, 14.3 / 16.5 for 49, 14.4 / 12.8 for 196, 22.6 / 16.8
// for 3920; k = 7 13.3 / 17.9 for 16.
int ffn_groups(const Shape &s) {
    if (!ffn_applies(s) || s.C == 128)
        return 1;
    const int64_t P = (int64_t)s.N * s.H * s.W;
    if (s.C == 256 && s.E == 1 && (P > 64 || (s.k <= 3 && P > 4 && P <= 32)))
        return 1;
    const int px = s.C == 256 ? 32 : 64;
    const int64_t tiles = (P + px - 1) / px, chunks = s.E * s.C / ffn::chunk(s.C);
    const int64_t most = s.C == 512 ? chunks / 2 : chunks;
    int64_t g = device_cu_count() / tiles;
    g = g > most ? most : g;
    const int64_t fit = ((int64_t)16 << 20) / (P * s.C * 4);
    g = g > fit ? fit : g;
    return ffn::filled_groups((int)chunks, (int)g);
}

int ffn_fitting_groups(const Shape &whole, size_t one, size_t bytes) {
    const int g = ffn_groups(whole);
    return g > 1 ? ffn::fitting_groups(whole.E * whole.C / ffn::chunk(whole.C), g, one, bytes) : 1;
}

// fp16 GELU of a block with groups.  The kernels of a handful of pixels work in
// fp32 (cf_slice.hip up to 64, cf_small.hip at C = 512 up to the some 70 that its
// LDS holds), and so do the groups over them, where it costs a launch of
// latencies little: 49 pixels at C = 256 13.7 us with the packed polynomial and
// 13.9 with fp32, at C = 512 23.0 and 22.9.  Above, the polynomial of the larger
// batches: 16 images of 14 x 14 at C = 256 26.6 and 27.5 us, 64 of 7 x 7 at C = 512
// 64.3 and 67.2, 4 of them over four groups 33.4 and 36.2.
int ffn_group_cfg(const Shape &whole) {
    return (int64_t)whole.N * whole.H * whole.W <= 128 ? CFG_FFN_F32 : CFG_FFN;
}

hipError_t launch_ffn_block(const void *x, void *y, const BlockW &w, const Shape &s, int groups, float *part,
                            hipStream_t st) {
    if (groups != ffn::filled_groups(s.E * s.C / ffn::chunk(s.C), groups))
        return hipErrorInvalidValue;  // the caller adds as many partials as it asks for
    return s.bf16 ? ffn::block<BF16>(x, y, w, s, groups, part, st) : ffn::block<F16>(x, y, w, s, groups, part, st);
}

}  // namespace cf
