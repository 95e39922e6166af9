// cf_ffn.h -- wide blocks (C = 128, 256, 512) as a depth-wise launch that
// writes D into y and one launch that runs the whole FFN and the residual on
// D in place (Sec. 5.3.1, eq. e:ffn-eff: expand, activation and project chunk
// by chunk, the hidden layer never leaves the registers).
//
// ffn_kernel: a workgroup owns PG * 16 * NT pixels; its PG * HS waves are PG
// pixel groups times HS shares (32 hidden channels each) of every chunk.  A
// wave keeps its pixels' D fragments and all C output accumulators in
// registers; with HS = 2 the two waves of a pixel group add their
// accumulators once, at the end.  Products are v_mfma_f32_16x16x32 with
// weights as the A operand and pixels as B.  W1's rows are taken in the order
// that leaves a lane eight consecutive hidden channels -- the project's B
// fragment -- and W2's in the order that leaves it eight consecutive output
// channels, one 16-byte store.  The order of every sum depends on neither the
// pixel tile nor the position of a pixel in it.
//
// Few pixels: grid.y splits the chunks into groups; each writes an fp32
// partial of s2 * project and the caller adds the groups in order.  Up to 128
// pixels these launches are chains of latencies, and the activation is the fp32
// GELU in fp16 too (ACT_GELU_F32): 7 x 7, C = 256 and 512, E = 4, fp16, relative
// error 7.9e-4 with the packed polynomial, 2.6e-4 this way.
//
// Chunks of W1 and W2 come by LDS-DMA into one of two slots while the other
// is used: one barrier per chunk.  A copy instruction moves 1 KB: whole rows
// of W1 (512 / C of them) or a 64 HS byte segment of 16 / HS rows of W2,
// always in address order; the kilobytes lie 1056 bytes apart.  A 16-byte LDS
// read serves its lanes in groups that mix two neighbouring q (fragment lanes
// j = 0-3, 12-15 of one with 4-11 of the other), so rows are dealt to
// kilobytes such that the two sets S0 = {0-3, 12-15} and S1 = {4-11} of j
// each cover the even 16-byte columns of the banks and q picks the parity: no
// conflicts (3.4 M conflict cycles of 7.7 M LDS cycles a launch with rows
// simply 16 bytes further along each kilobyte).  With j as the rank (0-7) in
// set S, share h and tile m:
//   W1 row 32 h + 8 (j / 4) + 4 m + j % 4: kilobyte rank + 8 S plus
//     16 h and row m of it (C = 256), row 2 h + m of it (C = 128), or plus
//     16 m (C = 512);
//   W2 row 32 o + 8 (j / 4) + 4 m + j % 4 (output pair o), HS = 2: kilobyte
//     rank % 4 + 4 o, segment rank / 4 + 2 S + 4 m of it; HS = 1: kilobyte
//     rank % 2 + 2 o, segment rank / 2 + 4 S + 8 m.
//
// A workgroup reads the D rows it owns before the first barrier and writes
// the same rows of y after the last, so D and y share the buffer and no
// workspace is needed (with groups the sums are written by a later launch).
#pragma once

#include "cf_ffn_plan.h"
#include "cf_fused_impl.h"

namespace cf {
namespace ffn {

enum { ACT_GELU_F32 = 3 };  // fp16 only, after ACT_GELU, ACT_RELU and ACT_NONE

struct Args {
    const uint16_t *x;
    uint16_t *y;  // D on entry, the block's output on return
    const uint16_t *w1, *w2;
    const float *s1, *b1, *s2, *b2;
    float *part;  // [groups][P][C], or null
    uint32_t P;
    int EC;
    int per;  // chunks per group
};

constexpr uint32_t PITCH = 1056;
constexpr uint32_t slot_bytes(int C) { return (uint32_t)(C / 8 * shares(C)) * PITCH; }
// LDS: two chunk slots, then s1 and b1 of the group's channels (fp16: a quarter of each)
constexpr uint32_t lds_bytes(int C, int channels) { return 2 * slot_bytes(C) + 8 * (uint32_t)channels; }

__device__ __forceinline__ void dma16s_at(const void *base, uint32_t voff, uint32_t lds_addr) {
    const uint32_t lds = (uint32_t)__builtin_amdgcn_readfirstlane(lds_addr);
    const uint64_t b = (uint64_t)(uintptr_t)base;
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
    const uint64_t bu = ((uint64_t)hi << 32) | (uint64_t)lo;
    uint32_t saved;
    asm volatile(
        "s_mov_b32 %0, m0\n\t"
        "s_mov_b32 m0, %3\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, %2\n\t"
        "s_mov_b32 m0, %0"
        : "=&s"(saved)
        : "v"(voff), "s"(bu), "s"(lds)
        : "memory");
}

// Wait for this wave's copies and LDS traffic, then the workgroup barrier.
__device__ __forceinline__ void copy_barrier() {
    __builtin_amdgcn_s_waitcnt(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

template <typename T, int C, int NT, int PG, int ACT>
__global__ __launch_bounds__(PG * shares(C) * 64) __attribute__((amdgpu_waves_per_eu(2, 2))) void ffn_kernel(Args a) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    constexpr int HS = shares(C), CHUNK = chunk(C), NW = PG * HS;
    constexpr int KS = C / 32, OP = C / 32;   // expand K steps; pairs of output tiles
    constexpr int NI = C / 16 * HS / NW;      // copies per wave of W1, and of W2, per chunk
    constexpr uint32_t CB = slot_bytes(C);
    static_assert((C / 16 * HS) % NW == 0 && (HS == 1 || NW * OP * NT * 1024 <= 2 * (int)CB),
                  "whole copies; the final exchange fits the slots");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int pg = wv % PG, hs = wv / PG;
    const int q = lane >> 4, jl = lane & 15;
    const int EC = a.EC;
    const int c0 = (int)blockIdx.y * a.per, nch = min(a.per, EC / CHUNK - c0);  // this group's chunks
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;

    // copies: this wave fills kilobytes b = wv + NW i of W1 and of W2.  A
    // lane's source offset holds the part of its row that depends on the lane,
    // the wave-uniform rest goes to the base address
    const uint32_t r1 = C == 512 ? 0 : lane / (C / 8 % 64);
    const uint32_t o1 = (32 * (r1 >> 1) + 4 * (r1 & 1)) * (C * 2) + (lane - r1 * (C / 8)) * 16;
    uint32_t o2;
    if constexpr (HS == 2) {
        const uint32_t r2 = lane >> 3, j4 = (r2 >> 1) & 1 ? 1 + (r2 & 1) : 3 * (r2 & 1);
        o2 = (8 * j4 + 4 * (r2 >> 2)) * (uint32_t)(EC * 2) + (lane & 7) * 16;
    } else {
        const uint32_t r2 = lane >> 2, hi = (r2 >> 1) & 1, j4 = (r2 >> 2) & 1 ? 1 + hi : 3 * hi;
        o2 = (8 * j4 + 4 * (r2 >> 3) + 2 * (r2 & 1)) * (uint32_t)(EC * 2) + (lane & 3) * 16;
    }
    // copy i (0 .. 2 NI - 1) of chunk c into a slot
    auto copy = [&](int c, uint32_t slot, int i) {
        const uint32_t b = (uint32_t)(wv + NW * (i % NI));
        const uint32_t dst = lds0 + slot * CB + b * PITCH;
        if (i < NI) {
            const uint32_t j = (b & 8) ? (b & 7) + 4 : (b & 4) ? (b & 7) + 8 : (b & 7);
            const uint32_t row = (C == 512 ? 4 : 32) * (b >> 4) + 8 * (j >> 2) + (j & 3);
            dma16s_at(a.w1 + ((size_t)(c0 + c) * CHUNK + row) * C, o1, dst);
        } else {
            const uint32_t row = HS == 2 ? 32 * (b >> 2) + (b & 3) : 32 * (b >> 1) + (b & 1);
            dma16s_at(a.w2 + (size_t)(c0 + c) * CHUNK + (size_t)row * EC, o2, dst + CB / 2);
        }
    };
#pragma unroll
    for (int i = 0; i < 2 * NI; i++)
        copy(0, 0, i);

    // D fragments, row-major loads (four adjacent lanes on 64 contiguous
    // bytes), then each dword to its fragment lane
    const uint32_t p0 = blockIdx.x * (PG * 16 * NT) + pg * (16 * NT);
    u32x4 df[KS][NT];
    {
        const int lr = lane >> 2, lp = lane & 3, perm = (4 * jl + q) * 4;
#pragma unroll
        for (int t = 0; t < NT; t++) {
            const uint32_t p = min(p0 + 16 * t + lr, a.P - 1);
            const uint16_t *dp = a.y + (size_t)p * C + 8 * lp;
#pragma unroll
            for (int k = 0; k < KS; k++)
                df[k][t] = *reinterpret_cast<const u32x4 *>(dp + 32 * k);
        }
#pragma unroll
        for (int k = 0; k < KS; k++)
#pragma unroll
            for (int t = 0; t < NT; t++)
#pragma unroll
                for (int d = 0; d < 4; d++)
                    df[k][t][d] = (uint32_t)__builtin_amdgcn_ds_bpermute(perm, (int)df[k][t][d]);
    }
    // s1, b1; the fp16 GELU works on u / 4 (exact powers of two)
    constexpr float QS = T::is_bf16 ? 1.0f : 0.25f;
    float *s1l = reinterpret_cast<float *>(smem + 2 * CB), *b1l = s1l + a.per * CHUNK;
    for (int i = tid; i < nch * CHUNK; i += NW * 64) {
        s1l[i] = (a.s1 ? a.s1[c0 * CHUNK + i] : 1.0f) * QS;
        b1l[i] = (a.b1 ? a.b1[c0 * CHUNK + i] : 0.0f) * QS;
    }

    // fragment addresses (see the layout above)
    const uint32_t set = ((jl >> 2) ^ (jl >> 3)) & 1, rank = set ? jl - 4 : jl < 4 ? jl : jl - 8;
    const uint32_t f1 = (rank + 8 * set + (C == 256 ? 16 * hs : 0)) * PITCH + (C == 128 ? hs * (4u * C) : 0u) + 16 * q;
    const uint32_t f2 = CB / 2 + (HS == 2 ? (rank & 3) * PITCH + ((rank >> 2) + 2 * set) * 128
                                          : (rank & 1) * PITCH + ((rank >> 1) + 4 * set) * 64) +
                        (uint32_t)(4 * hs + q) * 16;
    constexpr uint32_t F1M = C == 512 ? 16 * PITCH : C * 2, F2O = (HS == 2 ? 4 : 2) * PITCH;  // steps of m and o
    float4v out[2 * OP][NT];
#pragma unroll
    for (int o = 0; o < 2 * OP; o++)
#pragma unroll
        for (int t = 0; t < NT; t++)
            out[o][t] = float4v{0.f, 0.f, 0.f, 0.f};
    // of the two waves of a SIMD one runs ahead, so that its activation falls
    // beside the other's products
    if (HS == 2 && hs == 0)
        __builtin_amdgcn_s_setprio(1);
    for (int c = 0; c < nch; c++) {
        copy_barrier();  // chunk c has landed; every wave is done with the other slot
        // the next chunk's copies go out one at a time beside the expand's
        // products: the memory unit takes tens of cycles for each, and a wave
        // that issues them in one burst stands until the last is taken (the
        // last chunk copies itself again, into the free slot)
        const int cn = c + 1 < nch ? c + 1 : c;
        const uint32_t so = (uint32_t)((c + 1) & 1);
        const uint8_t *slot = smem + (uint32_t)(c & 1) * CB;
        // Weight fragments f = 0 .. 2 KS - 1 (expand, K step f / 2, tile f % 2)
        // and 2 KS .. 2 KS + 2 OP - 1 (project), read PF ahead of their use
        constexpr int FE = 2 * KS, FT = FE + 2 * OP, PF = T::is_bf16 && C * NT == 512 && C < 512 ? 2 : 4;
        u32x4 wf[PF];
        auto frag = [&](int f) {
            const int o = f - FE;
            return *reinterpret_cast<const u32x4 *>(
                f < FE ? slot + f1 + (f & 1) * F1M + (f >> 1) * 64 : slot + f2 + (o >> 1) * F2O + (o & 1) * 512);
        };
#pragma unroll
        for (int f = 0; f < PF; f++)
            wf[f] = frag(f);
        const float *sv = s1l + CHUNK * c + 32 * hs + 8 * q, *bv = b1l + CHUNK * c + 32 * hs + 8 * q;
        float4v sc[2], bi[2];
#pragma unroll
        for (int mt = 0; mt < 2; mt++) {
            sc[mt] = *reinterpret_cast<const float4v *>(sv + 4 * mt);
            bi[mt] = *reinterpret_cast<const float4v *>(bv + 4 * mt);
        }
        float4v hid[2][NT];
#pragma unroll
        for (int mt = 0; mt < 2; mt++)
#pragma unroll
            for (int t = 0; t < NT; t++)
                hid[mt][t] = float4v{0.f, 0.f, 0.f, 0.f};
        __builtin_amdgcn_sched_group_barrier(0x100, PF + 4, 0);
#pragma unroll
        for (int f = 0; f < FE; f++) {
#pragma unroll
            for (int t = 0; t < NT; t++)
                hid[f & 1][t] = T::mfma(wf[f % PF], df[f >> 1][t], hid[f & 1][t]);
            wf[f % PF] = frag(f + PF);
            __builtin_amdgcn_sched_group_barrier(0x008, NT, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            if (f * 2 * NI / FE != (f + 1) * 2 * NI / FE)
#pragma unroll
                for (int i = f * 2 * NI / FE; i < (f + 1) * 2 * NI / FE; i++)
                    copy(cn, so, i);
        }
        u32x4 hb[NT];
        auto activate = [&](int t) {
#pragma unroll
            for (int mt = 0; mt < 2; mt++)
#pragma unroll
                for (int e = 0; e < 2; e++) {
                    float u0 = fmaf(hid[mt][t][2 * e], sc[mt][2 * e], bi[mt][2 * e]);
                    float u1 = fmaf(hid[mt][t][2 * e + 1], sc[mt][2 * e + 1], bi[mt][2 * e + 1]);
                    uint32_t v;
                    if constexpr (T::is_bf16) {
                        if constexpr (ACT == ACT_GELU) {
                            u0 = gelu_f32(u0);
                            u1 = gelu_f32(u1);
                        } else if constexpr (ACT == ACT_RELU) {
                            u0 = fmaxf(u0, 0.0f);
                            u1 = fmaxf(u1, 0.0f);
                        }
                        v = T::pack2(u0, u1);
                    } else {
                        if constexpr (ACT == ACT_GELU_F32) {
                            u0 = gelu_f32<4>(u0);
                            u1 = gelu_f32<4>(u1);
                        }
                        half2v h = __builtin_bit_cast(half2v, T::pack2(u0, u1));
                        if constexpr (ACT == ACT_GELU)
                            h = gelu_pk_f16_quarter(h);
                        else if constexpr (ACT == ACT_RELU)
                            h = __builtin_elementwise_max(h, splat2(0.0f));
                        v = __builtin_bit_cast(uint32_t, h);
                    }
                    hb[t][2 * mt + e] = v;
                }
        };
#pragma unroll
        for (int t = 0; t < NT; t++)
            activate(t);
#pragma unroll
        for (int f = FE; f < FT; f++) {
#pragma unroll
            for (int t = 0; t < NT; t++)
                out[f - FE][t] = T::mfma(wf[f % PF], hb[t], out[f - FE][t]);
            __builtin_amdgcn_sched_group_barrier(0x008, NT, 0);
            if (f + PF < FT) {
                wf[f % PF] = frag(f + PF);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
        }
    }
    __builtin_amdgcn_s_setprio(0);
    copy_barrier();
    // with HS = 2 each wave hands half of its output tiles to the other
    float4v *ex = reinterpret_cast<float4v *>(smem) + (size_t)(pg * 2) * (OP * NT * 64) + lane;
    auto give = [&](auto first) {
        constexpr int O0 = decltype(first)::value;
#pragma unroll
        for (int o = 0; o < OP; o++)
#pragma unroll
            for (int t = 0; t < NT; t++)
                ex[(size_t)(hs * OP * NT + o * NT + t) * 64] = out[O0 + o][t];
    };
    // NO output tiles from tile O0 on: the group's partial, or y
    auto take = [&](auto first, auto count) {
        constexpr int O0 = decltype(first)::value, NO = decltype(count)::value;
        constexpr float OS = T::is_bf16 ? 1.0f : 4.0f;
#pragma unroll
        for (int op = 0; op < NO / 2; op++) {
            const int ch = 16 * O0 + 32 * op + 8 * q;
            float4v sc[2], bi[2];
#pragma unroll
            for (int m = 0; m < 2; m++) {
                sc[m] = a.s2 ? *reinterpret_cast<const float4v *>(a.s2 + ch + 4 * m) * OS : float4v{OS, OS, OS, OS};
                bi[m] = a.b2 && !a.part ? *reinterpret_cast<const float4v *>(a.b2 + ch + 4 * m) : float4v{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int t = 0; t < NT; t++) {
                const uint32_t p = p0 + 16 * t + jl;
                if (p < a.P) {
                    float4v z[2];
#pragma unroll
                    for (int m = 0; m < 2; m++) {
                        z[m] = out[O0 + 2 * op + m][t];
                        if constexpr (HS == 2)
                            z[m] += ex[(size_t)((1 - hs) * OP * NT + (2 * op + m) * NT + t) * 64];
#pragma unroll
                        for (int e = 0; e < 4; e++)
                            z[m][e] = fmaf(z[m][e], sc[m][e], bi[m][e]);
                    }
                    const size_t at = (size_t)p * C + ch;
                    if (a.part) {
                        float *pp = a.part + (size_t)blockIdx.y * a.P * C + at;
                        *reinterpret_cast<float4v *>(pp) = z[0];
                        *reinterpret_cast<float4v *>(pp + 4) = z[1];
                    } else {
                        const u32x4 xv = *reinterpret_cast<const u32x4 *>(a.x + at);
                        u32x4 v;
#pragma unroll
                        for (int i = 0; i < 4; i++)
                            v[i] = T::pack2(T::lo(xv[i]) + z[i >> 1][2 * (i & 1)], T::hi(xv[i]) + z[i >> 1][2 * (i & 1) + 1]);
                        *reinterpret_cast<u32x4 *>(a.y + at) = v;
                    }
                }
            }
        }
    };
    using std::integral_constant;
    if constexpr (HS == 1) {
        take(integral_constant<int, 0>{}, integral_constant<int, 2 * OP>{});
    } else {
        if (hs == 0)
            give(integral_constant<int, OP>{});
        else
            give(integral_constant<int, 0>{});
        __syncthreads();
        if (hs == 0)
            take(integral_constant<int, 0>{}, integral_constant<int, OP>{});
        else
            take(integral_constant<int, OP>{}, integral_constant<int, OP>{});
    }
}

}  // namespace ffn
}  // namespace cf
