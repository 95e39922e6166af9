// cf_down.hip -- the 2x2 stride-2 down-sampling conv between stages: a matrix
// product Out[p][o] = sd[o] * sum_k A[p][k] * W[o][k] + bd[o] over K = 4 Cin.
//
// Output pixel (n, i, j) reads input pixels (2i, 2j), (2i, 2j + 1) and the two
// below them: in NHWC that is two runs of 2 Cin contiguous elements, so row p
// of A needs no gather beyond a start address, and since Cin is a multiple of
// 32 a K step of 64 stays within a run.
//
// A workgroup makes BM = 32 FM pixels x BN outputs; its waves are 2 pixel
// halves times BN / 32 shares of the outputs.  Both operands come by
// LDS-DMA into a ring of three slots of one K step each, two steps ahead: the
// launch is short (K / 64 = 4 to 16 steps, one to three tiles per CU) and what
// bounds it is the latency of the loads, not their number.  Products are
// v_mfma_f32_16x16x32 with weights as the A operand and pixels as B; W's rows
// are dealt to tiles so that a lane ends up with eight consecutive outputs of
// a pixel, one 16-byte store.
//
// LDS layout (both operands): a copy instruction moves 8 row segments of 128
// bytes; 32 rows are four such kilobytes, PITCH apart.  Row j of tile m of the
// 32, with rank its place (0-7) within S0 = {0-3, 12-15} or S1 = {4-11}, lies in
// kilobyte rank % 4 at segment rank / 4 + 2 (j in S1) + 4 m: a 16-byte read
// serves S0 of one K quarter together with S1 of its neighbour, and this way
// they meet in no bank.
#include "cf_device.h"
#include "cf_kernels.h"

namespace cf {
namespace down {

struct Args {
    const uint16_t *x, *w;
    uint16_t *y;
    const float *scale, *bias;
    uint32_t P;           // output pixels, < 2^31
    uint32_t tiles;       // pixel tiles of the whole call
    uint32_t first;       // this launch's first eight of them
    int Wo, Cin, NO;
    FastDiv divWo, divNy;
};

constexpr uint32_t PITCH = 1056;
constexpr int GK = 64;
constexpr int S = 3;  // slots of the ring: two steps of copies under way while one is used
constexpr uint32_t slot_bytes(int BM, int BN) { return (uint32_t)(BM + BN) / 8 * PITCH; }

__device__ __forceinline__ void dma16(const uint16_t *src, uint32_t lds_addr) {
    const uint32_t lds = (uint32_t)__builtin_amdgcn_readfirstlane(lds_addr);
    uint32_t saved;
    asm volatile(
        "s_mov_b32 %0, m0\n\t"
        "s_mov_b32 m0, %2\n\t"
        "s_nop 0\n\t"
        "global_load_lds_dwordx4 %1, off\n\t"
        "s_mov_b32 m0, %0"
        : "=&s"(saved)
        : "v"(src), "s"(lds)
        : "memory");
}

// Wait until at most N of this wave's copies are under way, then the barrier.
template <int N>
__device__ __forceinline__ void copies_barrier() {
    static_assert(N < 64, "vmcnt");
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));  // and lgkmcnt 0
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

template <typename T, int FM, int BN>
__global__ __launch_bounds__(BN / 16 * 64) void down_kernel(Args a) {
    extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
    constexpr int BM = 32 * FM, NW = BN / 16;
    constexpr int CA = BM / 8, CW = BN / 8;                       // copies of a step
    constexpr int NA = (CA + NW - 1) / NW, NB = CW / NW, NC = NA + NB;  // per wave
    static_assert(CW % NW == 0 && (CA % NW == 0 || NW % CA == 0), "every wave makes as many copies");
    constexpr uint32_t SLOT = slot_bytes(BM, BN), OFFW = (uint32_t)CA * PITCH;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wv & 1, wn = wv >> 1;
    const int q = lane >> 4, jl = lane & 15;
    // the output tiles of one pixel tile follow each other on one XCD
    const uint32_t xcd = blockIdx.x & 7, s8 = blockIdx.x >> 3, pt8 = fdiv(s8, a.divNy);
    const uint32_t pt = (a.first + pt8) * 8 + xcd;
    if (pt >= a.tiles)
        return;
    const uint32_t p0 = pt * BM;
    const int o0 = (int)(s8 - pt8 * a.divNy.d) * BN;
    const int K = 4 * a.Cin, nk = K / GK, half = nk / 2;
    const size_t below = (size_t)(2 * a.Wo - 2) * a.Cin;  // from the end of one run to the start of the next
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t *)smem;

    // sources of this wave's copies; the lane's row of a kilobyte
    const uint16_t *sa[NA], *sw[NB];
    {
        const int r2 = lane >> 3, set = (r2 >> 1) & 1, m = r2 >> 2;
        auto row_j = [&](int kb) {
            const int rank = kb + 4 * (r2 & 1);
            return set ? rank + 4 : rank < 4 ? rank : rank + 8;
        };
#pragma unroll
        for (int i = 0; i < NA; i++) {
            const int b = (wv + NW * i) % CA;
            const uint32_t p = min(p0 + (uint32_t)(32 * (b >> 2) + 16 * m + row_j(b & 3)), a.P - 1);
            const uint32_t ni = fdiv(p, a.divWo), j = p - ni * (uint32_t)a.Wo;
            sa[i] = a.x + ((size_t)ni * 4 * a.Wo + 2 * j) * a.Cin + (lane & 7) * 8;
        }
#pragma unroll
        for (int i = 0; i < NB; i++) {
            const int b = wv + NW * i, j = row_j(b & 3);
            sw[i] = a.w + (size_t)(o0 + 32 * (b >> 2) + 8 * (j >> 2) + 4 * m + (j & 3)) * K + (lane & 7) * 8;
        }
    }
    uint32_t fill = 0;  // slot of the next step to be copied
    auto copy = [&](int kt) {
        const size_t ka = (size_t)kt * GK + (kt >= half ? below : 0);
#pragma unroll
        for (int i = 0; i < NA; i++)
            dma16(sa[i] + ka, lds0 + fill + (uint32_t)((wv + NW * i) % CA) * PITCH);
#pragma unroll
        for (int i = 0; i < NB; i++)
            dma16(sw[i] + kt * GK, lds0 + fill + OFFW + (uint32_t)(wv + NW * i) * PITCH);
        fill = fill + SLOT == S * SLOT ? 0 : fill + SLOT;
    };
    for (int kt = 0; kt < S - 1 && kt < nk; kt++)
        copy(kt);

    const uint32_t set = ((jl >> 2) ^ (jl >> 3)) & 1, rank = set ? jl - 4 : jl < 4 ? jl : jl - 8;
    const uint32_t f0 = (rank & 3) * PITCH + ((rank >> 2) + 2 * set) * 128 + 16 * q;
    float4v acc[2][FM];
#pragma unroll
    for (int o = 0; o < 2; o++)
#pragma unroll
        for (int t = 0; t < FM; t++)
            acc[o][t] = float4v{0.f, 0.f, 0.f, 0.f};
    uint32_t use = 0;
    for (int kt = 0; kt < nk; kt++) {
        // step kt has landed, and every wave is done with the slot of step kt - 1
        if (kt + 1 < nk)
            copies_barrier<NC>();
        else
            copies_barrier<0>();
        if (kt + S - 1 < nk)
            copy(kt + S - 1);
        const uint8_t *slot = smem + use + f0;
#pragma unroll
        for (int ks = 0; ks < GK / 32; ks++) {
            u32x4 fw[2], fa[FM];
#pragma unroll
            for (int o = 0; o < 2; o++)
                fw[o] = *reinterpret_cast<const u32x4 *>(slot + OFFW + (uint32_t)(4 * wn) * PITCH + o * 512 + 64 * ks);
#pragma unroll
            for (int t = 0; t < FM; t++) {
                const int r = wm * FM + t;
                fa[t] = *reinterpret_cast<const u32x4 *>(slot + (uint32_t)(4 * (r >> 1)) * PITCH + (r & 1) * 512 + 64 * ks);
            }
#pragma unroll
            for (int o = 0; o < 2; o++)
#pragma unroll
                for (int t = 0; t < FM; t++)
                    acc[o][t] = T::mfma(fw[o], fa[t], acc[o][t]);
        }
        use = use + SLOT == S * SLOT ? 0 : use + SLOT;
    }
    const int o = o0 + 32 * wn + 8 * q;
    float4v sc[2], bi[2];
#pragma unroll
    for (int m = 0; m < 2; m++) {
        sc[m] = a.scale ? *reinterpret_cast<const float4v *>(a.scale + o + 4 * m) : float4v{1.f, 1.f, 1.f, 1.f};
        bi[m] = a.bias ? *reinterpret_cast<const float4v *>(a.bias + o + 4 * m) : float4v{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int t = 0; t < FM; t++) {
        const uint32_t p = p0 + 16 * (wm * FM + t) + jl;
        if (p >= a.P)
            continue;
        u32x4 v;
#pragma unroll
        for (int i = 0; i < 4; i++) {
            const int m = i >> 1, e = 2 * (i & 1);
            v[i] = T::pack2(fmaf(acc[m][t][e], sc[m][e], bi[m][e]), fmaf(acc[m][t][e + 1], sc[m][e + 1], bi[m][e + 1]));
        }
        *reinterpret_cast<u32x4 *>(a.y + (size_t)p * a.NO + o) = v;
    }
}

template <typename T, int FM, int BN>
hipError_t go(Args a, hipStream_t st) {
    const void *k = (const void *)down_kernel<T, FM, BN>;
    hipError_t e = allow_full_lds(k);
    if (e != hipSuccess)
        return e;
    a.tiles = (a.P + 32 * FM - 1) / (32 * FM);
    const uint32_t ny = (uint32_t)(a.NO / BN), threads = BN / 16 * 64;
    a.divNy = make_fastdiv(ny);
    // a launch holds below 2^32 threads: eights of pixel tiles, in as many
    // launches as that takes
    const uint32_t eights = (a.tiles + 7) / 8;
    const uint32_t most = (uint32_t)((((uint64_t)1 << 32) - 1) / ((uint64_t)8 * ny * threads));
    if (most == 0)
        return hipErrorInvalidValue;
    for (a.first = 0; a.first < eights; a.first += most) {
        const uint32_t n = eights - a.first < most ? eights - a.first : most;
        void *args[] = {&a};
        e = hipLaunchKernel(k, dim3(n * 8 * ny), dim3(threads), args, S * slot_bytes(32 * FM, BN), st);
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

// Tiles of 64 pixels x 128 outputs, two workgroups of eight waves a CU, once
// they cover three quarters of the CUs; below that 32 x 64, four waves, for
// the shortest chain per workgroup.  In us, 64 x 128 against 32 x 64, and the
// register-staged kernel that both replaced: 128 images of 56 x 56 x 64 -> 128
// 18.1 / 22.7 / 28.9 (15.1 for its bytes at the copy rate), 28 x 28 x 128 ->
// 256 15.1 / 17.8 / 24.5, 14 x 14 x 256 -> 512 12.1 / 16.5 / 20.9; 32 images
// 5.9 / 6.9 / 9.5, 5.7 / 6.5 / 10.1, 8.2 / 6.5 / 14.6; 4 images 4.0 / 3.1 / 6.8,
// 5.3 / 3.9 / 9.3, 7.8 / 5.5 / 14.3.  128 x 128 24.0 / 15.9 / 12.7 for
// the first three; what is left of the larger ones is the 28 bytes a clock and
// CU that the copies bring from L2.  Outputs that are no multiple of 128 take
// 128 x 64 tiles instead (20.6 us for the first).
template <typename T>
hipError_t launch(const Args &a, hipStream_t st) {
    const int64_t tiles = (((int64_t)a.P + 63) / 64) * ((a.NO + 127) / 128);
    if (tiles * 4 < 3 * (int64_t)device_cu_count())
        return go<T, 1, 64>(a, st);
    return a.NO % 128 == 0 ? go<T, 2, 128>(a, st) : go<T, 4, 64>(a, st);
}

}  // namespace down

hipError_t launch_downsample(const void *x, void *y, const void *wd, const float *sd, const float *bd, int N, int H,
                             int W, int Cin, int Cout, int bf16, hipStream_t st) {
    down::Args a{};
    a.x = (const uint16_t *)x;
    a.w = (const uint16_t *)wd;
    a.y = (uint16_t *)y;
    a.scale = sd;
    a.bias = bd;
    a.Wo = W / 2;
    a.Cin = Cin;
    a.NO = Cout;
    const int64_t P = (int64_t)N * (H / 2) * a.Wo;
    if (P >= ((int64_t)1 << 31))
        return hipErrorInvalidValue;
    a.P = (uint32_t)P;
    a.divWo = make_fastdiv((uint32_t)a.Wo);
    return bf16 ? down::launch<BF16>(a, st) : down::launch<F16>(a, st);
}

}  // namespace cf
