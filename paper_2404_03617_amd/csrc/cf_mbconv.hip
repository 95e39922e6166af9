// cf_mbconv.hip -- block fusion of the paper's MBConv block with Squeeze &
// Excitation (Sec. 5.4 of Lavin, arXiv:2404.03617; the kernel of Sec. 5.4.1,
// Fig. f:mbconv-block-fusion-tensor-machine):
//   U = SiLU(s1 (X W1^T) + b1)                     expand to E*C hidden channels
//   V = SiLU(s2 gconv3x3(U) + b2)                  grouped conv, group width 8
//   g = sigmoid(We ReLU(Wr mean_hw(V) + br) + be)  squeeze & excitation
//   Y = X + s3 (W2 diag(g) V) + b3                 project, residual
//
// The squeeze is the one point where the whole image meets, so the block is
// cut there into two launches; U never leaves the chip, V crosses once.
//
// expand_conv_kernel, one workgroup per image and group of 64 hidden channels
// (as in the paper, expand and conv of a group need no other work item):
//  1. expand: the group's 64 rows of W1 (in LDS) against every pixel of the
//     image (v_mfma_f32_16x16x32, x read straight from global memory as B
//     fragments, the next batch of K steps in flight), SiLU in fp32, rounded
//     into an LDS buffer U with a zero border;
//  2. grouped conv (8 groups of 8, two per wave) as one product per tap
//     column: 16 columns x 2 output rows against K = 4 halo rows x 8 channels,
//     the next row pair's halo read ahead; SiLU; V overwrites the wave's own
//     channels of U one row and one column up, where no later row pair reads;
//  3. V (stride 2: its BlurPool) leaves LDS in whole 128-byte lines, its fp32
//     channel sums give the group's share of the squeeze, Wr[:, group] . mean.
// gate_project_kernel, one workgroup per 64 output pixels and up to 256 output
// channels:
//  4. the squeeze (shares added in group order), ReLU, excitation, sigmoid;
//  5. the projection over all E*C channels: V times the gates staged in LDS
//     256 channels at a time (two buffers, the next chunk's V in flight in
//     registers), W2 fragments straight from global memory two batches ahead,
//     each serving the tile's four 16-pixel columns; then s3, b3 and the
//     residual, and y is written once.
// Every sum has a fixed order that does not depend on how many images a
// launch holds, so results are deterministic and independent of the workspace
// size.  A pixel's x is read for the residual by the lane that writes it and
// every other read of x happens in the launch before, so y may be x itself.
//
// Bounds: the 2 * P * E*C SiLUs on the VALU (an exponential and a reciprocal
// each) for the first kernel, at three workgroups per CU; the chain of loads
// per workgroup (squeeze, gates, V, W2) for the second, two per CU.  N = 128,
// 16 x 16, C = 192, E = 4, fp16: 44 + 30 us (the pair 68 us, launched back to
// back), where one cooperative kernel with a barrier per image took 227 us:
// the barrier tied each image's work items to a chain of global round trips,
// four images deep, and the cooperative launch alone cost 17 us.
//
// Images up to 16 x 16 (the late-stage shapes the paper targets); C a
// multiple of 16; E*C a multiple of 64 and at most 4096; 1 <= R <= 256; C up
// to 768 at E = 2, 512 at E = 4, 256 at E = 8 (layout_bytes).
#include "cf_device.h"
#include "cf_kernels.h"


namespace cf {
namespace mbc {

constexpr int GH = 64;            // hidden channels per expand_conv workgroup
constexpr int HMAX = 16, WMAX = 16;
constexpr int UC = WMAX + 2;      // columns of the U buffer (zero border)
constexpr int PB = 2 * GH + 16;   // LDS bytes per pixel: an odd multiple of 16, conflict-free 16-B reads
constexpr int RMAX = 256;
constexpr int ECMAX = 4096;
constexpr int SLOTMAX = 2048;     // lines of the workspace header (reserved, stays zero)
constexpr int NT = 256;           // threads of both kernels: four waves
constexpr int TP = 64;            // output pixels per gate_project workgroup
constexpr int KC = 256;           // hidden channels per staged chunk of V
constexpr int VP = 2 * KC + 16;   // LDS bytes per staged pixel: an odd multiple of 16

struct Args {
    const uint16_t *x;
    uint16_t *y;
    const uint16_t *w1;            // [EC][C]
    const float *s1, *b1;
    const uint16_t *gw;            // [3][3][EC][8]
    const float *s2, *b2;
    const uint16_t *wr;            // [R][EC]
    const float *br;
    const uint16_t *we;            // [EC][R]
    const float *be;
    const uint16_t *w2;            // [K][EC]
    const float *s3, *b3;
    float *sq;                     // [N][G][R] squeeze shares
    uint16_t *vx;                  // [images of the launch][Po][EC] conv output (stride 2: after BlurPool)
    int H, W, C, EC, R, G;
    int K, Ho, Wo;                 // output channels and size (stride 1: C, H, W)
    int n0;                        // first image of the launch
    int tiles;                     // 64-pixel tiles per image
    uint32_t off_vec, off_part;    // LDS layout of expand_conv (W1, then U at 0)
    FastDiv dw, dwo, dg, dt;       // by W, Wo, G, tiles
};

__device__ __forceinline__ u32x4 ld16(const void *p) { return *reinterpret_cast<const u32x4 *>(p); }

__device__ __forceinline__ float silu_f32(float u) { return u * __builtin_amdgcn_rcpf(1.0f + __expf(-u)); }
__device__ __forceinline__ float sigmoid_f32(float u) { return __builtin_amdgcn_rcpf(1.0f + __expf(-u)); }

// Fragments read straight from global memory (x in the expand, W2 in the
// projection) are loaded with four adjacent lanes on 64 contiguous bytes of
// one row (lane l: row l / 4, piece l % 4) -- the memory unit merges only
// adjacent lanes, and in fragment order every lane would start a row of its
// own -- and each dword then moves to its fragment lane (q, jl), which takes
// row jl, piece q from lane 4 jl + q.
__device__ __forceinline__ u32x4 permute(int perm, const u32x4 &v) {
    u32x4 o;
#pragma unroll
    for (int d = 0; d < 4; d++)
        o[d] = (uint32_t)__builtin_amdgcn_ds_bpermute(perm, (int)v[d]);
    return o;
}

// Workgroup i runs on XCD i % 8: consecutive work items (an image's groups or
// tiles, which read the same x, W2 or V) share an XCD and its L2.
__device__ __forceinline__ uint32_t xcd_order() {
    const uint32_t m = gridDim.x, b = blockIdx.x;
    return m % 8 == 0 ? (b % 8) * (m / 8) + b / 8 : b;
}

template <typename T, int NPW, bool S2>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(3))) void expand_conv_kernel(Args a) {
    extern __shared__ __attribute__((aligned(256))) uint8_t smem[];
    constexpr int NWV = 4, NGG = 2;  // waves; 8-channel conv groups per wave
    constexpr int KE = NPW == 4 ? 1 : 2;  // expand K steps per load batch (two batches in flight)
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4, jl = lane & 15;
    const int lr = lane >> 2, lp = lane & 3;
    const int perm = (4 * jl + q) * 4;  // ds_bpermute source address
    const uint32_t lin = xcd_order();
    const int nl = (int)fdiv(lin, a.dg), g = (int)lin - nl * a.G, n = a.n0 + nl;
    const int C = a.C, EC = a.EC, R = a.R;
    const int P = a.H * a.W, Po = S2 ? a.Ho * a.Wo : P;
    const int RP = (a.H + 1) / 2;
    const int h0 = g * GH;  // first hidden channel of the group
    uint8_t *U = smem;
    float *s1l = reinterpret_cast<float *>(smem + a.off_vec);  // s1, b1, s2, b2, channel sums [64] each
    float *b1l = s1l + 64, *s2l = s1l + 128, *b2l = s1l + 192, *csum = s1l + 256;
    const uint16_t *xn = a.x + (size_t)n * P * C;
    const int ks = (C + 31) / 32, nbat = (ks + KE - 1) / KE;

    // x fragments of a batch, addresses clamped into the image (columns past
    // the last pixel are computed and never stored; K slices past C are
    // zeroed before use)
    const uint16_t *xp[NPW];
#pragma unroll
    for (int i = 0; i < NPW; i++)
        xp[i] = xn + (size_t)min(16 * (wv + NWV * i) + lr, P - 1) * C;
    auto loadb = [&](int b, u32x4 (&v)[KE][NPW]) {
#pragma unroll
        for (int j = 0; j < KE; j++) {
            const int k = min(32 * (KE * b + j) + 8 * lp, C - 8);
#pragma unroll
            for (int i = 0; i < NPW; i++)
                v[j][i] = ld16(xp[i] + k);
        }
    };
    u32x4 xA[KE][NPW], xB[KE][NPW];
    loadb(0, xA);

    if (tid < 64) {
        s1l[tid] = a.s1 ? a.s1[h0 + tid] : 1.0f;
        b1l[tid] = a.b1 ? a.b1[h0 + tid] : 0.0f;
        s2l[tid] = a.s2 ? a.s2[h0 + tid] : 1.0f;
        b2l[tid] = a.b2 ? a.b2[h0 + tid] : 0.0f;
    }
    // the group's 64 rows of W1 (pitch 2C + 16 bytes: an odd multiple of 16,
    // conflict-free fragment reads), over the bytes that U takes later: four
    // threads per row, eight loads of each in flight
    const uint32_t w1p = 2 * C + 16;
    uint8_t *w1l = smem;
    {
        const int row = tid >> 2, nc = C / 8;
        const uint16_t *src = a.w1 + (size_t)(h0 + row) * C;
        uint8_t *dst = w1l + (uint32_t)row * w1p;
        for (int c0 = tid & 3; c0 < nc; c0 += 32) {
            u32x4 v[8];
#pragma unroll
            for (int i = 0; i < 8; i++)
                v[i] = ld16(src + 8 * min(c0 + 4 * i, nc - 1));
#pragma unroll
            for (int i = 0; i < 8; i++)
                if (c0 + 4 * i < nc)
                    *reinterpret_cast<u32x4 *>(dst + (uint32_t)(c0 + 4 * i) * 16) = v[i];
        }
    }
    __syncthreads();

    // ---- 1. expand + SiLU into U; wave wv takes the 16-pixel tiles wv + NWV i
    u32x4 cav[NGG][3];
    bool tap_ok;
    {
        float4v acc[4][NPW];
#pragma unroll
        for (int mt = 0; mt < 4; mt++)
#pragma unroll
            for (int i = 0; i < NPW; i++)
                acc[mt][i] = float4v{0.f, 0.f, 0.f, 0.f};
        auto mmab = [&](int b, const u32x4 (&v)[KE][NPW]) {
#pragma unroll
            for (int j = 0; j < KE; j++) {
                const int kk = KE * b + j;
                if (kk >= ks)  // wave-uniform
                    break;
                const int k = 32 * kk + 8 * q;
                const bool in = k < C;  // false only in the half-padded last step
                u32x4 bv[NPW];
#pragma unroll
                for (int i = 0; i < NPW; i++) {
                    bv[i] = permute(perm, v[j][i]);
#pragma unroll
                    for (int d = 0; d < 4; d++)
                        bv[i][d] = in ? bv[i][d] : 0u;
                }
#pragma unroll
                for (int mt = 0; mt < 4; mt++) {
                    u32x4 av = *reinterpret_cast<const u32x4 *>(w1l + (uint32_t)(16 * mt + jl) * w1p +
                                                                (uint32_t)(in ? k : 0) * 2);
#pragma unroll
                    for (int i = 0; i < NPW; i++)
                        acc[mt][i] = T::mfma(av, bv[i], acc[mt][i]);
                }
            }
        };
        for (int b = 0; b < nbat; b += 2) {
            if (b + 1 < nbat)
                loadb(b + 1, xB);
            mmab(b, xA);
            if (b + 1 < nbat) {
                if (b + 2 < nbat)
                    loadb(b + 2, xA);
                mmab(b + 1, xB);
            }
        }
        // the conv taps of this wave's 8-channel groups, to registers
        const int cs = jl >> 3, co = jl & 7;
        const int ti = q - cs;  // the tap row this lane's K slice meets
        tap_ok = ti >= 0 && ti <= 2;
        const uint16_t *tp = a.gw + ((size_t)(tap_ok ? ti : 0) * 3 * EC + h0 + 8 * wv + co) * 8;
#pragma unroll
        for (int j = 0; j < NGG; j++)
#pragma unroll
            for (int dj = 0; dj < 3; dj++)
                cav[j][dj] = ld16(tp + ((size_t)dj * EC + 8 * NWV * j) * 8);
        __syncthreads();  // every wave has read its W1 fragments
        // the U border (row 0, rows past H, column 0, columns past W) is zero
        {
            const int cells = (2 * RP + 2) * UC;
            for (int i = tid; i < cells; i += NT) {
                const int row = i / UC, col = i - row * UC;
                if (row == 0 || row > a.H || col == 0 || col > a.W)
#pragma unroll
                    for (int c = 0; c < 8; c++)
                        *reinterpret_cast<u32x4 *>(U + (uint32_t)i * PB + 16 * c) = u32x4{0u, 0u, 0u, 0u};
            }
        }
#pragma unroll
        for (int i = 0; i < NPW; i++) {
            const int p = 16 * (wv + NWV * i) + jl;
            const int r = (int)fdiv((uint32_t)p, a.dw), c = p - r * a.W;
            uint8_t *cell = U + (uint32_t)((r + 1) * UC + c + 1) * PB;
            if (p < P) {
#pragma unroll
                for (int mt = 0; mt < 4; mt++) {
                    const int hl = 16 * mt + 4 * q;  // local hidden channels hl .. hl+3 of this lane
                    const float4v sc = *reinterpret_cast<const float4v *>(s1l + hl);
                    const float4v bi = *reinterpret_cast<const float4v *>(b1l + hl);
                    float u[4];
#pragma unroll
                    for (int e = 0; e < 4; e++)
                        u[e] = silu_f32(fmaf(acc[mt][i][e], sc[e], bi[e]));
                    *reinterpret_cast<u32x2 *>(cell + (uint32_t)hl * 2) =
                        u32x2{T::pack2(u[0], u[1]), T::pack2(u[2], u[3])};
                }
            }
        }
    }
    __syncthreads();
    // the squeeze weights of the group, needed last
    Pack8 wr[GH / 8];
#pragma unroll
    for (int c = 0; c < GH / 8; c++)
        wr[c].u = ld16(a.wr + (size_t)min(tid, R - 1) * EC + h0 + 8 * c);
#pragma unroll
    for (int j = 0; j < NGG; j++)
#pragma unroll
        for (int dj = 0; dj < 3; dj++)
#pragma unroll
            for (int d = 0; d < 4; d++)
                cav[j][dj][d] = tap_ok ? cav[j][dj][d] : 0u;

    // ---- 2. grouped conv + SiLU, V into U.  A rows (s, o): output row 2rp+s,
    //      channel o of the 8-group; K (t, j): halo row 2rp+t, input channel j.
    //      V of pixel (r, c) goes to cell (r, c), one row and column above the
    //      pixel's U: row pair rp writes rows 2rp, 2rp+1 of its own channels,
    //      and later row pairs read from row 2rp+2 on.
    {
        float4v sc[NGG], bi[NGG];
        float sum[NGG][4];
        uint32_t gb[NGG];
#pragma unroll
        for (int j = 0; j < NGG; j++) {
            const int hl = 8 * (wv + NWV * j) + 4 * (q & 1);  // output channels of this lane's D rows
            sc[j] = *reinterpret_cast<const float4v *>(s2l + hl);
            bi[j] = *reinterpret_cast<const float4v *>(b2l + hl);
            gb[j] = (uint32_t)(wv + NWV * j) * 16;
#pragma unroll
            for (int e = 0; e < 4; e++)
                sum[j][e] = 0.0f;
        }
        const uint8_t *hb = U + (uint32_t)(q * UC + jl) * PB;
        uint8_t *ob = U + (uint32_t)((q >> 1) * UC + jl) * PB + (uint32_t)(q & 1) * 8;
        u32x4 bv[NGG][3];
        auto halo = [&](int rp) {
#pragma unroll
            for (int j = 0; j < NGG; j++)
#pragma unroll
                for (int dj = 0; dj < 3; dj++)
                    bv[j][dj] = *reinterpret_cast<const u32x4 *>(hb + (uint32_t)(2 * rp * UC + dj) * PB + gb[j]);
        };
        halo(0);
        for (int rp = 0; rp < RP; rp++) {
            float4v acc[NGG];
#pragma unroll
            for (int j = 0; j < NGG; j++)
                acc[j] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int dj = 0; dj < 3; dj++)
#pragma unroll
                for (int j = 0; j < NGG; j++)
                    acc[j] = T::mfma(cav[j][dj], bv[j][dj], acc[j]);
            if (rp + 1 < RP)
                halo(rp + 1);
            if (2 * rp + (q >> 1) < a.H && jl < a.W) {
#pragma unroll
                for (int j = 0; j < NGG; j++) {
                    float u[4];
#pragma unroll
                    for (int e = 0; e < 4; e++) {
                        u[e] = silu_f32(fmaf(acc[j][e], sc[j][e], bi[j][e]));
                        sum[j][e] += u[e];
                    }
                    *reinterpret_cast<u32x2 *>(ob + (uint32_t)(2 * rp * UC) * PB + gb[j]) =
                        u32x2{T::pack2(u[0], u[1]), T::pack2(u[2], u[3])};
                }
            }
        }
        if constexpr (!S2) {
            // sum over the 16 columns (lane bits 0-3) and the two rows of a
            // pair (lane bit 5); lanes 0 and 16 hold channels hl .. hl+3
#pragma unroll
            for (int j = 0; j < NGG; j++) {
#pragma unroll
                for (int e = 0; e < 4; e++) {
#pragma unroll
                    for (int m = 1; m <= 8; m <<= 1)
                        sum[j][e] += __shfl_xor(sum[j][e], m);
                    sum[j][e] += __shfl_xor(sum[j][e], 32);
                }
                if (jl == 0 && q < 2)
#pragma unroll
                    for (int e = 0; e < 4; e++)
                        csum[8 * (wv + NWV * j) + 4 * q + e] = sum[j][e];
            }
        }
    }
    __syncthreads();

    // ---- 3. V to global memory, 128 contiguous bytes per pixel
    uint16_t *vx = a.vx + (size_t)nl * Po * EC + h0;
    if constexpr (!S2) {
        for (int idx = tid; idx < P * 8; idx += NT) {
            const int p = idx >> 3, c8 = idx & 7;
            const int r = (int)fdiv((uint32_t)p, a.dw), c = p - r * a.W;
            *reinterpret_cast<u32x4 *>(vx + (size_t)p * EC + 8 * c8) =
                *reinterpret_cast<const u32x4 *>(U + (uint32_t)(r * UC + c) * PB + 16 * c8);
        }
    } else {
        // BlurPool (Triangle-3 taps [1, 2, 1] / 4 in each direction, one pixel
        // of reflect padding, stride 2), rounded once; the channel sums of
        // the blurred map (fp32, before rounding) per thread over its pixels,
        // then over the threads in order
        float *part = reinterpret_cast<float *>(smem + a.off_part);  // [NT / 16][64]
        constexpr int NPG = NT / 16;
        const int c4 = tid & 15, pg = tid >> 4;  // channels 4 c4 .. 4 c4 + 3
        const uint8_t *vb = U + (uint32_t)c4 * 8;
        float s4[4] = {0.f, 0.f, 0.f, 0.f};
        for (int pp = pg; pp < Po; pp += NPG) {
            const int i = (int)fdiv((uint32_t)pp, a.dwo), j = pp - i * a.Wo;
            float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int ta = 0; ta < 3; ta++) {
                int r = 2 * i + ta - 1;
                r = r < 0 ? -r : (r >= a.H ? 2 * (a.H - 1) - r : r);
#pragma unroll
                for (int tb = 0; tb < 3; tb++) {
                    int c = 2 * j + tb - 1;
                    c = c < 0 ? -c : (c >= a.W ? 2 * (a.W - 1) - c : c);
                    const float wt = (ta == 1 ? 0.5f : 0.25f) * (tb == 1 ? 0.5f : 0.25f);
                    const u32x2 v = *reinterpret_cast<const u32x2 *>(vb + (uint32_t)(r * UC + c) * PB);
                    acc[0] = fmaf(wt, T::lo(v[0]), acc[0]);
                    acc[1] = fmaf(wt, T::hi(v[0]), acc[1]);
                    acc[2] = fmaf(wt, T::lo(v[1]), acc[2]);
                    acc[3] = fmaf(wt, T::hi(v[1]), acc[3]);
                }
            }
#pragma unroll
            for (int e = 0; e < 4; e++)
                s4[e] += acc[e];
            *reinterpret_cast<u32x2 *>(vx + (size_t)pp * EC + 4 * c4) =
                u32x2{T::pack2(acc[0], acc[1]), T::pack2(acc[2], acc[3])};
        }
#pragma unroll
        for (int e = 0; e < 4; e++)
            part[pg * 64 + 4 * c4 + e] = s4[e];
        __syncthreads();
        if (tid < 64) {
            float sm = 0.0f;
#pragma unroll
            for (int g2 = 0; g2 < NPG; g2++)
                sm += part[g2 * 64 + tid];
            csum[tid] = sm;
        }
        __syncthreads();
    }
    // the group's share of the squeeze: Wr[:, group] . mean(V)
    if (tid < R) {
        const float inv = 1.0f / (float)Po;
        float s = 0.0f;
#pragma unroll
        for (int c = 0; c < GH / 8; c++)
#pragma unroll
            for (int e = 0; e < 4; e++)
                s += T::lo(wr[c].w[e]) * csum[8 * c + 2 * e] + T::hi(wr[c].w[e]) * csum[8 * c + 2 * e + 1];
        a.sq[((size_t)n * a.G + g) * R + tid] = s * inv;
    }
}

// OTW: 16-channel output tiles per wave; blockIdx.y takes 4 OTW tiles.
template <typename T, int OTW, bool S2>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(2))) void gate_project_kernel(Args a) {
    extern __shared__ __attribute__((aligned(256))) uint8_t smem[];
    constexpr int KB = 2;  // K steps per W2 batch, two batches in flight
    const int tid = threadIdx.x, lane = tid & 63;
    const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4, jl = lane & 15;
    const int lr = lane >> 2, lp = lane & 3;
    const int perm = (4 * jl + q) * 4;
    const uint32_t lin = xcd_order();
    const int nl = (int)fdiv(lin, a.dt), tile = (int)lin - nl * a.tiles, n = a.n0 + nl;
    const int EC = a.EC, R = a.R, KO = a.K, OT = KO / 16;
    const int Po = a.Ho * a.Wo;
    const int ot0 = blockIdx.y * 4 * OTW + wv;  // this wave's tiles: ot0 + 4 i
    float *gate = reinterpret_cast<float *>(smem + 2 * TP * VP);  // [EC]
    float *zl = gate + EC;                                       // [R]
    const int nch = (EC + KC - 1) / KC, nbat = EC / (32 * KB);

    // V of a chunk: 64 pixels x 32 pieces of 16 bytes, eight per thread
    // (addresses clamped into the image and the row; what lies past them is
    // not read from LDS, or is a column that is not stored)
    const int vrow = tid >> 5, vc = tid & 31;
    const uint16_t *vbase = a.vx + (size_t)nl * Po * EC;
    u32x4 vr[8];
    auto loadv = [&](int c) {
        const int k = min(KC * c + 8 * vc, EC - 8);
#pragma unroll
        for (int i = 0; i < 8; i++)
            vr[i] = ld16(vbase + (size_t)min(TP * tile + vrow + 8 * i, Po - 1) * EC + k);
    };
    const uint16_t *wp[OTW];
#pragma unroll
    for (int i = 0; i < OTW; i++)
        wp[i] = a.w2 + (size_t)(16 * min(ot0 + 4 * i, OT - 1) + lr) * EC + 8 * lp;
    auto loadw = [&](int b, u32x4 (&w)[KB][OTW]) {
        const int bb = min(b, nbat - 1);
#pragma unroll
        for (int j = 0; j < KB; j++)
#pragma unroll
            for (int i = 0; i < OTW; i++)
                w[j][i] = ld16(wp[i] + 32 * (KB * bb + j));
    };
    u32x4 w[2][KB][OTW];
    loadv(0);
    loadw(0, w[0]);
    loadw(1, w[1]);

    // ---- 4. squeeze (shares in group order), excitation, gates of all channels
    for (int r = tid; r < R; r += NT) {
        const float *sp = a.sq + (size_t)n * a.G * R + r;
        float s = a.br ? a.br[r] : 0.0f;
        for (int g0 = 0; g0 < a.G; g0 += 16) {
            float v[16];
#pragma unroll
            for (int u = 0; u < 16; u++)
                v[u] = sp[(size_t)min(g0 + u, a.G - 1) * R];
#pragma unroll
            for (int u = 0; u < 16; u++)
                s += g0 + u < a.G ? v[u] : 0.0f;
        }
        zl[r] = s > 0.0f ? s : 0.0f;
    }
    __syncthreads();
    for (int c = tid; c < EC; c += NT) {
        const uint16_t *wrow = a.we + (size_t)c * R;
        float s = a.be ? a.be[c] : 0.0f;
        int r = 0;
        if ((R & 7) == 0) {
            for (; r + 32 <= R; r += 32) {  // four 16-byte loads in flight
                Pack8 v[4];
#pragma unroll
                for (int u = 0; u < 4; u++)
                    v[u].u = ld16(wrow + r + 8 * u);
#pragma unroll
                for (int u = 0; u < 4; u++)
#pragma unroll
                    for (int e = 0; e < 4; e++)
                        s += T::lo(v[u].w[e]) * zl[r + 8 * u + 2 * e] + T::hi(v[u].w[e]) * zl[r + 8 * u + 2 * e + 1];
            }
            for (; r < R; r += 8) {
                Pack8 v;
                v.u = ld16(wrow + r);
#pragma unroll
                for (int e = 0; e < 4; e++)
                    s += T::lo(v.w[e]) * zl[r + 2 * e] + T::hi(v.w[e]) * zl[r + 2 * e + 1];
            }
        }
        for (; r < R; r++)
            s += T::lo((uint32_t)wrow[r]) * zl[r];
        gate[c] = sigmoid_f32(s);
    }
    __syncthreads();

    // ---- 5. project
    float4v acc[OTW][4];
#pragma unroll
    for (int i = 0; i < OTW; i++)
#pragma unroll
        for (int t = 0; t < 4; t++)
            acc[i][t] = float4v{0.f, 0.f, 0.f, 0.f};
    for (int c = 0; c < nch; c++) {
        uint8_t *buf = smem + (uint32_t)(c & 1) * (TP * VP);
        {
            const int k = min(KC * c + 8 * vc, EC - 8);
            const float4v g0 = *reinterpret_cast<const float4v *>(gate + k);
            const float4v g1 = *reinterpret_cast<const float4v *>(gate + k + 4);
#pragma unroll
            for (int i = 0; i < 8; i++) {
                u32x4 o;
                o[0] = T::pack2(T::lo(vr[i][0]) * g0[0], T::hi(vr[i][0]) * g0[1]);
                o[1] = T::pack2(T::lo(vr[i][1]) * g0[2], T::hi(vr[i][1]) * g0[3]);
                o[2] = T::pack2(T::lo(vr[i][2]) * g1[0], T::hi(vr[i][2]) * g1[1]);
                o[3] = T::pack2(T::lo(vr[i][3]) * g1[2], T::hi(vr[i][3]) * g1[3]);
                *reinterpret_cast<u32x4 *>(buf + (uint32_t)(vrow + 8 * i) * VP + (uint32_t)vc * 16) = o;
            }
        }
        // one barrier per chunk: a buffer is rewritten two chunks later, after
        // the barrier in between
        __syncthreads();
        if (c + 1 < nch)
            loadv(c + 1);
        const int nb = min(KC / (32 * KB), nbat - c * (KC / (32 * KB)));
#pragma unroll
        for (int b = 0; b < KC / (32 * KB); b++) {
            if (b >= nb)  // uniform
                break;
            u32x4(&wb)[KB][OTW] = w[b & 1];
#pragma unroll
            for (int j = 0; j < KB; j++) {
                u32x4 bv[4];
#pragma unroll
                for (int t = 0; t < 4; t++)
                    bv[t] = *reinterpret_cast<const u32x4 *>(buf + (uint32_t)(16 * t + jl) * VP +
                                                             (uint32_t)((KB * b + j) * 64 + q * 16));
#pragma unroll
                for (int i = 0; i < OTW; i++) {
                    const u32x4 wf = permute(perm, wb[j][i]);
#pragma unroll
                    for (int t = 0; t < 4; t++)
                        acc[i][t] = T::mfma(wf, bv[t], acc[i][t]);
                }
            }
            loadw(c * (KC / (32 * KB)) + b + 2, wb);
        }
    }
#pragma unroll
    for (int i = 0; i < OTW; i++) {
        const int ot = ot0 + 4 * i, o = 16 * ot + 4 * q;
        if (ot >= OT)
            break;
        const float4v sc = a.s3 ? *reinterpret_cast<const float4v *>(a.s3 + o) : float4v{1.f, 1.f, 1.f, 1.f};
        const float4v bi = a.b3 ? *reinterpret_cast<const float4v *>(a.b3 + o) : float4v{0.f, 0.f, 0.f, 0.f};
        u32x2 xv[4];
#pragma unroll
        for (int t = 0; t < 4; t++) {
            const int p = TP * tile + 16 * t + jl;
            xv[t] = u32x2{0u, 0u};  // the residual (stride 1 only)
            if (!S2 && p < Po)
                xv[t] = *reinterpret_cast<const u32x2 *>(a.x + ((size_t)n * Po + p) * KO + o);
        }
#pragma unroll
        for (int t = 0; t < 4; t++) {
            const int p = TP * tile + 16 * t + jl;
            u32x2 out;
            out[0] = T::pack2(T::lo(xv[t][0]) + fmaf(acc[i][t][0], sc[0], bi[0]),
                              T::hi(xv[t][0]) + fmaf(acc[i][t][1], sc[1], bi[1]));
            out[1] = T::pack2(T::lo(xv[t][1]) + fmaf(acc[i][t][2], sc[2], bi[2]),
                              T::hi(xv[t][1]) + fmaf(acc[i][t][3], sc[3], bi[3]));
            if (p < Po)
                *reinterpret_cast<u32x2 *>(a.y + ((size_t)n * Po + p) * KO + o) = out;
        }
    }
}

// LDS of expand_conv.  First the group's rows of W1; then, over them, U: the
// border row above the image, its H rows, and zero rows below up to an even
// count of row pairs plus one (the conv reads halo rows 2rp .. 2rp+3 for every
// row pair rp).  Behind both s1, b1, s2, b2 and the channel sums of the group,
// and for stride 2 the BlurPool's partial sums.  16 x 16 images: 47,936 bytes
// (stride 2: 52,032), three workgroups per CU.
struct Layout {
    uint32_t off_vec, off_part, lds;
};

Layout layout(int H, int C, int K) {
    Layout l;
    const uint32_t ub = (uint32_t)(2 * ((H + 1) / 2) + 2) * UC * PB, w1b = 64 * (2 * (uint32_t)C + 16);
    l.off_vec = ub > w1b ? ub : w1b;
    l.off_part = l.off_vec + 5 * 64 * 4;
    l.lds = l.off_part + (K > 0 ? NT / 16 * 64 * 4 : 0);
    return l;
}

// The size rule of the accepted shapes: an image's padded U (or an even share
// of its gated V), the gates, the vectors, 64 rows of W1 and, for stride 2
// (K > 0), the group's full-resolution V within the 160 KB of a CU.
uint32_t layout_bytes(int H, int W, int C, int EC, int R, int K) {
    const int P = H * W, Po = K > 0 ? ((H + 1) / 2) * ((W + 1) / 2) : P, KO = K > 0 ? K : C;
    const int G = EC / GH, PT = (Po + 15) / 16;
    const uint32_t nu = G > PT ? 1 : (uint32_t)((PT + G - 1) / G);
    const uint32_t ubytes = (uint32_t)(2 * ((H + 1) / 2) + 2) * UC * PB, stage = nu * 16 * (2 * (uint32_t)EC + 16);
    return (ubytes > stage ? ubytes : stage) + (uint32_t)EC * 4 + (((uint32_t)R * 4 + 15) & ~15u) + GH * 4 +
           (4 * GH + 2 * (uint32_t)KO) * 4 + 64 * (2 * (uint32_t)C + 16) + (K > 0 ? (uint32_t)P * PB : 0u);
}

size_t head_bytes() { return 256 + (size_t)SLOTMAX * 128; }
size_t sq_bytes(int N, int G, int R) { return ((size_t)N * G * R * 4 + 255) & ~(size_t)255; }

// bytes of one image of the exchanged map: the block's output size
size_t image_bytes(int H, int W, int EC, int K) {
    return (K > 0 ? (size_t)((H + 1) / 2) * ((W + 1) / 2) : (size_t)H * W) * EC * 2;
}

template <typename T, bool S2>
const void *expand_kernel(int P) {
    return P > 128 ? (const void *)expand_conv_kernel<T, 4, S2>
                   : P > 64 ? (const void *)expand_conv_kernel<T, 2, S2> : (const void *)expand_conv_kernel<T, 1, S2>;
}

template <typename T, bool S2>
const void *project_kernel(int otw) {
    return otw == 1   ? (const void *)gate_project_kernel<T, 1, S2>
           : otw == 2 ? (const void *)gate_project_kernel<T, 2, S2>
           : otw == 3 ? (const void *)gate_project_kernel<T, 3, S2>
                      : (const void *)gate_project_kernel<T, 4, S2>;
}

}  // namespace mbc

bool mbconv_supported(int H, int W, int C, int E, int R, int K) {
    return H >= (K > 0 ? 2 : 1) && W >= (K > 0 ? 2 : 1) && H <= mbc::HMAX && W <= mbc::WMAX && C >= 16 &&
           C % 16 == 0 && E >= 1 && (E * C) % mbc::GH == 0 && E * C <= mbc::ECMAX && R >= 1 && R <= mbc::RMAX &&
           K >= 0 && K % 16 == 0 && K <= mbc::ECMAX && mbc::layout_bytes(H, W, C, E * C, R, K) <= 160 * 1024;
}

size_t mbconv_workspace_bytes(int N, int H, int W, int C, int E, int R, int K, int images) {
    return mbc::head_bytes() + mbc::sq_bytes(N, E * C / mbc::GH, R) +
           (size_t)images * mbc::image_bytes(H, W, E * C, K);
}

// V of a launch pair stays within 128 MiB, half the Infinity Cache: the second
// kernel reads it from there.
int mbconv_images_in_flight(int N, int H, int W, int C, int E, int K) {
    const size_t m = ((size_t)128 << 20) / mbc::image_bytes(H, W, E * C, K);
    return m < (size_t)N ? (m > 2 ? (int)m : 2) : (N > 2 ? N : 2);
}

hipError_t launch_mbconv(const void *x, void *y, const MBConvW &w, int N, int H, int W, int C, int E, int R, int K,
                         int bf16, void *ws, size_t ws_bytes, hipStream_t st) {
    mbc::Args a{};
    a.x = (const uint16_t *)x;
    a.y = (uint16_t *)y;
    a.w1 = (const uint16_t *)w.w1;
    a.s1 = w.s1;
    a.b1 = w.b1;
    a.gw = (const uint16_t *)w.gw;
    a.s2 = w.s2;
    a.b2 = w.b2;
    a.wr = (const uint16_t *)w.wr;
    a.br = w.br;
    a.we = (const uint16_t *)w.we;
    a.be = w.be;
    a.w2 = (const uint16_t *)w.w2;
    a.s3 = w.s3;
    a.b3 = w.b3;
    a.H = H;
    a.W = W;
    a.C = C;
    a.EC = E * C;
    a.R = R;
    a.G = a.EC / mbc::GH;
    a.K = K > 0 ? K : C;
    a.Ho = K > 0 ? (H + 1) / 2 : H;
    a.Wo = K > 0 ? (W + 1) / 2 : W;
    const int Po = a.Ho * a.Wo;
    a.tiles = (Po + mbc::TP - 1) / mbc::TP;
    a.dw = make_fastdiv((uint32_t)W);
    a.dwo = make_fastdiv((uint32_t)a.Wo);
    a.dg = make_fastdiv((uint32_t)a.G);
    a.dt = make_fastdiv((uint32_t)a.tiles);
    const mbc::Layout l = mbc::layout(H, C, K);
    a.off_vec = l.off_vec;
    a.off_part = l.off_part;
    const size_t fixed = mbc::head_bytes() + mbc::sq_bytes(N, a.G, R), per = mbc::image_bytes(H, W, a.EC, K);
    if (ws_bytes < fixed + 2 * per)
        return hipErrorInvalidValue;
    a.sq = (float *)((char *)ws + mbc::head_bytes());
    a.vx = (uint16_t *)((char *)ws + fixed);
    // as many images per launch pair as the workspace holds, in even passes
    size_t fit = (ws_bytes - fixed) / per;
    if (fit > 65536)
        fit = 65536;  // grid indices stay far below 2^31
    const int passes = (int)((N + fit - 1) / fit), nb = (N + passes - 1) / passes;
    // Output tiles per wave of the projection: a workgroup covers every output
    // channel (up to 256) when the pixel tiles alone fill the CUs; with fewer
    // it takes 64, so the chip holds up to four times as many workgroups, each
    // repeating the gates (a few microseconds of the launch either way).
    const int OT = a.K / 16;
    int otw = (OT + 3) / 4;
    otw = otw > 4 ? 4 : otw;
    if (nb * a.tiles < device_cu_count() / 2)
        otw = 1;
    const void *ka, *kb;
    if (K > 0) {
        ka = bf16 ? mbc::expand_kernel<BF16, true>(H * W) : mbc::expand_kernel<F16, true>(H * W);
        kb = bf16 ? mbc::project_kernel<BF16, true>(otw) : mbc::project_kernel<F16, true>(otw);
    } else {
        ka = bf16 ? mbc::expand_kernel<BF16, false>(H * W) : mbc::expand_kernel<F16, false>(H * W);
        kb = bf16 ? mbc::project_kernel<BF16, false>(otw) : mbc::project_kernel<F16, false>(otw);
    }
    const uint32_t ldsb = 2 * mbc::TP * mbc::VP + (uint32_t)(a.EC + ((R + 3) & ~3)) * 4;
    hipError_t e = allow_full_lds(ka);
    if (e == hipSuccess)
        e = allow_full_lds(kb);
    for (int n0 = 0; n0 < N && e == hipSuccess; n0 += nb) {
        const int m = N - n0 < nb ? N - n0 : nb;
        a.n0 = n0;
        void *args[] = {&a};
        e = hipLaunchKernel(ka, dim3(m * a.G), dim3(mbc::NT), args, l.lds, st);
        if (e == hipSuccess)
            e = hipLaunchKernel(kb, dim3(m * a.tiles, (OT + 4 * otw - 1) / (4 * otw)), dim3(mbc::NT), args, ldsb, st);
    }
    return e;
}

}  // namespace cf
