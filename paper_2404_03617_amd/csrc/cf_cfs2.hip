// cf_cfs2.hip -- the stride-2 ConvFirst block (Fig. f:convfirst-block (c))
// in one kernel: grouped 3 x 3 conv (group width 8) C -> C with its folded
// norm at the input size, BlurPool (Triangle-3 taps [1, 2, 1] / 4 per
// direction, one pixel of reflect padding, stride 2) of the conv output and
// of the block input, the two maps concatenated (2C channels, conv output
// first) into the expand, activation, project to K, no residual.
//
// A workgroup of eight waves takes tiles of TR output rows x 16 columns, one
// after the other; the taps, s0, b0, s1, b1, s2 and b2 are staged in LDS once
// per workgroup, and W1 and W2 as well when they fit.  Per tile, with a
// barrier between the steps:
//  1. the input window, rows 2i0 - 2 .. 2i0 + 2TR and columns 2j0 - 2 ..
//     2j0 + 32, zero outside the image (the conv's padding), from registers
//     to LDS; the next tile's window is then loaded into the same registers
//     (addresses clamped, the zeros selected at the LDS store);
//  2. the grouped conv at full resolution, rows 2i0 - 1 .. 2i0 + 2TR - 1 and
//     columns 2j0 - 1 .. 2j0 + 31 (the positions the blur reads, before
//     reflection), on v_mfma_f32_16x16x32: for group g and tap column dj, A
//     row m = 8s + o at K index 8R + t is the tap W[R - s][dj][8g + o][t]
//     (zero unless 0 <= R - s <= 2) and B column j at K index 8R + t is
//     window pixel (w0 + R, c + dj), channel 8g + t, so one product per tap
//     column gives conv rows w0 and w0 + 1 of 16 positions; the positions of
//     a row pair follow those of the last in one sequence of 33 per pair; s0,
//     b0; rounded to the I/O dtype;
//  3. the blur of both maps (fp32, rounded to the I/O dtype), each read at
//     the reflected positions, into a tile of 16 TR pixels x 2C channels,
//     zero-padded to a multiple of 32;
//  4. the expand on v_mfma_f32_16x16x32: a wave takes tiles of 16 hidden
//     channels over every pixel of the tile (A = W1 rows), s1, b1 and the
//     activation in fp32, rounded into LDS over the dead window and conv map;
//  5. the project: the products of 16 output channels (A = W2 rows) and 16
//     pixels dealt evenly to the waves; s2, b2; y stored once.
// Weights that are not in LDS are read from global memory (L2) one tile ahead
// with row-major loads -- lane 4r + p takes piece p of row r, four adjacent
// lanes on one contiguous run -- and ds_bpermute moves each dword to its
// fragment lane (a fragment-order load costs the memory unit several times
// more per byte).
// Conv positions outside the image are evaluated on the zero padding and
// never read: the blur's reflection of row -1 is row 1, of row H is H - 2,
// both inside the tile's rows (and likewise for columns).
//
// Bound by the chain of the five steps at eight or sixteen waves per CU.  A wave working
// alone on units of 16 pixels (the earlier form of this kernel) left room for
// four waves in the LDS at C = 48 and read every weight from L2 for each unit:
// N = 128, 64 x 64, C = 48, R = 288, K = 64, fp16: 151 us then, 84 us now.
#include "cf_device.h"
#include "cf_kernels.h"

namespace cf {
namespace cfs2 {

constexpr int XC = 35;          // window columns 2j0-2 .. 2j0+32
constexpr int VC = 33;          // conv columns 2j0-1 .. 2j0+31
constexpr int KMAX = 128;       // output channels
constexpr int RMAX = 1024;      // hidden channels
constexpr int NW = 8, NT = NW * 64;

struct Args {
    const uint16_t *x;
    uint16_t *y;
    const uint16_t *gw;  // [3][3][C][8]
    const float *s0, *b0;
    const uint16_t *w1;  // [R][2C]
    const float *s1, *b1;
    const uint16_t *w2;  // [K][R]
    const float *s2, *b2;
    int H, W, Ho, Wo, R, K, act;
    int tiles;                // N * it * jt
    FastDiv jt, it;           // tiles per row of tiles, rows of tiles per image
    uint32_t off_w1, off_w2;  // LDS: taps, s0, b0, s1, b1, s2, b2; W1 and W2 when staged;
    uint32_t off_x, off_z;    // then window and conv map (later the hidden tile); then the blurred tile
};

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// one pixel of reflect padding (-1 -> 1, n -> n - 2); past that (positions of
// a ragged tile whose outputs are not stored) the last one
__device__ __forceinline__ int refl(int v, int n) {
    int r = v < 0 ? -v : v;
    r = r == n ? n - 2 : r;
    return r < n ? r : n - 1;
}

__device__ __forceinline__ float act_f(float u, int act) {
    if (act == ACT_RELU)
        return fmaxf(u, 0.0f);
    if (act == ACT_GELU)
        return gelu_f32(u);
    return u;
}

__device__ __forceinline__ u32x4 ld16(const void *p) { return *reinterpret_cast<const u32x4 *>(p); }

// LDS bytes of the staged taps and vectors
__host__ __device__ inline uint32_t staged_bytes(int C, int R, int K) {
    return ((uint32_t)(9 * C * 16 + 4 * (2 * C + 2 * R + 2 * K)) + 255) & ~255u;
}

// row strides of W1 and W2 staged in LDS, and of the hidden tile: odd
// multiples of 16 bytes
__host__ __device__ inline uint32_t w1_stride(int C) { return (uint32_t)(4 * C + 16); }
__host__ __device__ inline uint32_t w2_stride(int R) { return (uint32_t)(2 * R + 16); }
__host__ __device__ inline uint32_t weights_bytes(int C, int R, int K) {
    return ((uint32_t)R * w1_stride(C) + (uint32_t)K * w2_stride(R) + 255) & ~255u;
}

// bytes per window / conv pixel: an odd multiple of 16
constexpr uint32_t pixel_bytes(int C) { return C % 16 ? 2 * C + 32 : 2 * C + 16; }
constexpr int row_pairs(int TR) { return TR + 1; }  // of the 2 TR + 1 conv rows

// LDS bytes of the window and conv map, or the hidden tile over them
inline uint32_t map_bytes(int C, int TR, int R) {
    const uint32_t xv = ((uint32_t)(2 * TR + 3) * XC + (uint32_t)(2 * TR + 1) * VC) * pixel_bytes(C);
    const uint32_t h = (uint32_t)(16 * TR) * w2_stride(R);
    return ((xv > h ? xv : h) + 255) & ~255u;
}
inline uint32_t tile_bytes(int C, int TR) { return (uint32_t)(16 * TR) * (2 * (uint32_t)((2 * C + 31) / 32 * 32) + 16); }

template <typename T, int C, int TR, bool WL>
struct Kern {
    static constexpr int G = C / 8;                      // groups of the conv
    static constexpr uint32_t PP = pixel_bytes(C);
    static constexpr int C2 = 2 * C, C2P = (C2 + 31) / 32 * 32;
    static constexpr int KS = C2P / 32;                  // expand K steps
    static constexpr uint32_t PZ = 2 * C2P + 16;         // LDS bytes per tile pixel
    static constexpr int RP = row_pairs(TR);
    static constexpr int XR = 2 * TR + 3;                // window rows
    static constexpr int VR = 2 * TR + 1;
    static constexpr uint32_t XB = (uint32_t)XR * XC * PP;
    static constexpr int NX = XR * XC * G, NIT = (NX + NT - 1) / NT;  // 16-byte pieces of the window, per thread
    static constexpr int NPOS = RP * VC, PT = (NPOS + 15) / 16;       // conv positions per group, tiles of 16

    struct Tile {
        int n, i0, j0;
    };
    static __device__ __forceinline__ Tile decode(const Args &a, int u) {
        const uint32_t r = fdiv((uint32_t)u, a.jt), n = fdiv(r, a.it);
        return Tile{(int)n, (int)(r - n * a.it.d) * TR, (int)((uint32_t)u - r * a.jt.d) * 16};
    }

    // this thread's pieces of a tile's window, positions clamped into the image
    static __device__ __forceinline__ void load_window(const Args &a, int u, int tid, u32x4 (&xv)[NIT]) {
        const Tile tl = decode(a, u);
        const uint16_t *xn = a.x + (size_t)tl.n * a.H * a.W * C;
#pragma unroll
        for (int it = 0; it < NIT; it++) {
            const int t = min(tid + NT * it, NX - 1);
            const int px = t / G, pc = t - px * G, rr = px / XC, cc = px - rr * XC;
            const int gr = clampi(2 * tl.i0 - 2 + rr, 0, a.H - 1), gc = clampi(2 * tl.j0 - 2 + cc, 0, a.W - 1);
            xv[it] = ld16(xn + ((size_t)gr * a.W + gc) * C + 8 * pc);
        }
    }
    static __device__ __forceinline__ void store_window(const Args &a, const Tile &tl, int tid,
                                                        const u32x4 (&xv)[NIT], uint8_t *X) {
#pragma unroll
        for (int it = 0; it < NIT; it++) {
            const int t = tid + NT * it;
            const int px = t / G, pc = t - px * G, rr = px / XC, cc = px - rr * XC;
            const int gr = 2 * tl.i0 - 2 + rr, gc = 2 * tl.j0 - 2 + cc;
            const bool in = gr >= 0 && gr < a.H && gc >= 0 && gc < a.W;
            if (t < NX)
                *reinterpret_cast<u32x4 *>(X + (uint32_t)px * PP + (uint32_t)pc * 16) = in ? xv[it] : u32x4{0u, 0u, 0u, 0u};
        }
    }

    static __device__ __forceinline__ u32x4 permute(int idx, const u32x4 &v) {
        u32x4 o;
#pragma unroll
        for (int d = 0; d < 4; d++)
            o[d] = (uint32_t)__builtin_amdgcn_ds_bpermute(idx, (int)v[d]);
        return o;
    }

    static __device__ void run(const Args &a, uint8_t *smem) {
        const int tid = threadIdx.x, lane = tid & 63;
        const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int q = lane >> 4, jl = lane & 15;
        const int lr = lane >> 2, lp = lane & 3, pidx = (4 * jl + q) * 4;  // row-major lane, its fragment source
        const int R = a.R, K = a.K, OT = (K + 15) / 16, HT = R / 16;
        const uint32_t PH = w2_stride(R);  // LDS bytes per pixel of the hidden tile
        u32x4 xv[NIT];
        load_window(a, blockIdx.x, tid, xv);
        // the taps [3][3][C][8] and the vectors, once per workgroup
        for (int i = tid; i < 9 * C; i += NT)
            *reinterpret_cast<u32x4 *>(smem + (uint32_t)i * 16) = ld16(a.gw + (size_t)i * 8);
        float *s0l = reinterpret_cast<float *>(smem + 9 * C * 16), *b0l = s0l + C, *s1l = b0l + C, *b1l = s1l + R,
              *s2l = b1l + R, *b2l = s2l + K;
        for (int c = tid; c < C; c += NT) {
            s0l[c] = a.s0 ? a.s0[c] : 1.0f;
            b0l[c] = a.b0 ? a.b0[c] : 0.0f;
        }
        for (int h = tid; h < R; h += NT) {
            s1l[h] = a.s1 ? a.s1[h] : 1.0f;
            b1l[h] = a.b1 ? a.b1[h] : 0.0f;
        }
        for (int o = tid; o < K; o += NT) {
            s2l[o] = a.s2 ? a.s2[o] : 1.0f;
            b2l[o] = a.b2 ? a.b2[o] : 0.0f;
        }
        if constexpr (WL) {
            // W1 [R][2C] and W2 [K][R] in 16-byte pieces, four in flight
            auto stage = [&](const uint16_t *w, int rows, int pieces, uint32_t off, uint32_t stride) {
                const int total = rows * pieces;
                for (int i0 = tid; i0 < total; i0 += 4 * NT) {
                    u32x4 v[4];
#pragma unroll
                    for (int u = 0; u < 4; u++)
                        v[u] = ld16(w + (size_t)min(i0 + NT * u, total - 1) * 8);
#pragma unroll
                    for (int u = 0; u < 4; u++) {
                        const int i = i0 + NT * u, r = i / pieces, pc = i - r * pieces;
                        if (i < total)
                            *reinterpret_cast<u32x4 *>(smem + off + (uint32_t)r * stride + (uint32_t)pc * 16) = v[u];
                    }
                }
            };
            stage(a.w1, R, C / 4, a.off_w1, w1_stride(C));
            stage(a.w2, K, R / 8, a.off_w2, w2_stride(R));
        }
        uint8_t *X = smem + a.off_x, *V = X + XB, *Z = smem + a.off_z, *Hd = X;

        for (int u = (int)blockIdx.x; u < a.tiles; u += (int)gridDim.x) {
            const Tile tl = decode(a, u);
            const int H = a.H, W = a.W;
            // 1. (the first time round also: the staged taps, vectors, weights)
            store_window(a, tl, tid, xv, X);
            __syncthreads();
            if (u + (int)gridDim.x < a.tiles)
                load_window(a, u + (int)gridDim.x, tid, xv);

            // 2. the grouped conv: this wave's run of (group, position tile) items
            {
                constexpr int ITEMS = G * PT, PER = (ITEMS + NW - 1) / NW;
                const int first = wv * PER, last = min(first + PER, ITEMS);
                const int di = q - (jl >> 3);  // A lane (row jl = 8s + o, K 8q .. 8q + 7): tap row q - s
                const bool tap = di >= 0 && di <= 2;
                u32x4 av[3];
                float4v sc, bi;
                for (int item = first; item < last; item++) {
                    const int g = item / PT, pt = item - g * PT;
                    const int cd = 8 * g + 4 * (q & 1);  // channels of D lane rows 4q .. 4q + 3
                    if (item == first || pt == 0) {  // wave-uniform
#pragma unroll
                        for (int dj = 0; dj < 3; dj++) {
                            const u32x4 v = *reinterpret_cast<const u32x4 *>(
                                smem + (uint32_t)((((tap ? di : 0) * 3 + dj) * C + 8 * g + (jl & 7)) * 16));
                            av[dj] = tap ? v : u32x4{0u, 0u, 0u, 0u};
                        }
                        sc = *reinterpret_cast<const float4v *>(s0l + cd);
                        bi = *reinterpret_cast<const float4v *>(b0l + cd);
                    }
                    const int pos = 16 * pt + jl, pp = min(pos, NPOS - 1);
                    const int rp = pp / VC, vc = pp - rp * VC;
                    // (the last pair's fourth row meets only the dropped
                    // second row's taps)
                    const uint8_t *bp = X + (uint32_t)(min(2 * rp + q, XR - 1) * XC + vc) * PP + (uint32_t)g * 16;
                    float4v d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int dj = 0; dj < 3; dj++)
                        d = T::mfma(av[dj], *reinterpret_cast<const u32x4 *>(bp + dj * PP), d);
                    const int vr = 2 * rp + (q >> 1);
                    if (pos < NPOS && vr < VR)
                        *reinterpret_cast<u32x2 *>(V + (uint32_t)(vr * VC + vc) * PP + (uint32_t)cd * 2) =
                            u32x2{T::pack2(fmaf(d[0], sc[0], bi[0]), fmaf(d[1], sc[1], bi[1])),
                                  T::pack2(fmaf(d[2], sc[2], bi[2]), fmaf(d[3], sc[3], bi[3]))};
                }
            }
            __syncthreads();

            // 3. BlurPool of the conv output and of the input (the conv map
            //    sits one row and one column inside the window), 8 channels
            //    of a pixel per thread
            for (int t = tid; t < 16 * TR * (C2P / 8); t += NT) {
                const int px = t / (C2P / 8), c = 8 * (t - px * (C2P / 8));
                const int i = tl.i0 + (px >> 4), j = tl.j0 + (px & 15);
                u32x4 out = {0u, 0u, 0u, 0u};  // zero padding past 2C
                if (c < C2) {
                    const bool isv = c < C;
                    const uint8_t *base = isv ? V + c * 2 : X + (c - C) * 2;
                    const int ro = 2 * tl.i0 - (isv ? 1 : 2), co = 2 * tl.j0 - (isv ? 1 : 2), wd = isv ? VC : XC;
                    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ta = 0; ta < 3; ta++) {
                        const uint32_t rb = (uint32_t)((refl(2 * i + ta - 1, H) - ro) * wd);
#pragma unroll
                        for (int tb = 0; tb < 3; tb++) {
                            const float wt = (ta == 1 ? 0.5f : 0.25f) * (tb == 1 ? 0.5f : 0.25f);
                            const u32x4 v = *reinterpret_cast<const u32x4 *>(
                                base + (rb + (uint32_t)(refl(2 * j + tb - 1, W) - co)) * PP);
#pragma unroll
                            for (int d = 0; d < 4; d++) {
                                acc[2 * d] = fmaf(wt, T::lo(v[d]), acc[2 * d]);
                                acc[2 * d + 1] = fmaf(wt, T::hi(v[d]), acc[2 * d + 1]);
                            }
                        }
                    }
#pragma unroll
                    for (int d = 0; d < 4; d++)
                        out[d] = T::pack2(acc[2 * d], acc[2 * d + 1]);
                }
                *reinterpret_cast<u32x4 *>(Z + (uint32_t)px * PZ + (uint32_t)c * 2) = out;
            }
            __syncthreads();

            // 4. expand: hidden tiles wv, wv + 8, ..; eight zeros behind each
            //    pixel's hidden values, for the project's K steps past R
            {
                if (tid < 16 * TR)
                    *reinterpret_cast<u32x4 *>(Hd + (uint32_t)tid * PH + (uint32_t)R * 2) = u32x4{0u, 0u, 0u, 0u};
                u32x4 zf[TR][KS];
#pragma unroll
                for (int t = 0; t < TR; t++)
#pragma unroll
                    for (int ks = 0; ks < KS; ks++)
                        zf[t][ks] = *reinterpret_cast<const u32x4 *>(Z + (uint32_t)(16 * t + jl) * PZ +
                                                                     (uint32_t)(32 * ks + 8 * q) * 2);
                u32x4 wn[KS];  // the next tile's fragments (from global memory: row-major pieces)
                auto fetch = [&](int ht) {
                    const int r0 = 16 * min(ht, HT - 1);
#pragma unroll
                    for (int ks = 0; ks < KS; ks++)
                        if constexpr (WL)
                            wn[ks] = *reinterpret_cast<const u32x4 *>(smem + a.off_w1 + (uint32_t)(r0 + jl) * w1_stride(C) +
                                                                      min(32 * ks + 8 * q, C2 - 8) * 2);
                        else
                            wn[ks] = ld16(a.w1 + (size_t)(r0 + lr) * C2 + min(32 * ks + 8 * lp, C2 - 8));
                };
                fetch(wv);
                for (int ht = wv; ht < HT; ht += NW) {
                    u32x4 wf[KS];
#pragma unroll
                    for (int ks = 0; ks < KS; ks++)
                        wf[ks] = WL ? wn[ks] : permute(pidx, wn[ks]);
                    fetch(ht + NW);
                    const float4v sc = *reinterpret_cast<const float4v *>(s1l + 16 * ht + 4 * q);
                    const float4v bi = *reinterpret_cast<const float4v *>(b1l + 16 * ht + 4 * q);
                    float4v h[TR];
#pragma unroll
                    for (int t = 0; t < TR; t++)
                        h[t] = float4v{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ks = 0; ks < KS; ks++)
#pragma unroll
                        for (int t = 0; t < TR; t++)
                            h[t] = T::mfma(wf[ks], zf[t][ks], h[t]);
#pragma unroll
                    for (int t = 0; t < TR; t++) {
                        float v[4];
#pragma unroll
                        for (int e = 0; e < 4; e++)
                            v[e] = act_f(fmaf(h[t][e], sc[e], bi[e]), a.act);
                        *reinterpret_cast<u32x2 *>(Hd + (uint32_t)(16 * t + jl) * PH + (uint32_t)(16 * ht + 4 * q) * 2) =
                            u32x2{T::pack2(v[0], v[1]), T::pack2(v[2], v[3])};
                    }
                }
            }
            __syncthreads();

            // 5. project: the OT x TR products of 16 channels x 16 pixels dealt
            //    evenly to the waves, in runs that share their W2 rows
            {
                const int n = OT * TR, u0 = wv * n / NW, u1 = (wv + 1) * n / NW;
                const int NK = (R + 31) / 32;
                for (int ot = u0 / TR; ot * TR < u1; ot++) {
                    const int ta = u0 - ot * TR, tb = u1 - ot * TR;  // pixel rows ta <= t < tb
                    float4v acc[TR];
#pragma unroll
                    for (int t = 0; t < TR; t++)
                        acc[t] = float4v{0.f, 0.f, 0.f, 0.f};
                    constexpr int KB = WL ? 2 : 4;  // K steps per batch, two batches of W2 in flight
                    u32x4 wb[2][KB];
                    const uint8_t *wl = smem + a.off_w2 + (uint32_t)min(16 * ot + jl, K - 1) * w2_stride(R);
                    const uint16_t *wr = a.w2 + (size_t)min(16 * ot + lr, K - 1) * R;
                    auto fetch = [&](int b, u32x4 (&w)[KB]) {
#pragma unroll
                        for (int k = 0; k < KB; k++)
                            if constexpr (WL)
                                w[k] = *reinterpret_cast<const u32x4 *>(wl + min(32 * (KB * b + k) + 8 * q, R - 8) * 2);
                            else
                                w[k] = ld16(wr + min(32 * (KB * b + k) + 8 * lp, R - 8));
                    };
                    auto use = [&](int b, const u32x4 (&w)[KB]) {
                        // a K step past R (R % 32 == 16, or the batch's end) repeats
                        // weights and meets the zeros behind the pixel's hidden values
                        u32x4 wf[KB];
#pragma unroll
                        for (int k = 0; k < KB; k++)
                            wf[k] = WL ? w[k] : permute(pidx, w[k]);
#pragma unroll
                        for (int t = 0; t < TR; t++)
                            if (t >= ta && t < tb) {  // uniform
                                u32x4 hv[KB];
                                const uint8_t *hp = Hd + (uint32_t)(16 * t + jl) * PH;
#pragma unroll
                                for (int k = 0; k < KB; k++)
                                    hv[k] = *reinterpret_cast<const u32x4 *>(hp + min(32 * (KB * b + k) + 8 * q, R) * 2);
#pragma unroll
                                for (int k = 0; k < KB; k++)
                                    acc[t] = T::mfma(wf[k], hv[k], acc[t]);
                            }
                    };
                    fetch(0, wb[0]);
                    for (int b = 0; KB * b < NK; b += 2) {
                        fetch(b + 1, wb[1]);
                        use(b, wb[0]);
                        if (KB * (b + 1) < NK) {
                            fetch(b + 2, wb[0]);
                            use(b + 1, wb[1]);
                        }
                    }
                    const int o = 16 * ot + 4 * q;
                    if (o < K) {
                        const float4v sc = *reinterpret_cast<const float4v *>(s2l + o);
                        const float4v bi = *reinterpret_cast<const float4v *>(b2l + o);
#pragma unroll
                        for (int t = 0; t < TR; t++)
                            if (t >= ta && t < tb && tl.i0 + t < a.Ho && tl.j0 + jl < a.Wo) {
                                float r[4];
#pragma unroll
                                for (int e = 0; e < 4; e++)
                                    r[e] = fmaf(acc[t][e], sc[e], bi[e]);
                                *reinterpret_cast<u32x2 *>(a.y + (((size_t)tl.n * a.Ho + tl.i0 + t) * a.Wo + tl.j0 + jl) * K + o) =
                                    u32x2{T::pack2(r[0], r[1]), T::pack2(r[2], r[3])};
                            }
                    }
                }
            }
            __syncthreads();  // the hidden tile's bytes are the next window's
        }
    }
};

template <typename T, int C, int TR, bool WL, int WE>
__global__ __launch_bounds__(NT) __attribute__((amdgpu_waves_per_eu(WE, WE))) void cfs2_kernel(Args a) {
    extern __shared__ __attribute__((aligned(256))) uint8_t smem[];
    Kern<T, C, TR, WL>::run(a, smem);
}

// Tile height and whether the weights are staged.  In order: staged weights
// with two workgroups on a CU (128 images of 128 x 128: C = 24 159 us, against
// 206 with one workgroup and four rows; C = 16 83); four rows with the weights
// (C = 32, 64 x 64: 60 us, against 74 without them and 68 with two rows); four
// rows without (C = 48, 64 x 64: 89 us, against 97 with two rows and the
// weights); two rows.  Fewer four-row tiles than CUs: two rows (4 images,
// C = 64: 12.6 against 16.6 us).
struct Plan {
    int tr;
    bool wl;
    uint32_t lds;
};
constexpr uint32_t PAIR_LDS = 80 * 1024, FULL_LDS = 160 * 1024;
// instances with registers for two workgroups on a CU
constexpr bool pairs(int C, int TR, bool wl) { return wl && (C == 16 || (TR == 2 && C <= 48)); }

inline Plan plan_for(int C, int R, int K, int64_t tiles4, int cus) {
    const uint32_t st = staged_bytes(C, R, K), wb = weights_bytes(C, R, K);
    auto need = [&](int tr, bool wl) { return st + (wl ? wb : 0u) + map_bytes(C, tr, R) + tile_bytes(C, tr); };
    const int top = tiles4 < cus ? 2 : 4;
    for (int tr = top; tr >= 2; tr -= 2)
        if (pairs(C, tr, true) && need(tr, true) <= PAIR_LDS)
            return Plan{tr, true, need(tr, true)};
    for (int tr = top; tr >= 2; tr -= 2)
        for (int wl = 1; wl >= 0; wl--)
            if (need(tr, wl != 0) <= FULL_LDS)
                return Plan{tr, wl != 0, need(tr, wl != 0)};
    return Plan{0, false, 0};
}

template <typename T, int C, int TR, bool WL, int WE>
hipError_t launch_e(const Args &a, size_t lds, int cus, hipStream_t st) {
    const void *k = (const void *)cfs2_kernel<T, C, TR, WL, WE>;
    hipError_t e = allow_full_lds(k);
    if (e != hipSuccess)
        return e;
    Args b = a;
    void *args[] = {&b};
    const int cap = cus * (WE / 2);  // persistent workgroups, WE / 2 per CU
    return hipLaunchKernel(k, dim3(a.tiles < cap ? a.tiles : cap), dim3(NT), args, lds, st);
}

template <typename T, int C, int TR, bool WL>
hipError_t launch_t(const Args &a, size_t lds, int cus, hipStream_t st) {
    if constexpr (pairs(C, TR, WL))
        if (lds <= PAIR_LDS)
            return launch_e<T, C, TR, WL, 4>(a, lds, cus, st);
    return launch_e<T, C, TR, WL, 2>(a, lds, cus, st);
}

template <typename T, int C>
hipError_t launch_c(const Args &a, const Plan &p, int cus, hipStream_t st) {
    if (p.tr == 4)
        return p.wl ? launch_t<T, C, 4, true>(a, p.lds, cus, st) : launch_t<T, C, 4, false>(a, p.lds, cus, st);
    return p.wl ? launch_t<T, C, 2, true>(a, p.lds, cus, st) : launch_t<T, C, 2, false>(a, p.lds, cus, st);
}

template <typename T>
hipError_t launch(const Args &a, int C, const Plan &p, int cus, hipStream_t st) {
    switch (C) {
    case 16: return launch_c<T, 16>(a, p, cus, st);
    case 24: return launch_c<T, 24>(a, p, cus, st);
    case 32: return launch_c<T, 32>(a, p, cus, st);
    case 48: return launch_c<T, 48>(a, p, cus, st);
    case 64: return launch_c<T, 64>(a, p, cus, st);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace cfs2

bool convfirst_s2_supported(int H, int W, int C, int R, int K) {
    return H >= 2 && W >= 2 && R >= 16 && R % 16 == 0 && R <= cfs2::RMAX && K >= 8 && K % 8 == 0 &&
           K <= cfs2::KMAX && (C == 16 || C == 24 || C == 32 || C == 48 || C == 64);
}

hipError_t launch_convfirst_s2(const void *x, void *y, const BlockW &w, int N, int H, int W, int C, int R, int K,
                               int bf16, int act, hipStream_t st) {
    if (!convfirst_s2_supported(H, W, C, R, K))
        return hipErrorInvalidConfiguration;
    cfs2::Args a{};
    a.x = (const uint16_t *)x;
    a.y = (uint16_t *)y;
    a.gw = (const uint16_t *)w.dw_w;
    a.s0 = w.s0;
    a.b0 = w.b0;
    a.w1 = (const uint16_t *)w.w1;
    a.s1 = w.s1;
    a.b1 = w.b1;
    a.w2 = (const uint16_t *)w.w2;
    a.s2 = w.s2;
    a.b2 = w.b2;
    a.H = H;
    a.W = W;
    a.Ho = (H + 1) / 2;
    a.Wo = (W + 1) / 2;
    a.R = R;
    a.K = K;
    a.act = act;
    const int cus = device_cu_count(), jt = (a.Wo + 15) / 16;
    const cfs2::Plan p = cfs2::plan_for(C, R, K, (int64_t)N * ((a.Ho + 3) / 4) * jt, cus);
    if (!p.tr)
        return hipErrorInvalidConfiguration;
    const int64_t tiles = (int64_t)N * ((a.Ho + p.tr - 1) / p.tr) * jt;
    if ((int64_t)N * a.Ho * jt > (int64_t)1 << 30)
        return hipErrorInvalidValue;
    a.tiles = (int)tiles;
    a.jt = make_fastdiv((uint32_t)jt);
    a.it = make_fastdiv((uint32_t)((a.Ho + p.tr - 1) / p.tr));
    a.off_w1 = cfs2::staged_bytes(C, R, K);
    a.off_w2 = a.off_w1 + (uint32_t)R * cfs2::w1_stride(C);
    a.off_x = a.off_w1 + (p.wl ? cfs2::weights_bytes(C, R, K) : 0u);
    a.off_z = a.off_x + cfs2::map_bytes(C, p.tr, R);
    return bf16 ? cfs2::launch<BF16>(a, C, p, cus, st) : cfs2::launch<F16>(a, C, p, cus, st);
}

}  // namespace cf
