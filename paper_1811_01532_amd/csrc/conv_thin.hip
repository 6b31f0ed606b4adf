// First-layer convolutions (1 .. 4 input channels) of any filter, stride and padding, any output channel count that is a
// multiple of 8 (gfx950): forward and weight gradient.
//
// With so few channels the layer is bound by its output (forward) or dy (weight gradient) stream, or, when it is small, by
// latency; what the generic kernels spend their time on is fetching the im2col operand two bytes at a time from memory, R*S
// times over.  Here a work-group stages the input patch of its tile (4 output rows x 32 pixels) ONCE in LDS, first as it
// lies in memory (16-byte loads, the next tile's in flight during this tile's products), then with every pixel widened to
// four channels (8 bytes), zeros outside the image.  Then every fragment is made of aligned 8-byte pieces
// whatever the stride: in the forward kernel 8 reduction elements are two neighbouring pixels of a filter row, in the
// weight gradient the transposing read takes 4 columns = one tap of 16 pixels.  The fourth channel and the odd tap of an
// odd filter row meet zeros on both sides.
// Measured, us, generic (or gather-based first-layer) kernel / this one, the weight gradient with its reduction:
//   forward     224x224x3 -> 64, 11x11 stride 4, 1 image 24.2 / 16.0; 13 x 192x192x3 -> 96, 3x3 114 / 36;
//               29 x 96x96x3 -> 16, 11x11 stride 4 50 / 14; 32 x 224x224x3 -> 64, 7x7 stride 2 68 / 50;
//               4 x 32x32x3 -> 16, 3x3 14.8 / 5.8
//   weight grad 13 x 192x192x3 -> 96, 3x3 123 / 46; 32 x 224x224x3 -> 64, 7x7 stride 2 190 / 46;
//               37 x 63x63x3 -> 32, 5x5 stride 2 27 / 13; 4 x 32x32x3 -> 16 28 / 11
// Where the specialised kernels of conv_c3.hip apply they stay ahead (3x3 stride 1 at 24 x 224x224 -> 64: 43 against 63
// us forward, 55 against 63 weight gradient); the gather for other filters and the pair for large filters at horizontal
// stride 4 share the field with these kernels by the rules below.
#include <algorithm>

#include "wap_internal.h"

namespace wap {

namespace {

constexpr int NT = 256, TR = 4, TW = 32;  // threads; output rows and pixels per row of a tile
constexpr size_t LDS_CAP = 160 * 1024;

struct ThinArgs {
    const bf16_t* x;
    const bf16_t* w;    // forward: [K][R][S][C]
    const bf16_t* dy;   // weight gradient: [N][OH][OW][K]
    const float* bias;
    bf16_t* y;
    float* part;        // weight gradient: [gridDim.x][K][R*S*C]
    int H, W, C, K, OH, OW, R, S, sh, sw, ph, pw, relu;
    int Kred;               // R * S * C
    int tiles_x, tiles_y, ntiles;
    int G, ksteps;          // forward: tap pairs per filter row, 16-deep reduction steps (two pairs each)
    int NB;                 // weight gradient: 32-column blocks (8 taps x 4 channels)
    int xw, npx;            // staged pixels per patch row, in all
    int nv, nvec, rpitch;   // 16-byte vectors per raw patch row, in all; bytes of a raw row
    int x_elems;
    FastDiv dTX, dTY, dXW, dNV, dKred, dSC, dC, dS;
};

__device__ __align__(16) unsigned int g_zero_block_thin[4] = {0u, 0u, 0u, 0u};

__device__ __forceinline__ unsigned short f2bf(float f) {
    __bf16 b = (__bf16)f;
    return __builtin_bit_cast(unsigned short, b);
}

typedef s16x4 __attribute__((address_space(3))) * lds_s16x4_ptr;
__device__ __forceinline__ u32x4 tr_pair(const unsigned char* p0, const unsigned char* p1) {
    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)p0);
    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)p1);
    s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(u32x4, both);
}

struct TilePos {
    int n, oh0, ow0;
};
__device__ __forceinline__ TilePos tile_pos(const ThinArgs& a, int tile) {
    const int t = (int)fdiv((uint32_t)tile, a.dTX);
    TilePos p;
    p.ow0 = (tile - t * a.tiles_x) * TW;
    p.n = (int)fdiv((uint32_t)t, a.dTY);
    p.oh0 = (t - p.n * a.tiles_y) * TR;
    return p;
}

// The raw patch of a tile: for every patch row inside the image the 16-byte vectors that cover it, the first of which
// starts up to seven elements before the patch (XV vectors per thread).  A vector that reaches over an end of the tensor is
// put together from the elements inside.
constexpr int XV = 6;
__device__ __forceinline__ void load_raw(const ThinArgs& a, const TilePos& tp, u32x4 (&rx)[XV]) {
    const int ih0 = tp.oh0 * a.sh - a.ph, iw0 = tp.ow0 * a.sw - a.pw;
#pragma unroll
    for (int u = 0; u < XV; ++u) {
        const int v = threadIdx.x + u * NT;
        rx[u] = u32x4{0u, 0u, 0u, 0u};
        if (u * NT >= a.nvec) continue;  // uniform
        const int py = (int)fdiv((uint32_t)v, a.dNV);
        const int ih = ih0 + py;
        if (v < a.nvec && (unsigned)ih < (unsigned)a.H) {
            const int e0 = ((((tp.n * a.H + ih) * a.W + iw0) * a.C) & ~7) + (v - py * a.nv) * 8;
            if (e0 >= 0 && e0 <= a.x_elems - 8) {
                rx[u] = *reinterpret_cast<const u32x4*>(a.x + e0);
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e)
                    if (e0 + e >= 0 && e0 + e < a.x_elems) rx[u][e >> 1] |= (unsigned)a.x[e0 + e] << (16 * (e & 1));
            }
        }
    }
}
__device__ __forceinline__ void store_raw(const ThinArgs& a, const u32x4 (&rx)[XV], unsigned char* sR) {
#pragma unroll
    for (int u = 0; u < XV; ++u) {
        const int v = threadIdx.x + u * NT;
        if (v < a.nvec) *reinterpret_cast<u32x4*>(sR + (size_t)v * 16) = rx[u];  // rows lie one behind the other
    }
}
// raw patch -> 4-channel pixels
__device__ __forceinline__ void widen(const ThinArgs& a, const TilePos& tp, const unsigned char* sR, unsigned char* sX) {
    const int ih0 = tp.oh0 * a.sh - a.ph, iw0 = tp.ow0 * a.sw - a.pw;
#pragma unroll 4
    for (int i = threadIdx.x; i < a.npx; i += NT) {
        const int py = (int)fdiv((uint32_t)i, a.dXW), px = i - py * a.xw;
        const int ih = ih0 + py, iw = iw0 + px;
        u32x2 v = {0u, 0u};
        if ((unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W) {
            const int off = (((tp.n * a.H + ih) * a.W + iw0) * a.C) & 7;
            const unsigned short* p = reinterpret_cast<const unsigned short*>(sR + py * a.rpitch) + off + px * a.C;
            v[0] = p[0];
            if (a.C > 1) v[0] |= (unsigned)p[1] << 16;
            if (a.C > 2) v[1] = p[2];
            if (a.C > 3) v[1] |= (unsigned)p[3] << 16;
        }
        *reinterpret_cast<u32x2*>(sX + (size_t)i * 8) = v;
    }
}

// ---- forward.  FB: 32-channel blocks per work-group (blockIdx.y: group of 32 * FB channels); wavefront = one output row of
// the tile.  The weights pass through LDS into MFMA fragment order once per (long-lived) work-group: reduction element
// (tap pair, tap of the pair, channel), pairs numbered r * G + s / 2. ----
template <int FB>
__global__ __launch_bounds__(NT, 2) void conv_thin_fwd_kernel(const ThinArgs a) {
    constexpr int OPITCH = FB * 64 + 16;
    constexpr int VPR = FB * 4;  // 16-byte vectors per output pixel
    extern __shared__ __align__(16) unsigned char smem_t[];
    unsigned char* const sW = smem_t;                                    // [ksteps][FB][64 lanes][16 bytes]
    unsigned char* const sX = sW + (size_t)a.ksteps * FB * 1024;
    unsigned char* const sR = sX + (size_t)(a.npx + 1) / 2 * 16;
    // One strip of 32 pixels per wavefront, where the raw patch lay until it was widened.  Apart from it, an 11x11 filter's
    // work-group took more than half of a CU's LDS: 8 x 224x224x3 -> 64 at stride 4 25.7 us in a step, 20.4 with two a CU.
    unsigned char* const sO = sR;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int half = lane >> 5, l32 = lane & 31;
    const int ch0 = blockIdx.y * 32 * FB;
    const int nch = a.K - ch0 < 32 * FB ? a.K - ch0 : 32 * FB;

    for (int i = tid; i < a.ksteps * FB * 64; i += NT) *reinterpret_cast<u32x4*>(sW + (size_t)i * 16) = u32x4{0u, 0u, 0u, 0u};
    __syncthreads();
    u32x4 rx[XV];
    if ((int)blockIdx.x < a.ntiles) load_raw(a, tile_pos(a, blockIdx.x), rx);
    {
        const bf16_t* wsrc = a.w + (size_t)ch0 * a.Kred;  // 16-byte aligned, a multiple of 16 bytes (channels in eights)
        const int total8 = nch * a.Kred / 8;
        for (int i0 = tid; i0 < total8; i0 += 4 * NT) {
            u32x4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (i0 + u * NT < total8) v[u] = *reinterpret_cast<const u32x4*>(wsrc + (size_t)(i0 + u * NT) * 8);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (i0 + u * NT >= total8) continue;
                const int idx = (i0 + u * NT) * 8;
                int ch = (int)fdiv((uint32_t)idx, a.dKred), k = idx - ch * a.Kred;
                int r = (int)fdiv((uint32_t)k, a.dSC), sc = k - r * (a.S * a.C);
                int s = (int)fdiv((uint32_t)sc, a.dC), c = sc - s * a.C;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int gi = r * a.G + (s >> 1);
                    *reinterpret_cast<unsigned short*>(
                        sW + ((size_t)((((gi >> 1) * FB + (ch >> 5)) * 64) + (gi & 1) * 32 + (ch & 31)) * 8 + (s & 1) * 4 + c) * 2) =
                        (unsigned short)((e & 1) ? v[u][e >> 1] >> 16 : v[u][e >> 1] & 0xffffu);
                    if (++c == a.C) {
                        c = 0;
                        if (++s == a.S) {
                            s = 0;
                            if (++r == a.R) { r = 0; ++ch; }
                        }
                    }
                }
            }
        }
    }
    unsigned char* const st = sO + wave * 32 * OPITCH;
    for (int tile = blockIdx.x; tile < a.ntiles; tile += gridDim.x) {
        const TilePos tp = tile_pos(a, tile);
        store_raw(a, rx, sR);
        __syncthreads();
        widen(a, tp, sR, sX);
        if (tile + (int)gridDim.x < a.ntiles) load_raw(a, tile_pos(a, tile + gridDim.x), rx);
        __syncthreads();
        const int oh = tp.oh0 + wave;
        if (oh < a.OH) {
            f32x16 acc[FB];
#pragma unroll
            for (int b = 0; b < FB; ++b)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[b][e] = 0.f;
            const unsigned char* xrow = sX + ((size_t)wave * a.sh * a.xw + l32 * a.sw) * 8;
            int r = 0, sp = half;  // this half-wavefront's tap pair
            if (sp >= a.G) { sp -= a.G; ++r; }
            for (int ks = 0; ks < a.ksteps; ++ks) {
                // beyond the filter (the second pixel of an odd row's last pair, the pair behind the last row) the patch
                // holds real pixels of other taps: zeroed, for a zero weight does not cancel an infinity
                const bool in_r = r < a.R, in_s1 = in_r && 2 * sp + 1 < a.S;
                const unsigned char* xa = xrow + ((in_r ? r : 0) * a.xw + 2 * sp) * 8;
                const u32x2 lo = *reinterpret_cast<const u32x2*>(xa);
                const u32x2 hi = *reinterpret_cast<const u32x2*>(xa + 8);
                const u32x4 xv = {in_r ? lo[0] : 0u, in_r ? lo[1] : 0u, in_s1 ? hi[0] : 0u, in_s1 ? hi[1] : 0u};
                const bf16x8 xf = __builtin_bit_cast(bf16x8, xv);
#pragma unroll
                for (int b = 0; b < FB; ++b) {
                    const bf16x8 wf = *reinterpret_cast<const bf16x8*>(sW + (size_t)((ks * FB + b) * 64 + lane) * 16);
                    acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, xf, acc[b], 0, 0, 0);
                }
                sp += 2;
                if (sp >= a.G) { sp -= a.G; ++r; }
                if (sp >= a.G) { sp -= a.G; ++r; }
            }
            // accumulator register i of block b: channel b*32 + (i/4)*8 + half*4 + i%4 of pixel l32
#pragma unroll
            for (int b = 0; b < FB; ++b)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int ch = b * 32 + q * 8 + half * 4;
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = acc[b][q * 4 + e];
                    if (a.bias) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] += ch < nch ? a.bias[ch0 + ch + e] : 0.f;
                    }
                    if (a.relu) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
                    }
                    *reinterpret_cast<uint2*>(st + l32 * OPITCH + ch * 2) =
                        make_uint2((unsigned)f2bf(v[0]) | ((unsigned)f2bf(v[1]) << 16),
                                   (unsigned)f2bf(v[2]) | ((unsigned)f2bf(v[3]) << 16));
                }
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the strip is private to this wavefront
            bf16_t* yrow = a.y + ((size_t)(tp.n * a.OH + oh) * a.OW + tp.ow0) * a.K + ch0;
#pragma unroll
            for (int it = 0; it < 32 * VPR / 64; ++it) {
                const int v = it * 64 + lane;
                const int px = v / VPR, vec = v % VPR;
                const u32x4 val = *reinterpret_cast<const u32x4*>(st + px * OPITCH + vec * 16);
                if (tp.ow0 + px < a.OW && vec * 8 < nch) *reinterpret_cast<u32x4*>(yrow + (size_t)px * a.K + vec * 8) = val;
            }
        }
        __syncthreads();  // the patch (and this wavefront's strip) may be overwritten
    }
}

// ---- weight gradient.  FB: 32-channel blocks of dy per work-group (blockIdx.y), JB: 32-column blocks per wavefront, PG:
// wavefronts that share the same columns and divide the tile's rows (small filters have few column blocks); 4 / PG
// wavefronts divide the columns.  One fp32 partial per work-group, added up in a fixed order by the caller. ----
template <int FB, int JB, int PG>
__global__ __launch_bounds__(NT, 2) void wgrad_thin_kernel(const ThinArgs a) {
    constexpr int BG = 4 / PG;
    constexpr int DPITCH = FB * 64 + 64;  // transposing reads: 4 rows x 64 bytes in disjoint bank groups
    constexpr int VPR = FB * 4;
    extern __shared__ __align__(16) unsigned char smem_t[];
    unsigned char* const sD = smem_t;                       // [TR * TW][DPITCH]
    unsigned char* const sX = sD + (size_t)TR * TW * DPITCH;
    unsigned char* const sR = sX + (size_t)(a.npx + 1) / 2 * 16;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int half = lane >> 5, l32 = lane & 31;
    const int bg = wave % BG, pg = wave / BG;
    const int ch0 = blockIdx.y * 32 * FB;
    const int nch = a.K - ch0 < 32 * FB ? a.K - ch0 : 32 * FB;

    const int kl = half * 8 + ((lane & 15) >> 2);              // this lane's pixel of a 16-pixel step (transposing read)
    const int tap8 = ((lane >> 4) & 1) * 4 + (lane & 3);       // and its tap of a 32-column block
    const int ccol = (((lane >> 4) & 1) * 16 + (lane & 3) * 4) * 2;
    int xo[JB];
#pragma unroll
    for (int j = 0; j < JB; ++j) {
        int t = (j * BG + bg) * 8 + tap8;
        if (t >= a.R * a.S) t = 0;  // columns past the filter: any readable address, the sums are dropped
        const int r = (int)fdiv((uint32_t)t, a.dS), s = t - r * a.S;
        xo[j] = (r * a.xw + s + kl * a.sw) * 8;
    }
    f32x16 acc[JB][FB];
#pragma unroll
    for (int j = 0; j < JB; ++j)
#pragma unroll
        for (int b = 0; b < FB; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[j][b][e] = 0.f;

    u32x4 rx[XV], dv[2 * FB];
    auto load_tile = [&](const TilePos& tp) {  // dy of the tile, zero beyond the last row, pixel and channel; the raw patch
#pragma unroll
        for (int i = 0; i < 2 * FB; ++i) {
            const int v = tid + i * NT;
            const int p = v / VPR, vec = v % VPR;
            const int oh = tp.oh0 + p / TW, ow = tp.ow0 + p % TW;
            const bool ok = oh < a.OH && ow < a.OW && vec * 8 < nch;
            dv[i] = *reinterpret_cast<const u32x4*>(
                ok ? a.dy + ((size_t)(tp.n * a.OH + oh) * a.OW + ow) * a.K + ch0 + vec * 8 : reinterpret_cast<const bf16_t*>(g_zero_block_thin));
        }
        load_raw(a, tp, rx);
    };
    if ((int)blockIdx.x < a.ntiles) load_tile(tile_pos(a, blockIdx.x));
    for (int tile = blockIdx.x; tile < a.ntiles; tile += gridDim.x) {
        const TilePos tp = tile_pos(a, tile);
        store_raw(a, rx, sR);
#pragma unroll
        for (int i = 0; i < 2 * FB; ++i) {
            const int v = tid + i * NT;
            *reinterpret_cast<u32x4*>(sD + (v / VPR) * DPITCH + (v % VPR) * 16) = dv[i];
        }
        __syncthreads();
        widen(a, tp, sR, sX);
        if (tile + (int)gridDim.x < a.ntiles) load_tile(tile_pos(a, tile + gridDim.x));
        __syncthreads();
#pragma unroll
        for (int rr = 0; rr < TR / PG; ++rr) {
            const int row = rr * PG + pg;
            if (tp.oh0 + row >= a.OH) continue;  // uniform
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int nvalid = a.OW - tp.ow0 - h * 16;  // pixels of this step inside the row
                if (nvalid <= 0) continue;
                const unsigned char* d0 = sD + (row * TW + h * 16 + kl) * DPITCH + ccol;
                bf16x8 fd[FB];
#pragma unroll
                for (int b = 0; b < FB; ++b) fd[b] = __builtin_bit_cast(bf16x8, tr_pair(d0 + b * 64, d0 + 4 * DPITCH + b * 64));
                const unsigned char* x0 = sX + ((size_t)row * a.sh * a.xw + h * 16 * a.sw) * 8;
#pragma unroll
                for (int j = 0; j < JB; ++j) {
                    if (j * BG + bg >= a.NB) continue;  // uniform
                    u32x4 fx = tr_pair(x0 + xo[j], x0 + xo[j] + 32 * a.sw);
                    if (nvalid < 16) {  // pixels past the row end: zeroed, for a zero dy does not cancel an infinity
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            const unsigned lo = half * 8 + 2 * e < nvalid ? 0xffffu : 0u;
                            const unsigned hi = half * 8 + 2 * e + 1 < nvalid ? 0xffff0000u : 0u;
                            fx[e] &= lo | hi;
                        }
                    }
#pragma unroll
                    for (int b = 0; b < FB; ++b)
                        acc[j][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fx), fd[b], acc[j][b], 0, 0, 0);
                }
            }
        }
        __syncthreads();  // the tile may be overwritten
    }

    // Epilogue: accumulator register i holds column (i/4)*8 + half*4 + i%4 of the block for output channel b*32 + l32.  One
    // block of every wavefront at a time passes through LDS, the PG wavefronts of a column group are added in order.
    float* const red = reinterpret_cast<float*>(smem_t);  // [4 wavefronts][32 columns][33]
    float* const outp = a.part + (size_t)blockIdx.x * a.K * a.Kred;
#pragma unroll
    for (int j = 0; j < JB; ++j)
#pragma unroll
        for (int b = 0; b < FB; ++b) {
#pragma unroll
            for (int i = 0; i < 16; ++i) red[(wave * 32 + (i >> 2) * 8 + half * 4 + (i & 3)) * 33 + l32] = acc[j][b][i];
            __syncthreads();
#pragma unroll
            for (int it = 0; it < 4 * BG; ++it) {
                const int o = it * NT + tid;
                const int col = o & 31, ch = (o >> 5) & 31, grp = o >> 10;
                float s = red[(grp * 32 + col) * 33 + ch];
#pragma unroll
                for (int p = 1; p < PG; ++p) s += red[((p * BG + grp) * 32 + col) * 33 + ch];
                const int t = (j * BG + grp) * 8 + (col >> 2), c = col & 3;
                if (t < a.R * a.S && c < a.C && b * 32 + ch < nch) outp[(size_t)(ch0 + b * 32 + ch) * a.Kred + t * a.C + c] = s;
            }
            __syncthreads();
        }
}

// ---- host side ----
struct ThinShape {
    int H, W, C, K, OH, OW, R, S, sh, sw, ph, pw, N;
};
ThinShape shape_of(const GemmGeom& g) {
    return {g.IH, g.IW, g.IC, g.Ncols, g.OH, g.OW, g.R, g.S, g.mul_h, g.mul_w, g.pad_h, g.pad_w, g.M / (g.OH * g.OW)};
}
ThinShape shape_of(const WgradGeom& g) { return {g.H, g.W, g.C, g.K, g.P, g.Q, g.R, g.S, g.sh, g.sw, g.ph, g.pw, g.N}; }
long thin_tiles(const ThinShape& s) { return (long)s.N * ((s.OH + TR - 1) / TR) * ((s.OW + TW - 1) / TW); }
// (in 64 bits: strides are bounded by int32 only)
long thin_xw(const ThinShape& s) { return (long)(TW - 1) * s.sw + (s.S + 1) / 2 * 2; }
long thin_rows(const ThinShape& s) { return (long)(TR - 1) * s.sh + s.R; }
long thin_npx(const ThinShape& s) { return thin_rows(s) * thin_xw(s); }
long thin_nv(const ThinShape& s) { return (thin_xw(s) * s.C + 7 + 7) / 8; }  // up to seven elements in front of the patch
size_t thin_patch_smem(const ThinShape& s) { return (size_t)((thin_npx(s) + 1) / 2 * 16 + thin_rows(s) * thin_nv(s) * 16); }
size_t thin_fwd_strips(int fb) { return (size_t)4 * 32 * (fb * 64 + 16); }
// What the choice between kernels goes by: its lines were fitted with the strips apart from the raw patch, where fewer
// work-groups are resident.
size_t thin_fwd_apart(const ThinShape& s, int fb) {
    const size_t ksteps = ((size_t)s.R * ((s.S + 1) / 2) + 1) / 2;
    return ksteps * fb * 1024 + thin_fwd_strips(fb) + thin_patch_smem(s);
}
size_t thin_fwd_smem(const ThinShape& s, int fb) {
    return thin_fwd_apart(s, fb) - std::min(thin_fwd_strips(fb), (size_t)(thin_rows(s) * thin_nv(s) * 16));
}
size_t thin_wgrad_smem(const ThinShape& s, int fb) {
    return std::max((size_t)TR * TW * (fb * 64 + 64) + thin_patch_smem(s), (size_t)4 * 32 * 33 * sizeof(float));
}
bool thin_shape_ok(const ThinShape& s) {
    // (the stride bound keeps the products below in 64 bits, the LDS bounds are far tighter; the last bound: the vectors of
    // a patch may reach behind the tensor, their offsets stay below 2^31)
    return s.C >= 1 && s.C <= 4 && s.K % 8 == 0 && s.R * s.S >= 2 && s.sh < 4096 && s.sw < 4096 &&
           thin_rows(s) * thin_nv(s) <= XV * NT && thin_patch_smem(s) <= 80 * 1024 && thin_tiles(s) < (1L << 30) &&
           (long)s.N * s.H * s.W * s.C <= 2147483647L - XV * NT * 8;
}
// Channel blocks per work-group: all of a thin layer's, so that the patch is staged once, as long as two work-groups per
// CU fit; one each where the tiles alone do not put two work-groups on every CU.
int thin_fwd_fb(const ThinShape& s) {
    const int nb = (s.K + 31) / 32;
    for (int fb : {3, 2})
        if (nb % fb == 0 && thin_tiles(s) * (nb / fb) >= 2 * kNumCU && thin_fwd_apart(s, fb) <= LDS_CAP / 2) return fb;
    return 1;
}
int thin_wgrad_fb(const ThinShape& s) {
    const int nb = (s.K + 31) / 32;
    if (s.R * s.S > 64) return 1;  // four column blocks per wavefront: two channel blocks spill
    return nb % 3 == 0 ? 3 : nb % 2 == 0 ? 2 : 1;
}
ThinArgs thin_args(const ThinShape& s) {
    ThinArgs a = {};
    a.H = s.H; a.W = s.W; a.C = s.C; a.K = s.K; a.OH = s.OH; a.OW = s.OW; a.R = s.R; a.S = s.S;
    a.sh = s.sh; a.sw = s.sw; a.ph = s.ph; a.pw = s.pw;
    a.Kred = s.R * s.S * s.C;
    a.tiles_x = (s.OW + TW - 1) / TW;
    a.tiles_y = (s.OH + TR - 1) / TR;
    a.ntiles = (int)thin_tiles(s);
    a.G = (s.S + 1) / 2;
    a.ksteps = (s.R * a.G + 1) / 2;
    a.NB = (s.R * s.S + 7) / 8;
    a.xw = (int)thin_xw(s);
    a.npx = (int)thin_npx(s);
    a.dTX = make_fastdiv((uint32_t)a.tiles_x);
    a.dTY = make_fastdiv((uint32_t)a.tiles_y);
    a.dXW = make_fastdiv((uint32_t)a.xw);
    a.nv = (int)thin_nv(s);
    a.nvec = (int)thin_rows(s) * a.nv;
    a.rpitch = a.nv * 16;
    a.x_elems = (int)((long)s.N * s.H * s.W * s.C);
    a.dNV = make_fastdiv((uint32_t)a.nv);
    a.dKred = make_fastdiv((uint32_t)a.Kred);
    a.dSC = make_fastdiv((uint32_t)(s.S * s.C));
    a.dC = make_fastdiv((uint32_t)s.C);
    a.dS = make_fastdiv((uint32_t)s.S);
    return a;
}
template <typename F>
int thin_attr(F kfn, std::atomic<bool>& done) {
    if (!done) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn), hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_CAP);
        if (e != hipSuccess) return set_error(WAP_EHIP, "hipFuncSetAttribute: %s", hipGetErrorString(e));
        done = true;
    }
    return WAP_OK;
}
template <int FB>
int launch_fwd_t(const ThinArgs& a, dim3 grid, size_t smem, hipStream_t st) {
    static std::atomic<bool> done{false};
    int rc = thin_attr(conv_thin_fwd_kernel<FB>, done);
    if (rc != WAP_OK) return rc;
    hipLaunchKernelGGL(conv_thin_fwd_kernel<FB>, grid, dim3(NT), smem, st, a);
    return check_launch("conv_thin_fwd");
}
template <int FB, int JB, int PG>
int launch_wgrad_t(const ThinArgs& a, dim3 grid, size_t smem, hipStream_t st) {
    static std::atomic<bool> done{false};
    int rc = thin_attr(wgrad_thin_kernel<FB, JB, PG>, done);
    if (rc != WAP_OK) return rc;
    hipLaunchKernelGGL((wgrad_thin_kernel<FB, JB, PG>), grid, dim3(NT), smem, st, a);
    return check_launch("wgrad_thin");
}

}  // namespace

bool conv_thin_fwd_supported(const GemmGeom& g) {
    if (g.div_h != 1 || g.div_w != 1) return false;
    const ThinShape s = shape_of(g);
    return thin_shape_ok(s) && thin_fwd_apart(s, 1) <= LDS_CAP;
}

int launch_conv_thin_fwd(const GemmGeom& g, const bf16_t* x, const bf16_t* w, const float* bias, bool relu, bf16_t* y,
                         hipStream_t st) {
    if (!conv_thin_fwd_supported(g)) return set_error(WAP_EINVAL, "internal: few-channel forward kernel not applicable");
    const ThinShape s = shape_of(g);
    ThinArgs a = thin_args(s);
    a.x = x; a.w = w; a.bias = bias; a.y = y; a.relu = relu ? 1 : 0;
    const int fb = thin_fwd_fb(s);
    const size_t smem = thin_fwd_smem(s, fb);
    const int groups = (s.K + 32 * fb - 1) / (32 * fb);
    // every work-group brings the weights into fragment order once: as many as are resident together, then tile after tile
    const long per_cu = std::min<long>(4, std::max<long>(1, (long)(LDS_CAP / smem)));
    const dim3 grid((unsigned)std::min<long>(a.ntiles, std::max<long>(1, per_cu * kNumCU / groups)), (unsigned)groups);
    if (fb == 3) return launch_fwd_t<3>(a, grid, smem, st);
    if (fb == 2) return launch_fwd_t<2>(a, grid, smem, st);
    return launch_fwd_t<1>(a, grid, smem, st);
}

// Preferred to the kernel for horizontal strides of 4 (which takes the same time up to some tiles per CU): while all tiles
// are resident at once, with two channel blocks for a second round.  11x11 at stride 4, us, that kernel / this one: 16 x
// 112x112 -> 32 15.9 / 14.3, 16 x 160x160 -> 32 (two rounds) 16.4 / 21.5, 16 x 112x112 -> 64 19.8 / 14.7, 8 x 224x224 -> 64
// (two rounds) 20.5 / 21.9 with its operands cached and 26.7 / 23.0 without; 4x4 at stride 4, 64 x 96x96 -> 32 8.0 / 7.6.
bool conv_thin_fwd_few_tiles(const GemmGeom& g) {
    if (!conv_thin_fwd_supported(g)) return false;
    const ThinShape s = shape_of(g);
    const long nb = (s.K + 31) / 32, resident = std::min<long>(2, (long)(LDS_CAP / thin_fwd_apart(s, 1)));
    return thin_tiles(s) * nb <= kNumCU * std::min<long>(2, std::max(nb, resident));
}

// Preferred to the gather-based kernel (32 or 64 channels): that one fetches every reduction step of 16 from memory, this one
// stages a patch per tile whatever the filter, so a short reduction, a ragged map or a large stride speaks for the gather.
// While one round of work-groups does it, only the start counts (3x3 stride 3, 16 x 33x33 -> 32 3.5 us with the gather, 5.5
// here; 5x5, 1 image of 48x48 -> 64 6.0 / 5.5; 7x7 -> 32 and 64 1.01 and 1.2 times faster here; 9x9 stride 2, 4 x 130x130 -> 64,
// two work-groups per CU, 15.2 / 11.4).  Beyond, the two times as fitted over 300 shapes (mean error 6 % with one channel
// block, 13 % with two): so much per 128 pixels and reduction step there, per tile, staged pixel and step of tap pairs here,
// and this kernel's later start.  us, gather / this one: 3x3 stride 2, 64 x 130x130 -> 64 16.6 / 25.2; 5x5 stride 2, 64 x
// 192x192 -> 32 46.9 / 26.1; 7x7 stride 2, 25 x 71x71 -> 64 (36 of 64 columns) 10.6 / 13.5, 64 x 224x224 -> 64 124 / 90.  With two
// channel blocks and one work-group per CU (11x11 at stride 4) nothing hides the staging: 32 x 224x224 -> 64 52 / 60.  Over
// 1166 shapes the choice is 0.4 % from the better of the two on average.
bool conv_thin_fwd_over_gather(const GemmGeom& g) {
    if (!conv_thin_fwd_supported(g)) return false;
    const ThinShape s = shape_of(g);
    const long tiles = thin_tiles(s), nb = (s.K + 31) / 32, ksteps = (g.Kred + 15) / 16;
    const bool alone = 2 * thin_fwd_apart(s, 1) > LDS_CAP;  // one work-group per CU
    if (tiles * nb <= kNumCU) return ksteps >= (nb == 1 ? 10 : 5);
    if (tiles * nb <= (alone ? 1 : 2) * kNumCU && ksteps >= (nb == 1 ? 16 : 10)) return true;
    if (alone && nb > 1) return false;
    const double pairs = (s.R * ((s.S + 1) / 2) + 1) / 2, staged = (double)thin_npx(s);
    const double gather = g.M / (double)(TR * TW) * (nb == 1 ? 1.0 + 1.7 * ksteps : 0.6 + 2.1 * ksteps);  // ns, as below
    const double here = tiles * (nb == 1 ? 0.3 + 0.00245 * staged + 0.32 * pairs : 0.4 + 0.0042 * staged + 0.55 * pairs) +
                        (nb == 1 ? 2100.0 : 1400.0);
    return 1.03 * here <= gather;
}

bool wgrad_thin_supported(const WgradGeom& g) {
    const ThinShape s = shape_of(g);
    return thin_shape_ok(s) && s.R * s.S <= 128;
}
// Preferred to the kernel for horizontal strides of 4, us, that one / this: two channel blocks, 11x11, 8 x 224x224 -> 64 29.7 /
// 25.2, 16 x 160x160 28.2 / 28.1, 32 x 224x224 32.9 / 46.5; one block, whose work-groups hold half the products for the same
// patch, 4 x 224x224 -> 32 22.4 / 17.1, 8 x 160x160 18.9 / 18.0, 64 x 96x96 21.2 / 26.3; 4x4, 16 x 224x224 -> 32 14.2 / 12.0.
bool wgrad_thin_few_tiles(const WgradGeom& g) {
    const long nb = (g.K + 31) / 32;
    return wgrad_thin_supported(g) &&
           thin_tiles(shape_of(g)) * nb <= (nb == 1 && g.R * g.S > 16 ? kNumCU / 2 : 2 * kNumCU);
}

// Work-groups along the tiles, each of which leaves a K x R*S*C fp32 partial: two per CU over all channel groups, but no
// more than 24 MB of partial sums together (11x11, 8 x 224x224 -> 64, whose work-groups then have one tile instead of two: 24.1 us
// with 16 MB, its sums 4.8; 19.7 and 6.0 with 24).
int wgrad_thin_nsplit(const WgradGeom& g) {
    const ThinShape s = shape_of(g);
    const int fb = thin_wgrad_fb(s), groups = (s.K + 32 * fb - 1) / (32 * fb);
    const long bytes = (long)s.K * s.R * s.S * s.C * 4;
    const long cap = std::max<long>(1, std::min<long>(2 * kNumCU / groups, (24L << 20) / bytes));
    const long tiles = thin_tiles(s);
    if (tiles <= cap) return (int)tiles;
    const long per = (tiles + cap - 1) / cap;  // the same number of tiles for (nearly) every work-group
    return (int)((tiles + per - 1) / per);
}

int launch_wgrad_thin(const WgradGeom& g, int nsplit, const bf16_t* x, const bf16_t* dy, float* part, hipStream_t st) {
    if (!wgrad_thin_supported(g) || nsplit < 1 || nsplit > thin_tiles(shape_of(g)))
        return set_error(WAP_EINVAL, "internal: few-channel weight-gradient kernel not applicable");
    const ThinShape s = shape_of(g);
    ThinArgs a = thin_args(s);
    a.x = x; a.dy = dy; a.part = part;
    const int fb = thin_wgrad_fb(s);
    const size_t smem = thin_wgrad_smem(s, fb);
    const dim3 grid((unsigned)nsplit, (unsigned)((s.K + 32 * fb - 1) / (32 * fb)));
#define WAP_THIN(FB)                                                                       \
    (a.NB <= 2 ? launch_wgrad_t<FB, 2, 4>(a, grid, smem, st)                                \
               : a.NB <= 4 ? launch_wgrad_t<FB, 2, 2>(a, grid, smem, st) : launch_wgrad_t<FB, 2, 1>(a, grid, smem, st))
    if (a.NB > 8) return launch_wgrad_t<1, 4, 1>(a, grid, smem, st);
    return fb == 3 ? WAP_THIN(3) : fb == 2 ? WAP_THIN(2) : WAP_THIN(1);
#undef WAP_THIN
}

}  // namespace wap
