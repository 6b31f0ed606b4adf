// Data gradient of a convolution whose INPUT has very few channels (the 3-channel image of the first layer):
//   dx[n,h,w,c] = sum over (k,r,s) of dy[n,p,q,k] * w[k,r,s,c]   with p*stride_h - pad_h + r = h, q likewise,
// the backward half of t_c (Eq. 1) of the first "primary" node of Section 3.2.2.
//
// As a product with one row per image pixel it has 3 (at most 4) columns, nine tenths of an MFMA tile would be padding.
// Turned around it is a good one: z[p,q][(r,s,c)] = sum over k of dy[p,q,k] * w[k,r,s,c] has one row per dy pixel and
// R*S*C columns (27 of 32 for a 3x3 filter), its operand dy is read as it lies in memory, and dx is the sum of the R*S
// values of z that land on a pixel.  z never leaves the LDS:
//   * a work-group (4 wavefronts) owns TH x TW pixels of dx; the filter is walked in groups of rows (and of taps of a
//     row, and of 64 channels) whose columns fit up to four 32-column blocks, e.g. the whole 3x3 filter in one block;
//   * for each group the wavefronts make z for the dy pixels under the tile, 32 pixels at a time: the pixel fragments
//     come straight from global memory (16 bytes of a pixel per lane, neighbouring pixels adjacent), the weight fragments
//     from the LDS, where the work-group put them in fragment order; out-of-image pixels load zeros;
//   * then each thread adds up the values of its PX pixels: for a stride above one only the taps that meet the pixel's
//     row and column phase.  The order of all sums is fixed: bitwise reproducible.
// Bound by reading dy once (plus the tiles' halo, from L2) for 3 x 3 filters: 64 channels at 224 x 224, minibatch 24
// (154 MB) 262 us on the vector ALUs (each dy element read once per tap, three multiply-adds each), now 44 us, 3.7 TB/s;
// for large strided filters by the latency of the groups' load - product - sum phases: 11 x 11 / 4 at minibatch 32 299 to
// 72 us (weights gathered with branches around the loads instead of out-of-range offsets: 123 us; one filter row per
// group: 131 us).
#include <algorithm>

#include "wap_internal.h"

namespace wap {

namespace {

constexpr int NT = 256;
constexpr int KC = 64;  // dy channels per pass: four MFMA reduction steps

struct ThinArgs {
    const bf16_t* dy;   // [N][IH][IW][K]
    const bf16_t* w;    // [K][R][S][C]
    bf16_t* dx;         // [N][OH][OW][C]
    int N, IH, IW, K, OH, OW, R, S, sh, sw, ph, pw;  // ph / pw: the forward pass's padding
    unsigned dy_bytes;       // below 2 GiB (host)
    int rg, sg;              // filter rows / taps of a row per group
    int zh, zw, zgroups;     // dy rows / columns under a tile for one group, 32-pixel groups of them
    int zp;                  // floats per z row: the columns rounded up to an odd number of 16-byte units (all banks)
    int tiles_w, tiles;      // tiles per row of dx, in all
    FastDiv dTW, dTI, dZW, dSH, dSW;   // division by tiles per row, tiles per image, zw, the strides
    int tiles_img;
};

__device__ __forceinline__ unsigned short f2bf(float f) {
    __bf16 b = (__bf16)f;
    return __builtin_bit_cast(unsigned short, b);
}

// smallest integer >= a / b for any a, b >= 1
__device__ __forceinline__ int ceil_div(int a, int b) { return a >= 0 ? (a + b - 1) / b : -((-a) / b); }

// C: channels of dx; NB: 32-column blocks of z; PX: pixels per thread (a tile is 8 x 32 for one, 16 x 64 for four)
template <int C, int NB, int PX>
__global__ __launch_bounds__(NT) void dgrad_thin_kernel(const ThinArgs a) {
    constexpr int TH = PX == 1 ? 8 : 16, TW = PX == 1 ? 32 : 64;
    constexpr int WF = NB * (KC / 16) * 64;  // 16-byte weight fragments of a group
    extern __shared__ __align__(16) unsigned char smem[];
    u32x4* const wf = reinterpret_cast<u32x4*>(smem);
    float* const z = reinterpret_cast<float*>(smem + WF * 16);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int ngr = (a.R + a.rg - 1) / a.rg, ngs = (a.S + a.sg - 1) / a.sg, nkc = (a.K + KC - 1) / KC;
    const int ngroups = ngr * ngs * nkc;
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.dy), 0, (int)a.dy_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrcW =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.w), 0, (int)((unsigned)a.K * a.R * a.S * C * 2u), 0x00020000);

    bool weights_in = false;
    for (int tile = blockIdx.x; tile < a.tiles; tile += gridDim.x) {
        const int n = (int)fdiv((uint32_t)tile, a.dTI);
        const int ti = tile - n * a.tiles_img;
        const int th = (int)fdiv((uint32_t)ti, a.dTW);
        const int h0 = th * TH, w0 = (ti - th * a.tiles_w) * TW;
        float acc[PX][C];
#pragma unroll
        for (int i = 0; i < PX; ++i)
#pragma unroll
            for (int c = 0; c < C; ++c) acc[i][c] = 0.f;
        // a pixel's row h meets the taps r = rf + sh * i at the dy rows hd - i, its column the taps sf + sw * j at wd - j
        int rf[PX], hd[PX], sf[PX], wd[PX];
#pragma unroll
        for (int i = 0; i < PX; ++i) {
            const int pix = tid + i * NT;
            const int hp = h0 + pix / TW + a.ph, wp = w0 + pix % TW + a.pw;
            hd[i] = (int)fdiv((uint32_t)hp, a.dSH);
            rf[i] = hp - hd[i] * a.sh;
            wd[i] = (int)fdiv((uint32_t)wp, a.dSW);
            sf[i] = wp - wd[i] * a.sw;
        }

        for (int grp = 0; grp < ngroups; ++grp) {
            const int k0 = (grp % nkc) * KC;
            const int s0 = (grp / nkc % ngs) * a.sg, r0 = grp / (nkc * ngs) * a.rg;
            const int rg = a.R - r0 < a.rg ? a.R - r0 : a.rg, sg = a.S - s0 < a.sg ? a.S - s0 : a.sg;
            // ---- weights of the group in fragment order: [block][reduction step][lane][8 channels], zero beyond ----
            if (ngroups > 1 || !weights_in) {
                unsigned short* const wl = reinterpret_cast<unsigned short*>(smem);
                // a thread keeps its column, so that neighbouring threads read runs of w; all its loads are in flight
                constexpr int KSTEP = NT / (NB * 32);
                const int col = tid % (NB * 32), kt = tid / (NB * 32);
                const int r = col / (sg * C);
                const bool in = r < rg;
                const unsigned row = (unsigned)(a.R * a.S * C) * 2u;
                const unsigned src = (unsigned)(k0 + kt) * row + (unsigned)((r0 + r) * (a.S * C) + s0 * C + (col - r * (sg * C))) * 2u;
                unsigned short v[KC / KSTEP];
#pragma unroll
                for (int i = 0; i < KC / KSTEP; ++i)
                    v[i] = __builtin_amdgcn_raw_buffer_load_b16(
                        rsrcW, in && k0 + kt + i * KSTEP < a.K ? src + (unsigned)(i * KSTEP) * row : 0x80000000u, 0, 0);
#pragma unroll
                for (int i = 0; i < KC / KSTEP; ++i) {
                    const int k = kt + i * KSTEP;
                    // lane = column within the block + 32 * (half of the 16-deep step)
                    wl[((((col >> 5) * (KC / 16) + (k >> 4)) * 64) + (col & 31) + ((k >> 3) & 1) * 32) * 8 + (k & 7)] = v[i];
                }
                weights_in = true;
            }
            __syncthreads();  // weights in place; the previous group's z is read
            // ---- z for the dy pixels under the tile ----
            const int p_lo = ceil_div(h0 + a.ph - (r0 + rg - 1), a.sh), q_lo = ceil_div(w0 + a.pw - (s0 + sg - 1), a.sw);
            for (int g = wave; g < a.zgroups; g += NT / 64) {
                const int px = g * 32 + (lane & 31);
                const int pr = (int)fdiv((uint32_t)px, a.dZW), pc = px - pr * a.zw;
                const int p = p_lo + pr, q = q_lo + pc;
                const bool in = pr < a.zh && (unsigned)p < (unsigned)a.IH && (unsigned)q < (unsigned)a.IW;
                const int kk = k0 + (lane >> 5) * 8;
                const unsigned base = (unsigned)(((n * a.IH + p) * a.IW + q) * a.K + kk) * 2u;
                bf16x8 fd[KC / 16];
#pragma unroll
                for (int ks = 0; ks < KC / 16; ++ks)  // outside the image or beyond K: beyond the buffer, i.e. zeros
                    fd[ks] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                                                            rsrc, in && kk + ks * 16 < a.K ? base + ks * 32u : 0x80000000u, 0, 0));
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    f32x16 d;
#pragma unroll
                    for (int e = 0; e < 16; ++e) d[e] = 0.f;
#pragma unroll
                    for (int ks = 0; ks < KC / 16; ++ks)
                        d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                            __builtin_bit_cast(bf16x8, wf[(b * (KC / 16) + ks) * 64 + lane]), fd[ks], d, 0, 0, 0);
#pragma unroll
                    for (int q4 = 0; q4 < 4; ++q4) {
                        const int col = b * 32 + q4 * 8 + (lane >> 5) * 4;
                        if (col < a.zp)
                            *reinterpret_cast<float4*>(z + px * a.zp + col) =
                                make_float4(d[q4 * 4], d[q4 * 4 + 1], d[q4 * 4 + 2], d[q4 * 4 + 3]);
                    }
                }
            }
            __syncthreads();
            // ---- the taps of the group that land on this thread's pixels ----
            const int ri = r0 / a.sh, rb = r0 - ri * a.sh, sj = s0 / a.sw, sb = s0 - sj * a.sw;
#pragma unroll
            for (int i = 0; i < PX; ++i) {
                // only taps whose dy pixel (hd - k, wd - j) lies in the image: its z is made of zeros beyond, which do not
                // cancel an infinite weight
                const int j0 = max(sj + (sf[i] < sb ? 1 : 0), wd[i] - a.IW + 1);
                const int s_first = sf[i] + a.sw * j0, s_end = min(s0 + sg, sf[i] + a.sw * wd[i] + 1);
                int k = max(ri + (rf[i] < rb ? 1 : 0), hd[i] - a.IH + 1);
                const int r_end = min(r0 + rg, rf[i] + a.sh * hd[i] + 1);
                for (int r = rf[i] + a.sh * k; r < r_end; r += a.sh, ++k) {
                    const float* src = z + ((hd[i] - k - p_lo) * a.zw + wd[i] - j0 - q_lo) * a.zp + ((r - r0) * sg + s_first - s0) * C;
                    for (int s = s_first; s < s_end; s += a.sw) {
#pragma unroll
                        for (int c = 0; c < C; ++c) acc[i][c] += src[c];
                        src += a.sw * C - a.zp;  // the next tap of this phase meets the dy pixel to the left
                    }
                }
            }
        }
#pragma unroll
        for (int i = 0; i < PX; ++i) {
            const int pix = tid + i * NT;
            const int h = h0 + pix / TW, wq = w0 + pix % TW;
            if (h < a.OH && wq < a.OW) {
                bf16_t* dst = a.dx + ((size_t)(n * a.OH + h) * a.OW + wq) * C;
#pragma unroll
                for (int c = 0; c < C; ++c) dst[c] = f2bf(acc[i][c]);
            }
        }
    }
}

// 3x3, stride 1, up to 64 channels of dy, whose 9 * C columns are one block: the whole product is one group, so
//   * the weight fragments stay in registers (the LDS holds z alone, four work-groups per CU instead of three), and
//   * the dy pixels of the next tile are fetched while the sums of the present one are made: a wavefront waited for its loads at
//     every tile, 12 KB of them in flight in its turn.
// 24 x 224 x 224 x 64 (154 MB) behind the pass that wrote it 59 -> 48 us (3.2 TB/s), bitwise the same.
constexpr int GW = 3;  // 32-pixel groups of a wavefront: 10 x 34 pixels lie under a tile, 11 groups

template <int C>
__global__ __launch_bounds__(NT, 4) void dgrad_thin_kernel(const ThinArgs a) {
    constexpr int TH = 8, TW = 32, ZH = TH + 2, ZW = TW + 2, KS = KC / 16;
    constexpr int ZU = (9 * C + 3) / 4, ZP = (ZU | 1) * 4;  // floats per z row: an odd number of 16-byte units
    static_assert((ZH * ZW + 31) / 32 <= GW * (NT / 64) && 9 * C <= 32, "one group");
    extern __shared__ __align__(16) unsigned char smem[];
    float* const z = reinterpret_cast<float*>(smem);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.dy), 0, (int)a.dy_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrcW =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.w), 0, (int)((unsigned)a.K * 9u * C * 2u), 0x00020000);
    auto lds_barrier = [&]() {  // leaves loads from memory in flight
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    // pixels of the groups of this wavefront, relative to the tile's first dy pixel, the same for all tiles
    int prow[GW], pcol[GW];
#pragma unroll
    for (int j = 0; j < GW; ++j) {
        const int px = (wave + j * (NT / 64)) * 32 + (lane & 31);
        prow[j] = px / ZW;
        pcol[j] = px - prow[j] * ZW;
        if (prow[j] >= ZH) prow[j] = -0x10000;  // above every image
    }
    const int kk = (lane >> 5) * 8;
    auto origin = [&](int tile, int* n, int* h0, int* w0) {
        *n = (int)fdiv((uint32_t)tile, a.dTI);
        const int ti = tile - *n * a.tiles_img, th = (int)fdiv((uint32_t)ti, a.dTW);
        *h0 = th * TH;
        *w0 = (ti - th * a.tiles_w) * TW;
    };
    bf16x8 fd[GW][KS];
    auto load_dy = [&](int tile) {
        int n, h0, w0;
        origin(tile, &n, &h0, &w0);
#pragma unroll
        for (int j = 0; j < GW; ++j) {
            const int p = h0 + a.ph - 2 + prow[j], q = w0 + a.pw - 2 + pcol[j];
            const bool in = tile < a.tiles && (unsigned)p < (unsigned)a.IH && (unsigned)q < (unsigned)a.IW;
            const unsigned base = (unsigned)(((n * a.IH + p) * a.IW + q) * a.K + kk) * 2u;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)  // outside the image or beyond K: beyond the buffer, i.e. zeros
                fd[j][ks] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                                                           rsrc, in && kk + ks * 16 < a.K ? base + ks * 32u : 0x80000000u, 0, 0));
        }
    };
    load_dy(blockIdx.x);
    bf16x8 wf[KS];  // column lane & 31, channels 8 * (lane >> 5) .. + 7 of each step; zero beyond
    {
        unsigned short v[KS][8];
        const int col = lane & 31;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int k = ks * 16 + kk + e;
                v[ks][e] = __builtin_amdgcn_raw_buffer_load_b16(rsrcW, col < 9 * C && k < a.K ? (unsigned)(k * 9 * C + col) * 2u : 0x80000000u, 0, 0);
            }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            u32x4 x;
#pragma unroll
            for (int d = 0; d < 4; ++d) x[d] = (unsigned)v[ks][2 * d] | ((unsigned)v[ks][2 * d + 1] << 16);
            wf[ks] = __builtin_bit_cast(bf16x8, x);
        }
    }

    const int trow = tid / TW, tcol = tid % TW;
    for (int tile = blockIdx.x; tile < a.tiles; tile += gridDim.x) {
        int n, h0, w0;
        origin(tile, &n, &h0, &w0);
#pragma unroll
        for (int j = 0; j < GW; ++j) {
            const int g = wave + j * (NT / 64), px = g * 32 + (lane & 31);
            f32x16 d;
#pragma unroll
            for (int e = 0; e < 16; ++e) d[e] = 0.f;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) d = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[ks], fd[j][ks], d, 0, 0, 0);
            if (px < ZH * ZW) {
#pragma unroll
                for (int q4 = 0; q4 < 4; ++q4) {
                    const int col = q4 * 8 + (lane >> 5) * 4;
                    if (col < ZP) *reinterpret_cast<float4*>(z + px * ZP + col) = make_float4(d[q4 * 4], d[q4 * 4 + 1], d[q4 * 4 + 2], d[q4 * 4 + 3]);
                }
            }
        }
        load_dy(tile + gridDim.x);
        __builtin_amdgcn_sched_barrier(0);
        lds_barrier();
        // tap (r, s) of this thread's pixel meets the dy pixel 2 - r rows below and 2 - s right of the first one under it
        const int h = h0 + trow, w = w0 + tcol, hp = h + a.ph, wp = w + a.pw;
        float acc[C];
#pragma unroll
        for (int c = 0; c < C; ++c) acc[c] = 0.f;
#pragma unroll
        for (int r = 0; r < 3; ++r)
#pragma unroll
            for (int t = 0; t < 3; ++t) {
                // only where the dy pixel lies in the image: its z is made of zeros beyond, which do not cancel an infinite weight
                const bool in = (unsigned)(hp - r) < (unsigned)a.IH && (unsigned)(wp - t) < (unsigned)a.IW;
                const float* src = z + ((trow + 2 - r) * ZW + tcol + 2 - t) * ZP + (r * 3 + t) * C;
#pragma unroll
                for (int c = 0; c < C; ++c) acc[c] += in ? src[c] : 0.f;
            }
        if (h < a.OH && w < a.OW) {
            bf16_t* dst = a.dx + ((size_t)(n * a.OH + h) * a.OW + w) * C;
#pragma unroll
            for (int c = 0; c < C; ++c) dst[c] = f2bf(acc[c]);
        }
        lds_barrier();
    }
}

template <int C>
int launch_3x3(const ThinArgs& a, hipStream_t st) {
    constexpr size_t smem = 10 * 34 * (((9 * C + 3) / 4) | 1) * 16;
    constexpr int most = kNumCU * 4;
    const int rounds = (a.tiles + most - 1) / most;
    hipLaunchKernelGGL(dgrad_thin_kernel<C>, dim3((a.tiles + rounds - 1) / rounds), dim3(NT), smem, st, a);
    return check_launch("dgrad_thin");
}

template <int C, int NB, int PX>
int launch_one(const ThinArgs& a, size_t smem, hipStream_t st) {
    auto kfn = dgrad_thin_kernel<C, NB, PX>;
    static std::atomic<bool> attr_done{false};
    if (!attr_done) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn), hipFuncAttributeMaxDynamicSharedMemorySize,
                                           160 * 1024);
        if (e != hipSuccess) return set_error(WAP_EHIP, "hipFuncSetAttribute: %s", hipGetErrorString(e));
        attr_done = true;
    }
    // as many work-groups as are resident at once (by LDS); they walk the tiles, so the weights are put in place once
    const int per_cu = (int)(160 * 1024 / smem);
    const int most = kNumCU * (per_cu < 6 ? per_cu : 6);
    hipLaunchKernelGGL(kfn, dim3(a.tiles < most ? a.tiles : most), dim3(NT), smem, st, a);
    return check_launch("dgrad_thin");
}

template <int C, int PX>
int launch_c(const ThinArgs& a, int cols, size_t smem, hipStream_t st) {
    if (cols <= 32) return launch_one<C, 1, PX>(a, smem, st);
    if (cols <= 64) return launch_one<C, 2, PX>(a, smem, st);
    return launch_one<C, 4, PX>(a, smem, st);
}

}  // namespace

// g: the data-gradient geometry (rows = input pixels, gathered tensor = dy, Ncols = input channels of the layer)
bool dgrad_thin_supported(const GemmGeom& g) {
    if (g.Ncols > 4 || (g.IC % 8) != 0 || g.mul_h != 1 || g.mul_w != 1) return false;
    // 32-bit byte offsets into dy and w
    return (double)(g.M / ((long)g.OH * g.OW)) * g.IH * g.IW * g.IC * 2.0 < 2147483648.0 &&
           (double)g.Kred * g.Ncols * 2.0 < 2147483648.0;
}

int launch_dgrad_thin(const GemmGeom& g, const bf16_t* dy, const bf16_t* w, bf16_t* dx, hipStream_t st) {
    if (!dgrad_thin_supported(g)) return set_error(WAP_EINVAL, "internal: thin data-gradient kernel not applicable");
    const int C = g.Ncols;
    ThinArgs a;
    a.dy = dy;
    a.w = w;
    a.dx = dx;
    a.N = g.M / (g.OH * g.OW);
    a.dy_bytes = (unsigned)((size_t)a.N * g.IH * g.IW * g.IC * 2);
    a.IH = g.IH; a.IW = g.IW; a.K = g.IC;
    a.OH = g.OH; a.OW = g.OW;
    a.R = g.R; a.S = g.S;
    // (with one row (column) of dy every stride past the map means the same; a larger one would wrap the tap counters)
    a.sh = g.IH == 1 ? (int)std::min<long>(g.div_h, (long)g.OH + g.R) : g.div_h;
    a.sw = g.IW == 1 ? (int)std::min<long>(g.div_w, (long)g.OW + g.S) : g.div_w;
    a.ph = g.R - 1 - g.pad_h; a.pw = g.S - 1 - g.pad_w;  // the geometry carries the flipped-filter padding
    // Strided both ways, a tile of 8 x 32 pixels lies over a handful of dy pixels: four times the pixels, less halo.
    const int px = a.sh > 1 && a.sw > 1 ? 4 : 1;
    const int TH = px == 1 ? 8 : 16, TW = px == 1 ? 32 : 64;
    // Groups: the fewest (each costs two barriers and a round of loads) whose columns fit four blocks and whose z leaves
    // room for two work-groups per CU; rows beyond 16 taps go in pieces, which bounds z by 105 KB.
    a.sg = a.S < 16 ? a.S : 16;
    a.zw = (TW - 1 + a.sg - 1) / a.sw + 1;
    size_t z_bytes = 0;
    for (int n = 1; n <= a.R; ++n) {
        a.rg = a.sg == a.S ? (a.R + n - 1) / n : 1;
        a.zh = (TH - 1 + a.rg - 1) / a.sh + 1;
        a.zgroups = (a.zh * a.zw + 31) / 32;
        a.zp = (a.rg * a.sg * C + 3) / 4 * 4;
        if ((a.zp & 4) == 0) a.zp += 4;
        z_bytes = (size_t)a.zgroups * 32 * a.zp * sizeof(float);
        if (a.rg == 1 || (a.rg * a.sg * C <= 128 && z_bytes <= 56 * 1024)) break;
    }
    const int cols = a.rg * a.sg * C;
    a.tiles_w = (a.OW + TW - 1) / TW;
    a.tiles_img = a.tiles_w * ((a.OH + TH - 1) / TH);
    a.tiles = a.N * a.tiles_img;
    a.dTW = make_fastdiv((uint32_t)a.tiles_w);
    a.dTI = make_fastdiv((uint32_t)a.tiles_img);
    a.dZW = make_fastdiv((uint32_t)a.zw);
    a.dSH = make_fastdiv((uint32_t)a.sh);
    a.dSW = make_fastdiv((uint32_t)a.sw);
    const size_t smem = (size_t)(cols <= 32 ? 1 : cols <= 64 ? 2 : 4) * (KC / 16) * 1024 + z_bytes;
    if (a.R == 3 && a.S == 3 && a.sh == 1 && a.sw == 1 && a.K <= KC && C <= 3)
        return C == 1 ? launch_3x3<1>(a, st) : C == 2 ? launch_3x3<2>(a, st) : launch_3x3<3>(a, st);
#define WAP_DISPATCH(C) (px == 1 ? launch_c<C, 1>(a, cols, smem, st) : launch_c<C, 4>(a, cols, smem, st))
    return C == 1 ? WAP_DISPATCH(1) : C == 2 ? WAP_DISPATCH(2) : C == 3 ? WAP_DISPATCH(3) : WAP_DISPATCH(4);
#undef WAP_DISPATCH
}

}  // namespace wap
