// Stride-1 convolution (forward, and data gradient with flipped weights) with the input PATCH resident in LDS
// (gfx950): every VGG-16 layer but the first, and the 13 x 13 / 27 x 27 AlexNet-style layers.
//
// The zero-padded input patch of a work-group's pixel tile (tile plus halo) is written to LDS one 32-channel slice
// at a time and every filter tap reads it through a shifted pointer, so activations cross L2 -> LDS once instead of
// R*S times; weights go from their packed copy straight into MFMA operand registers, one tap ahead.
//   * tiles: 8 x 32 / 16 x 16 pixels of one image (4 wavefronts = 2 pixel halves x 2 channel halves, 64 or 128
//     channels), 8 x 28 strips and flat runs of 224 raster-order pixels x 128 channels (4 channel wavefronts; the
//     runs may straddle rows and images; 64, 128, 160 or 192 pixels where those fill the CUs more evenly, tile2d_fill),
//     flat 192 x 64 tiles for thin outputs on maps nothing else divides;
//   * the patch is DOUBLE buffered: the global loads of slice c+1 are issued when the MFMA loop of slice c starts,
//     sit in registers for half of the taps and are written to the other buffer in the middle of the loop.  One
//     barrier per slice, placed in front of the last fragment read of the slice (which already targets the other
//     buffer), so no wavefront ever waits for a load or store phase.  (Two resident work-groups per CU that started
//     together reach such phases together: nobody covers them.)
//   * a 32-channel slice keeps a buffer near 30 KB (80-byte pixel rows: 64 bytes of data and 16 of padding, so 16
//     consecutive rows fall into 16 distinct 16-byte bank groups) and the staging registers at 24;
//   * patch rows are laid out with a BYTE stride chosen so that the first pixel of the next patch row lands in the
//     bank group that the pixel after this row's last tile pixel would have had (row stride = tile width x 80 plus a
//     multiple of 256 bytes): fragments that wrap from one patch row to the next still read conflict-free.
// UP variant (data gradient of a layer followed by a 2x2 / stride-2 max-pool): the input operand arrives as
// the gradient of the POOLED output plus the pool's argmax; the patch loader routes each window's value to
// the pixel its argmax names, so the max-pool backward costs no pass over the full-size gradient.
// Serves the "primary" convolution nodes of Section 3.2.2 (forward and backward halves of t_c, Eq. 1).
#include <algorithm>
#include <type_traits>
#include <utility>

#include "flat_runs.h"
#include "wap_internal.h"

namespace wap {

namespace {

constexpr int BK = 32, NT = 256;
constexpr int PITCH = 80;            // LDS bytes per padded pixel: 32 channels + 16 bytes
constexpr int VPP = BK / 8;          // 16-byte vectors per patch pixel
constexpr int MAX_PATCH = 352;       // padded pixels per 2-D tile patch (>= (tile h + R - 1) * (tile w + S - 1))
constexpr int MAX_PATCH_FLAT = 384;  // the same for flat (raster-order) 224-pixel tiles, which may straddle rows and images
constexpr int MAX_PATCH_FILL = 448;       // flat tiles of 160 and 192 pixels (56-wide maps, across images)
constexpr int MAX_PATCH_FLAT64 = 512;  // flat 192-pixel x 64-channel tiles (5x5 filters on 27-wide maps, across images)
constexpr size_t LDS_CAP = 160 * 1024;

struct TArgs {
    const bf16_t* A;
    const bf16_t* Wp;  // packed weights (see wo)
    const float* bias;
    const bf16_t* mask;  // optional: out = mask > 0 ? out : 0
    const uint8_t* up_am;  // UP: argmax (r * 2 + s) per pooling window; A is then N x IH/2 x IW/2 x IC
    bf16_t* out;         // may be NULL when only the pooled output is wanted
    bf16_t* pool_y;      // optional: 2x2 / stride-2 max-pool of the output tile ...
    uint8_t* pool_am;    // ... and the position r*2+s of the first maximum of every window
    float* colsum;       // optional: [tiles_m][Ncols] column sums of this tile's stored (masked) rows, for a bias gradient
    float* part;         // split reduction: fp32 partial sums [nsplit][M][Ncols], no epilogue here (flat tiles only)
    int nsplit, slices_per_split;  // 32-channel slices of the reduction that one work-group walks
    GemmGeom g;
    int tiles_x, tiles_y, tiles_img, tiles_m, tiles_n;
    int RWB, buf_bytes;  // LDS byte stride of a patch row, bytes of one patch buffer
    int patch_len;       // patch pixels to load (2-D tiles)
    int RW;              // patch row width in pixels: tile (flat tiles: image) width + S - 1
    FastDiv dRW, dRPHW;  // division by RW and (flat tiles) by PH * RW
    FastDiv dOW2;        // flat tiles with the fused pool: division by OW / 2
    int PH;              // flat tiles: padded image height
    int relu;
    unsigned a_bytes, w_bytes;
    WOrder wo;           // the tiles of small layers: where a weight lies
    FastDiv dTimg, dTx;
    FastDiv dOHW, dOW;   // flat tiles
    int UW, units;       // UP, 2-D tiles: pooling windows per patch row, windows per patch
    FastDiv dUW;
};

__device__ __forceinline__ int xcd_remap(int bid, int total) {
    int per = total / kNumXCD, rem = total % kNumXCD;
    int xcd = bid % kNumXCD, idx = bid / kNumXCD;
    return xcd < rem ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
}
__device__ __forceinline__ unsigned short f2bf(float f) {
    __bf16 b = (__bf16)f;
    return __builtin_bit_cast(unsigned short, b);
}

// keeps the bf16 lanes of v whose mask lane is > 0 (the ReLU derivative of the layer that produced the mask)
__device__ __forceinline__ u32x4 relu_mask8(u32x4 v, u32x4 mk) {
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const unsigned lo = __uint_as_float(mk[k] << 16) > 0.f ? 0xffffu : 0u;
        const unsigned hi = __uint_as_float(mk[k] & 0xffff0000u) > 0.f ? 0xffff0000u : 0u;
        v[k] &= (lo | hi);
    }
    return v;
}

// keeps the bf16 lanes of the pooled gradient v whose window's argmax byte equals this pixel's position code
__device__ __forceinline__ u32x4 unpool_select8(u32x4 v, u32x2 am, unsigned code) {
    const unsigned c4 = code * 0x01010101u;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const unsigned x = ((k < 2 ? am[0] : am[1]) >> ((k & 1) * 16)) ^ c4;  // a zero byte where argmax == code
        const unsigned lo = (x & 0xffu) == 0u ? 0xffffu : 0u;
        const unsigned hi = (x & 0xff00u) == 0u ? 0xffff0000u : 0u;
        v[k] &= (lo | hi);
    }
    return v;
}

template <typename F, int... T>
__device__ __forceinline__ void each_tap(F& f, std::integer_sequence<int, T...>) {
    (f(std::integral_constant<int, T>{}), ...);
}

// FN: 32-channel blocks per wavefront; TW: tile width in pixels; FM: 32-pixel fragments per wavefront;
// PG: wavefronts along the pixels (4 / PG along the channels).  Tile = 32*FM*PG pixels x 32*FN*(4/PG) channels.
// TW = 0: flat tiles, 32*FM*PG consecutive output pixels in raster order (they may straddle rows and images;
// the patch is then a run of the zero-padded image in raster order).  UP: pooled input operand.
// ST: filter side of the straight-line slice body (3 or 5), 0 = tap loop.
template <int FN, int TW, int FM, int PG, bool UP, int ST>
__device__ __forceinline__ void conv_tile2d_body(const TArgs& a) {
    constexpr bool FLAT = (TW == 0);
    constexpr bool SPLIT = FLAT && FM < 4;  // may walk a part of the reduction (the 224-pixel tiles have no register left for it)
    constexpr int BM = 32 * FM * PG;
    constexpr int CG = 4 / PG;
    constexpr int TWD = FLAT ? 1 : TW;  // divisor that is never zero
    constexpr int TH = BM / TWD;
    static_assert(FLAT || TH * TW == BM, "tile width must divide the tile");
    constexpr int PATCH_ROWS = FLAT ? (PG == 2 ? MAX_PATCH_FLAT64 : FM == 5 || FM == 6 ? MAX_PATCH_FILL : MAX_PATCH_FLAT) : MAX_PATCH;  // most patch pixels
    constexpr int PV = (PATCH_ROWS * VPP + NT - 1) / NT;  // 16-byte patch vectors per thread
    extern __shared__ __align__(16) unsigned char smem[];
    const GemmGeom& g = a.g;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int pg = wave % PG, cg = wave / PG;  // pixel group, channel group
    constexpr int BN = 32 * FN * CG;

    int logical = xcd_remap(blockIdx.x, a.tiles_m * a.tiles_n * (SPLIT ? a.nsplit : 1));
    int split = 0;
    if (SPLIT) {
        split = logical / (a.tiles_m * a.tiles_n);  // slowest: an XCD's work-groups share the weights of few splits
        logical -= split * (a.tiles_m * a.tiles_n);
    }
    const int tn = logical % a.tiles_n;
    const int tm = logical / a.tiles_n;
    const int img = (int)fdiv((uint32_t)tm, a.dTimg);
    const int trem = tm - img * a.tiles_img;
    const int tyi = (int)fdiv((uint32_t)trem, a.dTx);
    const int oh0 = tyi * TH, ow0 = (trem - tyi * a.tiles_x) * TW;
    const int n0 = tn * BN;
    const int OHW = g.OH * g.OW;
    // flat tiles: LDS byte position of output pixel m at tap (0,0) in the (unbounded) padded raster, rows RWB apart
    auto lbyte = [&](int m) {
        int n = (int)fdiv((uint32_t)m, a.dOHW);
        int rem = m - n * OHW;
        int oh = (int)fdiv((uint32_t)rem, a.dOW);
        return (n * a.PH + oh) * a.RWB + (rem - oh * g.OW) * PITCH;
    };
    const int m0 = tm * BM;
    const int m_last = (m0 + BM <= g.M ? m0 + BM : g.M) - 1;
    const int lds_lo = FLAT ? lbyte(m0) : 0;
    // the same in units of patch pixels (rows RW wide): what is loaded
    const int RPHW = a.PH * a.RW;
    auto rflat = [&](int m) {
        int n = (int)fdiv((uint32_t)m, a.dOHW);
        int rem = m - n * OHW;
        int oh = (int)fdiv((uint32_t)rem, a.dOW);
        return n * RPHW + oh * a.RW + (rem - oh * g.OW);
    };
    const int r_lo = FLAT ? rflat(m0) : 0;
    const int patch_len = FLAT ? rflat(m_last) + (g.R - 1) * a.RW + (g.S - 1) + 1 - r_lo : a.patch_len;
    const int RS = g.R * g.S;
    const int cs0 = SPLIT ? split * a.slices_per_split : 0;  // slices [cs0, ncs) of this work-group (never empty)
    const int ncs = SPLIT && cs0 + a.slices_per_split < g.IC / BK ? cs0 + a.slices_per_split : g.IC / BK;

    const __amdgpu_buffer_rsrc_t rsrcA =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.A), 0, (int)a.a_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrcW =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.Wp), 0, (int)a.w_bytes, 0x00020000);
    constexpr unsigned OOB = 0x80000000u;  // the activation tensor is below 2 GiB (checked on the host)
    const __amdgpu_buffer_rsrc_t rsrcM =  // UP: one argmax byte per pooled element, half the bytes of the pooled tensor
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(UP ? a.up_am : nullptr), 0, UP ? (int)(a.a_bytes / 2) : 0, 0x00020000);
    const int IH2 = g.IH >> 1, IW2 = g.IW >> 1;

    // ---- patch vectors of this thread: global byte offset of (padded pixel, 8-channel vector) or OOB, and the LDS
    // byte offset it goes to (-1: none, stored to the dump slot).  UP: the global offset is that of the pixel's pooling window in the pooled
    // tensor (the argmax byte sits at half of it), and pvcode holds the pixel's position (ih % 2) * 2 + iw % 2 inside
    // the window, 2 bits per vector ----
    constexpr bool UNITS = UP && !FLAT;  // 2-D tiles: a thread fetches whole pooling windows instead (below)
    unsigned pvoff[UNITS ? 1 : PV];
    int ploff[UNITS ? 1 : PV];
    unsigned pvcode = 0;
    // vectors with no patch pixel are stored unconditionally as well (no branches in the slice body), to a per-lane
    // slot behind the two buffers
    unsigned char* const dump = smem + 2 * a.buf_bytes + lane * 16;
#pragma unroll
    for (int i = 0; i < (UNITS ? 0 : PV); ++i) {
        int v = tid + i * NT;
        int q = v >> 2;
        unsigned off = OOB;
        ploff[i] = -1;
        if (q < patch_len) {
            if (FLAT) {
                int p = r_lo + q;
                int n = (int)fdiv((uint32_t)p, a.dRPHW);
                int rem = p - n * RPHW;
                int vh = (int)fdiv((uint32_t)rem, a.dRW);
                int pxp = rem - vh * a.RW;
                int ih = vh - g.pad_h, iw = pxp - g.pad_w;
                ploff[i] = (n * a.PH + vh) * a.RWB + pxp * PITCH - lds_lo + (v & 3) * 16;
                if (n * OHW < g.M && (unsigned)ih < (unsigned)g.IH && (unsigned)iw < (unsigned)g.IW) {
                    if (UP) {
                        off = (unsigned)(((n * IH2 + (ih >> 1)) * IW2 + (iw >> 1)) * g.IC + (v & 3) * 8) * 2u;
                        pvcode |= (unsigned)(((ih & 1) << 1) | (iw & 1)) << (2 * i);
                    } else {
                        off = (unsigned)(((n * g.IH + ih) * g.IW + iw) * g.IC + (v & 3) * 8) * 2u;
                    }
                }
            } else {
                int py = (int)fdiv((uint32_t)q, a.dRW);
                int px = q - py * a.RW;
                int ih = oh0 - g.pad_h + py, iw = ow0 - g.pad_w + px;
                ploff[i] = py * a.RWB + px * PITCH + (v & 3) * 16;
                if ((unsigned)ih < (unsigned)g.IH && (unsigned)iw < (unsigned)g.IW)
                    off = (unsigned)(((img * g.IH + ih) * g.IW + iw) * g.IC + (v & 3) * 8) * 2u;
            }
        }
        pvoff[i] = off;
    }

    // ---- UP, 2-D tiles: window `unit` = thread index / 4 (+ 64 per round) of the (UH x UW) windows that touch the
    // patch; one 16-byte load of the pooled gradient and one 8-byte load of the argmax serve its four pixels.
    // uq0 = LDS byte offset of the window's top-left pixel (it may lie one row / column outside the patch), uval =
    // which of the four pixels are inside the patch, 4 bits per window ----
    constexpr int UPV = 2;
    unsigned uoff[UNITS ? UPV : 1];
    int uq0[UNITS ? UPV : 1];
    unsigned uval = 0;
    if (UNITS) {
        const int ihf = oh0 - g.pad_h, iwf = ow0 - g.pad_w;  // image coordinates of patch pixel (0, 0)
        const int wy0 = ihf >> 1, wx0 = iwf >> 1;            // its window (floor division also below zero)
        const int PHt = TH + g.R - 1;
#pragma unroll
        for (int i = 0; i < UPV; ++i) {
            const int unit = (tid >> 2) + i * (NT / 4);
            const int uy = (int)fdiv((uint32_t)unit, a.dUW), ux = unit - uy * a.UW;
            const int wy = wy0 + uy, wx = wx0 + ux;
            const int py = 2 * wy - ihf, px = 2 * wx - iwf;
            unsigned off = OOB;
            if (unit < a.units && (unsigned)wy < (unsigned)IH2 && (unsigned)wx < (unsigned)IW2)
                off = (unsigned)(((img * IH2 + wy) * IW2 + wx) * g.IC + (tid & 3) * 8) * 2u;
            uoff[i] = off;
            uq0[i] = py * a.RWB + px * PITCH + (tid & 3) * 16;
            if (unit < a.units) {
                const unsigned vy0 = py >= 0, vy1 = py + 1 < PHt, vx0 = px >= 0, vx1 = px + 1 < a.RW;
                uval |= ((vy0 & vx0) | ((vy0 & vx1) << 1) | ((vy1 & vx0) << 2) | ((vy1 & vx1) << 3)) << (4 * i);
            }
        }
    }

    // ---- fragment rows of this lane: fragment j holds tile pixels (pg * FM + j) * 32 .. + 31 in raster order ----
    int frow[FM];
#pragma unroll
    for (int j = 0; j < FM; ++j) {
        const int idx = (pg * FM + j) * 32 + (lane & 31);
        if (FLAT) {
            const int m = m0 + idx <= m_last ? m0 + idx : m_last;  // tile tail: computed on a valid pixel, never stored
            frow[j] = lbyte(m) - lds_lo + (lane >> 5) * 16;
        } else {
            frow[j] = (idx / TWD) * a.RWB + (idx % TWD) * PITCH + (lane >> 5) * 16;
        }
    }

    // ---- weights: packed [channel block of 32][reduction step of 16][lane][8]; small layers' tiles take them unpacked as well ----
    const WOrder wo = SPLIT ? a.wo : w_packed(g.Kred);
    unsigned wrow[FN];
#pragma unroll
    for (int i = 0; i < FN; ++i)
        wrow[i] = (unsigned)(n0 + cg * 32 * FN + i * 32) / 32u * wo.block + (unsigned)(lane & 31) * wo.row + (unsigned)(lane >> 5) * wo.half;
    auto load_w = [&](int cs, int tap, bf16x8 (&wd)[2][FN]) {
        const unsigned koff = (unsigned)(tap * g.IC + cs * BK) / 16u * wo.step;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
            for (int i = 0; i < FN; ++i)
                wd[ks][i] = __builtin_bit_cast(
                    bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rsrcW, wrow[i] + koff + (unsigned)ks * wo.step, 0, 0));
    };

    // ---- patch slice: global -> registers (issue), registers -> LDS buffer (store) ----
    constexpr int NRP = UNITS ? UPV : PV;
    u32x4 rp[NRP];
    u32x2 ra[UP ? NRP : 1];  // an out-of-range offset halves to one that is still past the (half as long) argmax tensor
    auto issue_patch = [&](int cs) {
        const unsigned coff = (unsigned)(cs * BK) * 2u;
#pragma unroll
        for (int i = 0; i < NRP; ++i) {
            const unsigned o = (UNITS ? uoff[i] : pvoff[i]) + coff;
            rp[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrcA, o, 0, 0);
            if (UP) ra[i] = __builtin_amdgcn_raw_buffer_load_b64(rsrcM, o >> 1, 0, 0);
        }
    };
    auto store_patch = [&](unsigned char* buf) {
        if (UNITS) {
#pragma unroll
            for (int i = 0; i < UPV; ++i)
#pragma unroll
                for (int pos = 0; pos < 4; ++pos)
                    *reinterpret_cast<u32x4*>(((uval >> (4 * i + pos)) & 1u)
                                                  ? buf + uq0[i] + (pos >> 1) * a.RWB + (pos & 1) * PITCH
                                                  : dump) = unpool_select8(rp[i], ra[i], (unsigned)pos);
        } else {
#pragma unroll
            for (int i = 0; i < PV; ++i)
                *reinterpret_cast<u32x4*>(ploff[i] >= 0 ? buf + ploff[i] : dump) =
                    UP ? unpool_select8(rp[i], ra[i], (pvcode >> (2 * i)) & 3u) : rp[i];
        }
    };

    f32x16 acc[FN][FM];
#pragma unroll
    for (int i = 0; i < FN; ++i)
#pragma unroll
        for (int j = 0; j < FM; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    // Weight fragments: one register set per tap (two reduction steps).  What bounds the weight stream is how long a
    // load may stay in flight before its wavefront needs it, and a wavefront's loads return in order, so the first
    // weight load issued after the patch loads of the next slice drags those along: with sets filled one tap ahead
    // the patch latency (first touch: HBM or the memory-side cache) would be exposed once per slice.
    //   ST (square filters of 3 or 5 taps a side): the taps of a slice are straight-line code, the sets a ring of ST that
    //   is filled ST - 1 taps ahead and rotates without copies (ST divides the taps, so every slice starts at the same set),
    //   the patch loads go out right behind the weight loads of tap 0 (ST taps until a younger weight load is needed) and
    //   reach LDS after three quarters of the taps (3x3: after tap 7).  No branch in the slice body: the loads / stores /
    //   barrier of a slice beyond the last are issued anyway (clamped to the last slice, written to the idle buffer), so
    //   the compiler's counter waits are exact.
    //   otherwise: a tap loop with two sets, the new one copied over the current one at the end of every tap.
    constexpr int NSET = ST ? ST : 2;
    constexpr int STD = ST ? ST : 1, RSC = STD * STD;
    constexpr int STORE_TAP = ST == 3 ? 7 : RSC * 3 / 4;
    bf16x8 w[NSET][2][FN];
    issue_patch(cs0);
#pragma unroll
    for (int u = 0; u + 1 < NSET; ++u) load_w(cs0, u, w[u]);
    store_patch(smem);
    __syncthreads();
    // Fragment reads run one reduction step ahead of the MFMAs that consume them, in place: right after the MFMA that
    // consumed fragment j has been issued, the read of fragment j for the next step is issued into the same registers
    // (FM - 1 MFMAs, some 200 cycles, before it is needed), across taps and across slices.  The issue order is pinned:
    // the compiler's own order (read, wait, MFMA) leaves the LDS latency exposed in front of most MFMAs.
    bf16x8 fa[FM];
#pragma unroll
    for (int j = 0; j < FM; ++j) fa[j] = *reinterpret_cast<const bf16x8*>(smem + frow[j]);

    // one reduction step: consume fragment j with weight fragment wk, then fetch fragment j of the step after
    auto step = [&](bf16x8 (&wk)[FN], const unsigned char* next_base, int next_off, bool with_vmem) {
#pragma unroll
        for (int j = 0; j < FM; ++j) {
#pragma unroll
            for (int i = 0; i < FN; ++i)
                acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wk[i], fa[j], acc[i][j], 0, 0, 0);
            fa[j] = *reinterpret_cast<const bf16x8*>(next_base + frow[j] + next_off);
        }
    };
    // issue order of a step: one fragment read behind every FN MFMAs; the step's VMEM loads (weights of a later tap,
    // the next patch slice) ride in front of the first MFMA groups, one or more per group (where they sit within the
    // step measured the same: first, third or fifth group)
    auto pin_step = [&](auto vmem_tag) {
        constexpr int NV = decltype(vmem_tag)::value;  // VMEM loads to place
        constexpr int PER = NV > 0 ? (NV + FM - 1) / FM : 0;
#pragma unroll
        for (int q = 0; q < FM; ++q) {
            if (NV > 0 && q * PER < NV) __builtin_amdgcn_sched_group_barrier(0x020, PER, 0);  // VMEM read
            __builtin_amdgcn_sched_group_barrier(0x008, FN, 0);                                // MFMA
            __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                                 // DS read
        }
    };

    for (int cs = cs0; cs < ncs; ++cs) {
        const unsigned char* cur = smem + ((cs - cs0) & 1) * a.buf_bytes;
        unsigned char* nxt = smem + ((cs - cs0 + 1) & 1) * a.buf_bytes;
        const int csn = cs + 1 < ncs ? cs + 1 : cs;  // the next slice, clamped
        __builtin_amdgcn_s_setprio(1);
        if constexpr (ST != 0) {
            auto tap = [&](auto tap_tag) {
                constexpr int T = decltype(tap_tag)::value;
                constexpr int U = T % NSET;
                constexpr int PT = (T + NSET - 1) % RSC;  // the tap whose weights are fetched now
                const int tapoff = (T / STD) * a.RWB + (T % STD) * PITCH;
                const int tapoff1 = ((T + 1) / STD) * a.RWB + ((T + 1) % STD) * PITCH;
                __builtin_amdgcn_sched_barrier(0);
                load_w(T + NSET - 1 >= RSC ? csn : cs, PT, w[(U + NSET - 1) % NSET]);
                if (T == 0) issue_patch(csn);
                step(w[U][0], cur, tapoff + 32, true);
                if (T == 0) pin_step(std::integral_constant<int, 2 * FN + (UP ? 2 : 1) * NRP>{});
                else pin_step(std::integral_constant<int, 2 * FN>{});
                __builtin_amdgcn_sched_barrier(0);
                if (T == RSC - 1) {
                    // every wavefront has written its share of the next slice (after tap STORE_TAP; the LDS pipe executes a
                    // wavefront's operations in order and fragment reads issued after those writes have returned) and
                    // nobody reads the buffer that slice c+2 will overwrite before this point again
                    __builtin_amdgcn_s_barrier();
                    __builtin_amdgcn_sched_barrier(0);
                    step(w[U][1], nxt, 0, false);
                } else {
                    step(w[U][1], cur, tapoff1, false);
                }
                pin_step(std::integral_constant<int, 0>{});
                __builtin_amdgcn_sched_barrier(0);
                if (T == STORE_TAP) {
                    store_patch(nxt);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            each_tap(tap, std::make_integer_sequence<int, RSC>{});
        } else {
            const bool has_next = cs + 1 < ncs;
            if (has_next) issue_patch(cs + 1);
            const int mid = (RS - 1) >> 1;  // the tap after which the next slice goes to LDS (never the last tap)
            int r = 0, s2 = 0;
            // LAST: the slice's last tap, whose second step prefetches the first fragments of the next slice from the
            // other buffer, behind the slice's only barrier
            auto tap_body = [&](int tap, auto last_tag) {
                constexpr bool LAST = decltype(last_tag)::value;
                int s1 = s2 + 1, r1 = r;
                if (s1 == g.S) { s1 = 0; r1 = r + 1; }
                const int tapoff = r * a.RWB + s2 * PITCH;
                const int tapoff1 = r1 * a.RWB + s1 * PITCH;
                __builtin_amdgcn_sched_barrier(0);
                load_w(LAST ? csn : cs, LAST ? 0 : tap + 1, w[1]);  // (past the end: a harmless reload)
                step(w[0][0], cur, tapoff + 32, true);
                pin_step(std::integral_constant<int, 2 * FN>{});
                __builtin_amdgcn_sched_barrier(0);
                if (LAST) {
                    __builtin_amdgcn_s_barrier();  // see the note in the straight-line variant
                    __builtin_amdgcn_sched_barrier(0);
                    step(w[0][1], nxt, 0, false);
                } else {
                    step(w[0][1], cur, tapoff1, false);
                }
                pin_step(std::integral_constant<int, 0>{});
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                    for (int i = 0; i < FN; ++i) w[0][ks][i] = w[1][ks][i];
                r = r1;
                s2 = s1;
                if (!LAST && tap == mid && has_next) {
                    store_patch(nxt);
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            for (int tap = 0; tap + 1 < RS; ++tap) tap_body(tap, std::false_type{});
            tap_body(RS - 1, std::true_type{});
        }
        __builtin_amdgcn_s_setprio(0);
    }

    // ---- split reduction: the accumulators as they lie, four consecutive channels of a pixel per store ----
    if (SPLIT && a.part) {
        float* const po = a.part + (size_t)split * g.M * g.Ncols;
#pragma unroll
        for (int j = 0; j < FM; ++j) {
            const int m = m0 + (pg * FM + j) * 32 + (lane & 31);
            if (m > m_last) continue;
#pragma unroll
            for (int i = 0; i < FN; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<float4*>(po + (size_t)m * g.Ncols + n0 + cg * 32 * FN + i * 32 + q * 8 + (lane >> 5) * 4) =
                        make_float4(acc[i][j][q * 4], acc[i][j][q * 4 + 1], acc[i][j][q * 4 + 2], acc[i][j][q * 4 + 3]);
        }
        return;
    }

    // ---- epilogue: bias / ReLU / bf16, transposed through LDS (the patch buffers are dead) so that every global
    // store is 16 contiguous bytes per lane and a tile row of 32 pixels is one contiguous run.  The whole tile is
    // staged in one pass (the host sizes the LDS allocation for it): staged row = tile pixel index. ----
    constexpr int OPITCH = BN * 2 + 16;  // bytes per pixel row in the staging buffer
    constexpr int VPR = BN / 8;          // 16-byte vectors per pixel row
    constexpr int RPP = NT / VPR;        // pixel rows stored per pass
    constexpr int NR = BM / RPP;
    static_assert(NR * RPP == BM, "whole passes");
    // The mask of this thread's rows is fetched before the accumulators are converted: fetched row by row between the
    // stores (which the compiler may not move it over) every row waited for memory, 14 times per 224-pixel tile.
    u32x4 mk[NR];
    auto out_pixel = [&](int row) { return FLAT ? m0 + row : (img * g.OH + oh0 + row / TWD) * g.OW + ow0 + row % TWD; };
    if (a.mask) {
#pragma unroll
        for (int it = 0; it < NR; ++it) {
            int m = out_pixel(tid / VPR + it * RPP);
            if (FLAT && m > m_last) m = m_last;  // never stored
            mk[it] = *reinterpret_cast<const u32x4*>(a.mask + (size_t)m * g.Ncols + n0 + (tid % VPR) * 8);
        }
    }
    __syncthreads();  // the last readers of the patch are done
#pragma unroll
    for (int j = 0; j < FM; ++j) {
        const int srow = (pg * FM + j) * 32 + (lane & 31);
#pragma unroll
        for (int i = 0; i < FN; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int nl = cg * 32 * FN + i * 32 + q * 8 + (lane >> 5) * 4;  // channel within the tile
                float v[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[e] = acc[i][j][q * 4 + e];
                if (a.bias) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] += a.bias[n0 + nl + e];
                }
                if (a.relu) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
                }
                uint2 pk = make_uint2((unsigned)f2bf(v[0]) | ((unsigned)f2bf(v[1]) << 16),
                                      (unsigned)f2bf(v[2]) | ((unsigned)f2bf(v[3]) << 16));
                *reinterpret_cast<uint2*>(smem + srow * OPITCH + nl * 2) = pk;
            }
    }
    __syncthreads();
    float csum[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};  // column sums over this thread's rows (its 8 channels)
#pragma unroll
    for (int it = 0; it < NR; ++it) {
        const int row = tid / VPR + it * RPP;
        const int m = out_pixel(row);
        if (FLAT && m > m_last) continue;
        u32x4 vv = *reinterpret_cast<const u32x4*>(smem + row * OPITCH + (tid % VPR) * 16);
        const size_t o = (size_t)m * g.Ncols + n0 + (tid % VPR) * 8;
        if (a.mask) vv = relu_mask8(vv, mk[it]);
        if (a.out) *reinterpret_cast<u32x4*>(a.out + o) = vv;
        if (a.colsum) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                csum[2 * k] += __uint_as_float(vv[k] << 16);
                csum[2 * k + 1] += __uint_as_float(vv[k] & 0xffff0000u);
            }
        }
    }
    // ---- column sums of the stored tile (the bias gradient of the layer whose pre-activation gradient this is): the
    // RPP row groups are added in group order through LDS, one partial row per pixel tile; a second kernel adds the
    // tiles in a fixed order ----
    if (a.colsum) {
        __syncthreads();  // the staged tile has been read
        float* red = reinterpret_cast<float*>(smem);  // [RPP][BN]
#pragma unroll
        for (int e = 0; e < 8; ++e) red[(tid / VPR) * BN + (tid % VPR) * 8 + e] = csum[e];
        __syncthreads();
        if (tid < BN) {
            float t = red[tid];
            for (int k = 1; k < RPP; ++k) t += red[k * BN + tid];
            a.colsum[(size_t)tm * g.Ncols + n0 + tid] = t;
        }
    }
    // ---- fused 2x2 / stride-2 max-pool of the staged (bias / ReLU applied, bf16) tile: tile origin and size are
    // even and the whole tile is staged, so every window is complete.  A flat tile is a whole number of row pairs
    // (the host checks 224 % (2 OW) == 0 and even map sizes), possibly of two images.  Same rule as maxpool_fwd_kernel:
    // first maximum in (r, s) order. ----
    constexpr bool POOLS = FLAT ? (PG == 1) : ((PG == 2 && FM == 4) || TW == 28);
    if (POOLS && a.pool_y) {
        const int roww = FLAT ? g.OW : TWD;  // pixels per tile row
        const int PWT = roww >> 1;           // pooled pixels per tile row
        for (int item = tid; item < (BM / 4) * VPR; item += NT) {
            const int pp = item / VPR, vec = item % VPR;
            const int py = FLAT ? (int)fdiv((uint32_t)pp, a.dOW2) : pp / (TWD / 2);
            const int px = pp - py * PWT;
            const int idx00 = (2 * py) * roww + 2 * px;
            if (FLAT && m0 + idx00 + roww + 1 > m_last) continue;  // beyond the last pixel of the layer
            const int idx4[4] = {idx00, idx00 + 1, idx00 + roww, idx00 + roww + 1};
            unsigned short best[8];
            float bestf[8];
            unsigned char bi[8];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const u32x4 v = *reinterpret_cast<const u32x4*>(smem + idx4[k] * OPITCH + vec * 16);
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const unsigned short bits = (unsigned short)((e & 1) ? (v[e >> 1] >> 16) : (v[e >> 1] & 0xffffu));
                    const float f = __uint_as_float((unsigned)bits << 16);
                    if (k == 0 || f > bestf[e]) { bestf[e] = f; best[e] = bits; bi[e] = (unsigned char)k; }
                }
            }
            size_t po;
            if (FLAT) {
                const int m = m0 + idx00;
                const int n = (int)fdiv((uint32_t)m, a.dOHW);
                const int rem = m - n * OHW;
                const int oh = (int)fdiv((uint32_t)rem, a.dOW), ow = rem - oh * g.OW;
                po = ((size_t)(n * (g.OH / 2) + oh / 2) * (g.OW / 2) + ow / 2) * g.Ncols + n0 + vec * 8;
            } else {
                po = ((size_t)(img * (g.OH / 2) + oh0 / 2 + py) * (g.OW / 2) + ow0 / 2 + px) * g.Ncols + n0 + vec * 8;
            }
            u32x4 yo = {(unsigned)best[0] | ((unsigned)best[1] << 16), (unsigned)best[2] | ((unsigned)best[3] << 16),
                        (unsigned)best[4] | ((unsigned)best[5] << 16), (unsigned)best[6] | ((unsigned)best[7] << 16)};
            *reinterpret_cast<u32x4*>(a.pool_y + po) = yo;
            uint2 am;
            am.x = bi[0] | (bi[1] << 8) | (bi[2] << 16) | ((unsigned)bi[3] << 24);
            am.y = bi[4] | (bi[5] << 8) | (bi[6] << 16) | ((unsigned)bi[7] << 24);
            *reinterpret_cast<uint2*>(a.pool_am + po) = am;
        }
    }
}

template <int FN, int TW, int FM, int PG, bool UP, bool T9>
__global__ __launch_bounds__(NT, 2) void conv_tile2d_kernel(const TArgs a) {
    conv_tile2d_body<FN, TW, FM, PG, UP, T9 ? 3 : 0>(a);
}
template <int FN, int TW, int FM, int PG>
__global__ __launch_bounds__(NT, 2) void conv_tile2d_5x5_kernel(const TArgs a) {
    conv_tile2d_body<FN, TW, FM, PG, false, 5>(a);
}

template <typename F>
int launch_tile2d_k(F kfn, std::atomic<bool>& attr_done, const TArgs& ta, size_t smem, hipStream_t st) {
    if (!attr_done) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_CAP);
        if (e != hipSuccess) return set_error(WAP_EHIP, "hipFuncSetAttribute: %s", hipGetErrorString(e));
        attr_done = true;
    }
    hipLaunchKernelGGL(kfn, dim3(ta.tiles_m * ta.tiles_n * ta.nsplit), dim3(NT), smem, st, ta);
    return check_launch("conv_tile2d");
}
// flat tiles of FM x 32 pixels x 128 channels, picked to divide a layer evenly (3x3 only)
template <int FM>
int launch_tile2d_fill(const TArgs& ta, size_t smem, hipStream_t st) {
    static std::atomic<bool> done{false}, doneu{false};
    return ta.up_am ? launch_tile2d_k(conv_tile2d_kernel<1, 0, FM, 1, true, true>, doneu, ta, smem, st)
                    : launch_tile2d_k(conv_tile2d_kernel<1, 0, FM, 1, false, true>, done, ta, smem, st);
}
// straight-line 3x3 slices; 5x5 ones on the flat 192 x 64 tiles (the tilings such layers get); else the tap loop
constexpr int tile2d_st(int tw, int pg, bool up, int R, int S) {
    return R == 3 && S == 3 ? 3 : R == 5 && S == 5 && tw == 0 && pg == 2 && !up ? 5 : 0;
}
template <int FN, int TW, int FM, int PG, bool UP>
int launch_tile2d_u(const TArgs& ta, size_t smem, hipStream_t st) {
    static std::atomic<bool> done9{false}, done5{false}, done{false};
    const int side = tile2d_st(TW, PG, UP, ta.g.R, ta.g.S);
    if (side == 3) return launch_tile2d_k(conv_tile2d_kernel<FN, TW, FM, PG, UP, true>, done9, ta, smem, st);
    if constexpr (tile2d_st(TW, PG, UP, 5, 5) == 5)
        if (side == 5) return launch_tile2d_k(conv_tile2d_5x5_kernel<FN, TW, FM, PG>, done5, ta, smem, st);
    return launch_tile2d_k(conv_tile2d_kernel<FN, TW, FM, PG, UP, false>, done, ta, smem, st);
}
template <int FN, int TW, int FM, int PG>
int launch_tile2d_t(const TArgs& ta, size_t smem, hipStream_t st) {
    return ta.up_am ? launch_tile2d_u<FN, TW, FM, PG, true>(ta, smem, st) : launch_tile2d_u<FN, TW, FM, PG, false>(ta, smem, st);
}

}  // namespace

namespace {
struct TileCfg {
    int fn, tw, th, variant;  // variant 0: 256 pixels as 2 x 4 fragments; 1: 224 pixels (8 x 28) as 1 x 7 fragments,
                              // 128 channels; 2: the same with flat tiles (224 consecutive pixels); 3: flat tiles of
                              // 192 pixels x 64 channels (2 x 3 fragments) for thin outputs on maps no 2-D tile divides
    int RWB, buf_bytes;       // LDS layout: byte stride of a patch row, bytes of one patch buffer
    size_t smem;              // dynamic LDS of the launch: two patch buffers, or the staged output tile if larger
    int fm;                   // variant 2: 32-pixel fragments per wavefront (2 or 4 .. 7: tiles of 64 or 128 .. 224 pixels)
};
int tile_pixels(const TileCfg& c) { return c.variant == 3 ? 192 : c.variant == 2 ? 32 * c.fm : c.variant == 1 ? 224 : 256; }
// most patch pixels any bm-pixel raster-order tile of this geometry loads
int max_flat_patch(const GemmGeom& g, int bm) { return flat_patch(flat_runs(g.M, g.OH, g.OW, bm), g.OW, g.R, g.S); }
// most LDS bytes one patch buffer of such a tile spans when patch rows are rwb bytes apart
long max_flat_bytes(const GemmGeom& g, const FlatRuns& f, int rwb) {
    long worst = 0;
    for (int i = 0; i < f.n; ++i)
        worst = std::max(worst, (long)(f.run[i].pixels - 1 + g.S) * PITCH + (long)f.run[i].rows * (rwb - g.OW * PITCH) + (long)(f.run[i].images + 1) * (g.R - 1) * rwb);
    return worst;
}
// Row stride that keeps fragments conflict-free across a row wrap: the next row's first pixel must fall into the bank
// group (address mod 256) that pixel `width` of this row would have had.
int conflict_free_stride(int width, int S) { return width * PITCH + ((S - 1) * PITCH + 255) / 256 * 256; }

// LDS layout of a tile shape: the conflict-free row stride if two work-groups per CU still fit, else dense rows.
bool lds_layout(const GemmGeom& g, TileCfg* c) {
    const int bm = tile_pixels(*c);
    const int bn = c->variant == 3 ? 64 : c->variant >= 1 ? 128 : 64 * c->fn;
    const size_t stage = (size_t)bm * (bn * 2 + 16);
    const bool flat = c->variant >= 2;
    const int width = flat ? g.OW : c->tw;
    const int dense = (width + g.S - 1) * PITCH;
    const int cands[2] = {(flat || (c->tw != 32)) ? conflict_free_stride(width, g.S) : dense, dense};
    const FlatRuns runs = flat ? flat_runs(g.M, g.OH, g.OW, bm) : FlatRuns{};
    size_t best = 0;
    for (int pass = 0; pass < 2 && !best; ++pass)            // first two work-groups per CU, then one
        for (int k = 0; k < 2 && !best; ++k) {
            const int rwb = cands[k];
            const long buf = flat ? max_flat_bytes(g, runs, rwb)
                                  : (long)(c->th + g.R - 2) * rwb + (long)(c->tw + g.S - 1) * PITCH;
            const long bufa = (buf + 15) / 16 * 16;
            const size_t smem = std::max((size_t)(2 * bufa) + 1024, stage);  // + the dump slots of stores without a pixel
            if (smem <= (pass == 0 ? LDS_CAP / 2 : LDS_CAP)) {
                c->RWB = rwb;
                c->buf_bytes = (int)bufa;
                c->smem = smem;
                best = smem;
            }
        }
    return best != 0;
}
// Wide outputs at a small minibatch: the 128-channel tiles leave most CUs without work and conv_patch.hip does not
// apply, so the alternative is the generic tap-by-tap kernel with a split reduction (measured 270-390 TFLOP/s there,
// plus ~9 us for the launch of its reduction epilogue).  One 192 x 64 tile's serial reduction loop takes 5.4-6.6 us
// per 64-channel slice of a 3x3 filter whatever the minibatch, so the flat tiles win only once the layer holds
// enough work.
bool flat64_fits(const GemmGeom& g) {
    TileCfg c = {1, 0, 0, 3, 0, 0, 0, 0};
    return g.M >= 192 * 4 && max_flat_patch(g, 192) <= MAX_PATCH_FLAT64 && lds_layout(g, &c);
}
bool flat64_wins_small_batch(const GemmGeom& g) {
    if ((g.Ncols % 64) != 0 || g.Ncols <= 64 || g.M >= 224 * 32 || g.M < 192 * 4) return false;
    if ((long)((g.M + 191) / 192) * (g.Ncols / 64) < 64) return false;
    if (!flat64_fits(g)) return false;
    const double flops = 2.0 * g.M * (double)g.Ncols * g.Kred;
    const double t_generic = flops / 330e12 + 9e-6;
    const double floor_s = 5.5e-6 * (g.IC / 64.0) * (g.R * g.S / 9.0);
    const double t_flat = floor_s > flops / 900e12 ? floor_s : flops / 900e12;
    return t_flat < 0.85 * t_generic;
}
// The flat tilings a split reduction runs on: 64 pixels x 128 channels or 192 pixels x 64 channels.
TileCfg split_cfg(const GemmGeom& g, int tile) {
    const bool v3 = tile == kTileSplit192;
    TileCfg c = {1, 0, 0, v3 ? 3 : 2, 0, 0, 0, 2};
    if ((g.Ncols % (v3 ? 64 : 128)) != 0 || max_flat_patch(g, tile_pixels(c)) > (v3 ? MAX_PATCH_FLAT64 : MAX_PATCH_FLAT) ||
        !lds_layout(g, &c))
        c.fn = 0;
    return c;
}
// Tiles of 128 channels for a whole reduction of a 3x3 filter: flat ones of 32 * fm pixels, or (kTileStrips) the 8 x 28 strips.
TileCfg fill_cfg(const GemmGeom& g, int tile) {
    const bool strips = tile == kTileStrips;
    const int fm = tile - kTileFill;
    TileCfg c = {1, 0, 0, 2, 0, 0, 0, fm};
    if (strips) c = {1, 28, 8, 1, 0, 0, 0, 0};
    const bool fits = strips ? (g.OW % 28) == 0 && (g.OH % 8) == 0
                             : fm >= 4 && fm <= 6 && max_flat_patch(g, 32 * fm) <= (fm == 4 ? MAX_PATCH_FLAT : MAX_PATCH_FILL);
    if (!fits || g.R != 3 || g.S != 3 || (g.Ncols % 128) != 0 || !lds_layout(g, &c) || c.smem > LDS_CAP / 2) c.fn = 0;
    return c;
}
// Tile shape for this geometry (width must divide the map, patch must fit), fn = 0 if none.
TileCfg tile_cfg(const GemmGeom& g, int tile = 0) {
    if (tile >= kTileFill) return fill_cfg(g, tile);
    if (tile) return split_cfg(g, tile);
    TileCfg none = {0, 0, 0, 0, 0, 0, 0, 0};
    TileCfg c = none;
    if ((g.Ncols % 64) != 0) return none;
    const bool tiles128 = (g.Ncols % 128) == 0;  // 2-D tiles of 128 channels (64 output channels: conv_tile64.hip)
    for (int tw : {32, 16, 8}) {
        const int th = 256 / tw;
        if (tiles128 && (g.OH % th) == 0 && (g.OW % tw) == 0 && (th + g.R - 1) * (tw + g.S - 1) <= MAX_PATCH) {
            c = {2, tw, th, 0, 0, 0, 0, 0};
            if (lds_layout(g, &c)) return c;
            c = none;
        }
    }
    // maps of 28k x 8j pixels (56 x 56): 8 x 28 tiles, one 224-pixel strip per wavefront, 128-channel tiles
    if ((g.Ncols % 128) == 0 && (g.OW % 28) == 0 && (g.OH % 8) == 0 && (8 + g.R - 1) * (28 + g.S - 1) <= MAX_PATCH) {
        c = {1, 28, 8, 1, 0, 0, 0, 0};
        if (!lds_layout(g, &c)) c = none;
    }
    // Flat 128-channel tiles: 224 pixels per tile while that puts a work-group on at least three quarters of the CUs,
    // else 64 pixels (the serial reduction of a tile is what a small layer waits for: a short tile shortens every
    // reduction step four-fold and puts more work-groups on the chip; the weight stream per pixel grows, which a small
    // layer can afford).  Measured: conv4_2 at minibatch 8 55 -> 44 us, conv5_1 at 32 54 -> 44 us, at 16 37 -> 33 us;
    // 128 to 192 pixels where those divide the layer more evenly: tile2d_fill.  Short flat tiles
    // also replace the strips where those leave the chip under-filled.
    const long strips = c.fn ? (long)(g.M / 224) * (g.Ncols / 128) : 0;
    if ((c.fn == 0 || strips < kNumCU * 3 / 4) && (g.Ncols % 128) == 0 && g.M >= 64 * 4) {
        for (int fm : {7, 2}) {
            const int bm = 32 * fm;
            const long wgs = (long)((g.M + bm - 1) / bm) * (g.Ncols / 128);
            if (max_flat_patch(g, bm) > MAX_PATCH_FLAT || (fm > 2 && wgs < kNumCU * 3 / 4)) continue;
            if (c.fn != 0 && wgs <= strips) break;  // no better filled than the strips
            TileCfg f = {1, 0, 0, 2, 0, 0, 0, fm};
            if (lds_layout(g, &f)) { c = f; break; }
        }
    }
    // 192-pixel x 64-channel flat tiles where none of the above applies (64 or 192 output channels on maps no 2-D
    // tile divides), and for wide outputs at a small minibatch where they beat the generic kernel
    const bool use64 = (c.fn == 0 && flat64_fits(g)) ||
                       (c.fn != 0 && c.variant >= 1 && c.variant <= 2 &&
                        (long)((g.M + tile_pixels(c) - 1) / tile_pixels(c)) * (g.Ncols / 128) < kNumCU * 3 / 4 &&
                        flat64_wins_small_batch(g));
    if (use64) {
        c = {1, 0, 0, 3, 0, 0, 0, 0};
        if (!lds_layout(g, &c)) c = none;
    }
    return c;
}
}  // namespace

// 0 = not applicable, otherwise FN (32-channel blocks per wavefront)
int tile2d_supported(const GemmGeom& g, int tile) {
    if ((g.IC % BK) != 0 || g.div_h != 1 || g.div_w != 1 || g.mul_h != 1 || g.mul_w != 1) return 0;
    if (g.R * g.S < 2) return 0;
    long a_elems = (long)(g.M / ((long)g.OH * g.OW)) * g.IH * g.IW * g.IC;
    if (a_elems * 2 >= (1L << 31)) return 0;
    if (!tile && tile64_width(g)) return 1;  // 64 output channels on a map that 256-pixel tiles divide: conv_tile64.hip
    return tile_cfg(g, tile).fn;
}

// Shapes on which this kernel measured faster than conv_patch.hip: thin outputs on 256-pixel 2-D tiles, and the
// 224-pixel x 128-channel tiles (8 x 28 strips or flat) at any width once the map is large enough to fill the CUs.
bool tile2d_preferred(const GemmGeom& g) {
    if (!tile2d_supported(g)) return false;
    if (tile64_width(g)) return true;
    const TileCfg c = tile_cfg(g);
    if (c.variant == 0) return g.Ncols <= 128;
    if (c.variant == 3) {  // measured against the generic tap-by-tap kernel (64 channels) and conv_patch (wider)
        // 192 output channels on 13 x 13 maps (384 -> 192 data gradient): 27 against 38 us at minibatch 32 (87 tiles), 27
        // against 41 us at 64; at 16 and below (45 tiles and fewer) the generic kernel with a split reduction wins
        const long t3 = (long)((g.M + 191) / 192) * (g.Ncols / 64);
        return g.Ncols == 64 ? t3 >= 48 : (t3 >= 80 || flat64_wins_small_batch(g));
    }
    const long wgs = (long)((g.M + tile_pixels(c) - 1) / tile_pixels(c)) * (g.Ncols / 128);
    // 64-pixel flat tiles keep winning against the generic kernel well below a work-group per CU while the reduction is
    // short (13 x 13 layers of 192 .. 384 input channels at minibatch 8 .. 32: 23 against 36 us, 18 against 26 us, 17
    // against 21 us); with 512 input channels (reduction 4608) the generic kernel's split reduction draws level
    if (c.variant == 2 && c.fm == 2 && wgs >= 64 && g.Kred <= 3456) return true;
    return wgs >= kNumCU * 3 / 4;
}

// pixels and output channels of a work-group's tile
void tile2d_shape(const GemmGeom& g, int tile, int* pixels, int* channels) {
    if (!tile && tile64_width(g)) {
        *pixels = 256;
        *channels = 64;
        return;
    }
    const TileCfg c = tile_cfg(g, tile);
    *pixels = tile_pixels(c);
    *channels = c.variant == 3 ? 64 : c.variant >= 1 ? 128 : 64 * c.fn;
}

// How to divide the reduction of a layer too small to fill the chip: number of splits (1: don't) and the flat tiling.
// `generic`: the alternative is the tap-by-tap kernel, which splits its reduction as well but gathers every activation
// once per tap (3x3, weights packed before: 512 -> 512 channels on 14 x 14 at minibatch 8 32.4 -> 22.2, 256 -> 256 on 13 x 13
// at 8 19.0 -> 13.4, 384 -> 256 at 1 15.6 -> 10.2 us; other filters below).  Otherwise it is an unsplit tile of this
// kernel: a slice of a 3x3 filter takes a work-group about 2.2 us, the partial sums and their reduction about 9, so the
// split has to save 10 (384 -> 192 on 13 x 13 at 32 24.5 -> 22.7; 64 outputs of a 5x5 filter at 16 / 32 / 64 47 / 49 /
// 53 -> 27 / 36 / 44 us; 128 -> 64 on 56 x 56, four slices, would lose: 12.0 -> 15.7).
// Work-groups: just under one per CU for 3x3 filters (more splits only add partial sums: 384 -> 256 at 8 176 / 264
// work-groups 14.8 / 15.9 us), two per CU for larger filters, whose work per partial sum is higher.
int tile2d_split(const GemmGeom& g, bool generic, int* tile) {
    const int slices = g.IC / BK;
    if ((g.IC % BK) != 0 || slices < 2 || g.R * g.S < 2 || (g.Ncols % 64) != 0) return 1;
    *tile = (g.Ncols % 128) == 0 ? kTileSplit64 : kTileSplit192;
    // Against the tap-by-tap kernel (whose plan splits too), 1100 layers of 0.04 to 20 GFLOP, that kernel's time over this one's
    // with its packing: with straight-line taps 3x3 0.98 .. 1.30 and 5x5 on 192 x 64 tiles 0.96 .. 1.40; with the taps in a loop 2x2
    // 0.71 .. 0.98 up to two slices and mostly 1.0 .. 1.19 beyond, 5x5 on 64 x 128 tiles 0.64 .. 0.9 where the grid is small or few rows
    // pay for the packing, else 0.93 .. 1.52 (2704 x 128 x 128 17 us against 20, 5408 x 256 x 256 41 against 63) and 1.1 .. 1.3 with
    // sixteen slices, 7x7 0.48 .. 1.07.  The lines below are 0.5 % off the better of the two in the mean, 10 % at worst (5x5 and up).
    const int side = tile2d_st(0, *tile == kTileSplit192 ? 2 : 1, false, g.R, g.S), taps = g.R * g.S;
    if (generic && side == 0) {
        const bool wins = taps <= 9 ? slices * taps >= 16
                                    : taps <= 25 && (slices >= 16 || (g.M >= 600 && 2.0 * g.M * g.Ncols * g.Kred >= 1e9));
        if (!wins) return 1;
    }
    const long tiles = *tile == kTileSplit64 ? (long)((g.M + 63) / 64) * (g.Ncols / 128) : (long)((g.M + 191) / 192) * (g.Ncols / 64);
    const long target = g.R * g.S > 9 ? 2 * kNumCU : kNumCU * 27 / 32;
    long s = target / tiles;
    if (generic && s < 2 && tiles <= kNumCU * 3 / 4) s = 2;
    if (s > slices) s = slices;
    if (s < 2) return 1;
    const long per = (slices + s - 1) / s;
    s = (slices + per - 1) / per;  // none empty
    if (!generic && slices * (g.R * g.S / 9.0) * 2.2 * (1.0 - 1.0 / s) < 10.0) return 1;
    return tile2d_supported(g, *tile) ? (int)s : 1;
}

// The tile that divides a layer's pixels most evenly (0: the shape's own).  Two work-groups share a CU, so what counts is how many
// tiles the fullest CU gets, and every tile costs a start: 224 pixels leave most CUs half the work of the others where they make a
// few more tiles than CUs.  A 3x3 tile of 512 input channels takes a CU about 6 us for every 32 pixels and 4 beside, alone on its CU 5
// more (64-pixel tiles 18 in all).  us, packing included, 224 pixels / these: 22 x 28 x 28, 512 -> 512 89.7 / 75.0 (160), 512 -> 256 55.8
// (64 pixels) / 42.9, 256 -> 512 50.8 / 43.1, 45 x 14 x 14, 512 -> 512 58.1 (64) / 45.2, 11 x 28 x 28 58.4 (64) / 44.4, 45 x 27 x 27, 256 ->
// 256 50.9 / 42.1, 90 x 27 x 27 75.5 / 69.0 (192); strips of 56 x 56 maps / these, 256 -> 256 at 10 / 11 / 14 / 19 / 22 images 50.4 / 39.5
// (128), 51.4 / 44.1 (160), 54.8 / 52.1 (192), 76.6 / 66.0 (160), 78.2 / 74.5 (192).  With less than 8 % to gain nothing is left of
// it (64 x 28 x 28, 512 -> 512 188 / 186, 32 x 56 x 56, 256 -> 256 103.7 / 103.2: the clock under matrix load).
// With one slice of channels a tile is its start: 128 pixels gain nothing on 64 (88 layers 0.98 .. 1.08, 8 x 16 x 26, 32 -> 640 12.4 / 13.1).
// 256-pixel tiles: the 224-pixel strips where the fullest CU gets no more of them (112 x 112, 128 -> 128 at 3 / 6 / 8 / 11 / 16 / 22 / 32
// images 22.1 / 21.0, 34.6 / 32.2, 35.7 / 34.5, 49.4 / 46.7, 64.0 / 60.1, 78.2 / 75.6, 106.6 / 103.4; one more tile at 10 39.5 / 45.5, 64 201 / 203).
int tile2d_fill(const GemmGeom& g) {
    if (g.R != 3 || g.S != 3 || (g.Ncols % 128) != 0 || tile64_width(g)) return 0;
    const TileCfg own = tile_cfg(g);
    if (own.fn == 0 || own.variant > 2) return 0;
    auto fullest = [&](int pixels) {
        const long groups = (long)((g.M + pixels - 1) / pixels) * (g.Ncols / 128);
        return (groups + kNumCU - 1) / kNumCU;
    };
    if (own.variant == 0) return fullest(224) == fullest(256) && fill_cfg(g, kTileStrips).fn ? kTileStrips : 0;
    auto cost = [&](int fm) {
        const long n = fullest(32 * fm);
        return (double)n * (fm == 2 ? 18 : 6 * fm + 4) + (n == 1 ? 5 : 0);
    };
    int best = 0;
    double least = 0.92 * cost(own.variant == 1 ? 7 : own.fm);
    for (int fm : {6, 5, 4})
        if (!(fm == 4 && own.fm == 2 && g.IC <= 32) && cost(fm) < least && fill_cfg(g, kTileFill + fm).fn) {
            best = kTileFill + fm;
            least = cost(fm);
        }
    return best;
}

const char* tile2d_kernel_name(const GemmGeom& g, bool unpool, int tile) {
    if (!tile && tile64_width(g)) return tile64_kernel_name(g, unpool);
    const TileCfg c = tile_cfg(g, tile);
    const int u = unpool ? 1 : 0, t9 = (g.R == 3 && g.S == 3) ? 1 : 0;
    static const char* n1[2][2] = {{"conv_tile2d_kernel<1,28,7,1,false,false>", "conv_tile2d_kernel<1,28,7,1,false,true>"},
                                   {"conv_tile2d_kernel<1,28,7,1,true,false>", "conv_tile2d_kernel<1,28,7,1,true,true>"}};
    static const char* n2[2][2] = {{"conv_tile2d_kernel<1,0,7,1,false,false>", "conv_tile2d_kernel<1,0,7,1,false,true>"},
                                   {"conv_tile2d_kernel<1,0,7,1,true,false>", "conv_tile2d_kernel<1,0,7,1,true,true>"}};
    static const char* n3[2][2] = {{"conv_tile2d_kernel<1,0,3,2,false,false>", "conv_tile2d_kernel<1,0,3,2,false,true>"},
                                   {"conv_tile2d_kernel<1,0,3,2,true,false>", "conv_tile2d_kernel<1,0,3,2,true,true>"}};
    static const char* n22[2][2] = {{"conv_tile2d_kernel<1,0,2,1,false,false>", "conv_tile2d_kernel<1,0,2,1,false,true>"},
                                    {"conv_tile2d_kernel<1,0,2,1,true,false>", "conv_tile2d_kernel<1,0,2,1,true,true>"}};
    if (c.variant == 1) return n1[u][t9];
    static const char* nf[2][3] = {{"conv_tile2d_kernel<1,0,4,1,false,true>", "conv_tile2d_kernel<1,0,5,1,false,true>", "conv_tile2d_kernel<1,0,6,1,false,true>"},
                                   {"conv_tile2d_kernel<1,0,4,1,true,true>", "conv_tile2d_kernel<1,0,5,1,true,true>", "conv_tile2d_kernel<1,0,6,1,true,true>"}};
    if (c.variant == 2) return c.fm == 7 ? n2[u][t9] : c.fm == 2 ? n22[u][t9] : nf[u][c.fm - 4];
    if (c.variant == 3 && tile2d_st(0, 2, unpool, g.R, g.S) == 5) return "conv_tile2d_5x5_kernel<1,0,3,2>";
    if (c.variant == 3) return n3[u][t9];
    static const char* names[2][2][3] = {
        {{"conv_tile2d_kernel<2,32,4,2,false,false>", "conv_tile2d_kernel<2,16,4,2,false,false>", "conv_tile2d_kernel<2,8,4,2,false,false>"},
         {"conv_tile2d_kernel<2,32,4,2,false,true>", "conv_tile2d_kernel<2,16,4,2,false,true>", "conv_tile2d_kernel<2,8,4,2,false,true>"}},
        {{"conv_tile2d_kernel<2,32,4,2,true,false>", "conv_tile2d_kernel<2,16,4,2,true,false>", "conv_tile2d_kernel<2,8,4,2,true,false>"},
         {"conv_tile2d_kernel<2,32,4,2,true,true>", "conv_tile2d_kernel<2,16,4,2,true,true>", "conv_tile2d_kernel<2,8,4,2,true,true>"}}};
    return names[u][t9][c.tw == 32 ? 0 : c.tw == 16 ? 1 : 2];
}

// can the patch loader take the input operand pooled (2x2 / stride 2, whole windows) plus the argmax?
bool tile2d_fuses_unpool(const GemmGeom& g, int tile) {
    if (tile) return (g.IH % 2) == 0 && (g.IW % 2) == 0;
    if (tile64_width(g)) return tile64_fuses_unpool(g);
    if (!tile2d_supported(g) || (g.IH % 2) != 0 || (g.IW % 2) != 0) return false;
    const TileCfg c = tile_cfg(g);
    if (c.variant >= 2) return true;
    return ((c.th + g.R - 1) / 2 + 1) * ((c.tw + g.S - 1) / 2 + 1) <= 2 * (NT / 4);  // windows per patch: 2 per 4 threads
}

// partial rows (pixel tiles) the epilogue's column sums come in: [tile2d_colsum_rows][Ncols]
int tile2d_colsum_rows(const GemmGeom& g, int tile) {
    if (const int tw = tile ? 0 : tile64_width(g)) return (g.M / (g.OH * g.OW)) * (g.OW / tw) * (g.OH / (256 / tw));
    const TileCfg c = tile_cfg(g, tile);
    if (c.variant >= 2) return (g.M + tile_pixels(c) - 1) / tile_pixels(c);
    return (g.M / (g.OH * g.OW)) * (g.OW / c.tw) * (g.OH / c.th);
}

// can the epilogue also emit the 2x2 / stride-2 max-pool of the output?
bool tile2d_fuses_pool(const GemmGeom& g) {
    if (!tile2d_supported(g)) return false;
    if (tile64_width(g)) return true;  // even tile origin and size, whole tile staged
    const TileCfg c = tile_cfg(g);  // even tile origin and size, whole windows per staging pass
    if (c.variant == 0 || c.variant == 1) return true;  // strips stage the whole 224 x 128 tile in one pass
    // flat 224 x 128 tiles: whole row pairs per tile
    return c.variant == 2 && (g.OH % 2) == 0 && (g.OW % 2) == 0 && (tile_pixels(c) % (2 * g.OW)) == 0;
}

int launch_tile2d(const GemmGeom& g, const bf16_t* A, const void* Wp, const float* bias, bool relu, bf16_t* out,
                  hipStream_t st, const bf16_t* mask, bf16_t* pool_y, uint8_t* pool_am, const uint8_t* unpool_am,
                  float* colsum, int tile, int nsplit, float* part, bool w_raw) {
    if (colsum && pool_y) return set_error(WAP_EINVAL, "internal: column sums and the fused pool share the staging area");
    if (!tile && tile64_width(g)) return launch_tile64(g, A, Wp, bias, relu, out, st, mask, pool_y, pool_am, unpool_am, colsum);
    TArgs ta = {};
    ta.colsum = colsum;
    ta.mask = mask;
    if (unpool_am && !tile2d_fuses_unpool(g, tile))
        return set_error(WAP_EINVAL, "internal: fused max-pool backward not available for this shape");
    ta.up_am = unpool_am;
    if ((pool_y || pool_am) && !(pool_y && pool_am && (!tile || tile == kTileStrips) && tile2d_fuses_pool(g)))
        return set_error(WAP_EINVAL, "internal: fused pooling not available for this shape");
    if (!out && !pool_y && !part) return set_error(WAP_EINVAL, "internal: no output");
    if ((tile != 0 && tile < kTileFill) != (part != nullptr)) return set_error(WAP_EINVAL, "internal: split tiles write partial sums, others do not");
    ta.pool_y = pool_y;
    ta.pool_am = pool_am;
    if (!tile2d_supported(g, tile)) return set_error(WAP_EINVAL, "internal: 2-D tile kernel not applicable");
    const TileCfg c = tile_cfg(g, tile);
    ta.part = part;
    ta.nsplit = part ? nsplit : 1;
    ta.slices_per_split = (g.IC / BK + ta.nsplit - 1) / ta.nsplit;
    if ((long)(ta.nsplit - 1) * ta.slices_per_split >= g.IC / BK) return set_error(WAP_EINVAL, "internal: empty reduction split");
    ta.A = A;
    ta.Wp = reinterpret_cast<const bf16_t*>(Wp);
    ta.bias = bias;
    ta.out = out;
    ta.g = g;
    ta.tiles_n = c.variant == 3 ? g.Ncols / 64 : g.Ncols / 128;
    ta.RWB = c.RWB;
    ta.buf_bytes = c.buf_bytes;
    if (c.variant >= 2) {
        const int bm = tile_pixels(c);
        ta.tiles_x = ta.tiles_y = ta.tiles_img = 1;
        ta.tiles_m = (g.M + bm - 1) / bm;
        ta.PH = g.OH + g.R - 1;
        ta.RW = g.OW + g.S - 1;
        ta.dRPHW = make_fastdiv((uint32_t)(ta.PH * ta.RW));
        ta.patch_len = 0;  // per tile, computed in the kernel
        ta.dOHW = make_fastdiv((uint32_t)(g.OH * g.OW));
        ta.dOW = make_fastdiv((uint32_t)g.OW);
        ta.dOW2 = make_fastdiv((uint32_t)(g.OW / 2 > 0 ? g.OW / 2 : 1));
    } else {
        ta.tiles_x = g.OW / c.tw;
        ta.tiles_y = g.OH / c.th;
        ta.tiles_img = ta.tiles_x * ta.tiles_y;
        ta.tiles_m = ta.tiles_img * (g.M / (g.OH * g.OW));
        ta.RW = c.tw + g.S - 1;
        ta.patch_len = (c.th + g.R - 1) * ta.RW;
        // windows that can touch the patch: its first pixel may be the second of its window
        ta.UW = (c.tw + g.S - 1) / 2 + 1;
        ta.units = ((c.th + g.R - 1) / 2 + 1) * ta.UW;
        ta.dUW = make_fastdiv((uint32_t)ta.UW);
    }
    ta.relu = relu ? 1 : 0;
    ta.a_bytes = (unsigned)((size_t)(g.M / (g.OH * g.OW)) * g.IH * g.IW * g.IC * 2 / (unpool_am ? 4 : 1));
    if (w_raw && !part) return set_error(WAP_EINVAL, "internal: only split tiles take unpacked weights");
    ta.wo = w_raw ? w_unpacked(g.Kred) : w_packed(g.Kred);
    ta.w_bytes = w_raw ? (unsigned)((size_t)g.Ncols * g.Kred * 2) : (unsigned)wreg_wt_bytes(g);
    ta.dTimg = make_fastdiv((uint32_t)ta.tiles_img);
    ta.dTx = make_fastdiv((uint32_t)ta.tiles_x);
    ta.dRW = make_fastdiv((uint32_t)ta.RW);
    const size_t smem = c.smem;
    if (c.variant == 1) return launch_tile2d_t<1, 28, 7, 1>(ta, smem, st);
    if (c.variant == 2 && c.fm == 7) return launch_tile2d_t<1, 0, 7, 1>(ta, smem, st);
    if (c.variant == 2 && c.fm == 4) return launch_tile2d_fill<4>(ta, smem, st);
    if (c.variant == 2 && c.fm == 5) return launch_tile2d_fill<5>(ta, smem, st);
    if (c.variant == 2 && c.fm == 6) return launch_tile2d_fill<6>(ta, smem, st);
    if (c.variant == 2) return launch_tile2d_t<1, 0, 2, 1>(ta, smem, st);
    if (c.variant == 3) return launch_tile2d_t<1, 0, 3, 2>(ta, smem, st);
    const int TW = c.tw;  // 2-D tiles: two channel blocks per wavefront, 128-channel tiles
    if (TW == 32) return launch_tile2d_t<2, 32, 4, 2>(ta, smem, st);
    if (TW == 16) return launch_tile2d_t<2, 16, 4, 2>(ta, smem, st);
    return launch_tile2d_t<2, 8, 4, 2>(ta, smem, st);
}

}  // namespace wap
