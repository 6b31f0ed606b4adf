// Stride-1 convolution (forward, and data gradient with flipped weights) of layers too small for a chip full of large
// tiles (gfx950): flat tiles (runs of output pixels in raster order) whose REDUCTION is divided over the wavefronts of
// one work-group instead of over work-groups.
//
// A work-group of eight wavefronts owns 32 * FM pixels x 32 * CB channels.  The zero-padded input patch of the tile lies in
// LDS, a slice of 16 * KS channels at a time (double buffered), and every wavefront walks all filter taps of ONE
// 16-channel step of the slice: FM fragment reads, FM MFMAs and one weight load a tap, the same code for all, no wavefront
// waiting for another but at the slice's one barrier.  The KS partial sums of a tile meet in the LDS, are added in a fixed
// order and leave through the epilogue (bias, ReLU, mask, column sums): no partial sums in memory, no second launch.
//   * weights stream from their packed copy straight into operand registers, a ring of sets as long as the filter (3x3) or one
//     filter row (5x5), so a load has that many taps to arrive; they are read once per 32 * FM pixels;
//   * the loads of patch slice c + 2 go out when slice c + 1 is written to LDS, a whole slice ahead;
//   * neighbouring work-groups (on one XCD) share the weights where those are the larger operand, else the patch.
// Bound by the weights' way from the L2s to the CUs (22 x 14 x 14, 512 -> 512: 212 MB of weights and 50 MB of patches in 24 us;
// 64 x 128 tiles without the division read 321 MB in 32 us), the smallest by the start of a work-group: matrix pipes busy for 0.08 .. 0.30 of the
// time, LDS 0.08 .. 0.21, a third of the wavefronts' time spent waiting, 1.4 to 2.4 times the layer's bytes past the L2s (each of them reads the weights).  Against the divided
// reductions of conv_tile2d.hip with the launch that adds them up: 8 x 13 x 13, 384 -> 256 16.2 -> 10.0 us, 8 x 14 x 14, 512 -> 512
// 20.8 -> 15.0; unsplit ones 32 x 13 x 13, 384 -> 256 20.7 -> 14.3, 8 x 28 x 28, 512 -> 512 36 -> 30.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "wap_internal.h"

namespace wap {

namespace {

constexpr int NT = 512;
constexpr size_t LDS_CAP = 160 * 1024;

struct FlatArgs {
    const bf16_t* A;
    const bf16_t* Wp;      // packed weights, or the tensor itself (see wo)
    const float* bias;
    const bf16_t* mask;    // optional: out = mask > 0 ? out : 0
    const uint8_t* up_am;  // UP: argmax (r * 2 + s) per pooling window; A is then N x IH/2 x IW/2 x IC
    bf16_t* out;
    float* colsum;         // optional: [tiles_m][Ncols] column sums of this tile's stored (masked) rows
    GemmGeom g;
    int tiles_m, tiles_n, m_fast;  // m_fast: neighbouring work-groups differ in their pixels, not in their channels
    int RWB, buf_bytes;    // LDS byte stride of a patch row, bytes of one patch buffer
    int RW, PH;            // padded width and height of an image
    FastDiv dRW, dRPHW, dOHW, dOW;
    int relu;
    unsigned a_bytes, w_bytes;
    WOrder wo;
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

constexpr int pitch(int ks) { return ks * 32 + 16; }  // LDS bytes of a patch pixel: 16 rows fall into 16 bank groups of 16 bytes
// 16-byte patch vectors per thread, which bounds the patch pixels of a tile
constexpr int patch_vecs(int fm, int ks, int st) {
    return st == 5 ? (ks == 4 ? 8 : 4) : ks == 8 ? (fm == 1 ? 5 : 8) : ks == 4 ? (fm == 1 ? 3 : fm == 2 ? 4 : 5) : fm <= 2 ? 2 : 3;
}
constexpr int max_patch(int fm, int ks, int st) { return patch_vecs(fm, ks, st) * NT / (2 * ks); }

// KS wavefronts divide the reduction, CB = 8 / KS channel blocks; ST: filter side
template <int FM, int KS, bool UP, int ST>
__global__ __launch_bounds__(NT, FM <= 2 && KS <= 4 && ST == 3 && !UP ? 4 : 2) void conv_tile2d_flat_kernel(const FlatArgs a) {
    constexpr int CB = 8 / KS;
    constexpr int BM = 32 * FM, BN = 32 * CB;
    constexpr int PITCH = pitch(KS), VPP = 2 * KS, BK = 16 * KS;
    constexpr int PV = patch_vecs(FM, KS, ST);
    constexpr int RSC = ST * ST;
    constexpr int NSET = ST == 3 ? RSC : ST;  // weight sets
    constexpr int FSET = FM <= 2 ? ST : 1;    // fragment sets: taps that a fragment read is ahead of its MFMA
    constexpr int BAR_TAP = RSC - FSET;       // first tap whose fragment reads go to the next slice
    constexpr int STORE_TAP = BAR_TAP - 2;
    static_assert(RSC % NSET == 0 && RSC % FSET == 0, "a slice starts where the one before started");
    extern __shared__ __align__(16) unsigned char smem[];
    const GemmGeom& g = a.g;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave % KS, cg = wave / KS;

    const int logical = xcd_remap(blockIdx.x, a.tiles_m * a.tiles_n);
    const int tm = a.m_fast ? logical % a.tiles_m : logical / a.tiles_n;
    const int tn = a.m_fast ? logical / a.tiles_m : logical % a.tiles_n;
    const int n0 = tn * BN, m0 = tm * BM;
    const int m_last = (m0 + BM <= g.M ? m0 + BM : g.M) - 1;
    const int OHW = g.OH * g.OW, RPHW = a.PH * a.RW;
    // LDS byte position of output pixel m at tap (0,0) in the (unbounded) padded raster, rows RWB apart
    auto lbyte = [&](int m) {
        const int n = (int)fdiv((uint32_t)m, a.dOHW), rem = m - n * OHW, oh = (int)fdiv((uint32_t)rem, a.dOW);
        return (n * a.PH + oh) * a.RWB + (rem - oh * g.OW) * PITCH;
    };
    // the same in patch pixels (rows RW wide): what is loaded
    auto rflat = [&](int m) {
        const int n = (int)fdiv((uint32_t)m, a.dOHW), rem = m - n * OHW, oh = (int)fdiv((uint32_t)rem, a.dOW);
        return n * RPHW + oh * a.RW + (rem - oh * g.OW);
    };
    const int lds_lo = lbyte(m0), r_lo = rflat(m0);
    const int patch_len = rflat(m_last) + (ST - 1) * a.RW + ST - r_lo;
    const int ncs = g.IC / BK;

    const __amdgpu_buffer_rsrc_t rsrcA = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.A), 0, (int)a.a_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrcW = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.Wp), 0, (int)a.w_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrcM =  // UP: one argmax byte per pooled element, half the bytes of the pooled tensor
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(UP ? a.up_am : nullptr), 0, UP ? (int)(a.a_bytes / 2) : 0, 0x00020000);
    constexpr unsigned OOB = 0x80000000u;  // both operands are below 2 GiB (checked on the host)

    // ---- weights: packed [channel block of 32][reduction step of 16][lane][8], or [channel][reduction] ----
    const unsigned wrow = (unsigned)(tn * CB + cg) * a.wo.block + (unsigned)kg * a.wo.step + (unsigned)(lane & 31) * a.wo.row + (unsigned)(lane >> 5) * a.wo.half;
    const unsigned slicestep = KS * a.wo.step, tapstep = (unsigned)g.IC / 16u * a.wo.step;
    auto load_w = [&](unsigned row, unsigned cs, int tap) {
        return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rsrcW, row, cs * slicestep + (unsigned)tap * tapstep, 0));
    };
    bf16x8 w[NSET];
#pragma unroll
    for (int t = 0; t < NSET; ++t) w[t] = load_w(wrow, 0, t);

    // ---- patch vectors of this thread: global byte offset of (padded pixel, 8-channel vector) or OOB, and where it goes in
    // a buffer (none: to a slot of the lane's behind the buffers, so that the slice body has no branch).  UP: the offset is
    // that of the pixel's pooling window in the pooled tensor (the argmax byte sits at half of it), pvcode the pixel's
    // position (ih % 2) * 2 + iw % 2 inside the window, 2 bits per vector ----
    unsigned pvoff[PV];
    int ploff[PV];
    unsigned pvcode = 0;
    const int dump = 2 * a.buf_bytes + lane * 16;
#pragma unroll
    for (int i = 0; i < PV; ++i) {
        const int v = tid + i * NT, q = v / VPP, vec = v % VPP;
        const int p = r_lo + q;
        const int n = (int)fdiv((uint32_t)p, a.dRPHW), rem = p - n * RPHW;
        const int vh = (int)fdiv((uint32_t)rem, a.dRW), pxp = rem - vh * a.RW;
        const int ih = vh - g.pad_h, iw = pxp - g.pad_w;
        ploff[i] = q < patch_len ? (n * a.PH + vh) * a.RWB + pxp * PITCH - lds_lo + vec * 16 : -1;
        unsigned off = OOB;
        if (q < patch_len && n * OHW < g.M && (unsigned)ih < (unsigned)g.IH && (unsigned)iw < (unsigned)g.IW) {
            if (UP) {
                off = (unsigned)(((n * (g.IH >> 1) + (ih >> 1)) * (g.IW >> 1) + (iw >> 1)) * g.IC + vec * 8) * 2u;
                pvcode |= (unsigned)(((ih & 1) << 1) | (iw & 1)) << (2 * i);
            } else {
                off = (unsigned)(((n * g.IH + ih) * g.IW + iw) * g.IC + vec * 8) * 2u;
            }
        }
        pvoff[i] = off;
    }
    u32x4 rp[PV];
    u32x2 ra[UP ? PV : 1];  // an out-of-range offset halves to one that is still past the (half as long) argmax tensor
    auto issue_patch = [&](int cs) {
        const unsigned coff = (unsigned)(cs * BK) * 2u, none = cs < ncs ? 0u : OOB;
#pragma unroll
        for (int i = 0; i < PV; ++i) {
            const unsigned o = (pvoff[i] + coff) | none;
            rp[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrcA, o, 0, 0);
            if (UP) ra[i] = __builtin_amdgcn_raw_buffer_load_b64(rsrcM, o >> 1, 0, 0);
        }
    };
    auto store_patch = [&](int buf) {
#pragma unroll
        for (int i = 0; i < PV; ++i)
            *reinterpret_cast<u32x4*>(smem + (ploff[i] >= 0 ? buf + ploff[i] : dump)) =
                UP ? unpool_select8(rp[i], ra[i], (pvcode >> (2 * i)) & 3u) : rp[i];
    };
    issue_patch(0);

    // ---- fragment rows of this lane: fragment j holds tile pixels j * 32 .. + 31 ----
    int frow[FM];
#pragma unroll
    for (int j = 0; j < FM; ++j) {
        const int m = m0 + j * 32 + (lane & 31);  // past the tile's end: computed on a valid pixel, never stored
        frow[j] = lbyte(m <= m_last ? m : m_last) - lds_lo + (lane >> 5) * 16 + kg * 32;
    }
    f32x16 acc[FM];
#pragma unroll
    for (int j = 0; j < FM; ++j)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[j][e] = 0.f;

    // this wavefront's writes are done, then all wavefronts' are
    auto lds_barrier = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
    };
    store_patch(0);
    issue_patch(1);
    lds_barrier();
    bf16x8 fa[FSET][FM];
#pragma unroll
    for (int t = 0; t < FSET; ++t)
#pragma unroll
        for (int j = 0; j < FM; ++j) fa[t][j] = *reinterpret_cast<const bf16x8*>(smem + frow[j] + (t / ST) * a.RWB + (t % ST) * PITCH);

    int cur = 0, nxt = a.buf_bytes;
    for (int cs = 0; cs < ncs; ++cs) {
        const unsigned wnext = cs + 1 < ncs ? wrow : OOB;  // behind the last slice nothing is loaded (zeros, no access)
        auto tap = [&](auto tap_tag) {
            constexpr int T = decltype(tap_tag)::value;
            constexpr int TR = (T + FSET) % RSC, TW = (T + NSET) % RSC;  // tap whose fragments are read, whose weights are loaded
            const int base = (T + FSET < RSC ? cur : nxt) + (TR / ST) * a.RWB;
            __builtin_amdgcn_sched_barrier(0);
            if (T == BAR_TAP) {
                // every wavefront has written its share of the next slice, and nobody reads the buffer that the slice after
                // that will overwrite before this point again
                lds_barrier();
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int j = 0; j < FM; ++j) {
                acc[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[T % NSET], fa[T % FSET][j], acc[j], 0, 0, 0);
                fa[T % FSET][j] = *reinterpret_cast<const bf16x8*>(smem + frow[j] + base + (TR % ST) * PITCH);
            }
            w[T % NSET] = T + NSET < RSC ? load_w(wrow, cs, TW) : load_w(wnext, cs + 1, TW);
#pragma unroll
            for (int j = 0; j < FM; ++j) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);  // DS read
            }
            __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // VMEM read
            __builtin_amdgcn_sched_barrier(0);
            if (T == STORE_TAP) {
                store_patch(nxt);
                issue_patch(cs + 2);
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        each_tap(tap, std::make_integer_sequence<int, RSC>{});
        const int t = cur;
        cur = nxt;
        nxt = t;
    }

    // ---- the partial sums meet in the LDS: [kg][pixel][channel], 16 bytes of padding a row ----
    constexpr int CP = BN * 4 + 16;
    constexpr int VPR = BN / 8;             // 8-channel vectors per pixel
    constexpr int ITEMS = BM * VPR;
    constexpr int NR = (ITEMS + NT - 1) / NT;
    constexpr int RPP = NT / VPR;           // pixel rows per pass
    const int vec = tid % VPR, row0 = tid / VPR, ch = n0 + vec * 8;
    u32x4 mk[NR];
    if (a.mask) {  // fetched ahead of the stores
#pragma unroll
        for (int it = 0; it < NR; ++it) {
            int m = m0 + row0 + it * RPP;
            if (m > m_last) m = m_last;  // never stored
            mk[it] = ch < g.Ncols ? *reinterpret_cast<const u32x4*>(a.mask + (size_t)m * g.Ncols + ch) : u32x4{0u, 0u, 0u, 0u};
        }
    }
    __syncthreads();  // the last readers of the patch are done
#pragma unroll
    for (int j = 0; j < FM; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<f32x4*>(smem + (kg * BM + j * 32 + (lane & 31)) * CP + (cg * 32 + q * 8 + (lane >> 5) * 4) * 4) =
                f32x4{acc[j][q * 4], acc[j][q * 4 + 1], acc[j][q * 4 + 2], acc[j][q * 4 + 3]};
    __syncthreads();
    float bv[8], csum[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        csum[e] = 0.f;
        bv[e] = a.bias && ch + e < g.Ncols ? a.bias[ch + e] : 0.f;
    }
#pragma unroll
    for (int it = 0; it < NR; ++it) {
        const int row = row0 + it * RPP, m = m0 + row;
        if (row >= BM || m > m_last || ch >= g.Ncols) continue;
        f32x4 s[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            s[h] = *reinterpret_cast<const f32x4*>(smem + row * CP + vec * 32 + h * 16);
#pragma unroll
            for (int k = 1; k < KS; ++k) s[h] += *reinterpret_cast<const f32x4*>(smem + (k * BM + row) * CP + vec * 32 + h * 16);
        }
        u32x4 vv;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float lo = s[k >> 1][(k & 1) * 2], hi = s[k >> 1][(k & 1) * 2 + 1];
            if (a.bias) {
                lo += bv[2 * k];
                hi += bv[2 * k + 1];
            }
            if (a.relu) {
                lo = lo > 0.f ? lo : 0.f;
                hi = hi > 0.f ? hi : 0.f;
            }
            vv[k] = (unsigned)f2bf(lo) | ((unsigned)f2bf(hi) << 16);
        }
        if (a.mask) vv = relu_mask8(vv, mk[it]);
        *reinterpret_cast<u32x4*>(a.out + (size_t)m * g.Ncols + ch) = vv;
        if (a.colsum) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                csum[2 * k] += __uint_as_float(vv[k] << 16);
                csum[2 * k + 1] += __uint_as_float(vv[k] & 0xffff0000u);
            }
        }
    }
    // ---- column sums of the stored tile: the row groups added in group order, one partial row per pixel tile ----
    if (a.colsum) {
        constexpr int GROUPS = RPP < BM ? RPP : BM;
        __syncthreads();  // the sums have been read
        float* red = reinterpret_cast<float*>(smem);  // [GROUPS][BN]
        if (row0 < GROUPS) {
#pragma unroll
            for (int e = 0; e < 8; ++e) red[row0 * BN + vec * 8 + e] = csum[e];
        }
        __syncthreads();
        if (tid < BN && n0 + tid < g.Ncols) {
            float t = red[tid];
            for (int k = 1; k < GROUPS; ++k) t += red[k * BN + tid];
            a.colsum[(size_t)tm * g.Ncols + n0 + tid] = t;
        }
    }
}

// ---- host: layout and choice of a tiling ----
struct FlatCfg {
    int fm, ks;  // 0: none
    int RWB, buf_bytes;
    size_t smem;
};

// Most patch pixels that a bm-pixel tile loads, and most LDS bytes it spans with patch rows rwb bytes apart, wherever it starts: a run
// of bm pixels ends at most dr rows further down, dn images on.
void patch_extent(const GemmGeom& g, int bm, int rwb, int pit, long* pixels, long* bytes) {
    const long images = g.M / ((long)g.OH * g.OW), PW = g.OW + g.S - 1;
    if (bm > g.M) bm = g.M;
    const long dr = std::min((long)(bm + g.OW - 2) / g.OW, images * g.OH - 1);
    const long dn = std::min((dr + g.OH - 1) / g.OH, images - 1);
    const long rows = (dn + 1) * (g.R - 1);  // rows of padding in between, and the filter's
    *pixels = bm - 1 + dr * (PW - g.OW) + rows * PW + g.S;
    *bytes = (bm - 1) * (long)pit + dr * (rwb - (long)g.OW * pit) + rows * rwb + (long)g.S * pit;
}

bool flat_layout(const GemmGeom& g, int fm, int ks, FlatCfg* c) {
    if ((g.IC % (16 * ks)) != 0 || (g.R == 5 && ks == 8)) return false;
    const int bm = 32 * fm, pit = pitch(ks);
    const size_t sums = (size_t)ks * bm * (32 * (8 / ks) * 4 + 16);
    // rows a whole number of bank rounds beyond the row's last output pixel: fragments that wrap to the next row stay free
    // of conflicts; else as dense as they come
    const int cands[2] = {g.OW * pit + ((g.S - 1) * pit + 255) / 256 * 256, (g.OW + g.S - 1) * pit};
    for (int rwb : cands) {
        long px, by;
        patch_extent(g, bm, rwb, pit, &px, &by);
        if (px > max_patch(fm, ks, g.R)) return false;
        const long buf = (by + 15) / 16 * 16;
        const size_t smem = std::max((size_t)(2 * buf) + 1024, sums);  // + the slots of stores without a pixel
        if (smem > LDS_CAP) continue;
        *c = {fm, ks, rwb, (int)buf, smem};
        return true;
    }
    return false;
}

// the tilings there are
constexpr int kFlatTiles[] = {14, 18, 22, 24, 28, 32, 34, 42, 44};
bool flat_tile_exists(int tile) {
    for (int t : kFlatTiles)
        if (t == tile) return true;
    return false;
}

FlatCfg flat_cfg(const GemmGeom& g, int tile) {
    FlatCfg c = {0, 0, 0, 0, 0};
    const int fm = tile / 10, ks = tile % 10;
    if (!flat_tile_exists(tile)) return c;
    if (!flat_layout(g, fm, ks, &c)) c.fm = 0;
    return c;
}

template <typename F>
int launch_flat_k(F kfn, std::atomic<bool>& attr_done, const FlatArgs& fa, size_t smem, hipStream_t st) {
    if (!attr_done) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn), hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_CAP);
        if (e != hipSuccess) return set_error(WAP_EHIP, "hipFuncSetAttribute: %s", hipGetErrorString(e));
        attr_done = true;
    }
    hipLaunchKernelGGL(kfn, dim3(fa.tiles_m * fa.tiles_n), dim3(NT), smem, st, fa);
    return check_launch("conv_tile2d_flat");
}
template <int FM, int KS>
int launch_flat_t(const FlatArgs& fa, size_t smem, hipStream_t st) {
    static std::atomic<bool> done3{false}, done3u{false}, done5{false}, done5u{false};
    if (fa.g.R == 3 && fa.up_am) return launch_flat_k(conv_tile2d_flat_kernel<FM, KS, true, 3>, done3u, fa, smem, st);
    if (fa.g.R == 3) return launch_flat_k(conv_tile2d_flat_kernel<FM, KS, false, 3>, done3, fa, smem, st);
    if constexpr (KS != 8) {
        if (fa.g.R == 5 && fa.up_am) return launch_flat_k(conv_tile2d_flat_kernel<FM, KS, true, 5>, done5u, fa, smem, st);
        if (fa.g.R == 5) return launch_flat_k(conv_tile2d_flat_kernel<FM, KS, false, 5>, done5, fa, smem, st);
    }
    return set_error(WAP_EINVAL, "internal: flat tiles take 3x3 and 5x5 filters");
}
}  // namespace

bool flat_supported(const GemmGeom& g, int tile) {
    if ((g.IC % 32) != 0 || (g.Ncols % 8) != 0 || g.R != g.S || (g.R != 3 && g.R != 5)) return false;
    if (g.div_h != 1 || g.div_w != 1 || g.mul_h != 1 || g.mul_w != 1) return false;
    const double a_bytes = 2.0 * (g.M / ((long)g.OH * g.OW)) * g.IH * g.IW * g.IC;
    if (a_bytes >= 2147483648.0 || (double)wreg_wt_bytes(g) >= 2147483648.0) return false;
    return flat_cfg(g, tile).fm != 0;
}

// The tiling for a layer, and the time it takes in us.  The model is fitted to nine tilings of 351 products of 0.02 to 50 GFLOP (3x3 and
// 5x5, 32 to 512 channels, maps of 7 to 112 pixels, 1 to 64 images; rms error 9 %, the tiling it picks 0.4 % slower than the
// best in the mean): a start, and for every work-group a CU runs after another its own start, its MFMAs, its patch, and the
// weights and patches of all work-groups through the L2s.
int flat_pick(const GemmGeom& g, double* us_out) {
    int best = 0;
    double best_us = 0;
    for (int tile : kFlatTiles) {
        const int fm = tile / 10, ks = tile % 10;
        if (!flat_supported(g, tile)) continue;
        const FlatCfg c = flat_cfg(g, tile);
        const int bn = 32 * (8 / ks);
        const long groups = (long)((g.M + 32 * fm - 1) / (32 * fm)) * ((g.Ncols + bn - 1) / bn);
        long pixels, bytes;
        patch_extent(g, 32 * fm, c.RWB, pitch(ks), &pixels, &bytes);
        const bool two = c.smem <= LDS_CAP / 2 && (g.R == 3 ? fm <= 2 && tile != 28 : tile == 14);  // work-groups on a CU
        const long r = (groups + kNumCU - 1) / kNumCU;
        const double rounds = two ? 1.0 + 0.9 * (r - 1) : (double)r;
        const double fill = groups < kNumCU ? (double)groups / kNumCU : 1.0;
        const double mfma = (double)g.Kred / 16 / ks * fm * 0.032;                  // us at 2 GHz, two wavefronts a SIMD
        const double wmb = bn * 2e-6 * g.Kred, pmb = pixels * 2e-6 * g.IC;  // MB that a work-group reads
        const double us = 3.2 + rounds * (2.5 + 1.06 * mfma + 9.5 * pmb + fill * (2.1 * wmb + 5.1 * pmb));
        if (!best || us < best_us) {
            best = tile;
            best_us = us;
        }
    }
    *us_out = best_us;
    return best;
}

bool flat_fuses_unpool(const GemmGeom& g) { return (g.IH % 2) == 0 && (g.IW % 2) == 0; }
int flat_colsum_rows(const GemmGeom& g, int tile) { return (g.M + 32 * (tile / 10) - 1) / (32 * (tile / 10)); }

const char* flat_kernel_name(const GemmGeom& g, int tile, bool unpool) {
#define WAP_FLAT_ONE(FM, KS, UP, ST) "conv_tile2d_flat_kernel<" #FM "," #KS "," #UP "," #ST ">"
#define WAP_FLAT_KS(FM, KS) {WAP_FLAT_ONE(FM, KS, false, 3), WAP_FLAT_ONE(FM, KS, true, 3), WAP_FLAT_ONE(FM, KS, false, 5), WAP_FLAT_ONE(FM, KS, true, 5)}
#define WAP_FLAT(FM) {WAP_FLAT_KS(FM, 2), WAP_FLAT_KS(FM, 4), WAP_FLAT_KS(FM, 8)}
    static const char* names[4][3][4] = {WAP_FLAT(1), WAP_FLAT(2), WAP_FLAT(3), WAP_FLAT(4)};
#undef WAP_FLAT
#undef WAP_FLAT_KS
#undef WAP_FLAT_ONE
    return names[tile / 10 - 1][tile % 10 / 4][(g.R == 5 ? 2 : 0) + (unpool ? 1 : 0)];
}

int launch_flat(const GemmGeom& g, int tile, const bf16_t* A, const void* Wp, const float* bias, bool relu, bf16_t* out, hipStream_t st,
                const bf16_t* mask, const uint8_t* unpool_am, float* colsum, bool w_raw) {
    if (!flat_supported(g, tile) || (unpool_am && !flat_fuses_unpool(g))) return set_error(WAP_EINVAL, "internal: flat tiles not applicable");
    const FlatCfg c = flat_cfg(g, tile);
    FlatArgs fa = {};
    fa.A = A;
    fa.Wp = reinterpret_cast<const bf16_t*>(Wp);
    fa.bias = bias;
    fa.mask = mask;
    fa.up_am = unpool_am;
    fa.out = out;
    fa.colsum = colsum;
    fa.g = g;
    const int bm = 32 * c.fm, bn = 32 * (8 / c.ks);
    fa.tiles_m = (g.M + bm - 1) / bm;
    fa.tiles_n = (g.Ncols + bn - 1) / bn;
    fa.RWB = c.RWB;
    fa.buf_bytes = c.buf_bytes;
    fa.RW = g.OW + g.S - 1;
    fa.PH = g.OH + g.R - 1;
    fa.dRW = make_fastdiv((uint32_t)fa.RW);
    fa.dRPHW = make_fastdiv((uint32_t)(fa.PH * fa.RW));
    fa.dOHW = make_fastdiv((uint32_t)(g.OH * g.OW));
    fa.dOW = make_fastdiv((uint32_t)g.OW);
    fa.relu = relu ? 1 : 0;
    fa.a_bytes = (unsigned)((size_t)(g.M / (g.OH * g.OW)) * g.IH * g.IW * g.IC * 2 / (unpool_am ? 4 : 1));
    fa.wo = w_raw ? w_unpacked(g.Kred) : w_packed(g.Kred);
    fa.w_bytes = w_raw ? (unsigned)((size_t)g.Ncols * g.Kred * 2) : (unsigned)wreg_wt_bytes(g);
    fa.m_fast = fa.w_bytes > fa.a_bytes;
#define WAP_FLAT_TILE(FM, KS) \
    if (tile == FM * 10 + KS) return launch_flat_t<FM, KS>(fa, c.smem, st);
    WAP_FLAT_TILE(1, 4) WAP_FLAT_TILE(1, 8) WAP_FLAT_TILE(2, 2) WAP_FLAT_TILE(2, 4) WAP_FLAT_TILE(2, 8)
    WAP_FLAT_TILE(3, 2) WAP_FLAT_TILE(3, 4) WAP_FLAT_TILE(4, 2) WAP_FLAT_TILE(4, 4)
#undef WAP_FLAT_TILE
    return set_error(WAP_EINVAL, "internal: no such flat tile");
}

}  // namespace wap
