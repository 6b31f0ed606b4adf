// Forward-type implicit GEMM on bf16 MFMA (gfx950): rows = output pixels (gathered from an NHWC
// tensor), columns = output channels, reduction = filter taps x input channels.
//
// Serves the convolution forward pass, the convolution data gradient (rows = input pixels,
// gathered from dy; the weights are read with flipped taps and transposed through LDS) and both
// FC products that keep the batch as the row dimension (Section 3.2.2 "primary" nodes; the
// forward / backward halves of t_c in Eq. 1).
//
// Design for CDNA4:
// Bound by what a work-group does one thing after the other (12 x 57 x 57 x 72 -> 200, 3x3 stride 2, 158 work-groups of 11
// reduction tiles: addresses 0.6 us, first loads 1.5, 0.64 a tile, epilogue 1.4; with the address divisions and the loads of one
// tile ahead of four wavefronts' products, 0.93 a tile and 21.5 us for the call; this 12.8).
//   * block tile BM x BN x 64, 64-wide wavefronts each owning a (BM/WAVES_M) x (BN/WAVES_N)
//     sub-tile built from v_mfma_f32_32x32x16_bf16; the weight fragment is the MFMA "A" operand so
//     that each lane ends up with 4 consecutive output channels of one pixel (8-byte bf16 stores);
//   * operands staged through LDS, two stages, up to four more tiles in flight in registers; the step of a tile is one basic
//     block (no branch around a load or in the walk over the taps), so that address arithmetic, loads and LDS writes issue
//     between the MFMAs (one barrier per tile);
//   * where the grid leaves a CU one work-group, eight wavefronts share its tile, two for every sub-tile: each takes half of
//     the reduction steps and the sums meet in the LDS;
//   * LDS rows padded (144 B for reduction-contiguous tiles, +64 B for channel-contiguous tiles) so
//     ds_read_b128 / ds_read_b64_tr_b16 fragment reads are bank-conflict free;
//   * channel-contiguous weight tiles (data gradient) are transposed on the way out of LDS with
//     ds_read_b64_tr_b16 instead of a separate transpose pass over the weights;
//   * blockIdx is remapped so that each XCD (own L2) works on a contiguous range of tiles.
#include <algorithm>
#include <type_traits>

#include "wap_internal.h"

namespace wap {

namespace {

constexpr int BK = 64;
constexpr int A_PITCH = (BK + 8) * 2;  // bytes per LDS row of a reduction-contiguous tile

// Wavefronts that share a sub-tile and divide every reduction tile between them; their sums meet in the LDS at the end.  Two
// where a CU has one work-group (wavefronts of the same SIMD then cover each other's LDS and MFMA latency: 0.85 -> 0.64 us a
// tile); a grid of more than one work-group per CU has that from its neighbours, two of four wavefronts each (32 x 28 x 28,
// 512 <- 128 channels, 1x1: 17.1 us, 21.5 with eight wavefronts each in half the registers).
constexpr int waves_k(int bm, int bn, int variant) { return bm * bn <= 128 * 128 && !(variant & 8) ? 2 : 1; }

// One phase of a strided data gradient: the output pixels whose coordinates leave the same remainders (oh0, ow0) modulo
// the strides.  Only the filter taps r0, r0 + stride, ... meet a dy element there, so a phase is an ordinary stride-1
// product of its own, with R x S of the taps.
constexpr int kMaxPhases = 16;
struct Phase {
    int R, S, r0, s0, OH, OW, pad_h, pad_w, oh0, ow0, M;
    int tile0;  // first row tile
    FastDiv dOW, dOH;
};

struct KArgs {
    const bf16_t* A;
    const bf16_t* Bw;
    const float* bias;
    const bf16_t* mask;  // out = mask > 0 ? out : 0 (unsplit reductions)
    void* out;
    GemmGeom g;
    int tiles_m, tiles_n, nsplit, ktiles, ktiles_per_split;
    int relu, partial;
    unsigned a_bytes, b_bytes;  // of the operands
    int ICp;      // MODE 2: channels rounded up to 8, the reduction's length per tap (no group of 8 crosses a tap)
    FastDiv dICp;
    FastDiv dOW, dOH;  // row -> pixel (a phase has its own)
};
// (apart, so that the other launches do not carry the phases in their arguments: with them a short product, 302 x 256 ->
// 25088, took 35 instead of 22 us)
struct KPhaseArgs : KArgs {
    int nphase;
    Phase ph[kMaxPhases];
};

__device__ __forceinline__ int xcd_remap(int bid, int total) {
    int per = total / kNumXCD, rem = total % kNumXCD;
    int xcd = bid % kNumXCD, idx = bid / kNumXCD;
    return xcd < rem ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
}

// Out-of-image taps and tile tails load from beyond the buffer, which yields zeros and costs no access: the loaded
// registers then have no consumer until the LDS store, so the latency overlaps the compute of the tiles before.  (As loads of
// a block of zeros they all met in one L2 channel.)
constexpr unsigned kNowhere = 0xfffffff0u;  // operands of the modes 0 .. 2 end before (classify_mode)
// the same element by element
__device__ __align__(16) unsigned int g_zero_block[4] = {0u, 0u, 0u, 0u};

__device__ __forceinline__ unsigned short f2bf(float f) {
    __bf16 b = (__bf16)f;  // round to nearest even
    return __builtin_bit_cast(unsigned short, b);
}

__device__ __forceinline__ u32x4 pack8(const unsigned short* h) {
    u32x4 v = {(unsigned)h[0] | ((unsigned)h[1] << 16), (unsigned)h[2] | ((unsigned)h[3] << 16),
               (unsigned)h[4] | ((unsigned)h[5] << 16), (unsigned)h[6] | ((unsigned)h[7] << 16)};
    return v;
}

// MODE 0: fast  -- channel counts multiples of 64 / 8, unit tap divisor, 16-byte loads, one tap per tile
// MODE 1: vec   -- channel counts multiples of 8, any geometry
// MODE 2: odd   -- any channel counts of at least 8: unaligned 16-byte loads, every tap's channels rounded up to a multiple
//                  of 8 in the reduction (element by element, as MODE 3 does it, 288 x 4096 -> 3373 took 253 us for dx)
// MODE 3: scalar-- anything (2-byte loads)
// VARIANT: the mode, plus 8 where the grid has more than one work-group per CU (waves_k); plus 4 for PHASE: data gradient of a
// strided convolution, the row tiles grouped by phase (a.ph): a tap
// between dy elements costs nothing, where the unphased product multiplies stride_h * stride_w times as many zeros (12 x
// 57 x 57, 200 -> 72 channels, 3x3 stride 2: block forward and backward 141 -> 103 us)
// (One kernel, not two around a shared device function, behind whose call the compiler did not hoist the argument loads.)
template <int BM, int BN, int WAVES_M, int WAVES_N, bool B_TR, int VARIANT>
__global__ __launch_bounds__(64 * WAVES_M * WAVES_N * waves_k(BM, BN, VARIANT), (VARIANT & 8) ? 2 : 1) void igemm_kernel(
    const std::conditional_t<(VARIANT & 4) != 0, KPhaseArgs, KArgs> a) {
    constexpr bool PHASE = (VARIANT & 4) != 0;
    constexpr int MODE = VARIANT & 3;
    constexpr int WAVES_K = waves_k(BM, BN, VARIANT);
    constexpr int NT = 64 * WAVES_M * WAVES_N * WAVES_K;
    constexpr int WM = BM / WAVES_M, WN = BN / WAVES_N;
    constexpr int FM = WM / 32, FN = WN / 32;
    constexpr int A_RPP = NT / 8, A_PASSES = BM / A_RPP;
    constexpr int B_PITCH = B_TR ? (BN * 2 + 64) : A_PITCH;
    constexpr int B_VPR = B_TR ? BN / 8 : 8;  // 16-byte vectors per LDS row
    constexpr int B_RPP = NT / B_VPR;
    constexpr int B_ROWS = B_TR ? BK : BN;
    constexpr int B_PASSES = B_ROWS / B_RPP;
    constexpr int A_BYTES = BM * A_PITCH;
    constexpr int B_BYTES = B_ROWS * B_PITCH;
    constexpr int STAGE = A_BYTES + B_BYTES;
    static_assert(A_PASSES >= 1 && B_PASSES >= 1, "tile too small for the block");
    // Register sets for tiles in flight.  Four for the square tile (100 x 9216 -> 4096 22.6 us, 24.4 with two); the long ones, whose
    // loads take most of the memory's rate, start earlier with two (64 x 4096 -> 4096 18.4 us, 20.8 with four).
    constexpr int SETS = WAVES_K == 2 && MODE < 3 && BM == BN ? 4 : BM * BN <= 128 * 128 ? 2 : 1;

    extern __shared__ __align__(16) unsigned char smem[];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave % WAVES_M, wn = WAVES_K == 1 ? wave / WAVES_M : wave / WAVES_M % WAVES_N, wk = WAVES_K == 1 ? 0 : wave / (WAVES_M * WAVES_N);

    const int total = a.tiles_m * a.tiles_n * a.nsplit;
    // (phases differ in work: neighbouring work-groups go to different XCDs there)
    int logical = PHASE ? (int)blockIdx.x : xcd_remap(blockIdx.x, total);
    const int tn = logical % a.tiles_n;
    logical /= a.tiles_n;
    int tm = logical % a.tiles_m;
    const int split = logical / a.tiles_m;
    GemmGeom gp;
    int r0 = 0, s0 = 0, oh0 = 0, ow0 = 0;
    int ktiles = a.ktiles, kps = a.ktiles_per_split;
    FastDiv dOW = a.dOW, dOH = a.dOH;
    if constexpr (PHASE) {
        int c = 0;
        while (c + 1 < a.nphase && tm >= a.ph[c + 1].tile0) ++c;
        const Phase& p = a.ph[c];
        tm -= p.tile0;
        gp = a.g;
        gp.R = p.R; gp.S = p.S; gp.OH = p.OH; gp.OW = p.OW; gp.M = p.M;
        gp.pad_h = p.pad_h; gp.pad_w = p.pad_w;
        gp.mul_h = gp.mul_w = gp.div_h = gp.div_w = 1;
        gp.Kred = p.R * p.S * (MODE == 2 ? a.ICp : gp.IC);
        dOW = p.dOW; dOH = p.dOH;
        r0 = p.r0; s0 = p.s0; oh0 = p.oh0; ow0 = p.ow0;
        ktiles = (gp.Kred + BK - 1) / BK;
        kps = (ktiles + a.nsplit - 1) / a.nsplit;
    }
    const GemmGeom& g = PHASE ? gp : a.g;
    const int m0 = tm * BM, n0 = tn * BN;
    const int kt_begin = split * kps;
    int kt_end = kt_begin + kps;
    if (kt_end > ktiles) kt_end = ktiles;

    // ---- per-thread row state of the gathered operand ----
    const bool unit = MODE == 0 || PHASE || !B_TR || (g.div_h == 1 && g.div_w == 1);  // taps of neighbouring steps are neighbours in memory
    const int a_vec = tid & 7, a_row0 = tid >> 3;
    int hb[A_PASSES], wb[A_PASSES], abase[A_PASSES];  // unit: abase is the element of tap (0, 0), which may lie outside
#pragma unroll
    for (int i = 0; i < A_PASSES; ++i) {
        int m = m0 + a_row0 + i * A_RPP;
        if (m < g.M) {
            const int t = (int)fdiv((uint32_t)m, dOW), ow = m - t * g.OW;
            const int n = (int)fdiv((uint32_t)t, dOH), oh = t - n * g.OH;
            hb[i] = oh * g.mul_h - g.pad_h;
            wb[i] = ow * g.mul_w - g.pad_w;
            abase[i] = n * g.IH * g.IW * g.IC;
            if (unit) abase[i] += (hb[i] * g.IW + wb[i]) * g.IC;
        } else {
            hb[i] = -(1 << 28);
            wb[i] = -(1 << 28);
            abase[i] = 0;
        }
    }
    const int b_vec = tid % B_VPR, b_row0 = tid / B_VPR;
    const bf16_t* zero_src = reinterpret_cast<const bf16_t*>(g_zero_block);  // MODE 3
    const __amdgpu_buffer_rsrc_t rsrcA = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.A), 0, (int)a.a_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrcB = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.Bw), 0, (int)a.b_bytes, 0x00020000);
    auto ld8 = [](__amdgpu_buffer_rsrc_t r, bool ok, int off, unsigned past) {
        return __builtin_amdgcn_raw_buffer_load_b128(r, (ok ? (unsigned)off * 2u : kNowhere) | past, 0, 0);
    };

    // ---- walk over the reduction tiles: from an offset of the work-group's own, wrapping.  Work-groups running at the same
    // time then read different channel slices and filter taps, which spreads their requests over the L2 channels instead of
    // hammering the same few.  The fast mode walks channel-slice-major (all filter taps of one 64-channel slice before the
    // next slice): the 9 (or 25) shifted re-reads of the same input pixels then happen in consecutive tiles and hit in L2
    // instead of going back to HBM. ----
    const int nkt = kt_end - kt_begin;
    int cur = kt_begin + (nkt > 0 ? (int)(((unsigned)blockIdx.x / kNumXCD * 5u) % (unsigned)nkt) : 0);  // next tile to load
    int loaded = 0;                                                                                     // tiles loaded so far
    // MODE 0: tap and channel slice of that tile, and of the walk's first one
    int wr = 0, ws = 0, wc = 0, br = 0, bs = 0, bc = 0;
    if (MODE == 0 && nkt > 0) {
        const int RS = g.R * g.S;
        wc = cur / RS; ws = cur - wc * RS; wr = ws / g.S; ws -= wr * g.S; wc *= BK;
        bc = kt_begin / RS; bs = kt_begin - bc * RS; br = bs / g.S; bs -= br * g.S; bc *= BK;
    }
    // MODE 1, 2: lane l holds the decoded group of eight reduction elements l % 8 of the l / 8-th of the next eight tiles;
    // the loads fetch theirs from there.  (Divisions for every tile and pass took more time than the products: 12 x 57 x 57 x 72
    // -> 200, 3x3 stride 2, 27.8 us with them.)
    int t_rs = 0, t_c = 0, t_a = 0, t_b = 0;  // tap r | s << 8 | elements moved back << 16, -1: past the end; channel; offsets
    auto decode = [&]() {
        int kt = cur + (lane >> 3);
        while (kt >= kt_end) kt -= nkt;  // (lanes past the walk's end decode tiles again)
        const int kk = kt * BK + (lane & 7) * 8;
        const int tapk = MODE == 2 ? a.ICp : g.IC;
        const int tap = MODE == 2 ? (int)fdiv((uint32_t)kk, a.dICp) : kk / tapk;
        int c = kk - tap * tapk;
        const int r = tap / g.S, s = tap - r * g.S;
        if (B_TR) {  // (channel c of the group is its first reduction row here, whatever the row's length)
            const int rf = PHASE ? r0 + r * a.g.div_h : r, sf = PHASE ? s0 + s * a.g.div_w : s;
            t_b = ((c * a.g.R + (a.g.R - 1 - rf)) * a.g.S + (a.g.S - 1 - sf)) * g.Ncols;
        }
        t_c = c;
        const int over = MODE == 2 && c + 8 > g.IC ? c + 8 - g.IC : 0;
        c -= over;
        t_a = (r * g.IW + s) * g.IC + c;
        if (!B_TR) t_b = tap * g.IC + c;
        t_rs = tap < g.R * g.S ? r | (s << 8) | (over << 16) : -1;
    };
    auto beyond = [](int rs) { return (unsigned)(rs >> 31) & kNowhere; };
    auto from_lane = [](int v, int src) { return __builtin_amdgcn_ds_bpermute(src * 4, v); };

    auto load_global = [&](u32x4 (&ra)[A_PASSES], u32x4 (&rb)[B_PASSES]) {
        // past the walk's end: nothing (the loop's loads are unconditional, see there; a condition would become a branch)
        const unsigned past = loaded < nkt ? 0u : kNowhere;
        if constexpr (MODE == 0) {
            const int adelta = (wr * g.IW + ws) * g.IC + wc + a_vec * 8;
#pragma unroll
            for (int i = 0; i < A_PASSES; ++i) {
                const bool ok = (unsigned)(hb[i] + wr) < (unsigned)g.IH && (unsigned)(wb[i] + ws) < (unsigned)g.IW;
                ra[i] = ld8(rsrcA, ok, abase[i] + adelta, past);
            }
            if (!B_TR) {
                // Bw[n][kk]: LDS row = output channel, 8 vectors of 8 reduction elements per row
                const int kk = (wr * g.S + ws) * g.IC + wc + b_vec * 8;
#pragma unroll
                for (int i = 0; i < B_PASSES; ++i) {
                    const int n = n0 + b_row0 + i * B_RPP;
                    rb[i] = ld8(rsrcB, n < g.Ncols, n * g.Kred + kk, past);
                }
            } else {
                // Bw[k][R-1-r][S-1-s][n]: LDS row = reduction index k of one tap, BN/8 vectors of 8 channels
                const int rf = PHASE ? r0 + wr * a.g.div_h : wr, sf = PHASE ? s0 + ws * a.g.div_w : ws;
                const int n = n0 + b_vec * 8, tapoff = (a.g.R - 1 - rf) * a.g.S + (a.g.S - 1 - sf);
#pragma unroll
                for (int i = 0; i < B_PASSES; ++i) {
                    const int k = wc + b_row0 + i * B_RPP;
                    rb[i] = ld8(rsrcB, n < g.Ncols, (k * a.g.R * a.g.S + tapoff) * g.Ncols + n, past);
                }
            }
            const bool row = ws + 1 == g.S, slice = row && wr + 1 == g.R, wrap = cur + 1 == kt_end;
            cur = wrap ? kt_begin : cur + 1;
            wc = wrap ? bc : slice ? wc + BK : wc;
            wr = wrap ? br : slice ? 0 : row ? wr + 1 : wr;
            ws = wrap ? bs : row ? 0 : ws + 1;
            ++loaded;
        } else if constexpr (MODE <= 2) {
            if ((loaded & 7) == 0) decode();
            const int src0 = (loaded & 7) * 8;
            // ---------- gathered operand ----------
            {
                const int rs = from_lane(t_rs, src0 + a_vec), ad = from_lane(t_a, src0 + a_vec);
                const int r = rs & 255, s = (rs >> 8) & 255, over = (rs >> 16) & 7;
                const unsigned none = beyond(rs) | past;
                const int c = unit ? 0 : from_lane(t_c, src0 + a_vec) - over;
#pragma unroll
                for (int i = 0; i < A_PASSES; ++i) {
                    const int th = hb[i] + r, tw = wb[i] + s;
                    bool ok;
                    int off;
                    if (unit) {
                        ok = (unsigned)th < (unsigned)g.IH && (unsigned)tw < (unsigned)g.IW;
                        off = abase[i] + ad;
                    } else {
                        const int ih = th / g.div_h, iw = tw / g.div_w;
                        ok = th >= 0 && tw >= 0 && ih * g.div_h == th && iw * g.div_w == tw && ih < g.IH && iw < g.IW;
                        off = abase[i] + (ih * g.IW + iw) * g.IC + c;
                    }
                    ra[i] = ld8(rsrcA, ok, off, none);
                    if (MODE == 2) ra[i] = shift_down8(ra[i], over);
                }
            }
            // ---------- weight operand ----------
            if (!B_TR) {
                const int rs = from_lane(t_rs, src0 + b_vec), kk = from_lane(t_b, src0 + b_vec), over = (rs >> 16) & 7;
                const unsigned none = beyond(rs) | past;
#pragma unroll
                for (int i = 0; i < B_PASSES; ++i) {
                    const int n = n0 + b_row0 + i * B_RPP;
                    rb[i] = ld8(rsrcB, n < g.Ncols, n * g.Kred + kk, none);
                    if (MODE == 2) rb[i] = shift_down8(rb[i], over);
                }
            } else {
                // LDS row = reduction index (r,s,k): row j of the group's eight is its channel c + j
                const int n = n0 + b_vec * 8;
                const int nover = MODE == 2 && n + 8 > g.Ncols ? n + 8 - g.Ncols : 0;
#pragma unroll
                for (int i = 0; i < B_PASSES; ++i) {
                    const int row = b_row0 + i * B_RPP, src = src0 + (row >> 3), j = row & 7;
                    const int rs = from_lane(t_rs, src);
                    const int off = from_lane(t_b, src) + j * a.g.R * a.g.S * g.Ncols + n - nover;
                    const unsigned none = beyond(rs) | past;
                    if (MODE == 2) rb[i] = shift_down8(ld8(rsrcB, j + ((rs >> 16) & 7) < 8 && nover < 8, off, none), nover < 8 ? nover : 0);
                    else rb[i] = ld8(rsrcB, n < g.Ncols, off, none);
                }
            }
            ++loaded;
            if (++cur == kt_end) cur = kt_begin;
        } else {
            const int kk0 = past ? ktiles * BK : cur * BK;
            if (++cur == kt_end) cur = kt_begin;
            ++loaded;
            int rr[8], ss[8], cc[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                int kk = kk0 + a_vec * 8 + e;
                int tap = kk / g.IC;
                cc[e] = kk - tap * g.IC;
                rr[e] = tap / g.S;
                ss[e] = tap - rr[e] * g.S;
                if (kk >= g.Kred) rr[e] = -(1 << 20);  // forces the row test to fail
            }
#pragma unroll
            for (int i = 0; i < A_PASSES; ++i) {
                unsigned short h16[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int th = hb[i] + rr[e], tw = wb[i] + ss[e];
                    bool ok;
                    int off;
                    if (unit) {
                        ok = (unsigned)th < (unsigned)g.IH && (unsigned)tw < (unsigned)g.IW;
                        off = abase[i] + (rr[e] * g.IW + ss[e]) * g.IC + cc[e];
                    } else {
                        const int ih = th / g.div_h, iw = tw / g.div_w;
                        ok = th >= 0 && tw >= 0 && ih * g.div_h == th && iw * g.div_w == tw && ih < g.IH && iw < g.IW;
                        off = abase[i] + (ih * g.IW + iw) * g.IC + cc[e];
                    }
                    h16[e] = *(ok ? a.A + off : zero_src);
                }
                ra[i] = pack8(h16);
            }
            if (!B_TR) {
                int kk = kk0 + b_vec * 8;
#pragma unroll
                for (int i = 0; i < B_PASSES; ++i) {
                    int n = n0 + b_row0 + i * B_RPP;
                    unsigned short h16[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        bool ok = n < g.Ncols && (kk + e) < g.Kred;
                        h16[e] = *(ok ? a.Bw + (n * g.Kred + kk + e) : zero_src);
                    }
                    rb[i] = pack8(h16);
                }
            } else {
                int n = n0 + b_vec * 8;
#pragma unroll
                for (int i = 0; i < B_PASSES; ++i) {
                    int kk = kk0 + b_row0 + i * B_RPP;
                    int tap = kk / g.IC;
                    int k = kk - tap * g.IC;
                    int r = tap / g.S, s = tap - r * g.S;
                    if (PHASE) {
                        r = r0 + r * a.g.div_h;
                        s = s0 + s * a.g.div_w;
                    }
                    const int rowoff = ((k * a.g.R + (a.g.R - 1 - r)) * a.g.S + (a.g.S - 1 - s)) * g.Ncols;
                    unsigned short h16[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        bool ok = kk < g.Kred && (n + e) < g.Ncols;
                        h16[e] = *(ok ? a.Bw + (rowoff + n + e) : zero_src);
                    }
                    rb[i] = pack8(h16);
                }
            }
        }
    };

    auto store_lds = [&](int stage, const u32x4 (&ra)[A_PASSES], const u32x4 (&rb)[B_PASSES]) {
        unsigned char* sA = smem + stage * STAGE;
        unsigned char* sB = sA + A_BYTES;
#pragma unroll
        for (int i = 0; i < A_PASSES; ++i)
            *reinterpret_cast<u32x4*>(sA + (a_row0 + i * A_RPP) * A_PITCH + a_vec * 16) = ra[i];
#pragma unroll
        for (int i = 0; i < B_PASSES; ++i)
            *reinterpret_cast<u32x4*>(sB + (b_row0 + i * B_RPP) * B_PITCH + b_vec * 16) = rb[i];
    };

    f32x16 acc[FN][FM];
#pragma unroll
    for (int i = 0; i < FN; ++i)
#pragma unroll
        for (int j = 0; j < FM; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    auto compute = [&](int stage) {
        const unsigned char* sA = smem + stage * STAGE;
        const unsigned char* sB = sA + A_BYTES;
#pragma unroll
        for (int k2 = 0; k2 < BK / 16 / WAVES_K; ++k2) {
            const int ks = wk * (BK / 16 / WAVES_K) + k2;
            bf16x8 fa[FM], fw[FN];
#pragma unroll
            for (int j = 0; j < FM; ++j) {
                int row = wm * WM + j * 32 + (lane & 31);
                fa[j] = *reinterpret_cast<const bf16x8*>(sA + row * A_PITCH + (ks * 2 + (lane >> 5)) * 16);
            }
#pragma unroll
            for (int i = 0; i < FN; ++i) {
                if (!B_TR) {
                    int row = wn * WN + i * 32 + (lane & 31);
                    fw[i] = *reinterpret_cast<const bf16x8*>(sB + row * B_PITCH + (ks * 2 + (lane >> 5)) * 16);
                } else {
                    int col = wn * WN + i * 32 + ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
                    int krow = ks * 16 + (lane >> 5) * 8 + ((lane & 15) >> 2);
                    typedef s16x4 __attribute__((address_space(3))) * lds_s16x4_ptr;
                    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                        (lds_s16x4_ptr)(sB + krow * B_PITCH + col * 2));
                    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                        (lds_s16x4_ptr)(sB + (krow + 4) * B_PITCH + col * 2));
                    s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
                    fw[i] = __builtin_bit_cast(bf16x8, both);
                }
            }
#pragma unroll
            for (int i = 0; i < FN; ++i)
#pragma unroll
                for (int j = 0; j < FM; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[i], fa[j], acc[i][j], 0, 0, 0);
        }
    };

    // Tile it is in the LDS, tile it + 1 in one register set, and (where two sets fit) tile it + 2 in flight in the other: few
    // work-groups share a CU where this kernel is used, so one tile's loads do not cover the latency of the next.  The loads are
    // unconditional, or the compiler could not tell how many are in flight and would wait for all of them.
    if (nkt > 0) {
        u32x4 ra[SETS][A_PASSES], rb[SETS][B_PASSES];
#pragma unroll
        for (int i = 0; i < SETS; ++i) load_global(ra[i], rb[i]);
        // nothing is stored or loaded behind the last tile (the largest tiles have no registers for a second copy of the products)
        constexpr int LAST = BM * BN > 128 * 128 ? 0 : 1;
        store_lds(0, ra[0], rb[0]);
        int it = 0;
        if (nkt > 1 || LAST == 0) {
            load_global(ra[0], rb[0]);
            __syncthreads();
            auto step = [&](int stage, u32x4 (&xa)[A_PASSES], u32x4 (&xb)[B_PASSES]) {
                store_lds(stage ^ 1, xa, xb);
                load_global(xa, xb);
                compute(stage);
                __syncthreads();
            };
            constexpr int U = SETS < 2 ? 2 : SETS;
            for (; it + U + LAST <= nkt; it += U) {
#pragma unroll
                for (int u = 0; u < U; ++u) step(u & 1, ra[(u + 1) % SETS], rb[(u + 1) % SETS]);
            }
#pragma unroll
            for (int u = 0; u < U - 1; ++u)
                if (it + u + LAST < nkt) step(u & 1, ra[(u + 1) % SETS], rb[(u + 1) % SETS]);
        } else {
            __syncthreads();
        }
        if constexpr (LAST == 1) {
            compute((nkt - 1) & 1);
            __syncthreads();
        }
    }

    // ---- the halves of the reduction meet: each wavefront keeps every WAVES_K-th pixel block of its sub-tile ----
    if constexpr (WAVES_K == 2) {
        static_assert(FM % 2 == 0 && WAVES_M * WAVES_N * 2 * (FM / 2) * FN * 4096 <= 2 * STAGE, "does not fit the operand tiles");
        unsigned char* const mine = smem + wave * ((FM / 2) * FN * 4096) + lane * 16;
        unsigned char* const theirs = smem + (wave ^ (WAVES_M * WAVES_N)) * ((FM / 2) * FN * 4096) + lane * 16;
#pragma unroll
        for (int i = 0; i < FN; ++i)
#pragma unroll
            for (int j = 0; j < FM / 2; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<f32x4*>(mine + ((i * (FM / 2) + j) * 4 + q) * 1024) =
                        wk == 0 ? f32x4{acc[i][j + FM / 2][q * 4], acc[i][j + FM / 2][q * 4 + 1], acc[i][j + FM / 2][q * 4 + 2], acc[i][j + FM / 2][q * 4 + 3]}
                                : f32x4{acc[i][j][q * 4], acc[i][j][q * 4 + 1], acc[i][j][q * 4 + 2], acc[i][j][q * 4 + 3]};
        __syncthreads();
#pragma unroll
        for (int i = 0; i < FN; ++i)
#pragma unroll
            for (int j = 0; j < FM / 2; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 v = *reinterpret_cast<const f32x4*>(theirs + ((i * (FM / 2) + j) * 4 + q) * 1024);
#pragma unroll
                    for (int e = 0; e < 4; ++e)  // (the first half's sum first in both)
                        acc[i][j][q * 4 + e] = wk == 0 ? acc[i][j][q * 4 + e] + v[e] : v[e] + acc[i][j + FM / 2][q * 4 + e];
                }
    }

    // ---- epilogue.  A lane holds 4 consecutive channels of one pixel per register quad; a wavefront turns its blocks of 32
    // pixels around in LDS of its own, 16-byte groups exchanged within a row against bank conflicts, so that whole runs of
    // channels leave in 16-byte stores (8-byte stores to 32 rows each: 32 x 28 x 28, 512 <- 128 channels, 1x1, 21.0 us against 17.1;
    // partial sums in 32-byte runs: 4 x 14 x 14 x 512 -> 512, 1x1, 13.5 against 11.3). ----
    constexpr int JN = FM / WAVES_K, WNC = FN * 32;         // blocks of this wavefront, channels of a block
    constexpr int EP = 32 * WNC * 4;                        // bytes, as fp32
    static_assert((NT / 64) * EP <= 2 * STAGE || BM * BN > 128 * 128, "epilogue staging does not fit the operand tiles");
    if constexpr (WAVES_K == 2) __syncthreads();            // (the exchanged halves have been read)
    unsigned char* const ep = smem + wave * EP;
    const int l32 = lane & 31, half = lane >> 5;
    const int nw = n0 + wn * WNC;                           // first channel of the wavefront
#pragma unroll
    for (int j = 0; j < JN; ++j) {
        const int mw = m0 + wm * WM + (wk * JN + j) * 32;   // first pixel of the block
        auto row_of = [&](int p) {                          // output row of the block's pixel p
            int m = mw + p;
            if (PHASE) {  // back to the pixel of the whole map
                const int t = (int)fdiv((uint32_t)m, dOW), ow = m - t * g.OW;
                const int n = (int)fdiv((uint32_t)t, dOH), oh = t - n * g.OH;
                m = (n * a.g.OH + oh * a.g.div_h + oh0) * a.g.OW + ow * a.g.div_w + ow0;
            }
            return m;
        };
        if (a.partial) {
            constexpr int CH = WNC / 4;  // 16-byte groups per pixel
#pragma unroll
            for (int i = 0; i < FN; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int c = i * 8 + q * 2 + half;
                    *reinterpret_cast<f32x4*>(ep + l32 * (WNC * 4) + (c ^ (l32 & 15)) * 16) =
                        f32x4{acc[i][j][q * 4], acc[i][j][q * 4 + 1], acc[i][j][q * 4 + 2], acc[i][j][q * 4 + 3]};
                }
            __builtin_amdgcn_wave_barrier();  // LDS operations of one wavefront complete in order
#pragma unroll
            for (int it = 0; it < CH / 2; ++it) {
                const int v = it * 64 + lane, p = v / CH, c = v % CH, n = nw + c * 4;
                const f32x4 x = *reinterpret_cast<const f32x4*>(ep + p * (WNC * 4) + (c ^ (p & 15)) * 16);
                if (mw + p >= g.M || n >= g.Ncols) continue;
                float* o = reinterpret_cast<float*>(a.out) + ((size_t)split * a.g.M + row_of(p)) * g.Ncols + n;
                if (n + 4 <= g.Ncols) {
                    __builtin_memcpy(o, &x, 16);
                } else {
#pragma unroll
                    for (int e = 0; e < 3; ++e)
                        if (n + e < g.Ncols) o[e] = x[e];
                }
            }
        } else {
            constexpr int CH = WNC / 8;
            u32x4 mk[CH / 2];  // mask of the rows to be stored, fetched ahead
            if (a.mask) {
#pragma unroll
                for (int it = 0; it < CH / 2; ++it) {
                    const int v = it * 64 + lane, p = v / CH, n = nw + v % CH * 8;
                    mk[it] = u32x4{0u, 0u, 0u, 0u};
                    if (mw + p >= g.M || n >= g.Ncols) continue;
                    const bf16_t* src = a.mask + (size_t)row_of(p) * g.Ncols + n;
                    if (n + 8 <= g.Ncols) {
                        mk[it] = load8_unaligned(src);
                    } else {
#pragma unroll
                        for (int e = 0; e < 7; ++e)
                            if (n + e < g.Ncols) mk[it][e >> 1] |= (unsigned)src[e] << (16 * (e & 1));
                    }
                }
            }
#pragma unroll
            for (int i = 0; i < FN; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    float v[4];
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = acc[i][j][q * 4 + e];
                    const int n = nw + i * 32 + q * 8 + half * 4;
                    if (a.bias) {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (n + e < g.Ncols) v[e] += a.bias[n + e];
                    }
                    if (a.relu) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
                    }
                    const int c = i * 4 + q;
                    *reinterpret_cast<u32x2*>(ep + l32 * (WNC * 2) + (c ^ (l32 & 7)) * 16 + half * 8) =
                        u32x2{(unsigned)f2bf(v[0]) | ((unsigned)f2bf(v[1]) << 16), (unsigned)f2bf(v[2]) | ((unsigned)f2bf(v[3]) << 16)};
                }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int it = 0; it < CH / 2; ++it) {
                const int v = it * 64 + lane, p = v / CH, c = v % CH, n = nw + c * 8;
                u32x4 x = *reinterpret_cast<const u32x4*>(ep + p * (WNC * 2) + (c ^ (p & 7)) * 16);
                if (a.mask) {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        x[k] &= (__uint_as_float(mk[it][k] << 16) > 0.f ? 0xffffu : 0u) |
                                (__uint_as_float(mk[it][k] & 0xffff0000u) > 0.f ? 0xffff0000u : 0u);
                }
                if (mw + p >= g.M || n >= g.Ncols) continue;
                bf16_t* o = reinterpret_cast<bf16_t*>(a.out) + (size_t)row_of(p) * g.Ncols + n;
                if (n + 8 <= g.Ncols) {
                    __builtin_memcpy(o, &x, 16);
                } else {
#pragma unroll
                    for (int e = 0; e < 7; ++e)
                        if (n + e < g.Ncols) o[e] = (bf16_t)(x[e >> 1] >> (16 * (e & 1)));
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
}

// ---- tile configurations ----
struct Cfg {
    int BM, BN, NT;
};
constexpr Cfg kCfgs[] = {
    {256, 256, 512},  // 0: large
    {128, 128, 256},  // 1: medium / general
    {64, 256, 256},   // 2: few rows (small-batch FC)
    {256, 64, 256},   // 3: few output channels
    {256, 256, 256},  // 4: large, 4 wavefronts of 128x128 (less LDS traffic per MFMA)
    {256, 256, 256},  // 5: large, weights in registers (conv_wreg.hip)
    {224, 256, 256},  // 6: stride-1 multi-tap conv, input patch in LDS (conv_patch.hip)
    {256, 64, 256},   // 7: stride-1 multi-tap conv, 8 x 32-pixel tiles, 64 / 128 channels (conv_tile2d.hip)
};

size_t smem_bytes(const Cfg& c, bool b_tr) {
    size_t a = (size_t)c.BM * A_PITCH;
    size_t b = b_tr ? (size_t)BK * (c.BN * 2 + 64) : (size_t)c.BN * A_PITCH;
    return 2 * (a + b);
}

bool dense_grid(long groups) { return groups > kNumCU; }

template <typename F, typename A>
int launch_any(F kfn, std::atomic<bool>& attr_done, const A& ka, int threads, size_t smem, hipStream_t st) {
    if (!attr_done) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
        if (e != hipSuccess) return set_error(WAP_EHIP, "hipFuncSetAttribute: %s", hipGetErrorString(e));
        attr_done = true;
    }
    int total = ka.tiles_m * ka.tiles_n * ka.nsplit;
    hipLaunchKernelGGL(kfn, dim3(total), dim3(threads), smem, st, ka);
    return check_launch("igemm");
}
template <int BM, int BN, int WMv, int WNv, bool B_TR, int MODE>
int launch_one(const KArgs& ka, size_t smem, hipStream_t st) {
    static std::atomic<bool> attr_done{false}, attr_done2{false};  // one attribute call per instantiation
    constexpr int dense = BM * BN <= 128 * 128 && MODE < 3 ? 8 + MODE : MODE;
    if (dense != MODE && dense_grid((long)ka.tiles_m * ka.tiles_n * ka.nsplit))
        return launch_any(igemm_kernel<BM, BN, WMv, WNv, B_TR, dense>, attr_done2, ka, 64 * WMv * WNv * waves_k(BM, BN, dense), smem, st);
    return launch_any(igemm_kernel<BM, BN, WMv, WNv, B_TR, MODE>, attr_done, ka, 64 * WMv * WNv * waves_k(BM, BN, MODE), smem, st);
}
template <int BM, int BN, int WMv, int WNv, int MODE>
int launch_phase(const KPhaseArgs& ka, size_t smem, hipStream_t st) {
    static std::atomic<bool> attr_done{false}, attr_done2{false};
    constexpr int dense = MODE < 3 ? 12 + MODE : 4 + MODE;
    if (MODE < 3 && dense_grid((long)ka.tiles_m * ka.tiles_n * ka.nsplit))
        return launch_any(igemm_kernel<BM, BN, WMv, WNv, true, dense>, attr_done2, ka, 64 * WMv * WNv * waves_k(BM, BN, dense), smem, st);
    return launch_any(igemm_kernel<BM, BN, WMv, WNv, true, 4 + MODE>, attr_done, ka, 64 * WMv * WNv * waves_k(BM, BN, MODE), smem, st);
}

// (A 1x1 filter has one tap to skip and pays for writing every pixel's row apart from its neighbours': 64 <- 128 channels on
// 56 x 56 14.0 against 11.4 us.  3x3: 64 <- 64 on 112 x 112 27 against 52 us, 16 <- 64 on 64 x 64 11.7 against 27.)
bool phased(const GemmGeom& g, bool b_tr) {
    const long phases = (long)g.div_h * g.div_w;  // strides may be as large as an int holds
    return b_tr && g.R * g.S > 1 && phases > 1 && phases <= kMaxPhases;
}

int classify_mode(const GemmGeom& g, bool b_tr) {
    const size_t most = 2147483647u - 63;  // elements of an operand whose last 16 bytes lie below kNowhere
    if ((size_t)(g.M / (g.OH * g.OW)) * g.IH * g.IW * g.IC > most || (size_t)g.Kred * g.Ncols > most) return 3;
    bool vec_a = (g.IC % 8) == 0;
    bool vec_b = b_tr ? (g.Ncols % 8) == 0 : (g.Kred % 8) == 0;
    if (!(vec_a && vec_b)) {
        const long padded = (long)g.R * g.S * ((g.IC + 7L) / 8 * 8);  // the reduction of mode 2, counted in int
        return g.IC >= 8 && (!b_tr || g.Ncols >= 8) && padded <= 2147483647L - BK ? 2 : 3;
    }
    if ((g.IC % BK) == 0 && ((g.div_h == 1 && g.div_w == 1) || phased(g, b_tr))) return 0;
    return 1;
}

// A single forward call whose small tiles take the weights where they lie, without a packing launch (3 us, 10 of host time) in front.  An
// operand load is then 32 pieces of 32 bytes instead of one run of 1 KB, so the line lies where the tiles read the weights
// often enough to lose what the launch cost.  us, packed / as they are, by the weights' bytes times the tiles that read them: 7 MB (2 x 13 x 13,
// 256 -> 256) 10.9 / 9.2, 14 MB (8 x 56 x 56, 64 -> 64) 21.1 / 18.9, 19 MB (4 x 13 x 13, 384 -> 256) 13.2 / 12.3, 22 MB (32 x 20 x 20, 96 -> 64)
// 14.3 / 12.1, 28 MB (8 x 13 x 13, 192 -> 384) 10.6 / 11.4, 58 MB (56 x 56, 256 -> 256) 12.9 / 13.9, 115 MB (16 x 14 x 14, 512 -> 512) 25.5 / 40.2;
// 5x5 27 x 27, 64 -> 192 12.2 / 12.9.
bool reads_unpacked(const GemmGeom& g, bool b_tr, const GemmPlan& plan) {
    if (b_tr || !(plan.cfg == 16 || (plan.cfg == 7 && plan.nsplit > 1)) || g.R != 3 || g.S != 3) return false;
    const int pixels = plan.cfg == 16 ? 32 * (plan.tile / 10) : 64 * plan.tile;
    return (double)((g.M + pixels - 1) / pixels) * g.Ncols * g.Kred * 2.0 <= 24e6;
}

// The phases of a strided data gradient, those with the most taps first (the longest work-groups start first); returns the
// row tiles of bm pixels in all.
int make_phases(const GemmGeom& g, int bm, Phase* ph, int* nphase) {
    int n = 0;
    const int images = g.M / (g.OH * g.OW);
    for (int a = 0; a < g.div_h; ++a)
        for (int b = 0; b < g.div_w; ++b) {
            Phase p;
            p.oh0 = a; p.ow0 = b;
            p.OH = (g.OH - a + g.div_h - 1) / g.div_h;
            p.OW = (g.OW - b + g.div_w - 1) / g.div_w;
            if (a >= g.OH || b >= g.OW) continue;
            p.r0 = ((g.pad_h - a) % g.div_h + g.div_h) % g.div_h;
            p.s0 = ((g.pad_w - b) % g.div_w + g.div_w) % g.div_w;
            p.R = p.r0 < g.R ? (g.R - 1 - p.r0) / g.div_h + 1 : 0;
            p.S = p.s0 < g.S ? (g.S - 1 - p.s0) / g.div_w + 1 : 0;
            p.pad_h = (g.pad_h - a - p.r0) / g.div_h;  // exact
            p.pad_w = (g.pad_w - b - p.s0) / g.div_w;
            p.M = images * p.OH * p.OW;
            p.dOW = make_fastdiv((uint32_t)p.OW);
            p.dOH = make_fastdiv((uint32_t)p.OH);
            ph[n++] = p;
        }
    std::stable_sort(ph, ph + n, [](const Phase& x, const Phase& y) { return x.R * x.S > y.R * y.S; });
    int tiles = 0;
    for (int i = 0; i < n; ++i) {
        ph[i].tile0 = tiles;
        tiles += (ph[i].M + bm - 1) / bm;
    }
    *nphase = n;
    return tiles;
}

// us that the kernels of a plan take beside which the flat tiles stand: a start, the steps of a work-group's reduction (9 taps of 32
// channels, or 64 deep in the generic kernel), what a fuller chip and further rounds of work-groups add to each, and the partial sums through
// memory.  Fitted to 33 000 products with packed weights (3x3 and 5x5, 16 to 1024 channels, maps of 4 to 120 pixels, 1 to 128 images; rms error
// 4 to 8 %); 0: a tiling that the flat tiles beat wherever they were tried.
double us_beside_flat(const GemmGeom& g, int cfg, int nsplit, int tile, int ktiles, long tiles) {
    struct Line { double start, step, fill, round, mb; };
    static constexpr Line whole192 = {6.3, 0.83, 1.05, 0.69, 0}, split192 = {7.7, 0.84, 0.77, 0, 0.61};
    static constexpr Line whole64 = {5.35, 0.74, 0.61, 0.46, 0}, split64 = {6.9, 0.65, 0.70, 0.36, 0.54}, loop64 = {10.5, 0.12, 0.92, 0.92, 0.28};
    static constexpr Line whole_generic = {7.7, 0.38, 0.25, 0.46, 0}, split_generic = {9.7, 0.28, 0.31, 0, 0.49};
    const Line* l;
    double steps;
    if (cfg < 5) {
        l = nsplit > 1 ? &split_generic : &whole_generic;
        steps = (ktiles + nsplit - 1) / nsplit;
    } else {
        int pixels = 0, channels = 0;
        if (cfg == 7) tile2d_shape(g, tile, &pixels, &channels);
        if (channels == 64) l = nsplit > 1 ? &split192 : &whole192;
        else if (pixels == 64 && g.R == 3) l = nsplit > 1 ? &split64 : &whole64;
        else if (pixels == 64 && nsplit > 1) l = &loop64;
        else return 0;
        steps = (g.IC / 32 + nsplit - 1) / nsplit * (g.R * g.S / 9.0);
        tiles = (long)((g.M + pixels - 1) / pixels) * (g.Ncols / channels);
    }
    const long groups = tiles * nsplit, rounds = (groups + kNumCU - 1) / kNumCU;
    const double mb = nsplit > 1 ? nsplit * 4e-6 * g.M * g.Ncols : 0;
    return l->start + steps * (l->step + l->fill * groups / kNumCU + l->round * (rounds - 1)) + l->mb * mb;
}

}  // namespace

GemmPlan plan_fc_stream(const GemmGeom& g, bool lean) {
    GemmPlan p;
    p.cfg = 10;
    p.nsplit = 1;
    fc_fwd_plan(g, lean, &p.tile, &p.nsplit);
    if (g_force_nsplit >= 1) p.nsplit = g_force_nsplit;
    const int steps = (g.IC + 31) / 32;
    if (p.nsplit > steps) p.nsplit = steps;
    p.nsplit = (steps + (steps + p.nsplit - 1) / p.nsplit - 1) / ((steps + p.nsplit - 1) / p.nsplit);  // none empty
    p.ws_bytes = p.nsplit > 1 ? (size_t)p.nsplit * g.M * g.Ncols * sizeof(float) : 0;
    return p;
}

GemmPlan plan_fwd_like(const GemmGeom& g, bool b_tr, bool prepacked, bool lean, bool fc_stream) {
    GemmPlan p;
    if (!b_tr && (g_force_fwd_cfg < 0 || g_force_fwd_cfg == 8) && conv_c3_fwd_supported(g)) {
        p.cfg = 8;
        p.nsplit = 1;
        p.ws_bytes = 0;
        return p;
    }
    if (!b_tr && (g_force_fwd_cfg < 0 || g_force_fwd_cfg == 15) && conv_thin_fwd_supported(g)) {
        p.cfg = 15;
        p.nsplit = 1;
        p.ws_bytes = 0;
        return p;
    }
    if (b_tr && (g_force_fwd_cfg < 0 || g_force_fwd_cfg == 9) && dgrad_thin_supported(g)) {
        p.cfg = 9;  // at most four output columns (gradient w.r.t. a 3-channel image)
        p.nsplit = 1;
        p.ws_bytes = 0;
        return p;
    }
    if (g_force_fwd_cfg < 0 && b_tr && fc_dx_supported(g)) {
        p.cfg = 11;
        p.nsplit = 1;
        p.ws_bytes = 0;
        return p;
    }
    if (g_force_fwd_cfg < 0 && !b_tr && fc_stream && fc_fwd_supported(g, prepacked, lean)) {
        if (fc_fwd_odd_rows_slow(g, lean)) {  // (calls that bring no workspace stream where the generic kernel needs one)
            p = plan_fwd_like(g, b_tr, prepacked, lean, false);
            if (!lean || p.ws_bytes == 0) return p;
        }
        return plan_fc_stream(g, lean);
    }
    int mode = classify_mode(g, b_tr);
    int ktiles = ((mode == 2 ? g.R * g.S * ((g.IC + 7) / 8 * 8) : g.Kred) + BK - 1) / BK;
    const bool ph = phased(g, b_tr);
    if (ph) ktiles = (ktiles + g.div_h * g.div_w - 1) / (g.div_h * g.div_w);  // of the average phase
    auto tiles = [&](int c) {
        return (long)((g.M + kCfgs[c].BM - 1) / kCfgs[c].BM) * ((g.Ncols + kCfgs[c].BN - 1) / kCfgs[c].BN);
    };
    int cfg;
    if (mode != 0 || (ph && g.Ncols > 64)) {
        cfg = 1;
    } else if (g.Ncols <= 64) {
        cfg = 3;
    } else if (g.M <= 64) {
        cfg = 2;
    } else if (tiles(0) >= 200 && g.Ncols >= 192) {
        cfg = wreg_supported(g) ? 5 : 0;
    } else {
        cfg = 1;
    }
    if (g_force_fwd_cfg >= 0 && g_force_fwd_cfg < 8 && (mode == 0 || g_force_fwd_cfg == 1) &&
        (!ph || g_force_fwd_cfg == 1 || g_force_fwd_cfg == 3))
        cfg = g_force_fwd_cfg;
    long t = tiles(cfg);
    int nsplit = 1;
    // split the reduction when the tiles alone leave most CUs idle
    if (t < kNumCU * 3 / 4 && ktiles >= 8) {
        // about one work-group per CU in all (measured on the FC head: more splits only add partial-tile traffic and a
        // longer epilogue), at least 4 reduction tiles per split
        long want = kNumCU / t;
        long maxs = ktiles / 4;
        nsplit = (int)(want < maxs ? want : maxs);
        if (nsplit < 1) nsplit = 1;
        if (nsplit > 64) nsplit = 64;
    }
    if (g_force_nsplit >= 1) nsplit = g_force_nsplit < ktiles ? g_force_nsplit : ktiles;
    int kps = (ktiles + nsplit - 1) / nsplit;
    nsplit = (ktiles + kps - 1) / kps;
    if (cfg == 5 && !wreg_supported(g)) cfg = 0;
    if (g_force_fwd_cfg < 0 && patch_supported(g)) cfg = 6;
    if (cfg == 6 && !patch_supported(g)) cfg = 1;
    if (g_force_fwd_cfg < 0 && tile2d_preferred(g)) cfg = 7;
    if (cfg == 7 && !tile2d_supported(g)) cfg = 1;
    if (cfg == 6 || cfg == 7) nsplit = 1;
    // Reductions split over channel slices of the patch kernel.  A forward layer that pools in its epilogue stays whole,
    // and one whose partial sums would take it past the static scratch keeps the plan it had.
    if (g_force_fwd_cfg < 0 && g_force_nsplit < 0 && (cfg < 6 || cfg == 7)) {
        int tile = 0;
        const bool pools = !b_tr && cfg == 7 && (g.OH % 2) == 0 && (g.OW % 2) == 0 && tile2d_fuses_pool(g);
        // (A single call packs its weights in front, a launch more.  As a graph the split is 3 to 20 % ahead from 0.04 GFLOP on all
        // the same; called one by one, a layer of little work waits for the host, 4 us for every launch of a Python caller.  3x3
        // layers of 128 .. 512 channels, forward and both gradients, us without / with the split in both passes: 0.2 GFLOP 41 / 49,
        // 0.46 45 / 50, 0.6 49.5 / 49.4, 0.8 52 / 50, 1.6 59 / 53.  A forward pass runs ahead of the GPU earlier: AlexNet-style layers of
        // 0.2 .. 0.45 GFLOP, one image 115 / 113, two 116 / 113.)
        const bool worth = cfg == 7 || prepacked || 2.0 * g.M * g.Ncols * g.Kred >= (b_tr ? 6e8 : 1.9e8);
        const int sp = pools || !worth ? 1 : tile2d_split(g, cfg < 6, &tile);
        if (sp > 1 && (b_tr || (size_t)sp * g.M * g.Ncols * sizeof(float) + wreg_wt_bytes(g) <= WAP_STATIC_SCRATCH_BYTES)) {
            cfg = 7;
            p.tile = tile;
            nsplit = sp;
        }
    } else if ((g_force_fwd_cfg == 12 || g_force_fwd_cfg == 14) && g_force_nsplit >= 2 && g_force_nsplit <= g.IC / 32 &&
               tile2d_supported(g, g_force_fwd_cfg - 11)) {
        cfg = 7;
        p.tile = g_force_fwd_cfg - 11;
        const int slices = g.IC / 32, per = (slices + g_force_nsplit - 1) / g_force_nsplit;
        nsplit = (slices + per - 1) / per;
    }
    p.ws_bytes = nsplit > 1 ? (size_t)nsplit * g.M * g.Ncols * sizeof(float) : 0;
    if (cfg >= 5) p.ws_bytes += wreg_wt_bytes(g);  // weights repacked into MFMA fragment order
    // Small layers: tiles whose reduction is divided over the wavefronts of a work-group, so that no partial sums and no second launch are
    // needed.  us, kernels alone, the plan so far / the flat tiles, where the predictions for both say so (us_beside_flat; by the sizes alone
    // 2 900 of 33 000 products were 1.05 to 5 times slower: few pixels under a reduction of 512 channels and more, 2 x 6 x 58, 1024 -> 64
    // 14.5 / 36, 5x5 2 x 8 x 8, 928 -> 64 12.4 / 54, and two rounds of flat tiles for one of larger ones, 19 x 45 x 45, 64 -> 64 9.2 / 12.9):
    //   a split reduction of the patch kernel: 8 x 13 x 13, 256 -> 256 14.4 / 8.2, 8 x 14 x 14, 512 -> 512 20.8 / 15.0, 2 x 28 x 28,
    //     128 -> 128 15.8 / 6.2, 5x5 3 x 27 x 27, 192 -> 64 16.2 / 12.9;
    //   unsplit tiles of the patch kernel up to ten 32 x 32 blocks of outputs per CU (32 x 13 x 13, 384 -> 256 20.7 / 14.3, 22 x 14 x 14,
    //     512 -> 512 31.9 / 23.8), sixteen with 256 input channels (8 x 28 x 28, 512 -> 512 36 / 30; with 128 62 x 62 15 / 20), eight
    //     for 5x5 (32 x 27 x 27, 64 -> 192 20 / 26): beyond, the larger tiles read fewer weights per output;
    //   the generic kernel: where the predicted time, with a packing launch where there is one to pay for, is below that
    //     kernel's line of 9 us (14 with a split reduction) and 550 TFLOP/s (13 x 67 x 67, 384 -> 32 41 / 52, 28 x 10 x 10 20 / 8).
    // A forward layer that pools in its epilogue keeps the tiles that can.  Single data gradients of the whole-filter patch kernel with a
    // last block of channels that is not full keep theirs, though the flat tiles would often be faster there as well (90 x 90, 64 -> 200
    // 10 instead of 16 us): the tests of that kernel's weight order run these calls.  Single calls that split their reduction change over
    // from 700 pixels on, where 93 drawn layers took 0.47 to 0.9 of the time, 0.68 in the mean (us as a graph, split / flat: 28 x 28,
    // 512 -> 512 18.1 / 13.9, 256 -> 512 16.0 / 9.7, 4 x 44 x 44, 64 -> 32 15.2 / 9.4; gradient 4 x 30 x 30, 224 -> 160 18.7 / 13.0).  With
    // fewer, forward layers that read the weights as they are go from 0.5 to 1.5 times (5 x 9 x 9, 224 -> 192 9.1 / 13.7: four waits for
    // weights one after another, and too few work-groups to hide them), and layers of 169 and 196 pixels were level.  Beyond
    // 512 channels, where neither prediction was fitted, 13 of 110 layers were slower (gradient 64 x 14, 800 -> 928 31.1 / 34.8).  5x5 splits of
    // the patch kernel change over only with a reduction of 64 channels, where every wavefront has one turn, and a 32 x 32 block of outputs
    // a CU at most (27 x 27, 64 -> 192 11.7 / 9.5, 55 x 55, 64 -> 64 11.9 / 9.3); with 96 channels they were 3 to 12 % ahead, with more up to
    // half.  5x5 splits of the generic kernel whose reduction has more than 256 channels change over from four pixels for each of them on (gradient
    // 9 x 10 x 10, 384 -> 400 23.9 / 28.3, 30 x 6 x 6, 448 -> 432 27.9 / 32.7; 124 timings below that line 1.06 in the mean, 148 above it 0.90, none
    // of them above 1.06).  Where a single call needed no workspace, tiles that read a packed copy of the weights take over only if the caller
    // has one for it (not lean); where it needed some, only if that is enough (the two queries of a layer stay what they were).
    const bool split = !prepacked && nsplit > 1;
    const bool kept = !prepacked && ((nsplit > 1 && (g.M < 700 || std::max(g.IC, g.Ncols) > 512 || (cfg == 7 && g.R == 5 && (g.IC > 64 || (double)g.M * g.Ncols > 1024.0 * kNumCU)) ||
                                                       (cfg < 5 && g.R == 5 && g.IC > 256 && g.M < 4 * g.IC))) || (cfg == 6 && b_tr && g.Ncols % 32 != 0));
    if (g_force_fwd_cfg < 0 && g_force_nsplit < 0 && (cfg < 5 || cfg == 6 || cfg == 7) && !kept) {
        const double flops = 2.0 * g.M * g.Ncols * g.Kred, blocks = (double)g.M * g.Ncols / 1024.0 / kNumCU;
        size_t need = std::max(p.ws_bytes, wreg_wt_bytes(g));
        double us = 0;
        int tile = blocks <= 64.0 && (b_tr || need == p.ws_bytes || need <= WAP_STATIC_SCRATCH_BYTES) ? flat_pick(g, &us) : 0;
        GemmPlan flat;
        flat.cfg = 16;
        flat.nsplit = 1;
        flat.tile = tile;
        const bool raw = tile && !prepacked && reads_unpacked(g, b_tr, flat);
        if (!prepacked && p.ws_bytes == 0) {
            if (raw) need = 0;
            else if (lean) tile = 0;
        } else if (split && need > p.ws_bytes) {
            tile = 0;
        }
        bool wins;
        if (cfg == 7 && nsplit > 1) wins = true;
        else if (cfg < 5) wins = us + (prepacked ? 0.0 : 4.0) < (nsplit > 1 ? 14.0 : 9.0) + flops / 550e6;
        else wins = blocks <= (g.R == 5 ? 8.0 : g.IC >= 256 ? 16.0 : 10.0) && !(cfg == 7 && !b_tr && (g.OH % 2) == 0 && (g.OW % 2) == 0 && tile2d_fuses_pool(g));
        if (tile && wins) {
            // The flat tiles' own prediction falls short where the two are close, most for single fragments of a 5x5 filter; a packing launch takes 3.
            const double other = us_beside_flat(g, cfg, nsplit, p.tile, ktiles, t);
            const double short_of = g.R == 5 ? (tile == 14 && !(split && g.IC <= 64) ? 1.4 : 1.1) : cfg < 5 ? (nsplit > 1 ? 1.0 : 1.15) : nsplit > 1 ? 1.05 : 1.1;
            // Weights read as they are cost a wait of about 3 for every turn of a wavefront after its first; single calls leave a split for a tenth.
            const int turns = split && raw ? (g.IC / 32 - 1) / (tile % 10) : 0;
            wins = other == 0 || us * short_of + 3 * turns + (prepacked || raw ? 0 : 3) < (split ? 0.9 : 1.0) * (other + (prepacked || cfg < 5 ? 0 : 3));
        }
        if (tile && wins) {
            cfg = 16;
            p.tile = tile;
            nsplit = 1;
            p.ws_bytes = need;
        }
    }
    // (a launch that pools in its epilogue keeps the tiles that hold whole row pairs)
    if (g_force_fwd_cfg < 0 && g_force_nsplit < 0 && cfg == 7 && nsplit == 1) p.tile = tile2d_fill(g);
    if (g_force_fwd_cfg >= 200 && tile2d_supported(g, kTileFill + g_force_fwd_cfg - 200)) {
        cfg = 7;
        p.tile = kTileFill + g_force_fwd_cfg - 200;
        nsplit = 1;
        p.ws_bytes = wreg_wt_bytes(g);
    } else if (g_force_fwd_cfg >= 100 && g_force_fwd_cfg < 200 && flat_supported(g, g_force_fwd_cfg - 100)) {
        cfg = 16;
        p.tile = g_force_fwd_cfg - 100;
        nsplit = 1;
        p.ws_bytes = wreg_wt_bytes(g);
    }
    p.cfg = cfg;
    p.nsplit = nsplit;
    return p;
}

int launch_fwd_like(const GemmGeom& g, bool b_tr, const GemmPlan& plan, const bf16_t* A,
                    const bf16_t* Bw, const float* bias, bool relu, bf16_t* out, void* ws,
                    hipStream_t st, hipEvent_t ev_mid, const bf16_t* relu_mask, hipEvent_t ev_packed,
                    const void* prepacked, bf16_t* pool_y, uint8_t* pool_am, const uint8_t* unpool_am, float* colsum) {
    if (colsum && (fwd_like_colsum_rows(g, plan) == 0 || pool_y))
        return set_error(WAP_EINVAL, "internal: fused column sums not available for this plan");
    if ((pool_y || pool_am) && !(pool_y && pool_am && fwd_like_fuses_pool(g, plan)))
        return set_error(WAP_EINVAL, "internal: fused pooling not available for this plan");
    if (unpool_am && !fwd_like_fuses_unpool(g, plan))
        return set_error(WAP_EINVAL, "internal: fused max-pool backward not available for this plan");
    if (relu_mask && !fwd_like_fuses_mask(g, plan)) {
        // no fused epilogue for this tile configuration: plain product, then the element-wise mask
        int rc = launch_fwd_like(g, b_tr, plan, A, Bw, bias, relu, out, ws, st, ev_mid, nullptr, ev_packed, prepacked);
        if (rc != WAP_OK) return rc;
        return launch_relu_bwd(out, relu_mask, out, (size_t)g.M * g.Ncols, st);
    }
    if (plan.cfg == 8) return launch_conv_c3_fwd(g, A, Bw, bias, relu, out, st);
    if (plan.cfg == 15) return launch_conv_thin_fwd(g, A, Bw, bias, relu, out, st);
    if (plan.cfg == 9) return launch_dgrad_thin(g, A, Bw, out, st);
    if (plan.cfg == 10) {
        int rc10 = launch_fc_fwd(g, plan.nsplit, plan.tile, A, Bw, bias, relu, plan.nsplit > 1 ? ws : (void*)out, st);
        if (rc10 != WAP_OK || plan.nsplit == 1) return rc10;
        if (ev_mid) (void)hipEventRecord(ev_mid, st);
        return launch_reduce_bf16(reinterpret_cast<const float*>(ws), plan.nsplit, (size_t)g.M * g.Ncols, g.Ncols, bias,
                                  relu, out, st);
    }
    if (plan.cfg == 11) return launch_fc_dx(g, A, Bw, relu_mask, out, colsum, st);
    KArgs ka;
    ka.A = A;
    ka.Bw = Bw;
    ka.g = g;
    const Cfg& c = kCfgs[plan.cfg < 5 ? plan.cfg : 0];
    ka.tiles_m = (g.M + c.BM - 1) / c.BM;
    ka.tiles_n = (g.Ncols + c.BN - 1) / c.BN;
    const bool odd = plan.cfg == 1 && classify_mode(g, b_tr) == 2;
    ka.ICp = (g.IC + 7) / 8 * 8;
    ka.a_bytes = (unsigned)((size_t)(g.M / (g.OH * g.OW)) * g.IH * g.IW * g.IC * 2);
    ka.b_bytes = (unsigned)((size_t)g.Kred * g.Ncols * 2);
    ka.dICp = make_fastdiv((uint32_t)ka.ICp);
    ka.dOW = make_fastdiv((uint32_t)g.OW);
    ka.dOH = make_fastdiv((uint32_t)g.OH);
    ka.ktiles = ((odd ? g.R * g.S * ka.ICp : g.Kred) + BK - 1) / BK;
    ka.nsplit = plan.nsplit;
    ka.ktiles_per_split = (ka.ktiles + plan.nsplit - 1) / plan.nsplit;
    ka.partial = plan.nsplit > 1;
    ka.bias = ka.partial ? nullptr : bias;
    ka.mask = ka.partial ? nullptr : relu_mask;
    ka.relu = ka.partial ? 0 : (relu ? 1 : 0);
    ka.out = ka.partial ? ws : (void*)out;
    if (plan.cfg == 6 || plan.cfg == 7 || plan.cfg == 16) {
        const void* wp = prepacked;
        const bool raw = !prepacked && reads_unpacked(g, b_tr, plan);
        if (raw) wp = Bw;
        if (!wp) {
            int rc0 = launch_pack_weights(g, b_tr, Bw, ws, st);
            if (rc0 != WAP_OK) return rc0;
            wp = ws;
        }
        if (ev_packed) (void)hipEventRecord(ev_packed, st);
        if (plan.cfg == 16) return launch_flat(g, plan.tile, A, wp, bias, relu, out, st, relu_mask, unpool_am, colsum, raw);
        if (plan.cfg == 7 && plan.nsplit > 1) {
            float* part = reinterpret_cast<float*>(reinterpret_cast<unsigned char*>(ws) + wreg_wt_bytes(g));
            int rc7 = launch_tile2d(g, A, wp, nullptr, false, nullptr, st, nullptr, nullptr, nullptr, unpool_am, nullptr, plan.tile,
                                    plan.nsplit, part, raw);
            if (rc7 != WAP_OK) return rc7;
            if (ev_mid) (void)hipEventRecord(ev_mid, st);
            return launch_reduce_bf16(part, plan.nsplit, (size_t)g.M * g.Ncols, g.Ncols, bias, relu, out, st, relu_mask, colsum);
        }
        return plan.cfg == 6 ? launch_patch(g, A, wp, bias, relu, out, st, relu_mask)
                             : launch_tile2d(g, A, wp, bias, relu, out, st, relu_mask, pool_y, pool_am, unpool_am, colsum,
                                             pool_y && plan.tile != kTileStrips ? 0 : plan.tile);
    }
    if (plan.cfg == 5) {
        // the (small) weight tensor is first repacked into MFMA fragment order (taps flipped and
        // transposed for the data gradient); the partial tiles, if any, follow it in the workspace
        int rc0 = launch_pack_weights(g, b_tr, Bw, ws, st);
        if (rc0 != WAP_OK) return rc0;
        if (ev_packed) (void)hipEventRecord(ev_packed, st);
        void* part = reinterpret_cast<unsigned char*>(ws) + wreg_wt_bytes(g);
        int rc5 = launch_wreg(g, plan.nsplit, A, reinterpret_cast<const bf16_t*>(ws), bias, relu,
                              ka.partial ? part : (void*)out, ka.partial != 0, st);
        if (rc5 != WAP_OK) return rc5;
        if (ev_mid) (void)hipEventRecord(ev_mid, st);
        if (ka.partial)
            return launch_reduce_bf16(reinterpret_cast<const float*>(part), plan.nsplit, (size_t)g.M * g.Ncols,
                                      g.Ncols, bias, relu, out, st, relu_mask, colsum);
        return WAP_OK;
    }
    size_t smem = smem_bytes(c, b_tr);
    int mode = classify_mode(g, b_tr);
    int rc;
    if (phased(g, b_tr)) {
        KPhaseArgs kp;
        static_cast<KArgs&>(kp) = ka;
        kp.tiles_m = make_phases(g, c.BM, kp.ph, &kp.nphase);
        if (plan.cfg == 3 && mode == 0) rc = launch_phase<256, 64, 4, 1, 0>(kp, smem, st);
        else if (plan.cfg != 1) return set_error(WAP_EINVAL, "internal: strided data gradient on an unsuitable tile");
        else if (mode == 0) rc = launch_phase<128, 128, 2, 2, 0>(kp, smem, st);
        else if (mode == 1) rc = launch_phase<128, 128, 2, 2, 1>(kp, smem, st);
        else if (mode == 2) rc = launch_phase<128, 128, 2, 2, 2>(kp, smem, st);
        else rc = launch_phase<128, 128, 2, 2, 3>(kp, smem, st);
        if (rc != WAP_OK) return rc;
        if (ev_mid) (void)hipEventRecord(ev_mid, st);
        if (ka.partial)
            return launch_reduce_bf16(reinterpret_cast<const float*>(ws), plan.nsplit, (size_t)g.M * g.Ncols, g.Ncols, bias, relu,
                                      out, st, relu_mask, colsum);
        return WAP_OK;
    }
#define WAP_DISPATCH(BM, BN, WMv, WNv)                                                     \
    (b_tr ? (mode == 0 ? launch_one<BM, BN, WMv, WNv, true, 0>(ka, smem, st)                \
                       : mode == 1 ? launch_one<BM, BN, WMv, WNv, true, 1>(ka, smem, st)    \
                       : mode == 2 ? launch_one<BM, BN, WMv, WNv, true, 2>(ka, smem, st)    \
                                   : launch_one<BM, BN, WMv, WNv, true, 3>(ka, smem, st))   \
          : (mode == 0 ? launch_one<BM, BN, WMv, WNv, false, 0>(ka, smem, st)               \
                       : mode == 1 ? launch_one<BM, BN, WMv, WNv, false, 1>(ka, smem, st)   \
                       : mode == 2 ? launch_one<BM, BN, WMv, WNv, false, 2>(ka, smem, st)   \
                                   : launch_one<BM, BN, WMv, WNv, false, 3>(ka, smem, st)))
    if (plan.cfg == 0) {
        if (mode != 0) return set_error(WAP_EINVAL, "internal: large tile needs the fast mode");
        rc = b_tr ? launch_one<256, 256, 2, 4, true, 0>(ka, smem, st)
                  : launch_one<256, 256, 2, 4, false, 0>(ka, smem, st);
    } else if (plan.cfg == 4) {
        if (mode != 0) return set_error(WAP_EINVAL, "internal: large tile needs the fast mode");
        rc = b_tr ? launch_one<256, 256, 2, 2, true, 0>(ka, smem, st)
                  : launch_one<256, 256, 2, 2, false, 0>(ka, smem, st);
    } else if (plan.cfg == 1) {
        rc = WAP_DISPATCH(128, 128, 2, 2);
    } else if (plan.cfg == 2) {
        if (mode != 0) return set_error(WAP_EINVAL, "internal: row-thin tile needs the fast mode");
        rc = b_tr ? launch_one<64, 256, 1, 4, true, 0>(ka, smem, st)
                  : launch_one<64, 256, 1, 4, false, 0>(ka, smem, st);
    } else {
        if (mode != 0) return set_error(WAP_EINVAL, "internal: channel-thin tile needs the fast mode");
        rc = b_tr ? launch_one<256, 64, 4, 1, true, 0>(ka, smem, st)
                  : launch_one<256, 64, 4, 1, false, 0>(ka, smem, st);
    }
#undef WAP_DISPATCH
    if (rc != WAP_OK) return rc;
    if (ev_mid) (void)hipEventRecord(ev_mid, st);
    if (ka.partial)
        return launch_reduce_bf16(reinterpret_cast<const float*>(ws), plan.nsplit,
                                  (size_t)g.M * g.Ncols, g.Ncols, bias, relu, out, st, relu_mask, colsum);
    return WAP_OK;
}

}  // namespace wap

namespace wap {
bool fwd_like_packs_weights(const GemmPlan& plan) { return plan.cfg == 5 || plan.cfg == 6 || plan.cfg == 7 || plan.cfg == 16; }
bool fwd_like_fuses_pool(const GemmGeom& g, const GemmPlan& plan) {
    return plan.cfg == 7 && plan.nsplit == 1 && (g.OH % 2) == 0 && (g.OW % 2) == 0 && tile2d_fuses_pool(g);
}
bool fwd_like_fuses_unpool(const GemmGeom& g, const GemmPlan& plan) {
    return plan.cfg == 16 ? flat_fuses_unpool(g) : plan.cfg == 7 && tile2d_fuses_unpool(g, plan.tile);
}
int fwd_like_colsum_rows(const GemmGeom& g, const GemmPlan& plan) {
    if (plan.nsplit > 1 && plan.cfg != 10) return reduce_bf16_colsum_rows(g.M, g.Ncols);
    if (plan.cfg == 11) return fc_dx_sums(g) ? 1 : 0;
    if (plan.cfg == 16) return flat_colsum_rows(g, plan.tile);
    return plan.cfg == 7 && (g.Ncols % 8) == 0 ? tile2d_colsum_rows(g, plan.tile) : 0;
}
bool fwd_like_fuses_mask(const GemmGeom& g, const GemmPlan& plan) {
    if (plan.nsplit > 1 && plan.cfg != 10) return (g.Ncols % 4) == 0;  // by the kernel that adds up the splits
    return plan.cfg < 5 || ((plan.cfg == 6 || plan.cfg == 7) && (g.Ncols % 8) == 0) || plan.cfg == 11 || plan.cfg == 16;
}
// Label of the kernel instantiation a plan launches (matches the demangled kernel name).
const char* fwd_like_kernel_name(const GemmGeom& g, bool b_tr, const GemmPlan& plan, bool unpool) {
    if (plan.cfg == 5) return "conv_wreg_kernel";
    if (plan.cfg == 6) return patch_kernel_name(g);
    if (plan.cfg == 7) return tile2d_kernel_name(g, unpool, plan.tile);
    if (plan.cfg == 8) return conv_c3_fwd_kernel_name(g);
    if (plan.cfg == 9) return "dgrad_thin_kernel";
    if (plan.cfg == 10) return g.M <= 16 ? "fc_fwd_kernel" : g.M <= 32 ? "fc_fwd_kernel<2>" : "fc_fwd_kernel<4>";
    if (plan.cfg == 11) return "fc_dx_kernel";
    if (plan.cfg == 15) return "conv_thin_fwd_kernel";
    if (plan.cfg == 16) return flat_kernel_name(g, plan.tile, unpool);
    const int mode = classify_mode(g, b_tr);
    const Cfg& c = kCfgs[plan.cfg];
    Phase ph[kMaxPhases];
    int nphase;
    const long tm = phased(g, b_tr) ? make_phases(g, c.BM, ph, &nphase) : (g.M + c.BM - 1) / c.BM;
    const bool dense = mode < 3 && plan.cfg >= 1 && plan.cfg <= 3 && dense_grid(tm * ((g.Ncols + c.BN - 1) / c.BN) * plan.nsplit);
    const int variant = mode + (phased(g, b_tr) ? 4 : 0) + (dense ? 8 : 0);
#define WAP_IG(T, V) "igemm_kernel<" T "," V ">"
#define WAP_IG16(T) {WAP_IG(T, "0"), WAP_IG(T, "1"), WAP_IG(T, "2"), WAP_IG(T, "3"), WAP_IG(T, "4"), WAP_IG(T, "5"), WAP_IG(T, "6"), WAP_IG(T, "7"), \
                     WAP_IG(T, "8"), WAP_IG(T, "9"), WAP_IG(T, "10"), WAP_IG(T, "11"), WAP_IG(T, "12"), WAP_IG(T, "13"), WAP_IG(T, "14"), WAP_IG(T, "15")}
    static const char* names[5][2][16] = {
        {WAP_IG16("256,256,2,4,false"), WAP_IG16("256,256,2,4,true")}, {WAP_IG16("128,128,2,2,false"), WAP_IG16("128,128,2,2,true")},
        {WAP_IG16("64,256,1,4,false"), WAP_IG16("64,256,1,4,true")},   {WAP_IG16("256,64,4,1,false"), WAP_IG16("256,64,4,1,true")},
        {WAP_IG16("256,256,2,2,false"), WAP_IG16("256,256,2,2,true")},
    };
#undef WAP_IG16
#undef WAP_IG
    return names[plan.cfg][b_tr ? 1 : 0][variant];
}
}  // namespace wap
