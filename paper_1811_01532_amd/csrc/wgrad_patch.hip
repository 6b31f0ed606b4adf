// Weight gradient of a stride-1 3x3 or 5x5 convolution with the input PATCH resident in LDS (gfx950):
//   dw[k][(r,s,c)] = sum over pixels (n,p,q) of dy[n,p,q,k] * x[n, p-ph+r, q-pw+s, c]
// (backward half of t_c in Eq. 1; the output is the weight-sized tensor whose aggregation cost the
// platform model of Section 3.2.3 prices).
//
// The generic kernel in wgrad.hip gathers one x tile per filter tap, i.e. reads (and writes to LDS)
// every input pixel nine times.  Here a work-group owns 64*FD output channels x 64 input channels x
// ALL nine taps and walks a range of small 2-D pixel tiles (up to 128 pixels); per tile it writes the
// zero-padded x patch (tile plus halo, 64 channels) and the dy tile to LDS once, and every tap is the
// same patch read through a pointer shifted by (r * padded_width + s) pixels.  Both operands are stored
// as loaded (channel-contiguous) and transposed on the way to the MFMA with ds_read_b64_tr_b16, so an
// arbitrary pixel -> LDS row map costs nothing: a tile is a TH x TW rectangle, its width rounded up to a
// multiple of 4 (at least 16) columns whose surplus pixels carry dy = 0.
//   * 12 wavefronts, three per SIMD whatever the dispatcher's placement: wavefront (r, cb, kh) owns filter
//     row r, the 32-channel half cb of the x slice and FD 32-channel blocks of dy: 3 taps x FD tiles;
//     (5x5: ten wavefronts (r, cb) with 5 taps each and ONE 32-channel block of dy per work-group: two would need 160
//     accumulator registers beside three wavefronts per SIMD.  64 -> 192 channels on 27 x 27, generic kernel / this one
//     with their reductions, us: at 32 images 56 / 42, at 100 106 / 74; 64 -> 64 on 56 x 56 at 32 82 / 46);
//   * one work-group per CU.  LDS holds two tile buffers: while the wavefronts run the MFMAs of tile i out
//     of one buffer, their global loads of tile i+2 are in flight and tile i+1 (already in registers) is
//     written to the other buffer, so a tile costs one barrier and no exposed load or store phase;
//   * instruction count is what the kernel is built around (measured: the time of a tile is close to the
//     SUM of its MFMA time and the issue time of everything else, not their maximum): the loader works in
//     whole tile rows so that its address arithmetic is scalar, the reduction steps address LDS through
//     immediate offsets from two per-lane registers, and fragment reads are interleaved with the MFMAs one
//     step ahead;
//   * the pixel range is split across work-groups; every split writes an fp32 partial and the reduce
//     kernel adds them in a fixed order (bitwise reproducible).
// UP variant: dy is given as the gradient of a 2x2 / stride-2 max-pool OUTPUT plus the pool's argmax; the
// loader routes each window's value to the pixel the argmax names (the max-pool backward of the auxiliary
// node between two primary nodes, Section 3.2.2) on the way into LDS, so the full-size dy never exists.
#include "wap_internal.h"

namespace wap {

namespace {

constexpr int block_ko(int fd, int rf) { return rf == 3 ? 64 * fd : 32; }  // output channels per work-group
constexpr int wavefronts(int rf) { return rf == 3 ? 12 : 10; }
constexpr int XPITCH = 192;   // LDS bytes per patch pixel: 64 channels + 64 bytes, so that the 4 rows x 64 bytes a
                              // half-wavefront touches in one transposing read fall into 4 disjoint bank groups
constexpr int DCAP = 128;     // most dy rows (virtual pixels) per tile: 8 reduction steps of 16
constexpr int pv_max(int rf) { return rf == 3 ? 3 : 4; }  // most wavefront loads of the patch per wavefront and tile
constexpr unsigned OOB = 0x80000000u;  // both tensors are below 2 GiB (checked on the host)
constexpr size_t LDS_BYTES = 160 * 1024;

// How the 16 pixels of one reduction step lie in the tile.  Every mode keeps the LDS address of a step at a
// compile-time distance from the address of step 0, so the reduction loop holds no address arithmetic at all:
//   MODE 0: virtual tile width 16, a step is one tile row;
//   MODE 1: virtual tile width 32, a step is half a tile row;
//   MODE 2: any virtual width that is a multiple of 4, tile height 4, a step is a block of 4 rows x 4 columns.
template <int MODE> struct StepMap;
template <> struct StepMap<0> { static constexpr int VW = 16; };
template <> struct StepMap<1> { static constexpr int VW = 32; };

struct WPArgs {
    const bf16_t* x;
    const bf16_t* dy;
    float* out;
    WgradGeom g;
    int Kred;
    int TH, TWr, VW, PWp;       // tile rows, real / virtual tile columns, padded patch width
    int nk;                     // reduction steps per tile
    int NSEG, NXL;              // 8-pixel segments per patch row, wavefront loads per patch
    int DSEG, NDL;              // segments per dy tile row (UP: per row of pooling windows), wavefront loads per dy tile
    int tiles_x, tiles_img, tiles_total;
    int kgroups, ncombo, nsplit, tiles_per_split;
    int buf_bytes, d_off;       // bytes per LDS tile buffer, offset of the dy tile inside it
    unsigned x_bytes, dy_bytes;
    const uint8_t* am;  // UP: argmax (r * 2 + s) of every pooling window, same shape as the pooled dy
    int P2, Q2;         // UP: pooled map size
    FastDiv dNSEG, dDSEG, dTimg, dTx;
};

__device__ __forceinline__ int xcd_remap(int bid, int total) {
    int per = total / kNumXCD, rem = total % kNumXCD;
    int xcd = bid % kNumXCD, idx = bid / kNumXCD;
    return xcd < rem ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
}

typedef s16x4 __attribute__((address_space(3))) * lds_s16x4_ptr;
__device__ __forceinline__ bf16x8 tr_pair(const unsigned char* p0, const unsigned char* p1) {
    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)p0);
    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)p1);
    s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, both);
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

// FD: 32-channel dy blocks per wavefront; the work-group covers 64 * FD output channels.  UP: dy arrives pooled.
// NK: reduction steps per tile (tile pixels / 16).  RF: filter side; 5 with FD = 1 only, a work-group then covers 32
// output channels.
// Computes output channels ko0 .. and input channels c0 .. over the tiles t0 .. t1 - 1; element (k, tap, c) of the block goes to
// outp[k * ldk + tap * ldt + c].
template <int FD, bool UP, int MODE, int NK, int RF>
__device__ __forceinline__ void wgrad_patch_body(const WPArgs& a, int ko0, int c0, int t0, int t1, float* outp, int ldk, int ldt) {
    static_assert(RF == 3 || (RF == 5 && FD == 1 && !UP), "5x5: one dy block, full-size dy");
    constexpr int NW = wavefronts(RF);
    constexpr int KO = block_ko(FD, RF);                   // output channels per work-group
    constexpr int DPITCH = RF == 3 ? KO * 2 + 64 : 192;    // same bank argument as XPITCH
    constexpr int DVP = KO / 8;             // 16-byte vectors per dy pixel
    constexpr int PPW = 64 / DVP;           // dy pixels (UP: pooling windows) one wavefront load covers
    // wavefront loads per wavefront and tile: the wavefronts share (tile rows + RF - 1) x segments loads of the patch and
    // tile rows x segments loads of dy (pooled dy: one)
    constexpr int TVW = MODE == 0 ? 16 : MODE == 1 ? 32 : 4 * NK, TTH = NK * 16 / TVW;
    constexpr int PV = ((TTH + RF - 1) * ((TVW + RF - 1 + 7) / 8) + NW - 1) / NW;
    constexpr int DV = UP ? 1 : (TTH * ((TVW + PPW - 1) / PPW) + NW - 1) / NW;
    static_assert(PV <= pv_max(RF) && DV <= 3, "tile too large for the loader");
    extern __shared__ __align__(16) unsigned char smem[];
    const WgradGeom& g = a.g;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // uniform: everything derived from it stays scalar
    const int r = RF == 3 ? wave >> 2 : wave >> 1, cb = RF == 3 ? (wave >> 1) & 1 : wave & 1, kh = RF == 3 ? wave & 1 : 0;

    const __amdgpu_buffer_rsrc_t rsrcX =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.x), 0, (int)a.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrcD =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.dy), 0, (int)a.dy_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrcM =  // one argmax byte per pooled element: half the bytes of the pooled dy
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(UP ? a.am : nullptr), 0, UP ? (int)(a.dy_bytes / 2) : 0, 0x00020000);

    // ---- global loads of one tile.  A wavefront load covers a run of pixels of ONE tile row (8 patch pixels x 64
    // channels; 64 / DVP dy pixels or pooling windows x KO channels), so which row, which segment of it, whether the
    // row exists and where it starts in memory are all wavefront-uniform (scalar unit); a lane contributes a
    // constant offset and one comparison of its pixel against the row's valid columns.  The last segment of a row
    // is moved back so that it ends with the row: it then repeats a few pixels of its neighbour (both write the
    // same bytes to the same LDS address), and no lane ever falls outside its row.  Wavefront w takes the loads
    // w, w + NW, w + 2 NW, ... of the tile. ----
    auto seg_start = [](int seg, int per, int row_len) {  // first pixel of segment seg of a row of row_len >= per pixels
        const int p0 = seg * per;
        return p0 + per > row_len ? row_len - per : p0;
    };
    const int lx = lane >> 3;                                             // patch pixel within the segment
    const unsigned xv = (unsigned)(lx * g.C * 2 + (lane & 7) * 16);      // its bytes from the segment's first pixel
    const unsigned xs = (unsigned)(lx * XPITCH + (lane & 7) * 16);       // the same in LDS
    const int lp = lane / DVP, lc = lane % DVP;                           // dy pixel (window) within the segment, 16-byte chunk
    const unsigned dvv = (unsigned)((lp * g.K + lc * 8) * 2);            // bytes from the segment's first pixel (window)
    const unsigned dsl = (unsigned)((UP ? 2 * lp : lp) * DPITCH + lc * 16);  // the same in LDS (a window is two pixels wide)
    u32x4 rp[PV], rd[DV];
    u32x2 ra[1];
    auto load_tile = [&](int t) {
        const int img = (int)fdiv((uint32_t)t, a.dTimg);
        const int rem = t - img * a.tiles_img;
        const int tyi = (int)fdiv((uint32_t)rem, a.dTx);
        const int oh0 = tyi * a.TH, ow0 = (rem - tyi * a.tiles_x) * a.TWr;
        const int ih0 = oh0 - g.ph, iw0 = ow0 - g.pw;
        const int xbase = (((img * g.H + ih0) * g.W + iw0) * g.C + c0) * 2;  // first patch pixel (may lie before the tensor)
#pragma unroll
        for (int i = 0; i < PV; ++i) {
            const int j = wave + NW * i;
            const int py = (int)fdiv((uint32_t)j, a.dNSEG), px0 = seg_start(j - py * a.NSEG, 8, a.PWp);
            // columns of the segment that lie inside the image
            const int lo = -(iw0 + px0);
            const int hi = g.W - iw0 - px0;
            const bool rowok = j < a.NXL && (unsigned)(ih0 + py) < (unsigned)g.H;
            const bool ok = rowok && lx >= lo && lx < hi;
            const unsigned off = xv + (unsigned)(xbase + (py * g.W + px0) * g.C * 2);
            rp[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrcX, ok ? off : OOB, 0, 0);
        }
        if (UP) {
            // one load per wavefront: PPW pooling windows of one pooled row (16 bytes of pooled dy, 8 argmax bytes each);
            // the tile has even origin and size, so windows never straddle tiles
            const int j = wave;
            const int uy = (int)fdiv((uint32_t)j, a.dDSEG), ux0 = seg_start(j - uy * a.DSEG, PPW, a.VW / 2);
            const bool ok = j < a.NDL && oh0 + 2 * uy < g.P && 2 * (ux0 + lp) < a.TWr;
            const unsigned el = (unsigned)(((img * a.P2 + (oh0 >> 1) + uy) * a.Q2 + (ow0 >> 1) + ux0) * g.K + ko0);
            rd[0] = __builtin_amdgcn_raw_buffer_load_b128(rsrcD, ok ? dvv : OOB, el * 2u, 0);
            ra[0] = __builtin_amdgcn_raw_buffer_load_b64(rsrcM, ok ? dvv / 2u : OOB, el, 0);
        } else {
            const int dbase = (((img * g.P + oh0) * g.Q + ow0) * g.K + ko0) * 2;
#pragma unroll
            for (int i = 0; i < DV; ++i) {
                const int j = wave + NW * i;
                const int ty = (int)fdiv((uint32_t)j, a.dDSEG), tx0 = seg_start(j - ty * a.DSEG, PPW, a.VW);
                const bool ok = j < a.NDL && oh0 + ty < g.P && tx0 + lp < a.TWr;
                const unsigned soff = (unsigned)(dbase + (ty * g.Q + tx0) * g.K * 2);
                rd[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrcD, ok ? dvv : OOB, soff, 0);
            }
        }
    };
    // every patch pixel and every dy pixel of the tile is written (zeros where the load was masked), so every row
    // the MFMA loop reads holds either data or zeros
    auto store_tile = [&](int buf) {
        unsigned char* sX = smem + buf * a.buf_bytes;
        unsigned char* sD = sX + a.d_off;
#pragma unroll
        for (int i = 0; i < PV; ++i) {
            const int j = wave + NW * i;
            const int py = (int)fdiv((uint32_t)j, a.dNSEG), px0 = seg_start(j - py * a.NSEG, 8, a.PWp);
            if (j < a.NXL) *reinterpret_cast<u32x4*>(sX + (py * a.PWp + px0) * XPITCH + xs) = rp[i];
        }
        if (UP) {
            const int j = wave;
            const int uy = (int)fdiv((uint32_t)j, a.dDSEG), ux0 = seg_start(j - uy * a.DSEG, PPW, a.VW / 2);
            if (j < a.NDL) {
#pragma unroll
                for (int pos = 0; pos < 4; ++pos) {
                    const int q = (2 * uy + (pos >> 1)) * a.VW + 2 * ux0 + (pos & 1);
                    *reinterpret_cast<u32x4*>(sD + q * DPITCH + dsl) = unpool_select8(rd[0], ra[0], (unsigned)pos);
                    __builtin_amdgcn_sched_barrier(0);  // one pixel at a time: four selected copies at once do not fit
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < DV; ++i) {
                const int j = wave + NW * i;
                const int ty = (int)fdiv((uint32_t)j, a.dDSEG), tx0 = seg_start(j - ty * a.DSEG, PPW, a.VW);
                if (j < a.NDL) *reinterpret_cast<u32x4*>(sD + (ty * a.VW + tx0) * DPITCH + dsl) = rd[i];
            }
        }
    };

    f32x16 acc[RF][FD];  // [tap s of filter row r][32-channel block of dy]
#pragma unroll
    for (int s = 0; s < RF; ++s)
#pragma unroll
        for (int kb = 0; kb < FD; ++kb)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[s][kb][e] = 0.f;

    // transposing read: a lane supplies the address of pixel kl = (lane / 32) * 8 + (lane % 16) / 4 of the step's 16
    // (kl + 4 for the second read) and of the 4-channel chunk ((lane / 16) % 2) * 16 + (lane % 4) * 4 of its block
    const int kl = (lane >> 5) * 8 + ((lane & 15) >> 2);
    const int chunk = (((lane >> 4) & 1) * 16 + (lane & 3) * 4) * 2;
    // LDS offsets of the lane's first pixel in step 0: patch (tap s = 0 of filter row r) and dy; the second pixel
    // (kl + 4) lies at a compile-time distance (MODE 2: one tile row further, and the tile is 4 * NK columns wide)
    constexpr int XB = MODE == 2 ? (4 * NK + RF - 1) * XPITCH : 4 * XPITCH;
    constexpr int DB = MODE == 2 ? 4 * NK * DPITCH : 4 * DPITCH;
    int xa, da;
    if (MODE == 2) {     // pixel i of a step = row i / 4, column i % 4 of the block
        xa = ((r + (kl >> 2)) * a.PWp + (kl & 3)) * XPITCH + cb * 64 + chunk;
        da = a.d_off + ((kl >> 2) * a.VW + (kl & 3)) * DPITCH + kh * (FD * 64) + chunk;
    } else {             // pixel i of a step = column i of the row (half row)
        xa = (r * a.PWp + kl) * XPITCH + cb * 64 + chunk;
        da = a.d_off + kl * DPITCH + kh * (FD * 64) + chunk;
    }

    // ---- reduction over one tile, NK steps of 16 pixels.  Fragment reads run one step ahead of the MFMAs that
    // use them, inside the same wavefront, and mostly in place: a fragment is re-read for the next step as soon as
    // the last MFMA that uses it in this step has been issued, and the MFMAs are ordered so that every fragment then
    // has at least two of the wavefront's own MFMAs (about six of the SIMD's) between its read and its first use.
    // (The hardware arbitrates the MFMA pipe round-robin between the wavefronts of a SIMD, which keeps them in
    // lockstep: without the overlap inside a wavefront all of them wait for LDS at the same time.)  The tile's only
    // barrier sits in the LAST step, in front of the reads that fetch step 0 of the next tile from the other
    // buffer, so the pipeline never drains. ----
    bf16x8 fd[FD], fx[RF];  // dy fragments (one per 32-channel block), patch fragments (one per tap s)
    bf16x8 fdn[1];         // FD == 1 only: the single dy fragment is used by every MFMA of a step, so the next one gets registers of its own
    auto read_d = [&](bf16x8& f, int kb, const unsigned char* sB, int dO) {
        f = tr_pair(sB + da + dO + kb * 64, sB + da + dO + DB + kb * 64);
    };
    auto read_x = [&](int s, const unsigned char* sB, int xo) {
        fx[s] = tr_pair(sB + xa + xo + s * XPITCH, sB + xa + xo + XB + s * XPITCH);
    };
    auto step_x = [](int ks) {  // compile-time distance of step ks from step 0 in the patch
        return MODE == 0 ? ks * (StepMap<0>::VW + RF - 1) * XPITCH
             : MODE == 1 ? ((ks >> 1) * (StepMap<1>::VW + RF - 1) + (ks & 1) * 16) * XPITCH : ks * 4 * XPITCH;
    };
    auto step_d = [](int ks) { return (MODE == 2 ? ks * 4 : ks * 16) * DPITCH; };  // ... and in the dy tile
    auto tile_barrier = [&]() {
        // every wavefront's reads of this buffer have returned and its share of the next tile is in the other
        // buffer (its LDS counter is at zero) before anyone passes
        __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };
    auto mma = [&](int s, int kb, const bf16x8& d) {
        acc[s][kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fx[s], d, acc[s][kb], 0, 0, 0);
    };
    // 5x5: x of a surplus pixel (a tile's virtual columns, rows past the map) is zeroed in front of its product, for its
    // zero dy would not cancel an infinity.  Lane element e is pixel (lane / 32) * 8 + e of the step.
    auto pixel_mask = [&](int ks, int rows) {
        u32x4 m;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            unsigned w = 0;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int p = (lane >> 5) * 8 + 2 * k + h;
                const int row = MODE == 2 ? p >> 2 : MODE == 1 ? ks >> 1 : ks;
                const int col = MODE == 2 ? 4 * ks + (p & 3) : MODE == 1 ? (ks & 1) * 16 + p : p;
                if (row < rows && col < a.TWr) w |= h ? 0xffff0000u : 0xffffu;
            }
            m[k] = w;
        }
        return m;
    };
    auto tile_steps = [&](const unsigned char* sB, const unsigned char* sN, int rows) {
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) {
            const bool last = ks == NK - 1;
            const unsigned char* src = last ? sN : sB;  // where the fragments of the following step live
            const int xo = last ? 0 : step_x(ks + 1), dO = last ? 0 : step_d(ks + 1);
            if constexpr (FD == 2) {
                mma(0, 0, fd[0]); mma(1, 0, fd[0]); mma(2, 0, fd[0]);
                __builtin_amdgcn_sched_barrier(0);
                if (last) tile_barrier();
                read_d(fd[0], 0, src, dO);
                mma(0, 1, fd[1]);
                __builtin_amdgcn_sched_barrier(0);
                read_x(0, src, xo);
                mma(1, 1, fd[1]);
                __builtin_amdgcn_sched_barrier(0);
                read_x(1, src, xo);
                mma(2, 1, fd[1]);
                __builtin_amdgcn_sched_barrier(0);
                read_x(2, src, xo);
                read_d(fd[1], 1, src, dO);
                __builtin_amdgcn_sched_barrier(0);
            } else {
                if (last) tile_barrier();
                read_d((ks & 1) ? fd[0] : fdn[0], 0, src, dO);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (RF == 5) {
                    if (rows < a.TH || (MODE == 2 ? 4 * ks + 4 : MODE == 1 ? (ks & 1) * 16 + 16 : 16) > a.TWr) {
                        const u32x4 m = pixel_mask(ks, rows);
#pragma unroll
                        for (int s = 0; s < RF; ++s) fx[s] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(u32x4, fx[s]) & m);
                    }
                }
#pragma unroll
                for (int s = 0; s < RF; ++s) {
                    mma(s, 0, (ks & 1) ? fdn[0] : fd[0]);
                    read_x(s, src, xo);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
        if (FD == 1 && (NK & 1)) fd[0] = fdn[0];  // the next tile's step 0 sits in the second set: make it the current one
    };

    if (t0 < t1) {
        load_tile(t0);
        store_tile(0);
        if (t0 + 1 < t1) load_tile(t0 + 1);
    }
    __syncthreads();
#pragma unroll
    for (int kb = 0; kb < FD; ++kb) read_d(fd[kb], kb, smem, 0);
#pragma unroll
    for (int s = 0; s < RF; ++s) read_x(s, smem, 0);
    for (int t = t0; t < t1; ++t) {
        const int buf = (t - t0) & 1;
        // tile t+1 (in registers since the previous iteration) -> the other buffer, whose last readers finished
        // before the barrier in the previous tile's last step; then tile t+2 goes in flight
        if (t + 1 < t1) store_tile(buf ^ 1);
        if (t + 2 < t1) load_tile(t + 2);
        const unsigned char* sB = smem + buf * a.buf_bytes;
        const unsigned char* sN = smem + (buf ^ 1) * a.buf_bytes;
        int rows = a.TH;
        if (RF == 5) {  // rows of this tile inside the map
            const int rem = t - (int)fdiv((uint32_t)t, a.dTimg) * a.tiles_img;
            const int left = g.P - (int)fdiv((uint32_t)rem, a.dTx) * a.TH;
            rows = left < rows ? left : rows;
        }
        tile_steps(sB, sN, rows);
    }

    // ---- epilogue: a lane holds 4 consecutive input channels of one output channel per register quad ----
#pragma unroll
    for (int kb = 0; kb < FD; ++kb) {
        const int ko = kh * (FD * 32) + kb * 32 + (lane & 31);
#pragma unroll
        for (int s = 0; s < RF; ++s)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int col = (r * RF + s) * ldt + cb * 32 + q * 8 + (lane >> 5) * 4;
                *reinterpret_cast<float4*>(outp + (size_t)ko * ldk + col) =
                    make_float4(acc[s][kb][q * 4 + 0], acc[s][kb][q * 4 + 1], acc[s][kb][q * 4 + 2], acc[s][kb][q * 4 + 3]);
            }
    }
}

template <int FD, bool UP, int MODE, int NK, int RF>
__device__ __forceinline__ void wgrad_patch_split(const WPArgs& a) {
    const int logical = xcd_remap(blockIdx.x, a.ncombo * a.nsplit);
    const int combo = logical % a.ncombo, split = logical / a.ncombo;
    const int ko0 = (combo % a.kgroups) * block_ko(FD, RF), c0 = (combo / a.kgroups) * 64;
    const int t0 = split * a.tiles_per_split;
    int t1 = t0 + a.tiles_per_split;
    if (t1 > a.tiles_total) t1 = a.tiles_total;
    wgrad_patch_body<FD, UP, MODE, NK, RF>(a, ko0, c0, t0, t1, a.out + (size_t)split * a.g.K * a.Kred + (size_t)ko0 * a.Kred + c0,
                                           a.Kred, a.g.C);
}
template <int FD, bool UP, int MODE, int NK>
__global__ __launch_bounds__(64 * wavefronts(3), 3) void wgrad_patch_kernel(const WPArgs a) {
    wgrad_patch_split<FD, UP, MODE, NK, 3>(a);
}
template <int MODE, int NK>
__global__ __launch_bounds__(64 * wavefronts(5), 3) void wgrad_patch5_kernel(const WPArgs a) {
    wgrad_patch_split<1, false, MODE, NK, 5>(a);
}

// ---- several layers of a step in one launch.  Alone, a layer of little work pays for its share of the chip: one work-group per
// CU means a few tiles each, then 38 MB of partial sums written and read back and a launch for them (VGG-16 at 8 images, conv5_1
// .. 3: 3 x (19.4 + 13.3) us; so 44.3 + 24.6, the sums at 5.4 TB/s; the AlexNet-style conv3 .. 5 71 -> 32).  Here the blocks of all layers of a group are laid end to end, block after block the tiles of
// its reduction, and cut into equal runs of `per` tiles, one run per work-group (a run never spans two layers, so a layer's sums
// depend on `per` and its shape only).  A run that reaches over the end of a block goes on with the next one; every (run,
// block) pair leaves a partial tile in a slot of its own, number run + block of the layer, and a second launch adds up the few
// slots of each block, for all layers, in run order. ----
constexpr int kSlotFloats = 64 * 9 * 64;  // 64 output channels x nine taps x 64 input channels
struct WGroupArgs {
    int njobs, per;
    int first[kMaxWgradGroup + 1];  // first work-group of each layer
    int slot0[kMaxWgradGroup];
    float* part;
    WPArgs job[kMaxWgradGroup];
};
template <bool UP, int MODE, int NK>
__global__ __launch_bounds__(64 * wavefronts(3), 3) void wgrad_patch_group_kernel(const WGroupArgs ga) {
    int j = 0;
    while (j + 1 < ga.njobs && (int)blockIdx.x >= ga.first[j + 1]) ++j;
    const WPArgs& a = ga.job[j];
    const int run = xcd_remap((int)blockIdx.x - ga.first[j], ga.first[j + 1] - ga.first[j]);
    int u = run * ga.per;
    int end = u + ga.per;
    if (end > a.ncombo * a.tiles_total) end = a.ncombo * a.tiles_total;
    while (u < end) {  // at most `per` trips: a block has at least one tile
        const int combo = u / a.tiles_total, t0 = u - combo * a.tiles_total;
        int t1 = t0 + end - u;
        if (t1 > a.tiles_total) t1 = a.tiles_total;
        wgrad_patch_body<1, UP, MODE, NK, 3>(a, (combo % a.kgroups) * 64, (combo / a.kgroups) * 64, t0, t1,
                                             ga.part + (size_t)(ga.slot0[j] + run + combo) * kSlotFloats, 9 * 64, 64);
        u += t1 - t0;
        __syncthreads();  // the tile buffers may be overwritten
    }
}

// The sums of a group: a thread owns 16 bytes of a layer's dw, `spread` (1 or 8) threads share them, each every spread-th slot
// (a block cut into hundreds of runs is a small layer's: 16 KB of dw, walked slot by slot 0.2 us each), whose sums are added in
// order through LDS.
struct WGroupSum {
    int K, C, Kred, kgroups, tiles, runs, slot0, spread;
    FastDiv dRow, dC;   // by Kred / 4, C
    float* out;
    SgdFuse sgd;
};
struct WGroupSumArgs {
    int njobs, per;
    int first[kMaxWgradGroup + 1];  // first work-group of each layer
    const float* part;
    WGroupSum job[kMaxWgradGroup];
};
__global__ __launch_bounds__(256) void wgrad_group_sum_kernel(const WGroupSumArgs ga) {
    __shared__ float4 sm[256];
    int j = 0;
    while (j + 1 < ga.njobs && (int)blockIdx.x >= ga.first[j + 1]) ++j;
    const WGroupSum& a = ga.job[j];
    const int cols = 256 / a.spread, col = threadIdx.x % cols, grp = threadIdx.x / cols;
    const int v = ((int)blockIdx.x - ga.first[j]) * cols + col;
    const bool ok = v < a.K * (a.Kred / 4);
    const int ko = (int)fdiv((uint32_t)(ok ? v : 0), a.dRow);
    const int e = ((ok ? v : 0) - ko * (a.Kred / 4)) * 4;
    const int tap = (int)fdiv((uint32_t)e, a.dC), c = e - tap * a.C;
    const int combo = ko / 64 + c / 64 * a.kgroups;
    const int r0 = combo * a.tiles / ga.per, r1 = ((combo + 1) * a.tiles - 1) / ga.per;  // runs that hold a part of the block
    const float* src = ga.part + (size_t)(a.slot0 + combo) * kSlotFloats + (ko % 64) * (9 * 64) + tap * 64 + c % 64;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    for (int r = r0 + grp; r <= r1; r += 4 * a.spread) {
        float4 t[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int rk = r + k * a.spread;
            t[k] = *reinterpret_cast<const float4*>(src + (size_t)(rk <= r1 ? rk : r1) * kSlotFloats);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k)
            if (r + k * a.spread <= r1) { s.x += t[k].x; s.y += t[k].y; s.z += t[k].z; s.w += t[k].w; }
    }
    if (a.spread > 1) {  // (uniform)
        sm[threadIdx.x] = s;
        __syncthreads();
        if (grp == 0)
            for (int k = 1; k < a.spread; ++k) {
                const float4 t = sm[k * cols + col];
                s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
            }
    }
    if (grp != 0 || !ok) return;
    if (a.sgd.w32) sgd_apply4(a.sgd.w32 + (size_t)v * 4, a.sgd.wb + (size_t)v * 4, a.sgd.lr, s.x, s.y, s.z, s.w);
    else *reinterpret_cast<float4*>(a.out + (size_t)v * 4) = s;
}

struct TileShape {
    int TH, TWr, VW, mode;
    int nseg(int rf) const { return (VW + rf - 1 + 7) / 8; }  // 8-pixel segments per patch row
    int nk() const { return TH * VW / 16; }
};

bool choose_tile_fd(const WgradGeom& g, int fd, struct TileShape* out);
int fd_for(const WgradGeom& g);
size_t buf_bytes_for(int fd, const TileShape& ts, int rf) {
    return (size_t)(ts.TH + rf - 1) * (ts.VW + rf - 1) * XPITCH + (size_t)ts.TH * ts.VW * (rf == 3 ? fd * 128 + 64 : 192);
}
int ko_for(const WgradGeom& g, int fd) { return block_ko(fd, g.R); }

// Most real pixels per tile (the tile height need not divide the map: the last tile row of an image is then partly
// masked) among the tiles the kernel's three step maps cover and whose two LDS buffers fit; then the least padding.
bool choose_tile_fd(const WgradGeom& g, int fd, TileShape* out) {
    long best = 0;
    for (int twr = 1; twr <= g.Q && twr <= 32; ++twr) {
        if (g.Q % twr) continue;
        const int vw = twr <= 16 ? 16 : (twr + 3) / 4 * 4;
        if (vw > 32) continue;
        const int mode = vw == 16 ? 0 : vw == 32 ? 1 : 2;
        for (int th = 1; th <= g.P; ++th) {
            if ((mode == 2 && th != 4) || (mode == 1 && th != 4) || (mode == 0 && th != 7 && th != 8)) continue;
            const TileShape ts{th, twr, vw, mode};
            if (th * vw > DCAP || (th + g.R - 1) * ts.nseg(g.R) > wavefronts(g.R) * pv_max(g.R)) break;
            if (2 * buf_bytes_for(fd, ts, g.R) > LDS_BYTES) break;
            const int tiles_y = (g.P + th - 1) / th;
            // real pixels per tile first, then the least padding, then even tiles (whole pooling windows)
            long score = ((long)g.P * twr * 1024 / tiles_y + (1023 - th * (vw - twr))) * 2 + ((th % 2) == 0 && (twr % 2) == 0 ? 1 : 0);
            if (score > best) {
                best = score;
                *out = ts;
            }
        }
    }
    return best > 0;
}

// 32-channel dy blocks per wavefront: two where the layer has a multiple of 128 output channels, unless the pixel range
// is short (at most 28 tiles per work-group: small minibatches, the 14 x 14 layers): the fp32 partial tiles that every
// work-group writes and the reduction that reads them then weigh more than the better register tile saves, and
// 64-channel work-groups halve those bytes for the same number of work-groups (conv4_2 at minibatch 8: 75 -> 38 MB).
// Measured on whole steps with the limit at 8 / 16 / 28 tiles: VGG-16 -5.1 / -5.1 / -5.2 % at b = 8, -2.2 / -3.4 / -3.6 %
// at 16, -0.9 / -1.0 / -1.3 % at 32, 0 / 0 / -0.5 % at 64; the AlexNet-style step -2 .. -3 % at b = 8 .. 64.
int fd_for(const WgradGeom& g) {
    if (g.R != 3 || (g.K % 128) != 0 || g_force_wgrad_cfg == 6) return 1;
    if (g_force_wgrad_cfg == 5) return 2;
    TileShape ts;
    if (!choose_tile_fd(g, 2, &ts)) return 1;
    const long tiles = (long)g.N * ((g.P + ts.TH - 1) / ts.TH) * (g.Q / ts.TWr);
    const long ncombo2 = (long)(g.K / 128) * (g.C / 64);
    return tiles * ncombo2 <= 28L * kNumCU ? 1 : 2;
}
bool choose_tile(const WgradGeom& g, TileShape* out) { return choose_tile_fd(g, fd_for(g), out); }

}  // namespace

bool wgrad_patch_supported(const WgradGeom& g) {
    if (g.R != g.S || (g.R != 3 && g.R != 5) || g.sh != 1 || g.sw != 1) return false;
    if ((g.C % 64) != 0 || (g.K % (g.R == 3 ? 64 : 32)) != 0) return false;
    if ((size_t)g.N * g.H * g.W * g.C * 2 >= (1ull << 31) || (size_t)g.N * g.P * g.Q * g.K * 2 >= (1ull << 31)) return false;
    TileShape ts;
    if (!choose_tile(g, &ts)) return false;
    // 5x5: the prologue and the partial sums of one work-group per CU take about 18 us whatever the layer, the generic kernel
    // overtakes it below some 8 GFLOP (27 x 27, 64 -> 192: 4.3 / 17 GFLOP 31.6 against 25.5 and 41.6 against 56.5 us; 14 x 14,
    // 128 -> 128: 5.1 / 16 GFLOP 34 against 28 and 46 against 53; 28 x 28, 512 -> 64: 5.1 / 10 GFLOP 32 against 35 and 36
    // against 54).  (A single split could not apply the update by itself.)
    if (g.R == 5 && (wgrad_patch_nsplit(g) < 2 ||
                     (g_force_wgrad_cfg != 3 && 2.0 * g.N * g.P * g.Q * g.K * g.C * 25.0 < 8e9)))
        return false;
    return ts.TH * ts.TWr >= 64;  // tiny tiles: the generic kernel is no worse
}

namespace {
// the instantiated (step map, steps per tile) pairs
constexpr int kNumVariants = 6;
constexpr int kVariantMode[kNumVariants] = {0, 0, 1, 2, 2, 2};
constexpr int kVariantNK[kNumVariants] = {7, 8, 8, 5, 6, 7};
int variant_of(const TileShape& ts) {
    for (int v = 0; v < kNumVariants; ++v)
        if (kVariantMode[v] == ts.mode && kVariantNK[v] == ts.nk()) return v;
    return -1;
}
}  // namespace

const char* wgrad_patch_kernel_name(const WgradGeom& g, bool unpool) {
    static const char* names[2][2][kNumVariants] = {
        {{"wgrad_patch_kernel<1,false,0,7>", "wgrad_patch_kernel<1,false,0,8>", "wgrad_patch_kernel<1,false,1,8>",
          "wgrad_patch_kernel<1,false,2,5>", "wgrad_patch_kernel<1,false,2,6>", "wgrad_patch_kernel<1,false,2,7>"},
         {"wgrad_patch_kernel<1,true,0,7>", "wgrad_patch_kernel<1,true,0,8>", "wgrad_patch_kernel<1,true,1,8>",
          "wgrad_patch_kernel<1,true,2,5>", "wgrad_patch_kernel<1,true,2,6>", "wgrad_patch_kernel<1,true,2,7>"}},
        {{"wgrad_patch_kernel<2,false,0,7>", "wgrad_patch_kernel<2,false,0,8>", "wgrad_patch_kernel<2,false,1,8>",
          "wgrad_patch_kernel<2,false,2,5>", "wgrad_patch_kernel<2,false,2,6>", "wgrad_patch_kernel<2,false,2,7>"},
         {"wgrad_patch_kernel<2,true,0,7>", "wgrad_patch_kernel<2,true,0,8>", "wgrad_patch_kernel<2,true,1,8>",
          "wgrad_patch_kernel<2,true,2,5>", "wgrad_patch_kernel<2,true,2,6>", "wgrad_patch_kernel<2,true,2,7>"}}};
    static const char* names5[kNumVariants] = {"wgrad_patch5_kernel<0,7>", "wgrad_patch5_kernel<0,8>",
                                               "wgrad_patch5_kernel<1,8>", "wgrad_patch5_kernel<2,5>",
                                               "wgrad_patch5_kernel<2,6>", "wgrad_patch5_kernel<2,7>"};
    TileShape ts;
    if (!choose_tile(g, &ts) || variant_of(ts) < 0) return "wgrad_patch_kernel";
    if (g.R == 5) return names5[variant_of(ts)];
    return names[fd_for(g) - 1][unpool ? 1 : 0][variant_of(ts)];
}

// dy given as the gradient of the 2x2 / stride-2 pooled output plus the argmax: whole windows only, and one
// wavefront load of windows per wavefront
static int unpool_loads(const WgradGeom& g, const TileShape& ts) {
    const int ppw = fd_for(g) == 2 ? 4 : 8;
    return (ts.TH / 2) * ((ts.VW / 2 + ppw - 1) / ppw);
}
bool wgrad_patch_fuses_unpool(const WgradGeom& g) {
    TileShape ts;
    if (g.R != 3 || !wgrad_patch_supported(g) || (g.P % 2) != 0 || (g.Q % 2) != 0 || !choose_tile(g, &ts)) return false;
    if ((ts.TH % 2) != 0 || (ts.TWr % 2) != 0) return false;  // windows must not straddle tiles
    return unpool_loads(g, ts) <= wavefronts(3);
}

int wgrad_patch_nsplit(const WgradGeom& g) {
    TileShape ts;
    if (!choose_tile(g, &ts)) return 1;
    const long tiles = (long)g.N * ((g.P + ts.TH - 1) / ts.TH) * (g.Q / ts.TWr);
    const long ncombo = (long)(g.K / ko_for(g, fd_for(g))) * (g.C / 64);
    long want = kNumCU / ncombo;  // one resident work-group per CU, one round (never a second, nearly empty one)
    if (want < 1) want = 1;
    if (want > tiles) want = tiles;
    const long tps = (tiles + want - 1) / want;
    return (int)((tiles + tps - 1) / tps);
}

namespace {
template <int FD, bool UP>
const void* variant_fn(int v) {
    switch (v) {
        case 0: return (const void*)wgrad_patch_kernel<FD, UP, 0, 7>;
        case 1: return (const void*)wgrad_patch_kernel<FD, UP, 0, 8>;
        case 2: return (const void*)wgrad_patch_kernel<FD, UP, 1, 8>;
        case 3: return (const void*)wgrad_patch_kernel<FD, UP, 2, 5>;
        case 4: return (const void*)wgrad_patch_kernel<FD, UP, 2, 6>;
        default: return (const void*)wgrad_patch_kernel<FD, UP, 2, 7>;
    }
}
const void* variant5_fn(int v) {
    switch (v) {
        case 0: return (const void*)wgrad_patch5_kernel<0, 7>;
        case 1: return (const void*)wgrad_patch5_kernel<0, 8>;
        case 2: return (const void*)wgrad_patch5_kernel<1, 8>;
        case 3: return (const void*)wgrad_patch5_kernel<2, 5>;
        case 4: return (const void*)wgrad_patch5_kernel<2, 6>;
        default: return (const void*)wgrad_patch5_kernel<2, 7>;
    }
}
const void* kernel_fn(int fd, bool up, int v, int rf) {
    if (rf == 5) return variant5_fn(v);
    if (fd == 1) return up ? variant_fn<1, true>(v) : variant_fn<1, false>(v);
    return up ? variant_fn<2, true>(v) : variant_fn<2, false>(v);
}
}  // namespace

static int patch_args(const WgradGeom& g, int nsplit, const bf16_t* x, const bf16_t* dy, float* out, const uint8_t* unpool_am, WPArgs* args,
                      int* variant) {
    WPArgs& wa = *args;
    TileShape ts;
    if (!wgrad_patch_supported(g) || !choose_tile(g, &ts))
        return set_error(WAP_EINVAL, "internal: patch weight-gradient kernel not applicable");
    if (unpool_am && !wgrad_patch_fuses_unpool(g))
        return set_error(WAP_EINVAL, "internal: fused max-pool backward not available for this shape");
    const int fd = fd_for(g), rf = g.R, nw = wavefronts(rf);
    const int ppw = 512 / ko_for(g, fd);
    wa.am = unpool_am;
    wa.P2 = g.P / 2;
    wa.Q2 = g.Q / 2;
    wa.x = x;
    wa.dy = dy;
    wa.out = out;
    wa.g = g;
    wa.Kred = g.R * g.S * g.C;
    wa.TH = ts.TH;
    wa.TWr = ts.TWr;
    wa.VW = ts.VW;
    wa.PWp = ts.VW + rf - 1;
    wa.nk = ts.nk();
    wa.NSEG = ts.nseg(rf);
    wa.NXL = (ts.TH + rf - 1) * wa.NSEG;
    if (unpool_am) {
        wa.DSEG = (ts.VW / 2 + ppw - 1) / ppw;
        wa.NDL = unpool_loads(g, ts);
    } else {
        wa.DSEG = (ts.VW + ppw - 1) / ppw;
        wa.NDL = ts.TH * wa.DSEG;
    }
    // what the kernel's fixed loop counts and compile-time step distances assume
    const bool fits = variant_of(ts) >= 0 && wa.nk <= DCAP / 16 && wa.NXL <= nw * pv_max(rf) &&
                      wa.NDL <= (unpool_am ? nw : nw * (rf == 5 ? 1 : fd == 2 ? 3 : 2)) &&
                      ts.VW >= 16 && (ts.mode != 0 || ts.VW == StepMap<0>::VW) && (ts.mode != 1 || ts.VW == StepMap<1>::VW) &&
                      (ts.mode != 2 || (ts.TH == 4 && ts.VW == 4 * wa.nk));
    if (!fits) return set_error(WAP_EINVAL, "internal: patch weight-gradient tile outside the kernel's step maps");
    wa.tiles_x = g.Q / ts.TWr;
    wa.tiles_img = wa.tiles_x * ((g.P + ts.TH - 1) / ts.TH);
    wa.tiles_total = wa.tiles_img * g.N;
    wa.kgroups = g.K / ko_for(g, fd);
    wa.ncombo = wa.kgroups * (g.C / 64);
    wa.nsplit = nsplit;
    wa.tiles_per_split = (wa.tiles_total + nsplit - 1) / nsplit;
    wa.d_off = (ts.TH + rf - 1) * wa.PWp * XPITCH;
    wa.buf_bytes = (int)buf_bytes_for(fd, ts, rf);
    wa.x_bytes = (unsigned)((size_t)g.N * g.H * g.W * g.C * 2);
    wa.dy_bytes = (unsigned)((size_t)g.N * g.P * g.Q * g.K * 2 / (unpool_am ? 4 : 1));
    wa.dNSEG = make_fastdiv((uint32_t)wa.NSEG);
    wa.dDSEG = make_fastdiv((uint32_t)wa.DSEG);
    wa.dTimg = make_fastdiv((uint32_t)wa.tiles_img);
    wa.dTx = make_fastdiv((uint32_t)wa.tiles_x);
    *variant = variant_of(ts);
    if (2 * (size_t)wa.buf_bytes > LDS_BYTES) return set_error(WAP_EINVAL, "internal: patch weight-gradient tile does not fit LDS");
    return WAP_OK;
}

int launch_wgrad_patch(const WgradGeom& g, int nsplit, const bf16_t* x, const bf16_t* dy, float* out, hipStream_t st,
                       const uint8_t* unpool_am) {
    WPArgs wa;
    int variant;
    int rc = patch_args(g, nsplit, x, dy, out, unpool_am, &wa, &variant);
    if (rc != WAP_OK) return rc;
    const int fd = fd_for(g), rf = g.R;
    const size_t smem = 2 * (size_t)wa.buf_bytes;
    static std::atomic<bool> attr_done{false};
    if (!attr_done) {
        for (int k = 0; k < 5 * kNumVariants; ++k) {  // 3x3: one / two blocks, full-size / pooled dy; 5x5
            const int kind = k / kNumVariants;
            const void* f = kind == 4 ? kernel_fn(1, false, k % kNumVariants, 5) : kernel_fn(1 + kind / 2, (kind & 1) != 0, k % kNumVariants, 3);
            hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_BYTES);
            if (e != hipSuccess) return set_error(WAP_EHIP, "hipFuncSetAttribute: %s", hipGetErrorString(e));
        }
        attr_done = true;
    }
    void* kargs[] = {(void*)&wa};
    hipError_t le = hipLaunchKernel(kernel_fn(fd, unpool_am != nullptr, variant, rf), dim3(wa.ncombo * nsplit), dim3(64 * wavefronts(rf)), kargs, smem, st);
    if (le != hipSuccess) return set_error(WAP_EHIP, "wgrad_patch launch: %s", hipGetErrorString(le));
    return check_launch("wgrad_patch");
}

// ---- groups of layers (a step's) ----
// Layers of little work (one 32-channel dy block per wavefront) that run on the same instantiation may share a launch.
int wgrad_group_variant(const WgradGeom& g) {
    TileShape ts;
    if (g.R != 3 || plan_wgrad(g).cfg != 3 || fd_for(g) != 1 || !choose_tile(g, &ts)) return -1;
    return variant_of(ts);
}
long wgrad_group_units(const WgradGeom& g) {
    TileShape ts;
    if (!choose_tile(g, &ts)) return 0;
    return (long)g.N * ((g.P + ts.TH - 1) / ts.TH) * (g.Q / ts.TWr) * (g.K / 64) * (g.C / 64);
}
// Least tiles per work-group with which the layers (their units) need no more than one work-group per CU.
int wgrad_group_per(const long* units, int n) {
    long total = 0;
    for (int i = 0; i < n; ++i) total += units[i];
    for (long per = (total + kNumCU - 1) / kNumCU;; ++per) {
        long groups = 0;
        for (int i = 0; i < n; ++i) groups += (units[i] + per - 1) / per;
        if (groups <= kNumCU || per >= total) return (int)per;
    }
}
size_t wgrad_group_ws_bytes(const WgradGroup& wg) {
    size_t slots = 0;
    for (int i = 0; i < wg.n; ++i) slots += (wgrad_group_units(wg.g[i]) + wg.per - 1) / wg.per + (size_t)(wg.g[i].K / 64) * (wg.g[i].C / 64);
    return slots * kSlotFloats * sizeof(float);
}
const char* wgrad_group_kernel_name(const WgradGroup& wg, bool unpool, bool first) {
#define WAP_WG(U, V) {"wgrad_patch_group_kernel<" U "," V ">", "wgrad_patch_group_kernel<" U "," V "> (shared)"}
#define WAP_WG6(U) {WAP_WG(U, "0,7"), WAP_WG(U, "0,8"), WAP_WG(U, "1,8"), WAP_WG(U, "2,5"), WAP_WG(U, "2,6"), WAP_WG(U, "2,7")}
    static const char* names[2][kNumVariants][2] = {WAP_WG6("false"), WAP_WG6("true")};
#undef WAP_WG6
#undef WAP_WG
    const int v = wgrad_group_variant(wg.g[0]);
    return v < 0 ? "wgrad_patch_group_kernel" : names[unpool ? 1 : 0][v][first ? 0 : 1];
}
namespace {
template <bool UP>
const void* group_fn(int v) {
    switch (v) {
        case 0: return (const void*)wgrad_patch_group_kernel<UP, 0, 7>;
        case 1: return (const void*)wgrad_patch_group_kernel<UP, 0, 8>;
        case 2: return (const void*)wgrad_patch_group_kernel<UP, 1, 8>;
        case 3: return (const void*)wgrad_patch_group_kernel<UP, 2, 5>;
        case 4: return (const void*)wgrad_patch_group_kernel<UP, 2, 6>;
        default: return (const void*)wgrad_patch_group_kernel<UP, 2, 7>;
    }
}
}  // namespace

int launch_wgrad_group(const WgradGroup& wg, const WgradGroupPtrs* ptrs, float lr, void* ws, hipStream_t st, hipEvent_t ev_mid) {
    WGroupArgs ga;
    WGroupSumArgs gs;
    if (wg.n < 1 || wg.n > kMaxWgradGroup || wg.per < 1) return set_error(WAP_EINVAL, "internal: bad group of weight gradients");
    ga.njobs = gs.njobs = wg.n;
    ga.per = gs.per = wg.per;
    ga.part = reinterpret_cast<float*>(ws);
    gs.part = ga.part;
    ga.first[0] = gs.first[0] = 0;
    int variant = -1, slots = 0, smem = 0;
    for (int i = 0; i < wg.n; ++i) {
        const WgradGeom& g = wg.g[i];
        const WgradGroupPtrs& p = ptrs[i];
        WPArgs& wa = ga.job[i];
        int v;
        int rc = patch_args(g, 1, p.x, p.dy, nullptr, p.unpool_am, &wa, &v);
        if (rc != WAP_OK) return rc;
        if (fd_for(g) != 1 || g.R != 3 || (variant >= 0 && v != variant) || (p.unpool_am != nullptr) != (ptrs[0].unpool_am != nullptr) ||
            (long)wa.ncombo * wa.tiles_total > 2147483647L - wg.per || (long)g.K * wa.Kred / 4 > 2147483647L)
            return set_error(WAP_EINVAL, "internal: weight gradients of different kernels in one group");
        variant = v;
        smem = 2 * wa.buf_bytes > smem ? 2 * wa.buf_bytes : smem;
        const int runs = (wa.ncombo * wa.tiles_total + wg.per - 1) / wg.per;
        ga.first[i + 1] = ga.first[i] + runs;
        ga.slot0[i] = slots;
        WGroupSum& js = gs.job[i];
        js.K = g.K; js.C = g.C; js.Kred = wa.Kred; js.kgroups = wa.kgroups; js.tiles = wa.tiles_total; js.runs = runs; js.slot0 = slots;
        js.spread = wa.tiles_total / wg.per >= 8 ? 8 : 1;
        js.dRow = make_fastdiv((uint32_t)(wa.Kred / 4));
        js.dC = make_fastdiv((uint32_t)g.C);
        js.out = p.dw;
        js.sgd = SgdFuse{p.w32, p.wb, lr};
        const int cols = 256 / js.spread;
        gs.first[i + 1] = gs.first[i] + (g.K * (wa.Kred / 4) + cols - 1) / cols;
        slots += runs + wa.ncombo;
    }
    const bool up = ptrs[0].unpool_am != nullptr;
    static std::atomic<bool> attr_done{false};
    if (!attr_done) {
        for (int k = 0; k < 2 * kNumVariants; ++k) {
            hipError_t e = hipFuncSetAttribute(k < kNumVariants ? group_fn<false>(k) : group_fn<true>(k - kNumVariants),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS_BYTES);
            if (e != hipSuccess) return set_error(WAP_EHIP, "hipFuncSetAttribute: %s", hipGetErrorString(e));
        }
        attr_done = true;
    }
    void* kargs[] = {(void*)&ga};
    hipError_t le = hipLaunchKernel(up ? group_fn<true>(variant) : group_fn<false>(variant), dim3(ga.first[wg.n]), dim3(64 * wavefronts(3)),
                                    kargs, smem, st);
    if (le != hipSuccess) return set_error(WAP_EHIP, "wgrad_patch_group launch: %s", hipGetErrorString(le));
    int rc = check_launch("wgrad_patch_group");
    if (rc != WAP_OK) return rc;
    if (ev_mid) (void)hipEventRecord(ev_mid, st);
    hipLaunchKernelGGL(wgrad_group_sum_kernel, dim3(gs.first[wg.n]), dim3(256), 0, st, gs);
    return check_launch("wgrad_group_sum");
}

}  // namespace wap
