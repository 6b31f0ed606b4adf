// Weight-gradient implicit GEMM on bf16 MFMA (gfx950):
//   dw[k][(r,s,c)] = sum over pixels (n,p,q) of dy[n,p,q,k] * x[n, p*sh-ph+r, q*sw-pw+s, c]
// (backward half of t_c in Eq. 1; its output is the weight-sized tensor that the gradient
// aggregation of Section 3.2.3 would move).  Also serves the FC weight gradient (R=S=H=W=1).
//
// The reduction index (the pixel) is the slow axis of both operands in memory (NHWC), so both LDS
// tiles are kept channel-contiguous exactly as loaded and are transposed on the way to the MFMA
// with ds_read_b64_tr_b16.  The reduction is split across work-groups (the output is tiny, the
// reduction is N*P*Q long); every split writes an fp32 partial tile and a second kernel adds the
// partials in split order, so results are bitwise reproducible.  The x-column fragment is the MFMA
// "A" operand: each lane then owns 4 consecutive (r,s,c) columns of one output channel; the epilogue
// turns each wavefront's blocks around in LDS so that 16 lanes store one 256-byte run of a row.  With
// a parameter block the epilogue (or the reduction kernel of a split product) applies the SGD update
// with the finished sums instead of storing them.
#include <algorithm>

#include "wap_internal.h"

namespace wap {

namespace {

constexpr int BK = 64;  // pixels per reduction tile

struct WArgs {
    const bf16_t* x;
    const bf16_t* dy;
    float* out;
    WgradGeom g;
    int Kred, Mred;
    int tiles_c, tiles_k, nsplit, ktiles, ktiles_per_split;
    int Cp;      // MODE 1: channels rounded up to 8, the columns per tap (no group of 8 crosses a tap)
    FastDiv dCp;
    unsigned x_bytes, dy_bytes;
    bool once;       // host side, unsplit: the fp32 matrix passes the cache
    int max_groups;  // host side: most work-groups of the grid (0: one per tile)
    FastDiv dPQ, dQ;
    SgdFuse sgd;  // w32 != NULL (unsplit reduction, Kred % 4 == 0 only): update the parameters instead of storing dW
};

__device__ __forceinline__ int xcd_remap(int bid, int total) {
    int per = total / kNumXCD, rem = total % kNumXCD;
    int xcd = bid % kNumXCD, idx = bid / kNumXCD;
    return xcd < rem ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
}

// Masked-out elements load from beyond the buffer (no access, zeros), element by element from a zero block.
constexpr unsigned kNowhere = 0xfffffff0u;  // operands of the modes 0 and 1 end before (classify_mode)
__device__ __align__(16) unsigned int g_zero_block_w[4] = {0u, 0u, 0u, 0u};

__device__ __forceinline__ u32x4 pack8(const unsigned short* h) {
    u32x4 v = {(unsigned)h[0] | ((unsigned)h[1] << 16), (unsigned)h[2] | ((unsigned)h[3] << 16),
               (unsigned)h[4] | ((unsigned)h[5] << 16), (unsigned)h[6] | ((unsigned)h[7] << 16)};
    return v;
}

__device__ __forceinline__ bf16x8 tr_frag(const unsigned char* tile, int pitch, int colbase, int ks, int lane) {
    int col = colbase + ((lane >> 4) & 1) * 16 + (lane & 3) * 4;
    int krow = ks * 16 + (lane >> 5) * 8 + ((lane & 15) >> 2);
    typedef s16x4 __attribute__((address_space(3))) * lds_s16x4_ptr;
    s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(tile + krow * pitch + col * 2));
    s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(tile + (krow + 4) * pitch + col * 2));
    s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, both);
}

// MODE 0: C % 8 == 0 and K % 8 == 0 (16-byte loads); MODE 1: C and K of at least 8 (unaligned 16-byte loads, every tap's
// channels rounded up to a multiple of 8 columns; element by element, as MODE 2 does it, 195 x 4096 -> 250 took 23 us);
// MODE 2: anything (2-byte loads)
// VARIANT: the mode, plus 4 where the grid leaves a CU one work-group: two wavefronts for every sub-tile, each with half of the
// reduction steps (their sums meet in the LDS), and more tiles in flight, as in igemm.hip.
// ONCE: the fp32 matrix that it writes, with the update also reads, passes the cache (25088 -> 4096 at 22 rows with the update 212 ->
// 173 us; AlexNet-style step at 100 images, gradients stored, 989 -> 958)
template <int TC, int TK, int WAVES_C, int WAVES_K, int VARIANT, bool ONCE = false>
__global__ __launch_bounds__(64 * WAVES_C * WAVES_K * (VARIANT >= 4 ? 2 : 1), VARIANT >= 4 || TC * TK > 128 * 128 ? 1 : 2) void wgrad_kernel(const WArgs a) {
    constexpr int MODE = VARIANT & 3, HALVES = VARIANT >= 4 ? 2 : 1;
    constexpr int NT = 64 * WAVES_C * WAVES_K * HALVES;
    constexpr int SETS = HALVES == 2 ? 4 : 1;  // register sets for tiles in flight
    constexpr int WC = TC / WAVES_C, WK = TK / WAVES_K;
    constexpr int FC = WC / 32, FK = WK / 32;
    constexpr int X_PITCH = TC * 2 + 64, D_PITCH = TK * 2 + 64;
    constexpr int XV = TC / 8, DV = TK / 8;
    constexpr int X_RPP = NT / XV, D_RPP = NT / DV;
    constexpr int X_PASSES = BK / X_RPP, D_PASSES = BK / D_RPP;
    constexpr int X_BYTES = BK * X_PITCH, D_BYTES = BK * D_PITCH;
    constexpr int STAGE = X_BYTES + D_BYTES;
    static_assert(X_PASSES >= 1 && D_PASSES >= 1, "tile too small for the block");

    extern __shared__ __align__(16) unsigned char smem[];

    const WgradGeom& g = a.g;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wc = wave % WAVES_C, wk = HALVES == 1 ? wave / WAVES_C : wave / WAVES_C % WAVES_K, hf = HALVES == 1 ? 0 : wave / (WAVES_C * WAVES_K);

    const int total = a.tiles_c * a.tiles_k * a.nsplit;
    // (a grid of fewer work-groups than tiles walks them; see launch_wgrad's max_groups)
    for (int bid = blockIdx.x; bid < total; bid += gridDim.x) {
    int logical = xcd_remap(bid, total);
    const int tc = logical % a.tiles_c;
    logical /= a.tiles_c;
    const int tk = logical % a.tiles_k;
    const int split = logical / a.tiles_k;
    const int col0 = tc * TC, ko0 = tk * TK;
    const int kt_begin = split * a.ktiles_per_split;
    int kt_end = kt_begin + a.ktiles_per_split;
    if (kt_end > a.ktiles) kt_end = a.ktiles;

    // ---- fixed per-thread column decode of the x operand ----
    const int x_vec = tid % XV, x_row0 = tid / XV;
    const int d_vec = tid % DV, d_row0 = tid / DV;
    constexpr int NE = (MODE <= 1) ? 1 : 8;
    int xr[NE], xs[NE], xc[NE];
    int x_over = 0;
#pragma unroll
    for (int e = 0; e < NE; ++e) {
        int col = col0 + x_vec * 8 + e;
        if (MODE == 1) {
            const int tap = (int)fdiv((uint32_t)col, a.dCp);
            int c = col - tap * a.Cp;
            x_over = c + 8 > g.C ? c + 8 - g.C : 0;
            xc[e] = c - x_over;
            xr[e] = tap < g.R * g.S ? tap / g.S : -(1 << 20);
            xs[e] = tap - tap / g.S * g.S;
        } else if (col < a.Kred) {
            int tap = col / g.C;
            xc[e] = col - tap * g.C;
            xr[e] = tap / g.S;
            xs[e] = tap - xr[e] * g.S;
        } else {
            xc[e] = 0;
            xr[e] = -(1 << 20);  // fails the bounds test for every pixel
            xs[e] = 0;
        }
    }
    const int ko_d = ko0 + d_vec * 8;
    const int d_over = MODE == 1 && ko_d + 8 > g.K ? ko_d + 8 - g.K : 0;  // 8 and more: no channel of this group exists

    const bf16_t* zero_src = reinterpret_cast<const bf16_t*>(g_zero_block_w);  // MODE 2
    const __amdgpu_buffer_rsrc_t rsrcX = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.x), 0, (int)a.x_bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrcD = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.dy), 0, (int)a.dy_bytes, 0x00020000);
    auto ld8 = [](__amdgpu_buffer_rsrc_t r, bool ok, unsigned off) {
        return __builtin_amdgcn_raw_buffer_load_b128(r, ok ? off * 2u : kNowhere, 0, 0);
    };

    // (tiles past kt_end load nothing: no pixel there is below mend)
    const uint32_t mend = kt_end < a.ktiles ? (uint32_t)kt_end * BK : (uint32_t)a.Mred;
    int nxt = kt_begin;  // next tile to load
    auto load_global = [&](u32x4 (&rx)[X_PASSES], u32x4 (&rd)[D_PASSES]) {
        const uint32_t pix0 = (uint32_t)nxt++ * BK;
#pragma unroll
        for (int i = 0; i < X_PASSES; ++i) {
            const uint32_t pix = pix0 + x_row0 + i * X_RPP;
            const bool pok = pix < mend;
            const uint32_t upix = pok ? pix : 0u;
            int n = (int)fdiv(upix, a.dPQ);
            int rem = (int)upix - n * (g.P * g.Q);
            int p = (int)fdiv((uint32_t)rem, a.dQ);
            int q = rem - p * g.Q;
            int hb = p * g.sh - g.ph, wb = q * g.sw - g.pw;
            int base = n * g.H * g.W * g.C;
            if (MODE <= 1) {
                int h = hb + xr[0], w = wb + xs[0];
                bool ok = pok && (unsigned)h < (unsigned)g.H && (unsigned)w < (unsigned)g.W;
                int off = base + (h * g.W + w) * g.C + xc[0];
                rx[i] = ld8(rsrcX, ok, (unsigned)off);
                if (MODE == 1) rx[i] = shift_down8(rx[i], x_over);
            } else {
                unsigned short h16[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    int h = hb + xr[e], w = wb + xs[e];
                    bool ok = pok && (unsigned)h < (unsigned)g.H && (unsigned)w < (unsigned)g.W;
                    int off = base + (h * g.W + w) * g.C + xc[e];
                    h16[e] = *(ok ? a.x + off : zero_src);
                }
                rx[i] = pack8(h16);
            }
        }
#pragma unroll
        for (int i = 0; i < D_PASSES; ++i) {
            const uint32_t pix = pix0 + d_row0 + i * D_RPP;
            const bool pok = pix < mend;
            if (MODE == 1) {
                rd[i] = shift_down8(ld8(rsrcD, pok && d_over < 8, pix * g.K + ko_d - d_over), d_over < 8 ? d_over : 0);
            } else if (MODE == 0) {
                rd[i] = ld8(rsrcD, pok && ko_d < g.K, pix * g.K + ko_d);
            } else {
                unsigned short h16[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    bool ok = pok && (ko_d + e) < g.K;
                    h16[e] = *(ok ? a.dy + ((size_t)pix * g.K + ko_d + e) : zero_src);
                }
                rd[i] = pack8(h16);
            }
        }
    };

    auto store_lds = [&](int stage, const u32x4 (&rx)[X_PASSES], const u32x4 (&rd)[D_PASSES]) {
        unsigned char* sX = smem + stage * STAGE;
        unsigned char* sD = sX + X_BYTES;
#pragma unroll
        for (int i = 0; i < X_PASSES; ++i)
            *reinterpret_cast<u32x4*>(sX + (x_row0 + i * X_RPP) * X_PITCH + x_vec * 16) = rx[i];
#pragma unroll
        for (int i = 0; i < D_PASSES; ++i)
            *reinterpret_cast<u32x4*>(sD + (d_row0 + i * D_RPP) * D_PITCH + d_vec * 16) = rd[i];
    };

    f32x16 acc[FC][FK];
#pragma unroll
    for (int i = 0; i < FC; ++i)
#pragma unroll
        for (int j = 0; j < FK; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    auto compute = [&](int stage) {
        const unsigned char* sX = smem + stage * STAGE;
        const unsigned char* sD = sX + X_BYTES;
#pragma unroll
        for (int k2 = 0; k2 < BK / 16 / HALVES; ++k2) {
            const int ks = hf * (BK / 16 / HALVES) + k2;
            bf16x8 fx[FC], fd[FK];
#pragma unroll
            for (int i = 0; i < FC; ++i) fx[i] = tr_frag(sX, X_PITCH, wc * WC + i * 32, ks, lane);
#pragma unroll
            for (int j = 0; j < FK; ++j) fd[j] = tr_frag(sD, D_PITCH, wk * WK + j * 32, ks, lane);
#pragma unroll
            for (int i = 0; i < FC; ++i)
#pragma unroll
                for (int j = 0; j < FK; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fx[i], fd[j], acc[i][j], 0, 0, 0);
        }
    };

    const int nkt = kt_end - kt_begin;
    if (nkt > 0) {  // tile it in the LDS, the next SETS in registers or in flight; loads unconditional, see igemm.hip
        u32x4 rx[SETS][X_PASSES], rd[SETS][D_PASSES];
#pragma unroll
        for (int i = 0; i < SETS; ++i) load_global(rx[i], rd[i]);
        // nothing is stored or loaded behind the last tile (the largest tiles have no registers for a second copy of the products)
        constexpr int LAST = TC * TK > 128 * 128 ? 0 : 1;
        store_lds(0, rx[0], rd[0]);
        int it = 0;
        if (nkt > 1 || LAST == 0) {
            load_global(rx[0], rd[0]);
            __syncthreads();
            auto step = [&](int stage, u32x4 (&xx)[X_PASSES], u32x4 (&xd)[D_PASSES]) {
                store_lds(stage ^ 1, xx, xd);
                load_global(xx, xd);
                compute(stage);
                __syncthreads();
            };
            constexpr int U = SETS < 2 ? 2 : SETS;
            for (; it + U + LAST <= nkt; it += U) {
#pragma unroll
                for (int u = 0; u < U; ++u) step(u & 1, rx[(u + 1) % SETS], rd[(u + 1) % SETS]);
            }
#pragma unroll
            for (int u = 0; u < U - 1; ++u)
                if (it + u + LAST < nkt) step(u & 1, rx[(u + 1) % SETS], rd[(u + 1) % SETS]);
        } else {
            __syncthreads();
        }
        if constexpr (LAST == 1) {
            compute((nkt - 1) & 1);
            __syncthreads();
        }
    }

    // the halves of the reduction meet: each wavefront keeps half of the dy blocks of its sub-tile
    constexpr int FKK = FK / HALVES;
    if constexpr (HALVES == 2) {
        static_assert(FK % 2 == 0 && (NT / 64) * FC * FKK * 4096 <= 2 * STAGE, "does not fit the operand tiles");
        unsigned char* const mine = smem + wave * (FC * FKK * 4096) + lane * 16;
        unsigned char* const theirs = smem + (wave ^ (WAVES_C * WAVES_K)) * (FC * FKK * 4096) + lane * 16;
#pragma unroll
        for (int i = 0; i < FC; ++i)
#pragma unroll
            for (int j = 0; j < FKK; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<f32x4*>(mine + ((i * FKK + j) * 4 + q) * 1024) =
                        hf == 0 ? f32x4{acc[i][j + FKK][q * 4], acc[i][j + FKK][q * 4 + 1], acc[i][j + FKK][q * 4 + 2], acc[i][j + FKK][q * 4 + 3]}
                                : f32x4{acc[i][j][q * 4], acc[i][j][q * 4 + 1], acc[i][j][q * 4 + 2], acc[i][j][q * 4 + 3]};
        __syncthreads();
#pragma unroll
        for (int i = 0; i < FC; ++i)
#pragma unroll
            for (int j = 0; j < FKK; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 v = *reinterpret_cast<const f32x4*>(theirs + ((i * FKK + j) * 4 + q) * 1024);
#pragma unroll
                    for (int e = 0; e < 4; ++e)  // (the first half's sum first in both)
                        acc[i][j][q * 4 + e] = hf == 0 ? acc[i][j][q * 4 + e] + v[e] : v[e] + acc[i][j + FKK][q * 4 + e];
                }
        __syncthreads();
    }
    const int jb = hf * FKK;  // first dy block kept

    const bool vec4 = (a.Kred & 3) == 0 && (MODE != 1 || a.Cp == g.C);
    float* outp = a.out + (size_t)split * g.K * a.Kred;
    if (vec4) {
        // A lane of the MFMA accumulator holds 16-byte groups of 32 different output rows, so a direct store touches
        // 32 rows per instruction.  Each wave instead turns its 32 x 64 blocks around in a private LDS region (the
        // operand tiles are dead: the main loop ended with a barrier) and moves 256-byte row segments per 16 lanes.
        // With a parameter block the old master weights are fetched before the block goes through LDS.
        static_assert(FC % 2 == 0, "the epilogue stages 64 columns at a time");
        constexpr int EP_PITCH = 64 * 4 + 16;  // rows 16 bytes apart modulo the bank width: both phases conflict-free
        static_assert((NT / 64) * 32 * EP_PITCH <= (TC * TK == 128 * 128 && HALVES == 1 ? 1 : 2) * STAGE, "epilogue staging does not fit the operand tiles");
        unsigned char* const ep = smem + wave * (32 * EP_PITCH);
        const int r_rd = lane >> 4, c_rd = (lane & 15) * 4;
        const bool fused = a.sgd.w32 != nullptr;
        auto pack2bf = [](float lo, float hi) {
            return (unsigned)__builtin_bit_cast(unsigned short, (__bf16)lo) | ((unsigned)__builtin_bit_cast(unsigned short, (__bf16)hi) << 16);
        };
#pragma unroll
        for (int j = 0; j < FKK; ++j) {
#pragma unroll
            for (int ih = 0; ih < FC / 2; ++ih) {
                const int col = col0 + wc * WC + ih * 64 + c_rd;
                const int row0 = ko0 + wk * WK + (jb + j) * 32 + r_rd;
                float4 old[8];
                if (fused) {
#pragma unroll
                    for (int t = 0; t < 8; ++t) {
                        const int ko = row0 + t * 4;
                        old[t] = make_float4(0.f, 0.f, 0.f, 0.f);
                        if (ko < g.K && col < a.Kred) {
                            if constexpr (ONCE) old[t] = __builtin_bit_cast(float4, __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(a.sgd.w32 + (size_t)ko * a.Kred + col)));
                            else old[t] = *reinterpret_cast<const float4*>(a.sgd.w32 + (size_t)ko * a.Kred + col);
                        }
                    }
                }
#pragma unroll
                for (int ii = 0; ii < 2; ++ii) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int i = ih * 2 + ii;
                        *reinterpret_cast<float4*>(ep + (lane & 31) * EP_PITCH + (ii * 32 + q * 8 + (lane >> 5) * 4) * 4) =
                            make_float4(acc[i][j][q * 4 + 0], acc[i][j][q * 4 + 1], acc[i][j][q * 4 + 2],
                                        acc[i][j][q * 4 + 3]);
                    }
                }
                __builtin_amdgcn_wave_barrier();  // LDS operations of one wave complete in order
#pragma unroll
                for (int t = 0; t < 8; ++t) {
                    const int ko = row0 + t * 4;
                    const float4 v = *reinterpret_cast<const float4*>(ep + (t * 4 + r_rd) * EP_PITCH + c_rd * 4);
                    if (ko >= g.K || col >= a.Kred) continue;
                    const size_t e = (size_t)ko * a.Kred + col;
                    if constexpr (ONCE) {
                        f32x4 o = {v.x, v.y, v.z, v.w};
                        if (fused) {
                            o = f32x4{sgd_apply(old[t].x, v.x, a.sgd.lr), sgd_apply(old[t].y, v.y, a.sgd.lr), sgd_apply(old[t].z, v.z, a.sgd.lr), sgd_apply(old[t].w, v.w, a.sgd.lr)};
                            *reinterpret_cast<uint2*>(a.sgd.wb + e) = make_uint2(pack2bf(o[0], o[1]), pack2bf(o[2], o[3]));
                        }
                        __builtin_nontemporal_store(o, reinterpret_cast<f32x4*>((fused ? a.sgd.w32 : outp) + e));
                    } else if (fused) {
                        sgd_store4(a.sgd.w32 + e, a.sgd.wb + e, old[t], a.sgd.lr, v.x, v.y, v.z, v.w);
                    } else {
                        *reinterpret_cast<float4*>(outp + e) = v;
                    }
                }
                __builtin_amdgcn_wave_barrier();
            }
        }
    } else {
#pragma unroll
    for (int j = 0; j < FKK; ++j) {
        const int ko = ko0 + wk * WK + (jb + j) * 32 + (lane & 31);
        if (ko >= g.K) continue;
#pragma unroll
        for (int i = 0; i < FC; ++i) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int col = col0 + wc * WC + i * 32 + q * 8 + (lane >> 5) * 4;
                if constexpr (MODE == 1) {
                    const int tap = (int)fdiv((uint32_t)col, a.dCp), c = col - tap * a.Cp;
                    const int ncol = tap < g.R * g.S ? g.C - c : 0;  // columns of this group that exist
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        if (e >= ncol) continue;
                        const size_t o = (size_t)ko * a.Kred + tap * g.C + c + e;
                        if (a.sgd.w32) {
                            const float w = sgd_apply(a.sgd.w32[o], acc[i][j][q * 4 + e], a.sgd.lr);
                            a.sgd.w32[o] = w;
                            a.sgd.wb[o] = __builtin_bit_cast(unsigned short, (__bf16)w);
                        } else {
                            outp[o] = acc[i][j][q * 4 + e];
                        }
                    }
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (col + e < a.Kred) outp[(size_t)ko * a.Kred + col + e] = acc[i][j][q * 4 + e];
                }
            }
        }
    }
    }
    __syncthreads();  // the tiles in the LDS may be overwritten
    }
}

struct Cfg {
    int TC, TK, NT;
};
constexpr Cfg kCfgs[] = {
    {256, 256, 512},  // 0: large
    {128, 128, 256},  // 1: medium / general
    {256, 64, 256},   // 2: few output channels
};

size_t smem_bytes(const Cfg& c) { return 2 * ((size_t)BK * (c.TC * 2 + 64) + (size_t)BK * (c.TK * 2 + 64)); }

template <int TC, int TK, int WCv, int WKv, int VARIANT, bool ONCE = false>
int launch_variant(const WArgs& wa, size_t smem, hipStream_t st) {
    auto kfn = wgrad_kernel<TC, TK, WCv, WKv, VARIANT, ONCE>;
    static std::atomic<bool> attr_done{false};
    if (!attr_done) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kfn),
                                           hipFuncAttributeMaxDynamicSharedMemorySize,
                                           (int)smem_bytes({TC, TK, 0}));  // the most any launch takes, not this one's
        if (e != hipSuccess) return set_error(WAP_EHIP, "hipFuncSetAttribute: %s", hipGetErrorString(e));
        attr_done = true;
    }
    int total = wa.tiles_c * wa.tiles_k * wa.nsplit;
    if (wa.max_groups > 0 && total > wa.max_groups) total = wa.max_groups;
    hipLaunchKernelGGL(kfn, dim3(total), dim3(64 * WCv * WKv * (VARIANT >= 4 ? 2 : 1)), smem, st, wa);
    return check_launch("wgrad");
}
// (walks of one or two tiles gain nothing that pays for adding up the halves: 40 x 3000 -> 700 7.6 us, 9.6 so)
bool halves(long groups, int tiles) { return groups <= kNumCU && tiles >= 3; }
template <int TC, int TK, int WCv, int WKv, int MODE>
int launch_one(const WArgs& wa, size_t smem, hipStream_t st) {
    constexpr int lone = TC * TK <= 128 * 128 && MODE < 2 ? 4 + MODE : MODE;
    return halves((long)wa.tiles_c * wa.tiles_k * wa.nsplit, wa.ktiles_per_split) ? launch_variant<TC, TK, WCv, WKv, lone>(wa, smem, st)
                                                                 : launch_variant<TC, TK, WCv, WKv, MODE>(wa, smem, st);
}

int classify_mode(const WgradGeom& g) {
    const size_t most = 2147483647u - 63;  // elements of an operand whose last 16 bytes lie below kNowhere
    if ((size_t)g.N * g.H * g.W * g.C > most || (size_t)g.N * g.P * g.Q * g.K > most) return 2;
    if ((g.C % 8) == 0 && (g.K % 8) == 0) return 0;
    return g.C >= 8 && g.K >= 8 ? 1 : 2;
}
int padded_cols(const WgradGeom& g) { return classify_mode(g) == 1 ? g.R * g.S * ((g.C + 7) / 8 * 8) : g.R * g.S * g.C; }

}  // namespace

WgradPlan plan_wgrad(const WgradGeom& g, bool in_step, bool lean) {
    WgradPlan p;
    int mode = classify_mode(g);
    int Kred = g.R * g.S * g.C;
    long Mred = (long)g.N * g.P * g.Q;
    int cfg;
    if (mode != 0) cfg = 1;
    else if (g.K <= 64) cfg = 2;
    else if (g.K >= 192 && Kred >= 256) {
        // A short reduction over a large output (the FC layers at training minibatches) is bound by the epilogue's
        // stores: smaller tiles put several work-groups on a CU, whose store phases then overlap.
        // So does a layer of little work, whose few large tiles leave CUs idle or split the reduction thin (64 -> 192 channels,
        // 5x5 on 27 x 27 at 4 images 26.0 -> 19.6 us, at 8 30.2 -> 25.5, 256 -> 320 on 13 x 13 at 4 28.0 -> 23.0; from about
        // 6 GFLOP on the large tiles win: 14 GFLOP 56 against 61).
        const long small_tiles = (long)((Kred + 127) / 128) * ((g.K + 127) / 128);
        cfg = (Mred <= 256 && small_tiles >= kNumCU) || 2.0 * Mred * g.K * Kred < 6e9 ? 1 : 0;
    } else cfg = 1;
    if (g_force_wgrad_cfg >= 0 && g_force_wgrad_cfg < 3 && (mode == 0 || g_force_wgrad_cfg == 1)) cfg = g_force_wgrad_cfg;
    if ((g_force_wgrad_cfg < 0 || g_force_wgrad_cfg == 4) && wgrad_c3_supported(g)) {
        p.cfg = 4;
        p.nsplit = wgrad_c3_nsplit(g);
        p.ws_bytes = (size_t)p.nsplit * g.K * Kred * sizeof(float);  // always reduced from per-work-group partials
        return p;
    }
    if ((g_force_wgrad_cfg < 0 || g_force_wgrad_cfg == 7) && wgrad_thin_supported(g)) {
        p.cfg = 7;
        p.nsplit = wgrad_thin_nsplit(g);
        p.ws_bytes = (size_t)p.nsplit * g.K * Kred * sizeof(float);
        return p;
    }
    // (5 / 6: the patch kernel with two / one dy blocks per wavefront, for the tests)
    if ((g_force_wgrad_cfg < 0 || g_force_wgrad_cfg == 3 || g_force_wgrad_cfg == 5 || g_force_wgrad_cfg == 6) && mode == 0 &&
        wgrad_patch_supported(g)) {
        p.cfg = 3;
        p.nsplit = g_force_nsplit >= 1 ? g_force_nsplit : wgrad_patch_nsplit(g);
        long tiles_total = (long)g.N * g.P * g.Q / 64;  // every tile holds at least 64 pixels
        if (p.nsplit > tiles_total) p.nsplit = (int)tiles_total;
        p.ws_bytes = p.nsplit > 1 ? (size_t)p.nsplit * g.K * Kred * sizeof(float) : 0;
        return p;
    }
    if (g_force_wgrad_cfg < 0 && g_force_nsplit < 0 && fc_dw_supported(g, in_step)) {
        p.cfg = 8;
        p.nsplit = 1;
        p.ws_bytes = 0;
        return p;
    }
    const Cfg& c = kCfgs[cfg];
    long tiles = (long)((padded_cols(g) + c.TC - 1) / c.TC) * ((g.K + c.TK - 1) / c.TK);
    int ktiles = (int)((Mred + BK - 1) / BK);
    // about one work-group per CU, as fast with its eight wavefronts as two of four and with half the partial sums (24 x 27 x 27 x
    // 119 -> 200 49 us, 60 with two work-groups per CU; 16 x 80 x 80 x 48 -> 24, 5x5, 39.6 and 56)
    long want = tiles < kNumCU ? kNumCU / tiles : 1;
    long maxs = ktiles / 4;
    if (maxs < 1) maxs = 1;
    int nsplit = (int)(want < maxs ? want : maxs);
    // Few tiles and a short reduction fill few CUs with four steps a split: down to two, while the partial sums stay below 4.8 MB.  us, sums
    // included, four / two: 5 x 24 x 31, 256 -> 64 at stride 2 13.1 / 10.5, 4 x 20 x 20, 160 -> 64 13.5 / 10.9, 8 x 14 x 14, 128 -> 64, 1x1,
    // 12.9 / 8.8, 2 x 28 x 28, 96 -> 96 11.6 / 10.0; 4.9 and 7.4 MB (27 x 27, 64 -> 192, 5x5) 11.3 / 11.9 and 12.4, one step and 9 MB 12.5 for 10.9.  (What is
    // whole with four stays whole: the launch that adds up two halves costs 3.  1345 layers of 1x1 to 11x11 filters: 0.81 of the time
    // in the mean, 33 of them 1.02 to 1.06, most where one and a half times the splits make more than 3 MB of sums.)
    if (!lean && nsplit >= 2 && nsplit < want) {
        const long deeper = std::min({want, ((long)ktiles + 1) / 2, (long)(4.8e6 / (4.0 * g.K * Kred))});
        if (deeper > nsplit) nsplit = (int)deeper;
    }
    if (nsplit > 512) nsplit = 512;
    if (tiles >= kNumCU) nsplit = 1;
    if (g_force_nsplit >= 1) nsplit = g_force_nsplit < ktiles ? g_force_nsplit : ktiles;
    int kps = (ktiles + nsplit - 1) / nsplit;
    nsplit = (ktiles + kps - 1) / kps;
    p.cfg = cfg;
    p.nsplit = nsplit;
    p.ws_bytes = nsplit > 1 ? (size_t)nsplit * g.K * Kred * sizeof(float) : 0;
    return p;
}

size_t wgrad_query_bytes(const WgradGeom& g) {
    const WgradPlan p = plan_wgrad(g);
    return p.cfg == 4 ? (size_t)wgrad_c3_query_splits(g) * g.K * g.R * g.S * g.C * sizeof(float) : p.ws_bytes;
}

int launch_wgrad(const WgradGeom& g, const WgradPlan& plan, const bf16_t* x, const bf16_t* dy,
                 float* dw, void* ws, hipStream_t st, hipEvent_t ev_mid, const uint8_t* unpool_am,
                 const SgdFuse* sgd, int max_groups, bool once) {
    if (unpool_am && !wgrad_fuses_unpool(g, plan))
        return set_error(WAP_EINVAL, "internal: fused max-pool backward not available for this weight gradient");
    if (sgd && !wgrad_fuses_sgd(g, plan))
        return set_error(WAP_EINVAL, "internal: fused SGD update not available for this weight gradient");
    if (plan.cfg == 8) return launch_fc_dw(g, x, dy, dw, sgd, max_groups, once, st);
    WArgs wa;
    wa.sgd = SgdFuse{nullptr, nullptr, 0.f};
    if (sgd && plan.nsplit == 1) wa.sgd = *sgd;  // split reductions apply the update in the reduction kernel
    wa.max_groups = max_groups;
    wa.once = once && plan.nsplit == 1;  // (partial sums are read next)
    wa.x = x;
    wa.dy = dy;
    wa.g = g;
    wa.Kred = g.R * g.S * g.C;
    wa.Mred = g.N * g.P * g.Q;
    const Cfg& c = kCfgs[plan.cfg < 3 ? plan.cfg : 0];
    wa.Cp = (g.C + 7) / 8 * 8;
    wa.dCp = make_fastdiv((uint32_t)wa.Cp);
    wa.tiles_c = (padded_cols(g) + c.TC - 1) / c.TC;
    wa.tiles_k = (g.K + c.TK - 1) / c.TK;
    wa.ktiles = (wa.Mred + BK - 1) / BK;
    wa.nsplit = plan.nsplit;
    wa.ktiles_per_split = (wa.ktiles + plan.nsplit - 1) / plan.nsplit;
    wa.x_bytes = (unsigned)((size_t)g.N * g.H * g.W * g.C * 2);
    wa.dy_bytes = (unsigned)((size_t)wa.Mred * g.K * 2);
    wa.dPQ = make_fastdiv((uint32_t)(g.P * g.Q));
    wa.dQ = make_fastdiv((uint32_t)g.Q);
    wa.out = plan.nsplit > 1 ? reinterpret_cast<float*>(ws) : dw;
    if (plan.cfg == 4 || plan.cfg == 7) {
        int rc4 = plan.cfg == 4 ? launch_wgrad_c3(g, plan.nsplit, x, dy, reinterpret_cast<float*>(ws), st)
                                : launch_wgrad_thin(g, plan.nsplit, x, dy, reinterpret_cast<float*>(ws), st);
        if (rc4 != WAP_OK) return rc4;
        if (ev_mid) (void)hipEventRecord(ev_mid, st);
        return launch_reduce_f32(reinterpret_cast<const float*>(ws), plan.nsplit, (size_t)g.K * wa.Kred, dw, st, sgd);
    }
    if (plan.cfg == 3) {
        int rc3 = launch_wgrad_patch(g, plan.nsplit, x, dy, wa.out, st, unpool_am);
        if (rc3 != WAP_OK) return rc3;
        if (ev_mid) (void)hipEventRecord(ev_mid, st);
        if (plan.nsplit > 1)
            return launch_reduce_f32(reinterpret_cast<const float*>(ws), plan.nsplit, (size_t)g.K * wa.Kred, dw, st, sgd);
        return WAP_OK;
    }
    size_t smem = smem_bytes(c);
    if (plan.cfg == 1 && wa.ktiles_per_split == 1) smem /= 2;  // one tile: one stage (which holds the epilogue's blocks as well)
    int mode = classify_mode(g);
    int rc;
    if (plan.cfg == 0) {
        if (mode != 0) return set_error(WAP_EINVAL, "internal: large wgrad tile needs 16-byte loads");
        rc = launch_one<256, 256, 2, 4, 0>(wa, smem, st);
    } else if (plan.cfg == 1) {
        // (a fully-connected layer with whole vectors is all that a step has in this form)
        rc = mode == 0 && wa.once && !halves((long)wa.tiles_c * wa.tiles_k, wa.ktiles) ? launch_variant<128, 128, 2, 2, 0, true>(wa, smem, st)
             : mode == 0 ? launch_one<128, 128, 2, 2, 0>(wa, smem, st)
             : mode == 1 ? launch_one<128, 128, 2, 2, 1>(wa, smem, st)
                         : launch_one<128, 128, 2, 2, 2>(wa, smem, st);
    } else {
        if (mode != 0) return set_error(WAP_EINVAL, "internal: channel-thin wgrad tile needs 16-byte loads");
        rc = launch_one<256, 64, 4, 1, 0>(wa, smem, st);
    }
    if (rc != WAP_OK) return rc;
    if (ev_mid) (void)hipEventRecord(ev_mid, st);
    if (plan.nsplit > 1)
        return launch_reduce_f32(reinterpret_cast<const float*>(ws), plan.nsplit,
                                 (size_t)g.K * wa.Kred, dw, st, sgd);
    return WAP_OK;
}

}  // namespace wap

namespace wap {
bool wgrad_fuses_unpool(const WgradGeom& g, const WgradPlan& plan) {
    return plan.cfg == 3 && wgrad_patch_fuses_unpool(g);
}
// The update rides on whichever kernel holds the finished sums: the reduction kernel of a split product (the
// first-layer kernels always reduce), or the epilogue of an unsplit generic product whose accumulator rows are
// 16-byte groups of parameters.
bool wgrad_fuses_sgd(const WgradGeom& g, const WgradPlan& plan) {
    if (plan.cfg == 4 || plan.cfg == 7 || plan.cfg == 8 || plan.nsplit > 1) return true;
    return plan.cfg < 3 && ((g.R * g.S * g.C) & 3) == 0;
}
const char* wgrad_kernel_name(const WgradGeom& g, const WgradPlan& plan) { return wgrad_kernel_name(g, plan, false); }
const char* wgrad_kernel_name(const WgradGeom& g, const WgradPlan& plan, bool unpool) {
    if (plan.cfg == 3) return wgrad_patch_kernel_name(g, unpool);
    if (plan.cfg == 4) return wgrad_c3_kernel_name(g);
    if (plan.cfg == 7) return "wgrad_thin_kernel";
    if (plan.cfg == 8) return "fc_dw_kernel";
    static const char* names[3][6] = {
        {"wgrad_kernel<256,256,2,4,0>", "", "", "wgrad_kernel<256,256,2,4,0>", "", ""},
        {"wgrad_kernel<128,128,2,2,0>", "wgrad_kernel<128,128,2,2,1>", "wgrad_kernel<128,128,2,2,2>", "wgrad_kernel<128,128,2,2,4>",
         "wgrad_kernel<128,128,2,2,5>", "wgrad_kernel<128,128,2,2,2>"},
        {"wgrad_kernel<256,64,4,1,0>", "", "", "wgrad_kernel<256,64,4,1,4>", "", ""},
    };
    const Cfg& c = kCfgs[plan.cfg];
    const long groups = (long)((padded_cols(g) + c.TC - 1) / c.TC) * ((g.K + c.TK - 1) / c.TK) * plan.nsplit;
    const int ktiles = (int)(((long)g.N * g.P * g.Q + BK - 1) / BK);
    return names[plan.cfg][classify_mode(g) + (halves(groups, (ktiles + plan.nsplit - 1) / plan.nsplit) ? 3 : 0)];
}
}  // namespace wap
