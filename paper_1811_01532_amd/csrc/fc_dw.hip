// Weight gradient of a fully-connected layer at few batch rows (backward half of t_c in Eq. 1), with the SGD update where it is asked for:
//   dW[o][i] = sum over b of dy[b][o] * x[b][i]
// Ten bytes of memory traffic per weight with the update, four without, and a reduction of one to four MFMA depths: a
// stream of the weights.  No LDS and few registers, so that it runs beside the work-groups of other kernels (a step's convolutions):
//   * v_mfma_f32_16x16x32_bf16 with dy as the row operand: a lane's accumulators are one column of 4 rows.  Four MFMAs of a
//     block take the columns 4 n + c (c = 0 .. 3), so that a lane ends with float4s of the row-major matrix and a wavefront
//     moves whole 256-byte runs of four rows, with no pass through the LDS;
//   * a wavefront walks down the rows of its columns; the operand of x stays in registers, the old weights of the next
//     block are fetched as soon as those of the present one have been used;
//   * ONCE: the fp32 matrix, which nothing reads before it would have left the cache, passes it (non-temporal).  The bf16 copy then
//     stays there for the forward pass, and the cache holds fewer dirty lines that the next reads have to wait for: AlexNet-style
//     step at 8 / 32 images 395 / 520 -> 362 / 487 us (the copy past the cache as well: 374, 500), three in turn, whose copies the cache
//     does not hold, 399 / 530 -> 394 / 509; VGG-16 at 8 1383 -> 1369.
#include "wap_internal.h"

namespace wap {

namespace {

struct DwArgs {
    const bf16_t* x;   // [B][in]
    const bf16_t* dy;  // [B][out]
    float* dw;         // [out][in], stored here, or
    float* w32;        // ... applied to these
    bf16_t* wb;
    float lr;
    int B, in, out;
    int colb, rowb;    // blocks of CB * 64 columns and of 16 rows
    unsigned units, waves;
};

constexpr unsigned kNowhere = 0x80000000u;  // beyond every buffer here (all below 2 GiB): loads zeros, stores nothing

// NB: blocks of 32 batch rows; CB: blocks of 64 columns of a wavefront
template <int NB, int CB, bool SGD, bool ONCE>
__global__ __launch_bounds__(256, 2) void fc_dw_kernel(const DwArgs a) {
    constexpr int NT = ONCE ? 2 : 0;  // cache policy of the buffer accesses: non-temporal
    const int lane = threadIdx.x & 63, n = lane & 15, kg = lane >> 4;
    const unsigned wave = blockIdx.x * 4 + (unsigned)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    // units [u0, u1), down the rows of one block of columns after the other (side by side, 2 KB of a row to a work-group, 4096 x 4096
    // took 32 instead of 27 us)
    const unsigned u0 = (unsigned)((unsigned long long)a.units * wave / a.waves), u1 = (unsigned)((unsigned long long)a.units * (wave + 1) / a.waves);
    if (u0 >= u1) return;
    const __amdgpu_buffer_rsrc_t rX = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.x), 0, a.B * a.in * 2, 0x00020000);
    const __amdgpu_buffer_rsrc_t rG = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.dy), 0, a.B * a.out * 2, 0x00020000);
    const unsigned nbytes = (unsigned)a.out * (unsigned)a.in * 4u;
    const __amdgpu_buffer_rsrc_t rW = __builtin_amdgcn_make_buffer_rsrc(SGD ? a.w32 : a.dw, 0, (int)nbytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rB = __builtin_amdgcn_make_buffer_rsrc(a.wb, 0, SGD ? (int)(nbytes / 2) : 0, 0x00020000);

    unsigned g16[NB][8];  // eight batch rows of one output feature
    auto load_dy = [&](int rb) {
        const int o = rb * 16 + n;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int r = b * 32 + kg * 8 + j;
                g16[b][j] = __builtin_amdgcn_raw_buffer_load_b16(rG, o < a.out && r < a.B ? (unsigned)(r * a.out + o) * 2u : kNowhere, 0, 0);
            }
    };
    bf16x8 fx[CB][4][NB];
    auto load_x = [&](int cb) {
#pragma unroll
        for (int c = 0; c < CB; ++c)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int col = (cb * CB + c) * 64 + n * 4;
                u32x2 h[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) {
                    const int r = b * 32 + kg * 8 + j;
                    h[j] = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rX, col < a.in && r < a.B ? (unsigned)(r * a.in + col) * 2u : kNowhere, 0, 0));
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    u32x4 v;
#pragma unroll
                    for (int d = 0; d < 4; ++d)
                        v[d] = __builtin_amdgcn_perm(h[2 * d + 1][e >> 1], h[2 * d][e >> 1], (e & 1) ? 0x07060302u : 0x05040100u);
                    fx[c][e][b] = __builtin_bit_cast(bf16x8, v);
                }
            }
    };
    // byte offset of the float4 in row kg * 4 + e of the unit's c-th column block
    auto offset = [&](int cb, int rb, int c, int e) {
        const int o = rb * 16 + kg * 4 + e, col = (cb * CB + c) * 64 + n * 4;
        return o < a.out && col < a.in ? ((unsigned)o * (unsigned)a.in + (unsigned)col) * 4u : kNowhere;
    };
    f32x4 old[CB][4];
    auto load_old = [&](int cb, int rb, int c) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            old[c][e] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rW, offset(cb, rb, c, e), 0, NT));
    };

    int cb = (int)(u0 / (unsigned)a.rowb), rb = (int)(u0 - (unsigned)cb * (unsigned)a.rowb);
    load_x(cb);
    load_dy(rb);
    if (SGD) {
#pragma unroll
        for (int c = 0; c < CB; ++c) load_old(cb, rb, c);
    }
    for (unsigned u = u0; u < u1; ++u) {
        bf16x8 fg[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            u32x4 v;
#pragma unroll
            for (int d = 0; d < 4; ++d) v[d] = g16[b][2 * d] | (g16[b][2 * d + 1] << 16);
            fg[b] = __builtin_bit_cast(bf16x8, v);
        }
        const bool wrap = rb + 1 == a.rowb;
        const int ncb = u + 1 == u1 ? a.colb : wrap ? cb + 1 : cb, nrb = wrap ? 0 : rb + 1;  // (past the end: no column of it exists)
        load_dy(nrb);
#pragma unroll
        for (int c = 0; c < CB; ++c) {
            f32x4 acc[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int b = 0; b < NB; ++b) acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fg[b], fx[c][q][b], acc[q], 0, 0, 0);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const unsigned off = offset(cb, rb, c, e);
                f32x4 v = {acc[0][e], acc[1][e], acc[2][e], acc[3][e]};
                if (SGD) {
                    u32x2 pk;
#pragma unroll
                    for (int t = 0; t < 4; ++t) v[t] = sgd_apply(old[c][e][t], v[t], a.lr);
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        const __bf16 lo = (__bf16)v[2 * t], hi = (__bf16)v[2 * t + 1];
                        pk[t] = (unsigned)__builtin_bit_cast(unsigned short, lo) | ((unsigned)__builtin_bit_cast(unsigned short, hi) << 16);
                    }
                    __builtin_amdgcn_raw_buffer_store_b64(pk, rB, off >> 1, 0, 0);
                }
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), rW, off, 0, NT);
            }
            if (SGD) load_old(ncb, nrb, c);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (ncb != cb && u + 1 < u1) load_x(ncb);
        cb = ncb;
        rb = nrb;
    }
}

template <int NB, int CB>
int launch_dw(DwArgs a, int max_groups, bool once, hipStream_t st) {
    a.colb = (a.in + 64 * CB - 1) / (64 * CB);
    a.rowb = (a.out + 15) / 16;
    a.units = (unsigned)a.colb * (unsigned)a.rowb;
    unsigned groups = (a.units + 7) / 8;  // two units a wavefront
    if (groups > 4u * kNumCU) groups = 4u * kNumCU;
    if (max_groups > 0 && groups > (unsigned)max_groups) groups = (unsigned)max_groups;
    a.waves = groups * 4;
    if (a.w32 && once) hipLaunchKernelGGL((fc_dw_kernel<NB, CB, true, true>), dim3(groups), dim3(256), 0, st, a);
    else if (a.w32) hipLaunchKernelGGL((fc_dw_kernel<NB, CB, true, false>), dim3(groups), dim3(256), 0, st, a);
    else if (once) hipLaunchKernelGGL((fc_dw_kernel<NB, CB, false, true>), dim3(groups), dim3(256), 0, st, a);
    else hipLaunchKernelGGL((fc_dw_kernel<NB, CB, false, false>), dim3(groups), dim3(256), 0, st, a);
    return check_launch("fc_dw");
}

}  // namespace

// Where this is ahead of the tiles of wgrad.hip, stored and with the update, weights cached and from memory (8 800 calls at 1 .. 128 rows,
// geometric mean of the time here over the time there; what is not listed is 1.02 .. 1.3 in one of the four):
//   rows of x that are no whole 16-byte vectors (2052 -> 333), which the tiles load in pieces: 0.2 .. 0.75 at any number of batch rows;
//   up to 32 batch rows: 0.73 .. 0.92, up to 64 M weights of an even shape (25088 -> 4096, stored: 81.4 us here, 77.9 there; with
//     the update 215, 213).  A weight row that is not a whole number of lines is cut into runs that share their first and last line with
//     another wavefront's: from 14 M weights on, beyond what the caches hold together, 1.1 .. 1.3 from memory;
//   33 .. 64 rows: 0.83 .. 1.0 while 64 x 16 weights a unit make one round of work-groups, 0.92 .. 0.99 between 16 and 40 M weights
//     (4096 -> 1000, stored, 1.04, 9216 -> 512 1.12), 0.75 .. 0.98 where an odd number of outputs slows the tiles;
//   65 .. 96 rows: 0.91 .. 0.95 in one round (4096 -> 512 8.3 -> 7.6 us).
// Long rows of few outputs (9216 -> 104) leave the operand of x as the larger part: 1.05 .. 1.1 beyond 32 rows.
// In a step, behind and beside other kernels, the stream is ahead or level for all it was measured on, 4096 -> 1000 to 25088 -> 4096 up to
// 32 rows, to 64 M weights up to 64: stored gradients, tiles / stream, VGG-16 at 1 / 10 / 22 / 32 images 1204 / 1185, 2016 / 2000, 3052 / 3058,
// 3770 / 3755 us, AlexNet-style at 45 / 64 785 / 778, 864 / 856; beside the convolutions the tiles' LDS would keep these off the CUs.
bool fc_dw_supported(const WgradGeom& g, bool in_step) {
    if (g.H != 1 || g.W != 1 || g.P != 1 || g.Q != 1 || g.R != 1 || g.S != 1 || g.ph || g.pw) return false;
    const double weights = (double)g.K * g.C;
    if (g.N > 128 || (g.C % 4) != 0 || weights * 4.0 >= 2147483648.0 || (double)g.N * g.C * 2.0 >= 2147483648.0 || (double)g.N * g.K * 2.0 >= 2147483648.0)
        return false;
    if ((g.C % 8) != 0) return true;
    const bool odd = (g.K % 8) != 0, lines = (g.C % 32) == 0;
    if (in_step && (g.N <= 32 || (g.N <= 64 && weights <= 64e6))) return true;
    if (g.N <= 32) return lines ? odd || weights <= 64e6 : weights <= 14e6;
    const bool one_round = (long)((g.C + 63) / 64) * ((g.K + 15) / 16) <= 8 * kNumCU && g.C <= 8192;
    if (g.N <= 64 && odd) return g.K > 16 && (lines || weights <= 14e6);
    if (g.N <= 64) return lines && (one_round || (weights >= 16e6 && weights <= 40e6));
    return g.N <= 96 && one_round;
}

int launch_fc_dw(const WgradGeom& g, const bf16_t* x, const bf16_t* dy, float* dw, const SgdFuse* sgd, int max_groups, bool once, hipStream_t st) {
    DwArgs a = {x, dy, dw, nullptr, nullptr, 0.f, g.N, g.C, g.K, 0, 0, 0u, 0u};
    if (sgd) {
        a.w32 = sgd->w32;
        a.wb = sgd->wb;
        a.lr = sgd->lr;
    }
    // Beside the convolutions of a step (max_groups: a work-group per CU), one / two of them per CU: AlexNet-style at 32 images 542 / 544 us,
    // VGG-16 at 3 and 8 1062 / 1083, 1499 / 1508; at 64, where a wavefront's loads of x delay its stream, 718 / 700.  (Half of the
    // CUs: 585, 1146, 1588, 714.)
    if (g.N <= 32) return launch_dw<1, 2>(a, max_groups, once, st);
    max_groups *= 2;
    if (g.N <= 64) return launch_dw<2, 2>(a, max_groups, once, st);
    if (g.N <= 96) return launch_dw<3, 1>(a, max_groups, once, st);
    return launch_dw<4, 1>(a, max_groups, once, st);
}

}  // namespace wap
