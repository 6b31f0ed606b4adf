// Fully-connected layers at small minibatches (Section 3.2.2 "primary" nodes; the forward and the data half of the
// backward part of t_c in Eq. 1): y[B][out] = x[B][in] * Wt[out][in]^T and dx[B][in] = dy[B][out] * Wt[out][in].  Both
// are bound by reading Wt once, so the kernels are built as streams of Wt, not as tiles of a product:
//   * Wt goes from memory straight into the MFMA operand registers, never through the LDS: every byte of it is used by
//     one wavefront only.  The batch operand (L2-resident) is loaded beside it in the same layout.
//   * The reduction is divided over the wavefronts of ONE work-group, step by step in turn, so that the work-group as a
//     whole walks contiguous runs of Wt; the partial results meet in the LDS, are added in a fixed order (bitwise
//     reproducible) and leave with bias / ReLU / the ReLU derivative of the layer below applied.  The generic kernel
//     divides it over work-groups: fp32 partial sums through memory and a second launch of 5 .. 7 us.
//   * Every load of the next steps is issued before the products of the present ones, in two register sets.
//   * Row lengths that are no multiple of 8 are read with unaligned loads, the last vector moved back to end with the row.
// Forward (up to 64 rows): a work-group owns 16 output features (v_mfma_f32_16x16x32_bf16, 16 rows of Wt) or fewer, 16 wavefronts.
// Data gradient: the reduction runs over the rows of Wt.  A lane loads CPL neighbouring columns of eight rows and turns
// the 8 x CPL block around in registers (byte permutes); a work-group owns 16 * CPL columns, 8 wavefronts.
#include <algorithm>

#include "wap_internal.h"

namespace wap {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4_t;

struct FcArgs {
    const bf16_t* act;   // x [B][in] (forward) or dy [B][out] (data gradient)
    const bf16_t* w;     // [out][in]
    const float* bias;   // forward
    const bf16_t* mask;  // data gradient: dx = mask > 0 ? dx : 0
    void* res;           // bf16 result, or fp32 partial sums [split][B][out]
    int B, in, out;
    int relu, partial, steps_per_split;
    int feat;            // forward: output features of a work-group
    float* colsum;       // data gradient: optional, [in] column sums of the (masked) result
};

__device__ __forceinline__ unsigned short f2bf(float f) {
    __bf16 b = (__bf16)f;  // round to nearest even
    return __builtin_bit_cast(unsigned short, b);
}

__device__ __forceinline__ int xcd_remap(int bid, int total) {
    int per = total / kNumXCD, rem = total % kNumXCD;
    int xcd = bid % kNumXCD, idx = bid / kNumXCD;
    return xcd < rem ? xcd * (per + 1) + idx : rem * (per + 1) + (xcd - rem) * per + idx;
}

constexpr unsigned kNowhere = 0x80000000u;  // beyond every buffer here (all below 2 GiB): loads zeros

__device__ __forceinline__ bf16x8 ldb128(__amdgpu_buffer_rsrc_t r, unsigned off) {
    return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}

constexpr int FW_WAVES = 16;

// VEC8: rows are 16-byte aligned (in % 8 == 0); NB: blocks of 16 batch rows
template <bool VEC8, int NB>
__global__ __launch_bounds__(64 * FW_WAVES) void fc_fwd_kernel(const FcArgs a) {
    constexpr int U = NB == 1 ? 4 : 2;  // 32-deep steps per register set
    __shared__ f32x4_t red[NB][FW_WAVES][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int row = lane & 15, kg = lane >> 4;
    const int o0 = blockIdx.x * a.feat;
    const int orows = a.out - o0 < a.feat ? a.out - o0 : a.feat;
    const __amdgpu_buffer_rsrc_t rW = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(a.w + (size_t)o0 * a.in), 0, orows * a.in * 2, 0x00020000);
    const __amdgpu_buffer_rsrc_t rX =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.act), 0, a.B * a.in * 2, 0x00020000);
    const unsigned off = (unsigned)row * (unsigned)a.in * 2u;  // rows beyond the matrix lie beyond its buffer
    const int first = blockIdx.y * a.steps_per_split;
    const int steps = (a.in + 31) / 32;
    const int last = first + a.steps_per_split < steps ? first + a.steps_per_split : steps;

    // Two neighbouring steps of a row in turn, so that a wavefront reads whole 128-byte lines (one step is half a line, and the
    // other half went to the next wavefront).  us, one step / two, weights from memory: 1, 8 and 16 rows x 9216 -> 4096 17.5, 20.2,
    // 24.2 / 16.4, 18.2, 21.1; 4096 -> 4096 9.7, 10.7, 12.4 / 9.2, 9.9, 10.8; 6 x 25088 -> 4096 46.2 / 40.0.  Cached ones 1 to 2 %, short or
    // unaligned rows the same.
    auto step_of = [](int u) { return u / 2 * 2 * FW_WAVES + u % 2; };
    bf16x8 fw[2][U], fx[2][U][NB];
    auto load = [&](int set, int st) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = st + step_of(u);
            int k = s * 32 + kg * 8;
            const bool ok = s < last && k < a.in;
            if (!VEC8 && k > a.in - 8) k = a.in - 8;  // the row's last vector, moved back to end with the row
            fw[set][u] = ldb128(rW, ok ? off + (unsigned)k * 2u : kNowhere);
#pragma unroll
            for (int b = 0; b < NB; ++b) fx[set][u][b] = ldb128(rX, ok ? off + (unsigned)(b * 16 * a.in + k) * 2u : kNowhere);
        }
    };
    f32x4_t acc[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto mul = [&](int set, int st) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (!VEC8) {  // a vector that was moved back repeats elements of its neighbour: zeros on both sides, for a
                          // zero activation does not cancel an infinite weight
                const int k = (st + step_of(u)) * 32 + kg * 8;
#pragma unroll
                for (int e = 0; e < 7; ++e)
                    if (e < k - (a.in - 8)) {
                        fw[set][u][e] = (__bf16)0.f;
#pragma unroll
                        for (int b = 0; b < NB; ++b) fx[set][u][b][e] = (__bf16)0.f;
                    }
            }
#pragma unroll
            for (int b = 0; b < NB; ++b) acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fw[set][u], fx[set][u][b], acc[b], 0, 0, 0);
        }
    };
    constexpr int STRIDE = U * FW_WAVES;
    int st = first + 2 * wave;
    load(0, st);
    while (true) {
        load(1, st + STRIDE);
        __builtin_amdgcn_sched_barrier(0);  // the scheduler would move the loads down to their uses
        mul(0, st);
        st += STRIDE;
        if (st >= last) break;  // uniform in the wavefront; a set loaded beyond the range holds zeros and is dropped
        load(0, st + STRIDE);
        __builtin_amdgcn_sched_barrier(0);
        mul(1, st);
        st += STRIDE;
        if (st >= last) break;
    }

    // lane: batch row lane & 15 of the block, output features (lane >> 4) * 4 .. + 3; wavefront b adds up block b
#pragma unroll
    for (int b = 0; b < NB; ++b) red[b][wave][lane] = acc[b];
    __syncthreads();
    if (wave >= NB) return;
    f32x4_t s = red[wave][0][lane];
#pragma unroll
    for (int w = 1; w < FW_WAVES; ++w) s += red[wave][w][lane];
    const int o = o0 + kg * 4, bi = wave * 16 + row;
    if (bi >= a.B) return;
    const size_t e0 = (size_t)bi * a.out + o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if (o + e >= o0 + orows) continue;
        if (a.partial) {
            reinterpret_cast<float*>(a.res)[(size_t)blockIdx.y * a.B * a.out + e0 + e] = s[e];
        } else {
            float v = a.bias ? s[e] + a.bias[o + e] : s[e];
            if (a.relu) v = v > 0.f ? v : 0.f;
            reinterpret_cast<bf16_t*>(a.res)[e0 + e] = f2bf(v);
        }
    }
}

constexpr int DX_WAVES = 8;

// NB: blocks of 16 batch rows; CPL: columns of Wt per lane (a work-group owns 16 * CPL); VEC8: out % 8 == 0; SUM: column sums as well (as a flag of
// the launch they cost those without them 0.25 us: 96 x 500 -> 4096 7.50 / 7.76)
template <int NB, int CPL, bool VEC8, bool SUM>
__global__ __launch_bounds__(64 * DX_WAVES) void fc_dx_kernel(const FcArgs a) {
    constexpr int U = NB * CPL <= 4 ? 2 : 1;  // 32-deep steps per register set
    __shared__ f32x4_t red[DX_WAVES][CPL][64];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int il = lane & 15, og = lane >> 4;
    // neighbours in memory share an L2; the last work-group is moved back to end with the row (it repeats columns of its
    // neighbour, bit for bit)
    int i0 = xcd_remap(blockIdx.x, gridDim.x) * 16 * CPL;
    if (i0 > a.in - 16 * CPL) i0 = a.in - 16 * CPL;
    const int col = i0 + il * CPL;
    const __amdgpu_buffer_rsrc_t rW =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.w), 0, (int)((unsigned)a.out * (unsigned)a.in * 2u), 0x00020000);
    const __amdgpu_buffer_rsrc_t rG =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.act), 0, a.B * a.out * 2, 0x00020000);
    const unsigned rowb = (unsigned)a.in * 2u;
    const int steps = (a.out + 31) / 32;

    unsigned fw[2][U][8][CPL / 2];  // eight rows of Wt, CPL columns
    bf16x8 fg[2][U][NB];
    auto load1 = [&](int set, int u, int s) {
        const int o = s * 32 + og * 8;
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int bi = b * 16 + il;
            const int oo = !VEC8 && o > a.out - 8 ? a.out - 8 : o;  // the row's last vector, moved back to end with the row
            fg[set][u][b] = ldb128(rG, o < a.out && bi < a.B ? (unsigned)(bi * a.out + oo) * 2u : kNowhere);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const unsigned off = o + j < a.out ? (unsigned)(o + j) * rowb + (unsigned)col * 2u : kNowhere;
            if (CPL == 4) {
                const u32x2 v = __builtin_bit_cast(u32x2, __builtin_amdgcn_raw_buffer_load_b64(rW, off, 0, 0));
                fw[set][u][j][0] = v[0];
                fw[set][u][j][CPL / 2 - 1] = v[1];
            } else {
                fw[set][u][j][0] = __builtin_amdgcn_raw_buffer_load_b32(rW, off, 0, 0);
            }
        }
    };
    auto load = [&](int set, int s) {
#pragma unroll
        for (int u = 0; u < U; ++u) load1(set, u, s + u * DX_WAVES);
    };
    f32x4_t acc[CPL][NB];
#pragma unroll
    for (int c = 0; c < CPL; ++c)
#pragma unroll
        for (int b = 0; b < NB; ++b) acc[c][b] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    auto mul1 = [&](int set, int u, int s) {
        if (!VEC8) {  // a vector that was moved back: its elements d, d + 1, ... to the front, zeros behind
            const int d = s * 32 + og * 8 - (a.out - 8);
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                u32x4 v = __builtin_bit_cast(u32x4, fg[set][u][b]);
                if (d & 4) v = u32x4{v[2], v[3], 0u, 0u};
                if (d & 2) v = u32x4{v[1], v[2], v[3], 0u};
                if (d & 1) v = u32x4{(v[0] >> 16) | (v[1] << 16), (v[1] >> 16) | (v[2] << 16), (v[2] >> 16) | (v[3] << 16), v[3] >> 16};
                if (d > 0) fg[set][u][b] = __builtin_bit_cast(bf16x8, v);
            }
        }
#pragma unroll
        for (int c = 0; c < CPL; ++c) {
            u32x4 v;  // column c of the eight rows
#pragma unroll
            for (int d = 0; d < 4; ++d)
                v[d] = __builtin_amdgcn_perm(fw[set][u][2 * d + 1][c >> 1], fw[set][u][2 * d][c >> 1],
                                             (c & 1) ? 0x07060302u : 0x05040100u);
            const bf16x8 wv = __builtin_bit_cast(bf16x8, v);
#pragma unroll
            for (int b = 0; b < NB; ++b)
                acc[c][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv, fg[set][u][b], acc[c][b], 0, 0, 0);
        }
    };
    auto mul = [&](int set, int s) {
#pragma unroll
        for (int u = 0; u < U; ++u) mul1(set, u, s + u * DX_WAVES);
    };
    constexpr int STRIDE = U * DX_WAVES;
    int st = wave;
    load(0, st);
    while (true) {
        load(1, st + STRIDE);
        __builtin_amdgcn_sched_barrier(0);
        mul(0, st);
        st += STRIDE;
        if (st >= steps) break;
        load(0, st + STRIDE);
        __builtin_amdgcn_sched_barrier(0);
        mul(1, st);
        st += STRIDE;
        if (st >= steps) break;
    }

    float cs[4] = {0.f, 0.f, 0.f, 0.f};
    // lane: batch row lane & 15; accumulator element e of column block c is column ((lane >> 4) * 4 + e) * CPL + c, so a
    // lane holds 4 * CPL neighbouring columns, staged as CPL groups of four
#pragma unroll
    for (int b = 0; b < NB; ++b) {
#pragma unroll
        for (int h = 0; h < CPL; ++h) {
            f32x4_t v;
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] = acc[(h * 4 + t) % CPL][b][(h * 4 + t) / CPL];
            red[wave][h][lane] = v;
        }
        __syncthreads();
        if (tid < 64 * CPL) {
            const int h = tid >> 6;
            f32x4_t s = red[0][h][lane];
#pragma unroll
            for (int w = 1; w < DX_WAVES; ++w) s += red[w][h][lane];
            const int bi = b * 16 + il, i = i0 + og * 4 * CPL + h * 4;
            if (bi < a.B) {
                const size_t e = (size_t)bi * a.in + i;
                if (a.mask) {
                    u32x2 m;
                    __builtin_memcpy(&m, a.mask + e, 8);  // rows need not be 8-byte aligned
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        const float y = __uint_as_float((t & 1) ? m[t >> 1] & 0xffff0000u : m[t >> 1] << 16);
                        s[t] = y > 0.f ? s[t] : 0.f;
                    }
                }
                u32x2 pk = {(unsigned)f2bf(s[0]) | ((unsigned)f2bf(s[1]) << 16),
                            (unsigned)f2bf(s[2]) | ((unsigned)f2bf(s[3]) << 16)};
                __builtin_memcpy(reinterpret_cast<bf16_t*>(a.res) + e, &pk, 8);
#pragma unroll
                for (int t = 0; SUM && t < 4; ++t) cs[t] += __uint_as_float((t & 1) ? pk[t >> 1] & 0xffff0000u : pk[t >> 1] << 16);
            }
        }
        __syncthreads();
    }
    // the work-group has all rows of its columns: their sums are the bias gradient of the layer below
    if (SUM && tid < 64 * CPL) {
#pragma unroll
        for (int o = 1; o < 16; o <<= 1)
#pragma unroll
            for (int t = 0; t < 4; ++t) cs[t] += __shfl_xor(cs[t], o, 64);
        if (il == 0) __builtin_memcpy(a.colsum + i0 + og * 4 * CPL + (tid >> 6) * 4, cs, 16);
    }
}

// a fully-connected product: one pixel per image, one tap
bool is_fc(const GemmGeom& g) {
    return g.IH == 1 && g.IW == 1 && g.OH == 1 && g.OW == 1 && g.R == 1 && g.S == 1 && g.pad_h == 0 && g.pad_w == 0;
}
bool below_2g(double elems) { return elems * 2.0 < 2147483648.0; }

}  // namespace

// Every work-group reads the whole batch operand, through an L2 path that carries about 8.6 TB/s: with one block of 16
// rows that is as much traffic as Wt itself, with more it outweighs Wt, and the generic kernel's tiles (64 x 256, split
// reduction) are faster.  Up to 4096 features, one work-group per CU, this kernel is ahead (9216 -> 4096 at 8 rows 17.2
// us against 21.6; 4096 -> 1000 8.6 against 12.2) until the long rows of Wt outlast what the generic one spends on its
// second launch: 25088 -> 4096 at 2 / 8 / 16 rows 32.9 / 38.9 / 47.0 against 39.4, 16384 -> 4096 26.6 / 28.9 / 33.2 against
// 28.  Beyond that it runs in rounds of work-groups, each with a start of 3 us, which pays only while the reduction is long
// enough to be split there and short enough here: 64 -> 25088 17 against 4.5, 64 -> 6000 6.2 against 4.4, 512 -> 8192 7.1
// against 8.7, 2048 -> 8192 10.4 against 11.4, 4096 -> 9216 23.3 against 19.4.  Rows that are no multiple of 64, which
// the generic kernel loads more slowly, move that line: 600 -> 10000 8.7 against 10.1, 1000 -> 25088 20.0 against 19.6.
//
// 17 .. 64 rows: a wavefront multiplies its operand of Wt with two or four blocks of rows.  The batch operand is then most of what a
// work-group reads, so this is ahead while Wt is small or short (us, tiles of the generic kernel / this, Wt from memory: 32 rows, 4096 -> 1000
// 12.3 / 8.7, 9216 -> 512 14.6 / 10.5, 1000 -> 2000 9.8 / 5.3, 17 x 4096 -> 4096 14.8 / 12.1; 64 rows, 4096 -> 512 11.3 / 9.4) and far behind
// where it is large (32 x 9216 -> 4096 21.6 / 31.9, 64 x 25088 -> 4096 46 / 128).  The line is drawn by the two predictions: this kernel's
// (fc_fwd_plan), and the generic one's, fitted to 253 shapes of 17 .. 64 rows, 200 .. 25000 inputs and 64 .. 12000 outputs, cached and from memory
// (rms error 12 %): 175 of them come here, all shapes take 0.75 of their time (geometric mean; 0.74 with the better kernel for each) and
// only unaligned rows of a large Wt were slower (28 x 4387 -> 9504 91 instead of 52): these stay.  Steps, AlexNet-style at 32 and VGG-16 at
// 22 images, 512.4 / 508.3 and 2783.5 / 2780.4.
static double us_generic_rows(const GemmGeom& g) {
    const double k = g.IC, mb = 2e-6 * k * g.Ncols;
    return 7.6 + 0.13 * mb + 0.39e-3 * std::min(k, 16384.0) + 0.024 * g.M + ((g.IC % 64) == 0 ? 0.0 : 0.46 + 0.03 * mb) +
           ((g.IC % 8) != 0 || (g.Ncols % 4) != 0 ? 2.0 : 0.0) + ((g.IC % 8) != 0 ? 0.33 * mb : 0.0);
}
bool fc_fwd_supported(const GemmGeom& g, bool in_step, bool lean) {
    if (!is_fc(g) || g.M > 64 || g.IC < 8 || !below_2g((double)g.M * g.IC) || !below_2g(16.0 * g.IC)) return false;
    const bool quick = (g.IC % 64) == 0;  // the generic kernel's fast mode
    if (g.M > 16) {
        if ((g.IC % 8) != 0 && 2e-6 * g.IC * g.Ncols > 40.0) return false;
        int feat, nsplit;
        return fc_fwd_plan(g, lean, &feat, &nsplit) < 0.95 * us_generic_rows(g) + (in_step ? 2.0 : 0.0);  // (a step's next kernel waits for the second launch)
    }
    if (g.Ncols <= 4096) return !quick || g.M <= 6 || (double)g.IC * g.Ncols <= 50e6;
    return quick ? g.Ncols <= 8192 && g.IC >= 256 && g.IC <= 2048 : 25.0 * g.IC >= g.Ncols;
}
// Odd row lengths: a lane's 16 bytes begin between two dwords in every other row, and 512 of a row take 0.06 more for every batch row (rows of
// even length, also where they are no whole vectors, take what fc_fwd_plan says).  us, generic kernel / stream, Wt cached: 47 x 4789 -> 4096
// 28.7 / 49.2, 38 x 2013 -> 500 12.2 / 17.5, 64 x 6133 -> 1000 17.1 / 25.3; 43 x 7011 -> 512 17.4 / 15.6, 61 x 325 -> 174 13.4 / 7.8.  The generic kernel
// is behind its line, too, while the rows are short or few.  Of 981 timings with odd rows, cached and from memory, 799 stay here, at 0.64 of
// the generic kernel's time (6 of them more than 5 % slower, by 1.22 at most), and the other 182 took 1.14 of it.
bool fc_fwd_odd_rows_slow(const GemmGeom& g, bool lean) {
    if (g.M <= 16 || (g.IC & 1) == 0) return false;
    int feat, nsplit;
    const double us = fc_fwd_plan(g, lean, &feat, &nsplit);
    const long rounds = ((long)((g.Ncols + feat - 1) / feat) * nsplit + kNumCU - 1) / kNumCU;
    const bool behind = g.IC >= 256 && ((g.IC < 3000 && g.Ncols < 2000) || g.Ncols < 128);
    return us + 0.06 * g.M * rounds * (g.IC / 512.0 / nsplit) >= 0.95 * (us_generic_rows(g) + (behind ? 2.5 : 0.0));
}
// The same for the data gradient, whose work-groups share the batch operand among 64 (or 32) columns: up to 32 rows, and
// where the reduction is short (both kernels wait more than they stream) up to 128.  A work-group walks all rows of Wt with
// eight wavefronts, so few columns or many rows of Wt leave it waiting, most of all when Wt comes from memory and not
// from the 256 MB cache.  This kernel / the generic one in us, Wt cached (from memory), at 8 / 16 / 32 batch rows:
//   4096 rows of Wt x  4096 columns  10.9 / 12.1 / 15.4 (18.4 / 19.7 / 23.4)   14.3 / 15.5 / 16.7 (17.1 / 16.9 / 17.9)
//                      9216          15.6 / 16.5 / 18.9 (25.5 / 27.1 / 30.3)   21.1 / 21.3 / 22.7 (25.2 / 25.4 / 26.6)
//                     25088          35.0 / 36.7 / 40.2 (50.4 / 53.4 / 60.4)   44.6 / 45.1 / 46.5 (58.9 / 60.5 / 62.0)
//   8192             x   512         10.8 / 13.0 / 20.1 (19.7 / 22.0 / 27.6)   17.7 / 17.8 / 18.5 (18.2 / 18.4 / 19.1)
//                      8192          26.9 / 28.4 / 32.7 (43.4 / 46.4 / 52.2)   28.7 / 28.7 / 29.8 (34.3 / 34.2 / 35.6)
//  25088             x   512         28.1 / 41.8 / 82.9 (93 / 105 / 127)       27.9 / 28.3 / 28.0 (30.3 / 30.7 / 30.2)
//   1000             x  4096         4.0 / 3.9 / 4.6 (4.8 / 5.1 / 6.0)         10.2 / 10.6 / 11.4 (11.1 / 11.2 / 12.0)
//                      at 64 / 100 / 128 rows 5.9 / 9.6 / 10.1                 13.7 / 16.0 / 18.2
//   1024             x   512         at 64 / 100 / 128 rows 7.1 / 10.7 / 12.1  11.4 / 10.7 / 11.2
// The lines are drawn where the two times' geometric mean (cached, from memory) crosses.  The generic kernel is slower
// where it cannot load whole 64-channel slices (10000 x 9216 at 16 rows 36.7 against 70) and more so with odd rows
// (8192 x 4551 24 against 70), and the lines lie further out there.
bool fc_dx_supported(const GemmGeom& g) {
    if (!is_fc(g) || g.M > 128 || g.Ncols < 64 || g.IC < 8 || !below_2g((double)g.IC * g.Ncols) || !below_2g((double)g.M * g.IC))
        return false;
    const bool odd = (g.IC % 8) != 0 || (g.Ncols % 8) != 0, quick = !odd && (g.IC % 64) == 0;
    if (g.M > 32)
        return g.IC <= 1024 && (g.M <= 64 || g.Ncols <= 8192) && (!quick || g.M <= 80 || g.IC <= 768 || g.Ncols > 1024);
    if (odd) return g.IC <= 4096 || g.Ncols >= 2048 || (g.IC <= 8192 && g.M <= 16);
    if (!quick)
        return g.IC <= 4096 || (g.IC <= 12288 && g.Ncols >= 6144) || (g.IC <= 6144 && (g.M <= 16 || g.Ncols <= 1024));
    if (g.IC <= 4096) return g.M <= 16 || g.IC <= 2048 || g.Ncols <= 2048 || g.Ncols >= 9216;
    return g.IC <= 8192 && (g.Ncols >= 12288 || (g.M <= 16 && g.Ncols <= 512));
}

// How many output features a work-group owns (16, 8 or 4: the rows of the MFMA beyond them are zeros that no load is made for) and over
// how many work-groups the reduction is divided as well.  A work-group is bound by its CU's way to the L2: it starts in 3.5 us, and
// every 512-deep step of its 16 wavefronts takes 0.19 and 0.021 more for every row of Wt or of the batch (within 6 % of 13 shapes, 1 to
// 16 rows); a launch that adds up partial sums takes 2.3.  More work-groups than CUs run one after another.  us at 1 / 8 / 16 rows, weights from
// memory, 16 features and a division by 128 KB of Wt / this: 4096 -> 1000 7.7 / 9.1 / 10.3, 6.2 / 7.4 / 8.0; 9216 -> 512 10.4 / 11.8 / 13.3, 7.4 /
// 8.0 / 8.7; 11264 -> 609 11.5 / 13.3 / 15.0, 8.5 / 9.2 / 9.9.
// lean: divided only so far that a work-group of 16 features streams 128 KB of Wt and the work-groups are no more than the CUs; with more than 16
// rows not at all, for calls of that kind that needed no workspace take none.  More than 16 rows: half as many steps in flight, and a sum of
// twice or four times as many partial results (fitted to the 253 shapes above).  Returns the predicted us.
double fc_fwd_plan(const GemmGeom& g, bool lean, int* feat, int* nsplit) {
    const bool rows = g.M > 16;
    const double start = rows ? 4.2 : 3.5, step = rows ? 0.25 : 0.19, sum = rows ? 3.3 : 2.3;
    const int steps = (g.IC + 16 * 2 * FW_WAVES - 1) / (16 * 2 * FW_WAVES);
    const int most = lean && rows ? 1 : lean ? std::max(1, std::min(kNumCU / ((g.Ncols + 15) / 16), g.IC / 4096)) : 16;
    double least = 0, whole = 0;  // whole: 16 features, undivided; a gain on it of less than 0.4 is none
    for (int f : {16, 8, 4})
        for (int n = 1; n <= most && n <= steps; ++n) {
            const long groups = (long)((g.Ncols + f - 1) / f) * n;
            if ((f < 16 || n > 1) && groups > kNumCU) break;
            const long rounds = (groups + kNumCU - 1) / kNumCU;
            const double us = start * rounds + (rows ? rounds : 1) * ((steps + n - 1) / n) * (step + 0.021 * (f + g.M)) + (n > 1 ? sum + 0.05 * n : 0.0);
            if (least == 0 || (us < 0.97 * least && us < whole - 0.4)) {
                if (least == 0) whole = us;
                least = us;
                *feat = f;
                *nsplit = n;
            }
        }
    return least;
}

// The plan of 17 to 64 rows that needs no workspace, whatever the generic product takes; false where the stream cannot run.
bool fc_fwd_whole(const GemmGeom& g, GemmPlan* p) {
    if (!is_fc(g) || g.M <= 16 || g.M > 64 || g.IC < 8 || !below_2g((double)g.M * g.IC) || !below_2g(16.0 * g.IC)) return false;
    p->cfg = 10;
    p->ws_bytes = 0;
    fc_fwd_plan(g, true, &p->tile, &p->nsplit);
    return true;
}

namespace {
template <int NB>
int launch_fwd(const FcArgs& a, dim3 grid, hipStream_t st) {
    if ((a.in % 8) == 0) hipLaunchKernelGGL((fc_fwd_kernel<true, NB>), grid, dim3(64 * FW_WAVES), 0, st, a);
    else hipLaunchKernelGGL((fc_fwd_kernel<false, NB>), grid, dim3(64 * FW_WAVES), 0, st, a);
    return check_launch("fc_fwd");
}
}  // namespace

int launch_fc_fwd(const GemmGeom& g, int nsplit, int feat, const bf16_t* x, const bf16_t* w, const float* bias, bool relu, void* out,
                  hipStream_t st) {
    FcArgs a = {x, w, bias, nullptr, out, g.M, g.IC, g.Ncols, relu ? 1 : 0, nsplit > 1 ? 1 : 0, 0, feat, nullptr};
    a.steps_per_split = ((g.IC + 31) / 32 + nsplit - 1) / nsplit;
    const dim3 grid((g.Ncols + a.feat - 1) / a.feat, nsplit);
    if (g.M <= 16) return launch_fwd<1>(a, grid, st);
    if (g.M <= 32) return launch_fwd<2>(a, grid, st);
    return launch_fwd<4>(a, grid, st);
}

namespace {
template <int CPL, bool VEC8, bool SUM = false>
int launch_dx(const FcArgs& a, hipStream_t st) {
    const dim3 grid((a.in + 16 * CPL - 1) / (16 * CPL)), block(64 * DX_WAVES);
    if (a.B <= 16) hipLaunchKernelGGL((fc_dx_kernel<1, CPL, VEC8, SUM>), grid, block, 0, st, a);
    else if (a.B <= 32) hipLaunchKernelGGL((fc_dx_kernel<2, CPL, VEC8, SUM>), grid, block, 0, st, a);
    else if (a.B <= 64) hipLaunchKernelGGL((fc_dx_kernel<4, CPL, VEC8, SUM>), grid, block, 0, st, a);
    else if constexpr (CPL == 2) hipLaunchKernelGGL((fc_dx_kernel<8, 2, VEC8, SUM>), grid, block, 0, st, a);
    else return set_error(WAP_EINVAL, "internal: more than 64 batch rows need two columns per lane");
    return check_launch("fc_dx");
}
}  // namespace

bool fc_dx_sums(const GemmGeom& g) { return (g.IC % 8) == 0 && (g.Ncols % 64) == 0; }  // whole work-groups of columns

// Four columns per lane read whole 128-byte lines of a row.  Where that gives fewer than 96 work-groups (4096 columns at
// 8 rows: 12.7 us), or the sums of more than 64 batch rows would not fit the registers, two columns per lane (10.7 us;
// the other half of the line comes from the L2).  9216 columns: 15.2 us with four, 22.4 us with two.
int launch_fc_dx(const GemmGeom& g, const bf16_t* dy, const bf16_t* w, const bf16_t* mask, bf16_t* dx, float* colsum, hipStream_t st) {
    const FcArgs a = {dy, w, nullptr, mask, dx, g.M, g.Ncols, g.IC, 0, 0, 0, 0, colsum};
    const bool wide = g.Ncols >= 96 * 64 && g.M <= 64, vec8 = (g.IC % 8) == 0;
    if (colsum) {
        if (!fc_dx_sums(g)) return set_error(WAP_EINVAL, "internal: no column sums from this fully-connected data gradient");
        return wide ? launch_dx<4, true, true>(a, st) : launch_dx<2, true, true>(a, st);
    }
    if (wide) return vec8 ? launch_dx<4, true>(a, st) : launch_dx<4, false>(a, st);
    return vec8 ? launch_dx<2, true>(a, st) : launch_dx<2, false>(a, st);
}

}  // namespace wap
