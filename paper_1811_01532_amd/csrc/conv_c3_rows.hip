// First layer of the AlexNet-style network: 11x11 filter at stride 4, three input channels (gfx950), forward.
//
// As in conv_c3.hip the input rows lie in LDS, but with every 4 x 4 pixels together (96 bytes, in a slot of 112): with the filter
// padded to 12x12 by zero weights the layer is a 3x3 one at stride 1 of 48 channels, and the operand of a pixel is 16 aligned
// bytes in slots that 16 neighbouring pixels find in different banks.  (As rows of pixels, 24 bytes from one to the next, the
// operand took two 8-byte reads: the LDS was busy for 71 % of the time, the matrix pipes for 37, 256 images 71 us; this 65.)
// What a work-group does one thing after the other is cut down:
//   * it takes G neighbouring output rows of an image at a time, whose 4 G + 7 input rows overlap: one pass through memory, LDS and
//     barrier for all of them, the rows of the next group on their way meanwhile;
//   * weights pass through the LDS a filter row a thread (element by element a work-group started 8 us later; gathered from
//     memory by unaligned 16-byte loads 7 us later);
//   * an output tile leaves through LDS of the wavefront's own: the rows are all that the work-group waits for.
// 224 x 224 -> 64 channels, us at 1 / 8 / 32 / 100 / 256 images, the kernels that had them before (conv_thin.hip to 8, an output row with all
// its input rows at a time beyond) and this: 15.2 / 18.6 / 30.0 / 53 / 101, 8.2 / 11.5 / 19.2 / 35 / 65; the output alone takes 20 at 256.
// The twelfth row and column of a window are masked out of the operand: the zero weights alone would make a NaN of an infinity there
// (256 images 61 -> 65 us, 32 18.9 -> 19.2).  Wavefront: one block of 32 output channels, its weights in
// registers for the whole kernel, and every second of the (row, 32 pixels) tiles.
#include "wap_internal.h"

namespace wap {

namespace {

constexpr int NT = 256;
constexpr int R = 11, S3 = 33, ST = 4;    // filter rows, elements of one, stride
constexpr int KS = 27;                    // reduction steps: 3 x 3 blocks of 48 elements
constexpr int BP = 112, BRP = 66 * BP;    // LDS bytes of a block of 4 x 4 pixels, of a row of them (64 output pixels and two more)
constexpr int OP = 32 * 2 + 16;           // ... of a pixel of a wavefront's output tile
constexpr int WRP = 72;                    // ... of a filter row of the weights
constexpr int MAX_VECS = 87;              // 16-byte vectors of an input row with its left border (228 pixels)

struct RowsArgs {
    const bf16_t* x;
    const bf16_t* w;
    const float* bias;
    bf16_t* y;
    int N, H, W3, OH, OW, K, ph, pw, relu;
    int groups, units, nvx;  // row groups of an image, of all images; vectors of an input row
    unsigned x_bytes;
    FastDiv dGroups, dNVX;
};

__device__ __forceinline__ unsigned short f2bf(float f) {
    __bf16 b = (__bf16)f;
    return __builtin_bit_cast(unsigned short, b);
}

// Elements e and e + 1 of a block of 4 x 4 taps at reduction step ks: ones where the tap is one of the filter's 11 x 11.
__device__ constexpr unsigned pair_mask(int ks, int e) {
    const int r = ks / 9 * 4, s = ks / 3 % 3 * 4;  // the block's first tap
    const bool lo = r + e / 12 < R && s + e % 12 / 3 < R, hi = r + (e + 1) / 12 < R && s + (e + 1) % 12 / 3 < R;
    return (lo ? 0xffffu : 0u) | (hi ? 0xffff0000u : 0u);
}
constexpr int rows_of(int g) { return (g - 1) * ST + R; }
// the rows, the output tiles and the bias, or before them the weights
constexpr size_t smem_of(int fb, int g) {
    const size_t rows = (size_t)(g + 2) * BRP + 4 * 32 * OP + 256, weights = (size_t)fb * 32 * R * WRP;
    return rows > weights ? rows : weights;
}

// FB: 32-channel blocks; G: output rows of a group
template <int FB, int G>
__global__ __launch_bounds__(NT, 2) void conv_c3_fwd_strided_kernel(const RowsArgs a) {
    constexpr int NR = rows_of(G);
    constexpr int XV = (NR * MAX_VECS + NT - 1) / NT;
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, l32 = lane & 31;
    const int b = wave % FB, wi = wave / FB;
    const __amdgpu_buffer_rsrc_t rX = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(a.x), 0, (int)a.x_bytes, 0x00020000);
    constexpr unsigned OOB = 0x80000000u;

    // ---- this thread's vectors of a group of rows, the same for all groups: vector j of a row covers dwords 4 j .. of the row behind
    // its left border.  One that sticks out of the row is loaded from inside and shifted (vshift: dwords up, negative: down) ----
    int vrow[XV], vsrc[XV], vshift[XV];
    unsigned vdst[XV];  // where its two halves go: eight bytes are two thirds of a pixel row of a block
    const int border = a.pw * 3 / 2, rowd = a.W3 / 2;  // dwords
#pragma unroll
    for (int i = 0; i < XV; ++i) {
        const int v = tid + i * NT;
        const int r = (int)fdiv((uint32_t)v, a.dNVX), j = v - r * a.nvx;
        const int d = 4 * j - border;
        const int up = d < 0 ? -d : 0, down = d + 4 > rowd ? d + 4 - rowd : 0;
        const bool some = r < NR && up < 4 && down < 4;
        vrow[i] = some ? r : 1 << 20;  // none: outside every image
        vshift[i] = up - down;
        vsrc[i] = (r * rowd + d + up - down) * 4;
        const int base = (r >> 2) * BRP + (r & 3) * 24;
        const int h0 = 2 * j, h1 = 2 * j + 1;
        vdst[i] = some ? (unsigned)(base + h0 / 3 * BP + h0 % 3 * 8) | ((unsigned)(base + h1 / 3 * BP + h1 % 3 * 8) << 16) : 0xffffffffu;
    }
    u32x4 rx[XV];
    auto load_rows = [&](int u) {  // (of a group past the last one: nothing)
        const int n = (int)fdiv((uint32_t)u, a.dGroups), g = u - n * a.groups;
        const int ih0 = g * (G * ST) - a.ph;
        const int base = (n * a.H + ih0) * a.W3 * 2;
#pragma unroll
        for (int i = 0; i < XV; ++i) {
            const bool ok = (unsigned)(ih0 + vrow[i]) < (unsigned)a.H && u < a.units;
            rx[i] = __builtin_amdgcn_raw_buffer_load_b128(rX, ok ? (unsigned)(base + vsrc[i]) : OOB, 0, 0);
        }
    };
    load_rows(blockIdx.x);

    // ---- weights: a filter row a thread into the LDS, where the next one starts 8-byte aligned, then four elements at a time ----
    for (int i = tid; i < FB * 32 * R; i += NT) {
        u32x4 t[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) t[k] = load8_unaligned(a.w + i * S3 + k * 8);
        const unsigned last = a.w[i * S3 + 32];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            *reinterpret_cast<u32x2*>(smem + i * WRP + k * 16) = u32x2{t[k][0], t[k][1]};
            *reinterpret_cast<u32x2*>(smem + i * WRP + k * 16 + 8) = u32x2{t[k][2], t[k][3]};
        }
        *reinterpret_cast<u32x2*>(smem + i * WRP + 64) = u32x2{last, 0u};
    }
    __syncthreads();
    bf16x8 wf[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const int tap = ks / 3, sub = ks % 3;  // block of 4 x 4 taps, 16 of its 48 elements
        u32x4 v;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int e = sub * 16 + half * 8 + q * 4, r = tap / 3 * 4 + e / 12, j = tap % 3 * 12 + e % 12;  // elements j .. j + 3 of filter row r
            u32x2 t = *reinterpret_cast<const u32x2*>(smem + ((b * 32 + l32) * R + (r < R ? r : R - 1)) * WRP + j * 2);
            if (r >= R) t = u32x2{0u, 0u};
            v[2 * q] = t[0];
            v[2 * q + 1] = t[1];
        }
        wf[ks] = __builtin_bit_cast(bf16x8, v);
    }
    __syncthreads();  // every wavefront has its weights: the area takes the rows
    // borders, and what is read past the rows: zeros
    for (int i = tid; i < (G + 2) * BRP / 16; i += NT) *reinterpret_cast<u32x4*>(smem + i * 16) = u32x4{0u, 0u, 0u, 0u};
    float* const sB = reinterpret_cast<float*>(smem + (G + 2) * BRP + 4 * 32 * OP);
    if (tid < FB * 32) sB[tid] = a.bias ? a.bias[tid] : 0.f;
    __syncthreads();

    unsigned char* const sO = smem + (G + 2) * BRP + wave * (32 * OP);
    for (int u = blockIdx.x; u < a.units; u += gridDim.x) {
#pragma unroll
        for (int i = 0; i < XV; ++i) {
            if (vdst[i] == 0xffffffffu) continue;
            u32x4 v = rx[i];
            if (vshift[i] != 0) {
                u32x4 t = {0u, 0u, 0u, 0u};
#pragma unroll
                for (int k = 0; k < 4; ++k)
#pragma unroll
                    for (int m = 0; m < 4; ++m)
                        if (k - m == vshift[i]) t[k] = v[m];
                v = t;
            }
            *reinterpret_cast<u32x2*>(smem + (vdst[i] & 0xffffu)) = u32x2{v[0], v[1]};
            *reinterpret_cast<u32x2*>(smem + (vdst[i] >> 16)) = u32x2{v[2], v[3]};
        }
        __syncthreads();
        load_rows(u + gridDim.x);
        const int n = (int)fdiv((uint32_t)u, a.dGroups), oh0 = (u - n * a.groups) * G;
        const int rows = a.OH - oh0 < G ? a.OH - oh0 : G;
        for (int t = wi; t < rows * 2; t += 4 / FB) {
            const int j = t >> 1, pt = t & 1;
            const unsigned char* const x0 = smem + j * BRP + (pt * 32 + l32) * BP + half * 16;
            f32x16 acc, odd;  // two sums: an MFMA does not wait for the one before
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[e] = odd[e] = 0.f;
            // reads AHEAD steps before their MFMA, or every one of these waits for the LDS
            constexpr int AHEAD = 4;
            bf16x8 xf[AHEAD];
            auto read = [&](int ks) { return *reinterpret_cast<const bf16x8*>(x0 + ks / 9 * BRP + ks / 3 % 3 * BP + ks % 3 * 32); };
            // the operand without the twelfth row and column
            auto inside = [&](bf16x8 v, int ks) {
                u32x4 x = __builtin_bit_cast(u32x4, v);
#pragma unroll
                for (int d = 0; d < 4; ++d) x[d] &= half ? pair_mask(ks, ks % 3 * 16 + 8 + 2 * d) : pair_mask(ks, ks % 3 * 16 + 2 * d);
                return __builtin_bit_cast(bf16x8, x);
            };
#pragma unroll
            for (int ks = 0; ks < AHEAD; ++ks) xf[ks] = read(ks);
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) {
                __builtin_amdgcn_sched_barrier(0);
                f32x16& sum = ks & 1 ? odd : acc;
                sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[ks], inside(xf[ks % AHEAD], ks), sum, 0, 0, 0);
                if (ks + AHEAD < KS) xf[ks % AHEAD] = read(ks + AHEAD);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[e] += odd[e];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float v[4];
                const f32x4 bv = *reinterpret_cast<const f32x4*>(sB + b * 32 + q * 8 + half * 4);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    v[e] = a.bias ? acc[q * 4 + e] + bv[e] : acc[q * 4 + e];
                    if (a.relu) v[e] = v[e] > 0.f ? v[e] : 0.f;
                }
                *reinterpret_cast<u32x2*>(sO + l32 * OP + q * 16 + half * 8) =
                    u32x2{(unsigned)f2bf(v[0]) | ((unsigned)f2bf(v[1]) << 16), (unsigned)f2bf(v[2]) | ((unsigned)f2bf(v[3]) << 16)};
            }
            __builtin_amdgcn_wave_barrier();  // LDS operations of one wavefront complete in order
            bf16_t* const yrow = a.y + ((size_t)(n * a.OH + oh0 + j) * a.OW + pt * 32) * a.K + b * 32;
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                const int p = it * 16 + (lane >> 2);
                const u32x4 v = *reinterpret_cast<const u32x4*>(sO + p * OP + (lane & 3) * 16);
                if (pt * 32 + p < a.OW) *reinterpret_cast<u32x4*>(yrow + (size_t)p * a.K + (lane & 3) * 8) = v;
            }
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();  // the rows have been read
    }
}

int row_vecs(const GemmGeom& g) { return (int)((6L * g.IW + 6L * g.pad_w + 15) / 16); }
// Output rows of a group: as few as one round of work-groups takes, two on a CU.
int group_rows(const GemmGeom& g) {
    const int images = g.M / (g.OH * g.OW);
    for (int k : {1, 2})
        if ((long)images * ((g.OH + k - 1) / k) <= 2 * kNumCU) return k;
    return 4;
}

template <int FB, int G>
int launch_rows(RowsArgs a, hipStream_t st) {
    a.groups = (a.OH + G - 1) / G;
    a.units = a.N * a.groups;
    a.dGroups = make_fastdiv((uint32_t)a.groups);
    constexpr size_t smem = smem_of(FB, G);
    static_assert(smem <= 64 * 1024, "two work-groups per CU, and no attribute to set");
    const int grid = a.units < 2 * kNumCU ? a.units : 2 * kNumCU;
    hipLaunchKernelGGL((conv_c3_fwd_strided_kernel<FB, G>), dim3(grid), dim3(NT), smem, st, a);
    return check_launch("conv_c3_fwd_strided");
}

}  // namespace

// Rows of 33 to 64 output pixels: with one tile of 32 a row conv_thin.hip's tiles of whole pixels are as fast.
bool conv_c3_rows_supported(const GemmGeom& g) {
    if (g.IC != 3 || g.R != R || g.S != R || g.mul_h != ST || g.mul_w != ST || g.div_h != 1 || g.div_w != 1) return false;
    if ((g.Ncols != 32 && g.Ncols != 64) || g.OW <= 32 || g.OW > 64 || (g.IW % 2) != 0 || (g.pad_w % 2) != 0) return false;
    if (row_vecs(g) > MAX_VECS) return false;
    const double images = g.M / ((double)g.OH * g.OW);
    return images * g.IH * g.IW * 6.0 < 2147483648.0 && g.OH <= 1 << 15;
}
const char* conv_c3_rows_kernel_name(const GemmGeom& g) {
    static const char* names[2][3] = {{"conv_c3_fwd_strided_kernel<1,1>", "conv_c3_fwd_strided_kernel<1,2>", "conv_c3_fwd_strided_kernel<1,4>"},
                                      {"conv_c3_fwd_strided_kernel<2,1>", "conv_c3_fwd_strided_kernel<2,2>", "conv_c3_fwd_strided_kernel<2,4>"}};
    return names[g.Ncols / 64][group_rows(g) / 2];
}

int launch_conv_c3_rows(const GemmGeom& g, const bf16_t* x, const bf16_t* w, const float* bias, bool relu, bf16_t* y, hipStream_t st) {
    if (!conv_c3_rows_supported(g)) return set_error(WAP_EINVAL, "internal: strided 3-channel kernel not applicable");
    RowsArgs a = {};
    a.x = x; a.w = w; a.bias = bias; a.y = y;
    a.N = g.M / (g.OH * g.OW); a.H = g.IH; a.W3 = g.IW * 3; a.OH = g.OH; a.OW = g.OW; a.K = g.Ncols;
    a.ph = g.pad_h; a.pw = g.pad_w; a.relu = relu ? 1 : 0;
    a.nvx = row_vecs(g);
    a.x_bytes = (unsigned)((size_t)a.N * g.IH * a.W3 * 2);
    a.dNVX = make_fastdiv((uint32_t)a.nvx);
    switch (group_rows(g) * 2 + g.Ncols / 64) {
        case 2: return launch_rows<1, 1>(a, st);
        case 3: return launch_rows<2, 1>(a, st);
        case 4: return launch_rows<1, 2>(a, st);
        case 5: return launch_rows<2, 2>(a, st);
        case 8: return launch_rows<1, 4>(a, st);
        default: return launch_rows<2, 4>(a, st);
    }
}

}  // namespace wap
