// Memory-bound kernels of the training step (gfx950): split-reduction epilogues, ReLU backward,
// max-pool forward / backward, softmax cross-entropy, SGD, casts.  These are the "auxiliary
// computation nodes" of Section 3.2.2 and the weight update of Section 3.2.3; all are streaming
// kernels with 16-byte accesses where the shape allows and a grid sized to cover the chip.
#include <algorithm>

#include "wap_internal.h"

namespace wap {

namespace {

constexpr int kThreads = 256;

// One item a thread, up to `walk` items in 4096 work-groups at most, which walk the tensor.  More work-groups walk large tensors together (max-pool
// of 64 x 224 x 224 x 64 forward / backward 107 / 125 us in 4096, 101 / 115 so), but their starts cost something: each launch has its line.
inline int grid_for(size_t work_items, size_t walk = SIZE_MAX) {
    const size_t cap = work_items <= walk ? (size_t)kNumCU * 16 : (size_t)1 << 22;
    return (int)std::max((size_t)1, std::min((work_items + kThreads - 1) / kThreads, cap));
}

// of updates and ReLU derivatives that do not pass the cache, us walking / one vector a thread, same tensors again: ReLU derivative of 10.1 M elements
// 10.2 / 10.7, in place 9.1 / 9.7, of 12.5 M level, of 22 M 20.5 / 20.1; update of 5.6 M weights without a copy 10.8 / 11.5, of 7 M level, of 15 M 26.9 / 26.0
constexpr size_t kWalk = (size_t)3 << 19;

__device__ __forceinline__ float bf2f(unsigned short h) { return __uint_as_float((unsigned)h << 16); }
__device__ __forceinline__ unsigned short f2bf(float f) {
    __bf16 b = (__bf16)f;  // round to nearest even
    return __builtin_bit_cast(unsigned short, b);
}

// ---- out[r][c] = bf16(act(bias[c] + sum_k part[k][r][c])), summed in split order; with `mask`, zeroed where the mask is
// not positive (ReLU derivative of the layer below); with `colsum`, also the column sums of what is stored, one partial
// row per work-group row range (the bias gradient of that layer).  Bound by the launch and the latency of the loads: the
// partial sums of a layer small enough to be split are a few MB that the caches still hold.  A thread owns 16 bytes of a
// row, `vpb` (a power of two) threads lie side by side, U splits are in flight, the last batch with its absent splits
// loaded from the last one and left out (a loop over them waited for each: 2.9 us without, 3.8 with, 400 x 128 in 4 splits;
// 96 x 1000 in 32 4.9 us, 9.7 with a load at a time).  The separate mask and column-sum passes that this replaces took 5 us
// each at 1568 x 512. ----
template <int U, bool COLSUM>
__global__ __launch_bounds__(256) void reduce_bf16_kernel(const float* __restrict__ part, int nsplit, int rows, int ncols,
                                                          const float* __restrict__ bias, int relu,
                                                          const bf16_t* __restrict__ mask, bf16_t* __restrict__ out,
                                                          float* __restrict__ colsum, int log_vpb, int rows_per_block) {
    const int rb = blockIdx.y, vpb = 1 << log_vpb;
    const int vec = threadIdx.x & (vpb - 1), rsub = threadIdx.x >> log_vpb, rp = 256 >> log_vpb;
    const int c = ((int)blockIdx.x * vpb + vec) * 4;
    const size_t elems = (size_t)rows * ncols;
    float4 cs = make_float4(0.f, 0.f, 0.f, 0.f);
    if (c < ncols) {
        float4 bv = make_float4(0.f, 0.f, 0.f, 0.f);
        if (bias) bv = make_float4(bias[c], bias[c + 1], bias[c + 2], bias[c + 3]);
        const int r1 = (rb + 1) * rows_per_block < rows ? (rb + 1) * rows_per_block : rows;
        for (int r = rb * rows_per_block + rsub; r < r1; r += rp) {
            const size_t o = (size_t)r * ncols + c;
            const float* p = part + o;
            uint2 mk = make_uint2(0u, 0u);
            if (mask) mk = *reinterpret_cast<const uint2*>(mask + o);
            float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
            for (int k = 0; k < nsplit; k += U) {
                float4 t[U];
#pragma unroll
                for (int u = 0; u < U; ++u) t[u] = *reinterpret_cast<const float4*>(p + (size_t)(k + u < nsplit ? k + u : nsplit - 1) * elems);
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (k + u == 0) s = t[0];
                    else if (k + u < nsplit) { s.x += t[u].x; s.y += t[u].y; s.z += t[u].z; s.w += t[u].w; }
                }
            }
            if (bias) { s.x += bv.x; s.y += bv.y; s.z += bv.z; s.w += bv.w; }
            if (relu) {
                s.x = s.x > 0.f ? s.x : 0.f; s.y = s.y > 0.f ? s.y : 0.f;
                s.z = s.z > 0.f ? s.z : 0.f; s.w = s.w > 0.f ? s.w : 0.f;
            }
            unsigned short h0 = f2bf(s.x), h1 = f2bf(s.y), h2 = f2bf(s.z), h3 = f2bf(s.w);
            if (mask) {
                h0 = __uint_as_float(mk.x << 16) > 0.f ? h0 : 0;
                h1 = __uint_as_float(mk.x & 0xffff0000u) > 0.f ? h1 : 0;
                h2 = __uint_as_float(mk.y << 16) > 0.f ? h2 : 0;
                h3 = __uint_as_float(mk.y & 0xffff0000u) > 0.f ? h3 : 0;
            }
            *reinterpret_cast<uint2*>(out + o) = make_uint2((unsigned)h0 | ((unsigned)h1 << 16), (unsigned)h2 | ((unsigned)h3 << 16));
            if (!COLSUM) break;  // one row per thread
            cs.x += bf2f(h0); cs.y += bf2f(h1); cs.z += bf2f(h2); cs.w += bf2f(h3);
        }
    }
    if constexpr (COLSUM) {  // the row slots of a column as a tree through LDS: order fixed by the shape
        __shared__ float4 red[256];
        red[threadIdx.x] = cs;
        __syncthreads();
        for (int o = rp / 2; o > 0; o >>= 1) {
            if (rsub < o) {
                const float4 t = red[threadIdx.x + o * vpb];
                cs.x += t.x; cs.y += t.y; cs.z += t.z; cs.w += t.w;
                red[threadIdx.x] = cs;
            }
            __syncthreads();
        }
        if (rsub == 0 && c < ncols) *reinterpret_cast<float4*>(colsum + (size_t)rb * ncols + c) = cs;
    }
}

// the same for row lengths that are no multiple of 4, element by element
__global__ void reduce_bf16_scalar_kernel(const float* __restrict__ part, int nsplit, size_t elems, int ncols,
                                          const float* __restrict__ bias, int relu, bf16_t* __restrict__ out) {
    size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < elems; i += stride) {
        float s = part[i];
        for (int k = 1; k < nsplit; ++k) s += part[(size_t)k * elems + i];
        if (bias) s += bias[i % (size_t)ncols];
        if (relu) s = s > 0.f ? s : 0.f;
        out[i] = f2bf(s);
    }
}

// With a parameter block (sgd.w32 != NULL) the sums update the parameters instead of being stored.
__global__ void reduce_f32_kernel(const float* __restrict__ part, int nsplit, size_t elems,
                                  float* __restrict__ out, const SgdFuse sgd) {
    size_t stride = (size_t)gridDim.x * blockDim.x;
    if ((elems & 3) == 0) {
        size_t n4 = elems / 4;
        for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += stride) {
            float4 s = reinterpret_cast<const float4*>(part)[i];
            for (int k = 1; k < nsplit; ++k) {
                float4 t = reinterpret_cast<const float4*>(part + (size_t)k * elems)[i];
                s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w;
            }
            if (sgd.w32) sgd_apply4(sgd.w32 + i * 4, sgd.wb + i * 4, sgd.lr, s.x, s.y, s.z, s.w);
            else reinterpret_cast<float4*>(out)[i] = s;
        }
    } else {
        for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < elems; i += stride) {
            float s = part[i];
            for (int k = 1; k < nsplit; ++k) s += part[(size_t)k * elems + i];
            if (sgd.w32) {
                float a = sgd_apply(sgd.w32[i], s, sgd.lr);
                sgd.w32[i] = a;
                sgd.wb[i] = f2bf(a);
            } else {
                out[i] = s;
            }
        }
    }
}

// Many splits of a small tensor: G groups of threads each add the splits k = g, g + G, g + 2G, ... of one 16-byte column
// (V = float4; one element where the tensor is no multiple of four) in increasing k (four independent loads in flight), then
// the G partial sums are added in group order through LDS.  The summation tree is fixed by (nsplit, G), so results are bitwise
// reproducible.  (A thread per element that walks all splits takes 0.2 us for each: the bias gradient of 50176 x 33 in 784
// chunks 176 us.)
__device__ __forceinline__ void acc4(float4& s, const float4& t) { s.x += t.x; s.y += t.y; s.z += t.z; s.w += t.w; }
__device__ __forceinline__ void acc4(float& s, float t) { s += t; }
template <int G, typename V>
__global__ __launch_bounds__(256) void reduce_f32_grouped_kernel(const float* __restrict__ part, int nsplit, size_t elems,
                                                               float* __restrict__ out, const SgdFuse sgd) {
    constexpr int COLS = 256 / G, VEC = sizeof(V) / sizeof(float);
    __shared__ V sm[G][COLS];
    const int col = threadIdx.x % COLS, grp = threadIdx.x / COLS;
    const size_t nv = elems / VEC;
    const size_t i = (size_t)blockIdx.x * COLS + col;
    V s = {};
    if (i < nv) {
        const V* p = reinterpret_cast<const V*>(part) + i;
        int k = grp;
        for (; k + 3 * G < nsplit; k += 4 * G) {
            const V t0 = p[(size_t)k * nv], t1 = p[(size_t)(k + G) * nv], t2 = p[(size_t)(k + 2 * G) * nv],
                    t3 = p[(size_t)(k + 3 * G) * nv];
            acc4(s, t0); acc4(s, t1); acc4(s, t2); acc4(s, t3);
        }
        for (; k < nsplit; k += G) acc4(s, p[(size_t)k * nv]);
    }
    sm[grp][col] = s;
    __syncthreads();
    if (grp == 0 && i < nv) {
#pragma unroll
        for (int g2 = 1; g2 < G; ++g2) acc4(s, sm[g2][col]);
        if constexpr (VEC == 4) {
            if (sgd.w32) sgd_apply4(sgd.w32 + i * 4, sgd.wb + i * 4, sgd.lr, s.x, s.y, s.z, s.w);
            else reinterpret_cast<float4*>(out)[i] = s;
        } else if (sgd.w32) {
            const float a = sgd_apply(sgd.w32[i], s, sgd.lr);
            sgd.w32[i] = a;
            sgd.wb[i] = f2bf(a);
        } else {
            out[i] = s;
        }
    }
}

// ---- bias gradient, first stage: column sums of a chunk of rows (blockIdx.y) for a block of column vectors
// (blockIdx.x) of VEC channels.  `vpb` vectors lie side by side in a work-group, `rp` rows below each other (its threads
// cover whole rows, or runs of them, whatever their length), eight loads in flight each (the loop is bound by load latency,
// not by bytes: a whole FC layer's gradient is 0.8 MB; the last batch loads its absent rows from the last one and leaves
// them out), and the rp partial sums of a column are added as a tree through LDS.  The order is fixed by (rows, cols):
// bitwise reproducible.  Few wide work-groups with one load in flight and a serial sum over rp took 17 us for 100 x 4096, 18
// for 67600 x 256 and 55 for 50176 x 33; this takes 3.2, 9.2 and 6.2. ----
template <int VEC> struct BiasVec;
template <> struct BiasVec<8> { using type = u32x4; };
template <> struct BiasVec<4> { using type = u32x2; };
template <> struct BiasVec<1> { using type = bf16_t; };
template <int VEC>
__device__ __forceinline__ void add_vec(float* s, const typename BiasVec<VEC>::type u) {
    if constexpr (VEC == 1) {
        s[0] += bf2f(u);
    } else {
#pragma unroll
        for (int k = 0; k < VEC / 2; ++k) {
            s[2 * k] += __uint_as_float(u[k] << 16);
            s[2 * k + 1] += __uint_as_float(u[k] & 0xffff0000u);
        }
    }
}

template <int VEC>
__global__ __launch_bounds__(1024) void bias_grad_kernel(const bf16_t* __restrict__ dy, float* __restrict__ part,
                                                        uint32_t rows, uint32_t cols, uint32_t rows_per_chunk, int vpb, int rp) {
    using V = typename BiasVec<VEC>::type;
    __shared__ float red[VEC][1024];
    const int cv = (int)(cols / VEC);              // vectors per row
    const int rsub = threadIdx.x / vpb, vec = threadIdx.x - rsub * vpb;
    const int v = blockIdx.x * vpb + vec;
    // (32-bit offsets: a tensor has at most 2^31 - 1 elements)
    const uint32_t r0 = blockIdx.y * rows_per_chunk, r1 = r0 + rows_per_chunk < rows ? r0 + rows_per_chunk : rows;
    float s[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) s[e] = 0.f;
    if (v < cv && rsub < rp) {
        const bf16_t* p = dy + (size_t)v * VEC;
        for (uint32_t r = r0 + rsub; r < r1; r += 8u * rp) {
            V t[8];
            if (r + 7u * rp < r1) {
#pragma unroll
                for (int k = 0; k < 8; ++k) t[k] = *reinterpret_cast<const V*>(p + (r + (uint32_t)k * rp) * cols);
#pragma unroll
                for (int k = 0; k < 8; ++k) add_vec<VEC>(s, t[k]);
            } else {
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const uint32_t rk = r + (uint32_t)k * rp;
                    t[k] = *reinterpret_cast<const V*>(p + (rk < r1 ? rk : r1 - 1) * cols);
                }
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    if (r + (uint32_t)k * rp < r1) add_vec<VEC>(s, t[k]);
            }
        }
    }
    if (rp > 1) {  // (uniform)
#pragma unroll
        for (int e = 0; e < VEC; ++e) red[e][threadIdx.x] = s[e];
        for (int n = rp; n > 1;) {  // four rows into one: half the barriers of a tree of pairs
            const int h = (n + 3) >> 2;
            __syncthreads();
            if (rsub < h) {
#pragma unroll
                for (int q = 1; q < 4; ++q)
                    if (rsub + q * h < n) {
#pragma unroll
                        for (int e = 0; e < VEC; ++e) s[e] += red[e][threadIdx.x + q * h * vpb];
                    }
#pragma unroll
                for (int e = 0; e < VEC; ++e) red[e][threadIdx.x] = s[e];
            }
            n = h;
        }
    }
    if (rsub == 0 && v < cv) {
        float* o = part + (size_t)blockIdx.y * cols + (size_t)v * VEC;
        if constexpr (VEC == 1) {
            *o = s[0];
        } else {
#pragma unroll
            for (int e = 0; e < VEC; e += 4) *reinterpret_cast<float4*>(o + e) = make_float4(s[e], s[e + 1], s[e + 2], s[e + 3]);
        }
    }
}

// vector(i) for this thread's i < n, single(i - n) for the `rest` items behind them; with WALK for every one of its items
template <bool WALK, typename V, typename S>
__device__ __forceinline__ void walk_items(size_t n, size_t rest, V&& vector, S&& single) {
    size_t i = (size_t)blockIdx.x * kThreads + threadIdx.x;
    if constexpr (WALK)
        for (const size_t stride = (size_t)gridDim.x * kThreads; i < n; i += stride) vector(i);
    else if (i < n) {
        vector(i);
        return;
    }
    if (i - n < rest) single(i - n);
}

// ---- ReLU backward: bound by memory.  One 16-byte vector a thread; ONCE: the operands pass the cache (beyond_cache), what is
// written, which the next kernels read, does not.  Walk of 4096 work-groups / this, us: 16.8 M elements 13.9 / 13.8, 67 M 78 / 56,
// 77 M 89 / 63, 268 M 361 / 253 (6.4 TB/s). ----
template <bool ONCE, bool WALK>
__global__ __launch_bounds__(kThreads) void relu_bwd_kernel(const bf16_t* dy, const bf16_t* __restrict__ y, bf16_t* dx, size_t n) {
    const size_t n8 = n / 8;
    walk_items<WALK>(n8, n & 7, [&](size_t i) {
        const u32x4 *gp = reinterpret_cast<const u32x4*>(dy) + i, *vp = reinterpret_cast<const u32x4*>(y) + i;
        u32x4 g, v;
        if constexpr (ONCE) {
            g = __builtin_nontemporal_load(gp);
            v = __builtin_nontemporal_load(vp);
        } else {
            g = *gp;
            v = *vp;
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const unsigned lo = (bf2f((unsigned short)(v[k] & 0xffff)) > 0.f) ? (g[k] & 0xffffu) : 0u;
            const unsigned hi = (bf2f((unsigned short)(v[k] >> 16)) > 0.f) ? (g[k] & 0xffff0000u) : 0u;
            g[k] = lo | hi;
        }
        reinterpret_cast<u32x4*>(dx)[i] = g;
    }, [&](size_t i) {
        const size_t j = n8 * 8 + i;
        dx[j] = (bf2f(y[j]) > 0.f) ? dy[j] : (bf16_t)0;
    });
}

// ---- max-pool forward: VEC channels of one window per thread, the window's loads issued together.  Bound by the input
// stream; index arithmetic in 64 bits (a software division per coordinate) held it to 2.2 TB/s: 100 x 55 x 55 x 64,
// window 3, 23.8 -> 12.4 us. ----
struct PoolArgs {
    int H, W, C, P, Q, st;
    uint32_t items;        // threads' work items
    FastDiv dCV, dX, dY;   // item -> channel vector, x, y, image: divisions by vectors per pixel, items per row, rows
};

// VEC maxima (fp32 bits) and their window positions at element o
template <int VEC>
__device__ __forceinline__ void pool_store_max(bf16_t* y, uint8_t* am, size_t o, const unsigned* best, const unsigned* bi) {
    if constexpr (VEC == 8) {
        u32x4 yo;
#pragma unroll
        for (int k = 0; k < 4; ++k) yo[k] = (best[2 * k] >> 16) | best[2 * k + 1];
        *reinterpret_cast<u32x4*>(y + o) = yo;
        const u32x2 ao = {bi[0] | (bi[1] << 8) | (bi[2] << 16) | (bi[3] << 24), bi[4] | (bi[5] << 8) | (bi[6] << 16) | (bi[7] << 24)};
        *reinterpret_cast<u32x2*>(am + o) = ao;
    } else {
        y[o] = (bf16_t)(best[0] >> 16);
        am[o] = (uint8_t)bi[0];
    }
}

template <int VEC, int WIN>
__global__ void maxpool_fwd_kernel(const bf16_t* __restrict__ x, bf16_t* __restrict__ y, uint8_t* __restrict__ am,
                                   const PoolArgs a) {
    const uint32_t CV = a.C / VEC;
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < a.items; i += stride) {
        uint32_t t = fdiv(i, a.dCV);
        const uint32_t cv = i - t * CV;
        const uint32_t t2 = fdiv(t, a.dX);
        const int q = (int)(t - t2 * a.Q);
        const uint32_t n = fdiv(t2, a.dY);
        const int p = (int)(t2 - n * a.P);
        const bf16_t* src = x + (((size_t)n * a.H + (size_t)p * a.st) * a.W + (size_t)q * a.st) * a.C + (size_t)cv * VEC;
        u32x4 v8[WIN * WIN];
        unsigned short v1[WIN * WIN];
#pragma unroll
        for (int k = 0; k < WIN * WIN; ++k) {
            const bf16_t* s = src + ((size_t)(k / WIN) * a.W + k % WIN) * a.C;
            if (VEC == 8) v8[k] = *reinterpret_cast<const u32x4*>(s);
            else v1[k] = *s;
        }
        unsigned best[VEC];  // as fp32 bits
        unsigned bi[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
#pragma unroll
            for (int k = 0; k < WIN * WIN; ++k) {
                const unsigned f = VEC == 8 ? ((e & 1) ? (v8[k][e >> 1] & 0xffff0000u) : (v8[k][e >> 1] << 16)) : (unsigned)v1[k] << 16;
                const bool take = k == 0 || __uint_as_float(f) > __uint_as_float(best[e]);  // the first maximum
                best[e] = take ? f : best[e];
                bi[e] = take ? (unsigned)k : bi[e];
            }
        }
        pool_store_max<VEC>(y, am, (size_t)t * a.C + (size_t)cv * VEC, best, bi);
    }
}

// any other window side (VEC channels by one load, as above: element by element 8 x 40 x 40 x 64, window 5, took 21 us for 12)
template <int VEC>
__global__ void maxpool_fwd_any_kernel(const bf16_t* __restrict__ x, bf16_t* __restrict__ y, uint8_t* __restrict__ am, int win,
                                       const PoolArgs a) {
    const uint32_t CV = a.C / VEC;
    const uint32_t stride = gridDim.x * blockDim.x;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < a.items; i += stride) {
        uint32_t t = fdiv(i, a.dCV);
        const uint32_t cv = i - t * CV;
        const uint32_t t2 = fdiv(t, a.dX);
        const int q = (int)(t - t2 * a.Q);
        const uint32_t n = fdiv(t2, a.dY);
        const int p = (int)(t2 - n * a.P);
        const bf16_t* src = x + (((size_t)n * a.H + (size_t)p * a.st) * a.W + (size_t)q * a.st) * a.C + (size_t)cv * VEC;
        unsigned best[VEC], bi[VEC];  // best: as fp32 bits
        for (int r = 0; r < win; ++r)
            for (int q2 = 0; q2 < win; ++q2) {
                const bf16_t* x1 = src + ((size_t)r * a.W + q2) * a.C;
                unsigned f[VEC];
                if constexpr (VEC == 8) {
                    const u32x4 u = *reinterpret_cast<const u32x4*>(x1);
#pragma unroll
                    for (int e = 0; e < VEC; ++e) f[e] = (e & 1) ? u[e >> 1] & 0xffff0000u : u[e >> 1] << 16;
                } else {
                    f[0] = (unsigned)*x1 << 16;
                }
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    const bool take = (r | q2) == 0 || __uint_as_float(f[e]) > __uint_as_float(best[e]);
                    best[e] = take ? f[e] : best[e];
                    bi[e] = take ? (unsigned)(r * win + q2) : bi[e];
                }
            }
        pool_store_max<VEC>(y, am, (size_t)t * a.C + (size_t)cv * VEC, best, bi);
    }
}

// ---- max-pool backward as a gather over the windows covering each input element (zero where ry is given and not
// positive).  VEC channels of one gradient window as fp32 plus the argmax; an absent window names no pixel. ----
template <int VEC>
struct PoolWindow {
    float g[VEC];
    unsigned am[VEC];
    __device__ __forceinline__ void load(const bf16_t* dy, const uint8_t* amp, const bf16_t* ry, size_t o, bool ok) {
        if (VEC == 8) {
            u32x4 gv = {0u, 0u, 0u, 0u}, yv = {0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u};
            u32x2 av = {0xffffffffu, 0xffffffffu};
            if (ok) {
                gv = *reinterpret_cast<const u32x4*>(dy + o);
                av = *reinterpret_cast<const u32x2*>(amp + o);
                if (ry) yv = *reinterpret_cast<const u32x4*>(ry + o);
            }
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                const unsigned yb = (e & 1) ? (yv[e >> 1] & 0xffff0000u) : (yv[e >> 1] << 16);
                const unsigned gb = (e & 1) ? (gv[e >> 1] & 0xffff0000u) : (gv[e >> 1] << 16);
                g[e] = __uint_as_float(gb);
                am[e] = __uint_as_float(yb) > 0.f ? ((e < 4 ? av[0] : av[1]) >> ((e & 3) * 8)) & 0xffu : 0xffu;
            }
        } else {
            g[0] = ok ? bf2f(dy[o]) : 0.f;
            am[0] = ok && (!ry || bf2f(ry[o]) > 0.f) ? amp[o] : 0xffu;
        }
    }
    __device__ __forceinline__ void add(float* sum, unsigned code) const {
#pragma unroll
        for (int e = 0; e < VEC; ++e) sum[e] += am[e] == code ? g[e] : 0.f;
    }
};
template <int VEC>
__device__ __forceinline__ void pool_store(bf16_t* dx, const float* s, float* cs = nullptr) {  // cs: sums of what is stored
    if (VEC == 8) {
        u32x4 v;
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = (unsigned)f2bf(s[2 * k]) | ((unsigned)f2bf(s[2 * k + 1]) << 16);
        *reinterpret_cast<u32x4*>(dx) = v;
        if (cs) {
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                cs[2 * k] += __uint_as_float(v[k] << 16);
                cs[2 * k + 1] += __uint_as_float(v[k] & 0xffff0000u);
            }
        }
    } else {
        *dx = f2bf(s[0]);
    }
}

// sum of the row losses as a tree of 256, by any number of threads from 128 on: the same order everywhere
__device__ __forceinline__ void loss_mean(const LossMean m, float* sh) {
    for (int v = threadIdx.x; v < 256; v += blockDim.x) {
        float s = 0.f;
        for (int j = v; j < m.B; j += 256) s += m.row_loss[j];
        sh[v] = s;
    }
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) *m.loss = sh[0] / (float)m.B;
}

// Stride 2 (every pool of the two networks): a thread owns a 2 x 2 block of input pixels, which only the windows ending
// in it (WIN 3: and the ones before, above and left) can reach: one (four) window loads for four pixels, where a thread
// per pixel loads 4 (9).  100 x 55 x 55 x 64, window 3: 30.7 -> 17.3 us.
// COLSUM (work-groups of whole pixels, so that a thread keeps its channels): a row of column sums of what the work-group stores, for the
// bias gradient of the layer below, which otherwise takes a pass over the tensor and a launch for its partial sums.  The sums take 107 registers
// instead of 94 (window 3: four wavefronts a SIMD instead of five), so that the three pools of an AlexNet-style step at 100 images take 43 instead
// of 38 us, for three passes of 6 us and as many sums of 5.6.  MEAN: the last
// work-group takes the mean of the row losses; it waits for nothing here, and nothing for it.  (A flag of the launch instead, which every
// work-group waits for: 12 x 29 x 29 x 200 5.1 -> 5.5 us.)
template <int VEC, int WIN, bool COLSUM, bool MEAN>
__device__ __forceinline__ void maxpool_bwd_s2(const bf16_t* __restrict__ dy, const uint8_t* __restrict__ am, const bf16_t* __restrict__ ry,
                                               bf16_t* __restrict__ dx, const PoolArgs& a, uint32_t threads, float* __restrict__ colsum, const LossMean& mean) {
    __shared__ __align__(16) float red[COLSUM ? kThreads * VEC : MEAN ? kThreads : 4];
    const uint32_t groups = gridDim.x - (MEAN ? 1 : 0);
    if constexpr (MEAN) {
        if (blockIdx.x == groups) {
            loss_mean(mean, red);
            return;
        }
    }
    float cs[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) cs[e] = 0.f;
    const uint32_t CV = a.C / VEC;
    const uint32_t WB = (a.W + 1) / 2, HB = (a.H + 1) / 2;
    const uint32_t stride = groups * threads;
    for (uint32_t i = blockIdx.x * threads + threadIdx.x; i < a.items; i += stride) {
        const uint32_t t = fdiv(i, a.dCV);
        const uint32_t cv = i - t * CV;
        const uint32_t t2 = fdiv(t, a.dX);
        const int q = (int)(t - t2 * WB);
        const uint32_t n = fdiv(t2, a.dY);
        const int p = (int)(t2 - n * HB);
        constexpr int NB = WIN == 3 ? 2 : 1;  // windows per direction
        PoolWindow<VEC> w[NB][NB];            // [1]: the window of (p, q), [0]: the one before
#pragma unroll
        for (int u = 0; u < NB; ++u)
#pragma unroll
            for (int v = 0; v < NB; ++v) {
                const int pw = p - (NB - 1) + u, qw = q - (NB - 1) + v;
                w[u][v].load(dy, am, ry, (((size_t)n * a.P + pw) * a.Q + qw) * a.C + (size_t)cv * VEC,
                             (unsigned)pw < (unsigned)a.P && (unsigned)qw < (unsigned)a.Q);
            }
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int h = 2 * p + r, x = 2 * q + s;
                if (h >= a.H || x >= a.W) continue;
                float sum[VEC];
#pragma unroll
                for (int e = 0; e < VEC; ++e) sum[e] = 0.f;
                if (WIN == 3) {
                    if (r == 0 && s == 0) w[0][0].add(sum, 2 * WIN + 2);
                    if (r == 0) w[0][NB - 1].add(sum, 2 * WIN + s);
                    if (s == 0) w[NB - 1][0].add(sum, r * WIN + 2);
                }
                w[NB - 1][NB - 1].add(sum, r * WIN + s);
                pool_store<VEC>(dx + (((size_t)n * a.H + h) * a.W + x) * a.C + (size_t)cv * VEC, sum, COLSUM ? cs : nullptr);
            }
    }
    if constexpr (COLSUM) {  // the pixels of the work-group in order of a tree: fixed by the shape
        const uint32_t np = threads / CV, px = threadIdx.x / CV;
        f32x4* const mine = reinterpret_cast<f32x4*>(red + threadIdx.x * VEC);
        auto put = [&]() {
#pragma unroll
            for (int q = 0; q < VEC / 4; ++q) mine[q] = f32x4{cs[4 * q], cs[4 * q + 1], cs[4 * q + 2], cs[4 * q + 3]};
        };
        put();
        for (uint32_t h = np; h > 1;) {
            const uint32_t half = (h + 1) / 2;
            __syncthreads();
            if (px < half && px + half < h) {
#pragma unroll
                for (int q = 0; q < VEC / 4; ++q) {
                    const f32x4 o = mine[half * CV * (VEC / 4) + q];
#pragma unroll
                    for (int e = 0; e < 4; ++e) cs[4 * q + e] += o[e];
                }
                put();
            }
            h = half;
        }
        if (px == 0) {
#pragma unroll
            for (int q = 0; q < VEC / 4; ++q)
                *reinterpret_cast<f32x4*>(colsum + (size_t)blockIdx.x * a.C + threadIdx.x * VEC + 4 * q) = f32x4{cs[4 * q], cs[4 * q + 1], cs[4 * q + 2], cs[4 * q + 3]};
        }
    }
}

// Alone, with work-groups of a constant size, and with what rides along: one kernel for both read the size and its longer arguments at every
// work-group's start (31 x 19 x 19 x 200, window 3, 5.8 us, 5.5 so; 11 x 51 x 51 x 344, window 2, 9.7 / 9.3).
template <int VEC, int WIN>
__global__ __launch_bounds__(kThreads) void maxpool_bwd_s2_kernel(const bf16_t* __restrict__ dy, const uint8_t* __restrict__ am,
                                                                  const bf16_t* __restrict__ ry, bf16_t* __restrict__ dx, const PoolArgs a) {
    maxpool_bwd_s2<VEC, WIN, false, false>(dy, am, ry, dx, a, kThreads, nullptr, LossMean{nullptr, nullptr, 0});
}
template <int WIN, bool COLSUM, bool MEAN>
__global__ __launch_bounds__(kThreads) void maxpool_bwd_s2_sums_kernel(const bf16_t* __restrict__ dy, const uint8_t* __restrict__ am,
                                                                       const bf16_t* __restrict__ ry, bf16_t* __restrict__ dx, const PoolArgs a,
                                                                       uint32_t threads, float* __restrict__ colsum, const LossMean mean) {
    maxpool_bwd_s2<8, WIN, COLSUM, MEAN>(dy, am, ry, dx, a, COLSUM ? threads : kThreads, colsum, mean);
}

// any other stride or window: a thread per input pixel walks the windows that cover it
template <int VEC>
__global__ void maxpool_bwd_kernel(const bf16_t* __restrict__ dy, const uint8_t* __restrict__ am,
                                   const bf16_t* __restrict__ ry, bf16_t* __restrict__ dx, int win, const PoolArgs a) {
    const uint32_t CV = a.C / VEC;
    const uint32_t stride = gridDim.x * blockDim.x;
    const int st = a.st;
    for (uint32_t i = blockIdx.x * blockDim.x + threadIdx.x; i < a.items; i += stride) {
        const uint32_t t = fdiv(i, a.dCV);
        const uint32_t cv = i - t * CV;
        const uint32_t t2 = fdiv(t, a.dX);
        const int w = (int)(t - t2 * a.W);
        const uint32_t n = fdiv(t2, a.dY);
        const int h = (int)(t2 - n * a.H);
        float sum[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) sum[e] = 0.f;
        int p_lo = (h - win + 1 + st - 1);
        p_lo = p_lo > 0 ? p_lo / st : 0;
        int p_hi = h / st; if (p_hi > a.P - 1) p_hi = a.P - 1;
        int q_lo = (w - win + 1 + st - 1);
        q_lo = q_lo > 0 ? q_lo / st : 0;
        int q_hi = w / st; if (q_hi > a.Q - 1) q_hi = a.Q - 1;
        for (int p = p_lo; p <= p_hi; ++p)
            for (int q = q_lo; q <= q_hi; ++q) {
                PoolWindow<VEC> wd;
                wd.load(dy, am, ry, (((size_t)n * a.P + p) * a.Q + q) * a.C + (size_t)cv * VEC, true);
                wd.add(sum, (unsigned)((h - p * st) * win + (w - q * st)));
            }
        pool_store<VEC>(dx + (size_t)t * a.C + (size_t)cv * VEC, sum);
    }
}

// ---- softmax cross-entropy: one work-group per example ----
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__global__ __launch_bounds__(256) void softmax_xent_kernel(const bf16_t* __restrict__ z,
                                                           const int32_t* __restrict__ labels, int B,
                                                           int classes, float* __restrict__ row_loss,
                                                           bf16_t* __restrict__ dz) {
    __shared__ float red[4];
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const bf16_t* zb = z + (size_t)b * classes;
    float m = -3.0e38f;
    for (int j = tid; j < classes; j += 256) m = fmaxf(m, bf2f(zb[j]));
    m = wave_max(m);
    if (lane == 0) red[wave] = m;
    __syncthreads();
    m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
    __syncthreads();
    float s = 0.f;
    for (int j = tid; j < classes; j += 256) s += expf(bf2f(zb[j]) - m);
    s = wave_sum(s);
    if (lane == 0) red[wave] = s;
    __syncthreads();
    s = (red[0] + red[1]) + (red[2] + red[3]);
    const float inv = 1.f / s, invB = 1.f / (float)B;
    // a label outside [0, classes) names no class: the row gets no one-hot term and contributes no loss (and no
    // out-of-range read)
    const int lab = labels[b];
    const bool lab_ok = (unsigned)lab < (unsigned)classes;
    for (int j = tid; j < classes; j += 256) {
        float p = expf(bf2f(zb[j]) - m) * inv;
        dz[(size_t)b * classes + j] = f2bf((p - (j == lab ? 1.f : 0.f)) * invB);
    }
    if (tid == 0) row_loss[b] = lab_ok ? -(bf2f(zb[lab]) - m - logf(s)) : 0.f;
}

__global__ __launch_bounds__(kThreads) void loss_mean_kernel(const LossMean m) {
    __shared__ float sh[kThreads];
    loss_mean(m, sh);
}

// ---- SGD on fp32 master weights, re-deriving the bf16 compute copy: bound by memory.  One 16-byte group a thread and as many
// threads, so that the work-groups in flight walk the tensors together (138 M weights, a walk of 4096 work-groups 465 us, 4.2 TB/s;
// this 341); ONCE: gradient and master weights pass the cache (beyond_cache), the bf16 copy, which the next forward pass reads, does
// not (308 us, 6.3 TB/s; in a VGG-16 step at 22 images 394 -> 290). ----
template <bool ONCE, bool WALK>
__global__ __launch_bounds__(kThreads) void sgd_kernel(size_t n, float* __restrict__ w, const float* __restrict__ dw, float lr,
                                                       bf16_t* __restrict__ wb) {
    const size_t n4 = n / 4;
    walk_items<WALK>(n4, n & 3, [&](size_t i) {
        f32x4* const wp = reinterpret_cast<f32x4*>(w) + i;
        const f32x4* const gp = reinterpret_cast<const f32x4*>(dw) + i;
        f32x4 a, g;
        if constexpr (ONCE) {
            a = __builtin_nontemporal_load(wp);
            g = __builtin_nontemporal_load(gp);
        } else {
            a = *wp;
            g = *gp;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) a[e] = sgd_apply(a[e], g[e], lr);
        if constexpr (ONCE) __builtin_nontemporal_store(a, wp);
        else *wp = a;
        if (wb) {
            uint2 pk;
            pk.x = (unsigned)f2bf(a[0]) | ((unsigned)f2bf(a[1]) << 16);
            pk.y = (unsigned)f2bf(a[2]) | ((unsigned)f2bf(a[3]) << 16);
            reinterpret_cast<uint2*>(wb)[i] = pk;
        }
    }, [&](size_t i) {
        const size_t j = n4 * 4 + i;
        const float a = sgd_apply(w[j], dw[j], lr);
        w[j] = a;
        if (wb) wb[j] = f2bf(a);
    });
}

__global__ void cast_kernel(size_t n, const float* __restrict__ src, bf16_t* __restrict__ dst) {
    size_t stride = (size_t)gridDim.x * blockDim.x;
    size_t n4 = n / 4;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += stride) {
        float4 a = reinterpret_cast<const float4*>(src)[i];
        uint2 pk;
        pk.x = (unsigned)f2bf(a.x) | ((unsigned)f2bf(a.y) << 16);
        pk.y = (unsigned)f2bf(a.z) | ((unsigned)f2bf(a.w) << 16);
        reinterpret_cast<uint2*>(dst)[i] = pk;
    }
    for (size_t i = n4 * 4 + (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        dst[i] = f2bf(src[i]);
}

// deterministic small values in (-1, 1) for profiling buffers
__global__ void fill_kernel(bf16_t* p, size_t n, uint32_t seed) {
    size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        uint32_t h = (uint32_t)i * 2654435761u + seed;
        h ^= h >> 15; h *= 2246822519u; h ^= h >> 13;
        float f = ((float)(h & 0xffff) - 32768.f) * (1.f / 32768.f);
        p[i] = f2bf(f);
    }
}

// n elements, an item for every whole vector of `vec` and for every element behind them: launch(first, elements, grid, whether it walks),
// in pieces of whole vectors where one grid (fewer than 2^32 threads) does not do; `walk` as in grid_for.
template <typename F>
void in_pieces(size_t n, size_t vec, size_t walk, F&& launch) {
    const size_t most = vec << 30;
    for (size_t at = 0; at < n; at += most) {
        const size_t m = std::min(n - at, most), items = m / vec + m % vec;
        const int groups = grid_for(items, walk);
        launch(at, m, dim3((unsigned)groups), (size_t)groups * kThreads < items);
    }
}

}  // namespace

// Threads side by side in a row: the largest power of two up to 64 that divides the row into whole vectors, unless that
// falls below 16 (then the smallest that covers the row, some threads of the last column block idle).
static int reduce_vpb(int ncols) {
    const int cv = ncols / 4;
    int vpb = 64;
    while (vpb > 16 && cv % vpb != 0) vpb /= 2;
    if (cv % vpb != 0 || cv < 16) {
        vpb = 1;
        while (vpb < cv && vpb < 64) vpb *= 2;
    }
    return vpb;
}
// rows of one work-group: one per thread, four where column sums are wanted (fewer partial rows to add up later)
static int reduce_rows_per_block(int ncols, bool colsum) { return 256 / reduce_vpb(ncols) * (colsum ? 4 : 1); }
int reduce_bf16_colsum_rows(int rows, int ncols) {
    const int rpb = reduce_rows_per_block(ncols, true);
    return (ncols & 3) == 0 ? (rows + rpb - 1) / rpb : 0;
}

int launch_reduce_bf16(const float* part, int nsplit, size_t elems, int ncols, const float* bias,
                       bool relu, bf16_t* out, hipStream_t st, const bf16_t* mask, float* colsum) {
    if ((ncols & 3) != 0) {
        if (mask || colsum) return set_error(WAP_EINVAL, "internal: split reduction with a mask needs rows of whole 16-byte vectors");
        hipLaunchKernelGGL(reduce_bf16_scalar_kernel, dim3(grid_for(elems)), dim3(kThreads), 0, st, part, nsplit, elems, ncols,
                           bias, relu ? 1 : 0, out);
        return check_launch("reduce_bf16_scalar");
    }
    const int rows = (int)(elems / ncols), vpb = reduce_vpb(ncols), rpb = reduce_rows_per_block(ncols, colsum != nullptr);
    const int colblocks = (ncols / 4 + vpb - 1) / vpb;
    int log_vpb = 0;
    while ((1 << log_vpb) < vpb) ++log_vpb;
    // (a split product has at most 192 tiles of 256 rows: fewer than 65536 row blocks)
    const dim3 grid((unsigned)colblocks, (unsigned)((rows + rpb - 1) / rpb));
#define WAP_REDUCE(U)                                                                                                        \
    hipLaunchKernelGGL((colsum ? reduce_bf16_kernel<U, true> : reduce_bf16_kernel<U, false>), grid, dim3(256), 0, st, part, \
                       nsplit, rows, ncols, bias, relu ? 1 : 0, mask, out, colsum, log_vpb, rpb)
    if (nsplit <= 2) WAP_REDUCE(2);
    else if (nsplit <= 4) WAP_REDUCE(4);
    else WAP_REDUCE(8);
#undef WAP_REDUCE
    return check_launch("reduce_bf16");
}

int launch_reduce_f32(const float* part, int nsplit, size_t elems, float* out, hipStream_t st, const SgdFuse* sgdp) {
    SgdFuse sgd = {nullptr, nullptr, 0.f};
    if (sgdp) sgd = *sgdp;
    if (nsplit >= 8) {
        const bool vec = (elems & 3) == 0;
        const size_t nv = vec ? elems / 4 : elems;
#define WAP_GROUPED(G, V) \
    hipLaunchKernelGGL((reduce_f32_grouped_kernel<G, V>), dim3((unsigned)((nv + 256 / G - 1) / (256 / G))), dim3(256), 0, st, part, nsplit, elems, out, sgd)
        if (nsplit >= 64 && vec) WAP_GROUPED(32, float4);
        else if (nsplit >= 64 && elems <= 4096) WAP_GROUPED(32, float);  // (rows of 32 bytes)
        else if (vec) WAP_GROUPED(8, float4);
        else WAP_GROUPED(8, float);
#undef WAP_GROUPED
        return check_launch("reduce_f32_grouped");
    }
    hipLaunchKernelGGL(reduce_f32_kernel, dim3(grid_for(elems / 4 + 1)), dim3(kThreads), 0, st, part,
                       nsplit, elems, out, sgd);
    return check_launch("reduce_f32");
}

int launch_fill_bf16(bf16_t* p, size_t n, uint32_t seed, hipStream_t st) {
    hipLaunchKernelGGL(fill_kernel, dim3(grid_for(n)), dim3(kThreads), 0, st, p, n, seed);
    return check_launch("fill");
}

// ---- fixed-order column sums of fp32 or bf16 matrices [rows][cols], cols % 4 == 0 (the per-tile partial sums that other kernels'
// epilogues leave for the bias gradients, and the gradient of the logits itself), every matrix of a step in one launch.  First stage: a
// work-group adds a chunk of rows of up to 16 vectors of four columns, a thread every RP-th row, then the RP partial sums in a tree.
// Second stage: a thread adds the chunks of one column vector in order.  (Rows in one piece, a load at a time and the RP sums one after
// the other: 15.0 and 8.5 us for the layers of VGG-16 at 22 and of the AlexNet-style network at 100 images; 4.9 and 6.0 so.) ----
static __host__ __device__ int colsum_vpb(int cols) { return cols / 4 < 16 ? cols / 4 : 16; }
__global__ __launch_bounds__(256) void colsum_multi_kernel(const ColsumJobs js, unsigned char* __restrict__ base) {
    __shared__ float4 red[256];
    int j = 0;
    while (j + 1 < js.n && (int)blockIdx.x >= js.first[j + 1]) ++j;
    const ColsumJob& jb = js.job[j];
    const int local = (int)blockIdx.x - js.first[j];
    const int cv = jb.cols / 4, vpb = colsum_vpb(jb.cols);
    const int colblocks = (cv + vpb - 1) / vpb;
    const int chunk = local / colblocks, cb = local - chunk * colblocks;
    const int rp = 256 / vpb;
    const int vec = threadIdx.x % vpb, rsub = threadIdx.x / vpb;
    const int v = cb * vpb + vec;
    float* part2 = reinterpret_cast<float*>(base + jb.part2_off);
    const int rpc = (jb.rows + jb.chunks - 1) / jb.chunks;
    const int r0 = chunk * rpc, r1 = r0 + rpc < jb.rows ? r0 + rpc : jb.rows;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (rsub < rp && v < cv) {
        for (int r = r0 + rsub; r < r1; r += 8 * rp) {  // eight loads in flight, absent rows loaded from the last one and left out
            float4 t[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const size_t o = (size_t)(r + k * rp < r1 ? r + k * rp : r1 - 1) * jb.cols + (size_t)v * 4;
                if (jb.bf16) {
                    const uint2 u = *reinterpret_cast<const uint2*>(reinterpret_cast<const bf16_t*>(base + jb.part_off) + o);
                    t[k] = make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16), __uint_as_float(u.y & 0xffff0000u));
                } else {
                    t[k] = *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(base + jb.part_off) + o);
                }
            }
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (r + k * rp < r1) acc4(s, t[k]);
        }
    }
    red[threadIdx.x] = s;
    for (int h = rp; h > 1;) {
        const int half = (h + 1) / 2;
        __syncthreads();
        if (rsub < half && rsub + half < h) {
            acc4(s, red[threadIdx.x + half * vpb]);
            red[threadIdx.x] = s;
        }
        h = half;
    }
    if (rsub == 0 && v < cv) *reinterpret_cast<float4*>(part2 + (size_t)chunk * jb.cols + (size_t)v * 4) = s;
}

// 16 column vectors (of the concatenation of all matrices) per work-group, 16 threads per vector that each add every
// 16th chunk; their sums are added in order.  (One thread per vector walked up to 64 chunks one load after the other:
// 20 us for VGG-16's twelve layers at minibatch 22; this takes 6.)
__global__ __launch_bounds__(256) void colsum_finish_kernel(const ColsumJobs js, unsigned char* __restrict__ base) {
    __shared__ float4 red[256];
    const int sub = threadIdx.x >> 4;
    const int t = blockIdx.x * 16 + (threadIdx.x & 15);
    int j = 0, v0 = 0;
    while (j < js.n && t >= v0 + js.job[j].cols / 4) { v0 += js.job[j].cols / 4; ++j; }
    const ColsumJob& jb = js.job[j < js.n ? j : 0];
    const int v = t - v0;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (j < js.n) {
        const float* part2 = reinterpret_cast<const float*>(base + jb.part2_off) + (size_t)v * 4;
#pragma unroll 4
        for (int k = sub; k < jb.chunks; k += 16) {
            const float4 u = *reinterpret_cast<const float4*>(part2 + (size_t)k * jb.cols);
            s.x += u.x; s.y += u.y; s.z += u.z; s.w += u.w;
        }
    }
    red[threadIdx.x] = s;
    __syncthreads();
    if (sub == 0 && j < js.n) {
#pragma unroll
        for (int k = 1; k < 16; ++k) {
            const float4 u = red[k * 16 + threadIdx.x];
            s.x += u.x; s.y += u.y; s.z += u.z; s.w += u.w;
        }
        *reinterpret_cast<float4*>(reinterpret_cast<float*>(base + jb.out_off) + (size_t)v * 4) = s;
    }
}

// chunks of up to eight rows a thread, 64 of them at most (then of more rows)
int colsum_chunks(int rows, int cols) {
    const int per = 8 * (256 / colsum_vpb(cols));
    return std::max(1, std::min(64, (rows + per - 1) / per));
}

int colsum_jobs_add(ColsumJobs& js, int rows, int cols, bool bf16, size_t part_off, size_t part2_off, size_t out_off) {
    if (js.n >= kMaxColsumJobs || (cols & 3) != 0 || rows < 1) return -1;
    ColsumJob& jb = js.job[js.n];
    jb.rows = rows; jb.cols = cols; jb.chunks = colsum_chunks(rows, cols); jb.bf16 = bf16 ? 1 : 0;
    jb.part_off = part_off; jb.part2_off = part2_off; jb.out_off = out_off;
    const int cv = cols / 4, vpb = colsum_vpb(cols);
    if (js.n == 0) js.first[0] = 0;
    js.first[js.n + 1] = js.first[js.n] + jb.chunks * ((cv + vpb - 1) / vpb);
    return js.n++;
}

int launch_colsum_multi(const ColsumJobs& js, void* base, hipStream_t st) {
    if (js.n < 1) return WAP_OK;
    hipLaunchKernelGGL(colsum_multi_kernel, dim3(js.first[js.n]), dim3(256), 0, st, js, (unsigned char*)base);
    int rc = check_launch("colsum_multi");
    if (rc != WAP_OK) return rc;
    int vecs = 0;
    for (int j = 0; j < js.n; ++j) vecs += js.job[j].cols / 4;
    hipLaunchKernelGGL(colsum_finish_kernel, dim3((vecs + 15) / 16), dim3(256), 0, st, js, (unsigned char*)base);
    return check_launch("colsum_finish");
}

// How the first stage is laid out: 16-byte vectors where the row length allows it (8-byte, else 2-byte).  A few rows are
// summed in one chunk, whose sums are the result (no second launch of about 4.6 us): up to 512 rows, and
// while a thread of a 1024-thread work-group walks at most 16 rows, i.e. two batches of loads.  Up to 16 vectors (64 elements)
// lie side by side: 256-byte runs of a row, fewer threads per row mean more rows in flight and more work-groups.  More rows
// are divided into chunks of 16 rows per thread of 256-thread work-groups.  Rows that are no whole 128-byte lines go to a
// work-group in one piece there, 32 rows per thread: narrower blocks fetch their border lines twice, from two L2s (50176 x 1000
// 28.5 us in 256-byte runs, 21.6 in whole rows; 802816 x 200 80 and 59; 12544 x 500, where the fetches hide, 7.0 and 7.6).
struct BiasGradShape {
    int vecw, vpb, colblocks, chunks, rp;
    size_t rpc;  // rows per chunk
};
static BiasGradShape bias_grad_shape(size_t rows, int cols) {
    BiasGradShape b;
    b.vecw = (cols & 7) == 0 ? 8 : (cols & 3) == 0 ? 4 : 1;
    const int cv = cols / b.vecw;
    auto blocks = [&](int most) {
        b.colblocks = (cv + most - 1) / most;
        b.vpb = (cv + b.colblocks - 1) / b.colblocks;
    };
    blocks(b.vecw == 1 ? 64 : 16);
    b.chunks = 1;
    b.rpc = rows;
    b.rp = 1024 / b.vpb;
    if (rows > 512 && rows > (size_t)16 * b.rp) {
        const bool lines = (cols & 63) == 0;
        if (!lines) blocks(b.vecw == 1 ? 256 : 128);
        b.rp = 256 / b.vpb;
        const size_t per = (size_t)(lines ? 16 : 32) * b.rp;
        size_t cap = (size_t)kNumCU * 8 / b.colblocks;  // at most ~8 work-groups per CU
        if (cap < 1) cap = 1;
        b.chunks = (int)std::min((rows + per - 1) / per, cap);
        b.rpc = (rows + b.chunks - 1) / b.chunks;
    }
    b.rp = (int)std::min<size_t>((size_t)b.rp, (b.rpc + 7) / 8);  // one batch of loads is enough: a shorter tree
    return b;
}
int bias_grad_chunks(size_t rows, int cols) { return bias_grad_shape(rows, cols).chunks; }

int launch_bias_grad(size_t rows, int cols, const bf16_t* dy, float* db, float* part, hipStream_t st) {
    const BiasGradShape b = bias_grad_shape(rows, cols);
    float* dst = b.chunks == 1 ? db : part;  // a single chunk writes the result itself
    const dim3 grid(b.colblocks, b.chunks), block((b.vpb * b.rp + 63) / 64 * 64);
    if (b.vecw == 8)
        hipLaunchKernelGGL(bias_grad_kernel<8>, grid, block, 0, st, dy, dst, (uint32_t)rows, (uint32_t)cols, (uint32_t)b.rpc, b.vpb, b.rp);
    else if (b.vecw == 4)
        hipLaunchKernelGGL(bias_grad_kernel<4>, grid, block, 0, st, dy, dst, (uint32_t)rows, (uint32_t)cols, (uint32_t)b.rpc, b.vpb, b.rp);
    else
        hipLaunchKernelGGL(bias_grad_kernel<1>, grid, block, 0, st, dy, dst, (uint32_t)rows, (uint32_t)cols, (uint32_t)b.rpc, b.vpb, b.rp);
    int rc = check_launch("bias_grad");
    if (rc != WAP_OK || b.chunks == 1) return rc;
    return launch_reduce_f32(part, b.chunks, (size_t)cols, db, st);
}

int launch_relu_bwd(const bf16_t* dy, const bf16_t* y, bf16_t* dx, size_t n, hipStream_t st) {
    // (us through / past the cache: 46 M elements 39.7 / 42.4, 50 M 46.2 / 46.4, 56 M 56.3 / 52.1; in place 76 M 65.3 / 69.7, 88 M 82.3 / 80.1, 96 M 97 / 87)
    const bool once = beyond_cache((dy == dx ? 3.0 : 5.35) * n);
    in_pieces(n, 8, once ? 0 : kWalk, [&](size_t at, size_t m, dim3 grid, bool walks) {
        if (once) hipLaunchKernelGGL((relu_bwd_kernel<true, false>), grid, dim3(kThreads), 0, st, dy + at, y + at, dx + at, m);
        else if (walks) hipLaunchKernelGGL((relu_bwd_kernel<false, true>), grid, dim3(kThreads), 0, st, dy + at, y + at, dx + at, m);
        else hipLaunchKernelGGL((relu_bwd_kernel<false, false>), grid, dim3(kThreads), 0, st, dy + at, y + at, dx + at, m);
    });
    return check_launch("relu_bwd");
}

// items = one per channel vector of `rows` x `cols` positions per image
static PoolArgs pool_args(int N, int H, int W, int C, int win, int st, int vec, int rows, int cols) {
    PoolArgs a;
    a.H = H; a.W = W; a.C = C; a.st = st;
    a.P = (H - win) / st + 1;
    a.Q = (W - win) / st + 1;
    a.items = (uint32_t)((size_t)N * rows * cols * (C / vec));
    a.dCV = make_fastdiv((uint32_t)(C / vec));
    a.dX = make_fastdiv((uint32_t)cols);
    a.dY = make_fastdiv((uint32_t)rows);
    return a;
}

int launch_maxpool_fwd(int N, int H, int W, int C, int win, int stp, const bf16_t* x, bf16_t* y,
                       uint8_t* am, hipStream_t st) {
    const int vec = (C & 7) == 0 ? 8 : 1;
    const PoolArgs a = pool_args(N, H, W, C, win, stp, vec, (H - win) / stp + 1, (W - win) / stp + 1);
    // (element by element they walk: 256 x 70 x 70 x 45, window 2, 34.4 us, 43.5 with an item a thread, 28 x 87 x 87 x 81, stride 1, 37.4 / 48.3)
    const dim3 grid(grid_for(a.items, vec == 8 ? 0 : SIZE_MAX)), block(kThreads);
    if (win != 2 && win != 3) {
        if (vec == 8) hipLaunchKernelGGL(maxpool_fwd_any_kernel<8>, grid, block, 0, st, x, y, am, win, a);
        else hipLaunchKernelGGL(maxpool_fwd_any_kernel<1>, grid, block, 0, st, x, y, am, win, a);
    } else if (vec == 8 && win == 2) hipLaunchKernelGGL((maxpool_fwd_kernel<8, 2>), grid, block, 0, st, x, y, am, a);
    else if (vec == 8) hipLaunchKernelGGL((maxpool_fwd_kernel<8, 3>), grid, block, 0, st, x, y, am, a);
    else if (win == 2) hipLaunchKernelGGL((maxpool_fwd_kernel<1, 2>), grid, block, 0, st, x, y, am, a);
    else hipLaunchKernelGGL((maxpool_fwd_kernel<1, 3>), grid, block, 0, st, x, y, am, a);
    return check_launch("maxpool_fwd");
}

// Two items a thread, so that the partial rows are fewer than the work-groups in flight (100 x 55 x 55 x 64, window 3: 1225 rows).
static int pool_colsum_threads(int C) { return kThreads / (C / 8) * (C / 8); }
int maxpool_bwd_colsum_rows(int N, int H, int W, int C, int win, int stp) {
    if (stp != 2 || (win != 2 && win != 3) || (C & 7) != 0 || C > kThreads * 4) return 0;
    const size_t items = (size_t)N * ((H + 1) / 2) * ((W + 1) / 2) * (C / 8), per = 2 * pool_colsum_threads(C);
    return (int)std::min((items + per - 1) / per, (size_t)1 << 22);
}

int launch_maxpool_bwd(int N, int H, int W, int C, int win, int stp, const bf16_t* dy, const uint8_t* am,
                       const bf16_t* ry, bf16_t* dx, hipStream_t st, float* colsum, const LossMean* mean) {
    const int vec = (C & 7) == 0 ? 8 : 1;
    const dim3 block(kThreads);
    const LossMean lm = mean ? *mean : LossMean{nullptr, nullptr, 0};
    const int rows = maxpool_bwd_colsum_rows(N, H, W, C, win, stp);
    if ((colsum || mean) && !rows) return set_error(WAP_EINVAL, "internal: no column sums from this max-pool");
    if (stp == 2 && (win == 2 || win == 3)) {
        const PoolArgs a = pool_args(N, H, W, C, win, stp, vec, (H + 1) / 2, (W + 1) / 2);
        // (walking element by element as in the forward pass: 256 x 49 x 49 x 42, window 2, 35.0 / 38.8)
        const dim3 grid((colsum ? rows : grid_for(a.items, vec == 8 ? 0 : SIZE_MAX)) + (mean ? 1 : 0));
        const dim3 threads(colsum ? pool_colsum_threads(C) : kThreads);
#define WAP_POOL_SUMS(COLSUM, MEAN)                                                                                                             \
    hipLaunchKernelGGL((win == 2 ? maxpool_bwd_s2_sums_kernel<2, COLSUM, MEAN> : maxpool_bwd_s2_sums_kernel<3, COLSUM, MEAN>), grid, threads, 0, \
                       st, dy, am, ry, dx, a, threads.x, colsum, lm)
        if (colsum && mean) WAP_POOL_SUMS(true, true);
        else if (colsum) WAP_POOL_SUMS(true, false);
        else if (mean) WAP_POOL_SUMS(false, true);
        else if (vec == 8) hipLaunchKernelGGL((win == 2 ? maxpool_bwd_s2_kernel<8, 2> : maxpool_bwd_s2_kernel<8, 3>), grid, threads, 0, st, dy, am, ry, dx, a);
        else hipLaunchKernelGGL((win == 2 ? maxpool_bwd_s2_kernel<1, 2> : maxpool_bwd_s2_kernel<1, 3>), grid, threads, 0, st, dy, am, ry, dx, a);
#undef WAP_POOL_SUMS
        return check_launch("maxpool_bwd");
    }
    const PoolArgs a = pool_args(N, H, W, C, win, stp, vec, H, W);
    const dim3 grid(grid_for(a.items, 0));
    if (vec == 8) hipLaunchKernelGGL(maxpool_bwd_kernel<8>, grid, block, 0, st, dy, am, ry, dx, win, a);
    else hipLaunchKernelGGL(maxpool_bwd_kernel<1>, grid, block, 0, st, dy, am, ry, dx, win, a);
    return check_launch("maxpool_bwd");
}

int launch_softmax_xent(int B, int classes, const bf16_t* z, const int32_t* labels, float* loss,
                        float* row_loss, bf16_t* dz, hipStream_t st) {
    hipLaunchKernelGGL(softmax_xent_kernel, dim3(B), dim3(256), 0, st, z, labels, B, classes, row_loss, dz);
    int rc = check_launch("softmax_xent");
    if (rc != WAP_OK || !loss) return rc;
    hipLaunchKernelGGL(loss_mean_kernel, dim3(1), dim3(kThreads), 0, st, LossMean{row_loss, loss, B});
    return check_launch("loss_mean");
}

// Update of a call of its own, us through / past the cache: 24 M weights 47.4 / 50.7, 32 M 64.7 / 67.2, 36 M 73.5 / 74.0, 40 M 93.5 / 83.8; without a
// bf16 copy 28 M 46.5 / 51.6, 44 M 76.9 / 80.4, 46 M 87.4 / 84.0.
bool sgd_once(size_t n, bool copy) { return beyond_cache((copy ? 7.4 : 5.95) * n); }

int launch_sgd(size_t n, float* w, const float* dw, float lr, bf16_t* wb, bool once, hipStream_t st) {
    in_pieces(n, 4, once ? 0 : kWalk, [&](size_t at, size_t m, dim3 grid, bool walks) {
        bf16_t* const b = wb ? wb + at : nullptr;
        if (once) hipLaunchKernelGGL((sgd_kernel<true, false>), grid, dim3(kThreads), 0, st, m, w + at, dw + at, lr, b);
        else if (walks) hipLaunchKernelGGL((sgd_kernel<false, true>), grid, dim3(kThreads), 0, st, m, w + at, dw + at, lr, b);
        else hipLaunchKernelGGL((sgd_kernel<false, false>), grid, dim3(kThreads), 0, st, m, w + at, dw + at, lr, b);
    });
    return check_launch("sgd");
}

int launch_cast(size_t n, const float* src, bf16_t* dst, hipStream_t st) {
    // (us walking / one vector a thread: 8.7 M elements 11.8 / 12.6, 13.1 M 16.3 / 17.6, 52 M 48.8 / 52.5, 64 M 68 / 66, 103 M 118 / 106)
    hipLaunchKernelGGL(cast_kernel, dim3(grid_for(n / 4 + 1, (size_t)15 << 20)), dim3(kThreads), 0, st, n, src, dst);
    return check_launch("cast");
}

}  // namespace wap
