// Elementwise glue and small reductions: GELU (erf form) forward/backward, column sums for the
// bias gradient, and the fixed-order sum of split-K partial products.
#include <algorithm>

#include "lrd_internal.hpp"
#include "lrd_measure.h"

namespace lrd {
namespace {

// 8 bf16 (16 bytes) per thread per step; n8 = number of whole groups of 8.
__global__ __launch_bounds__(256) void gelu_fwd_bf16(const bf16_t* __restrict__ Z, bf16_t* __restrict__ A, int64_t n)
{
    int64_t n8 = n / 8;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < n8; g += stride) {
        bf16x8 z = *reinterpret_cast<const bf16x8*>(Z + g * 8);
        bf16x8 a;
#pragma unroll
        for (int e = 0; e < 8; ++e) a[e] = (bf16_t)gelu_bf16_f((float)z[e]);
        *reinterpret_cast<bf16x8*>(A + g * 8) = a;
    }
    if (blockIdx.x == 0 && threadIdx.x < n - n8 * 8) {
        int64_t i = n8 * 8 + threadIdx.x;
        A[i] = (bf16_t)gelu_bf16_f((float)Z[i]);
    }
}

__global__ __launch_bounds__(256) void gelu_bwd_bf16(const bf16_t* dA, const bf16_t* __restrict__ Z,
                                                     bf16_t* dZ, int64_t n)   // dZ may alias dA
{
    int64_t n8 = n / 8;
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < n8; g += stride) {
        bf16x8 z = *reinterpret_cast<const bf16x8*>(Z + g * 8);
        bf16x8 d = *reinterpret_cast<const bf16x8*>(dA + g * 8);
        bf16x8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = (bf16_t)((float)d[e] * gelu_grad_bf16_f((float)z[e]));
        *reinterpret_cast<bf16x8*>(dZ + g * 8) = o;
    }
    if (blockIdx.x == 0 && threadIdx.x < n - n8 * 8) {
        int64_t i = n8 * 8 + threadIdx.x;
        dZ[i] = (bf16_t)((float)dA[i] * gelu_grad_bf16_f((float)Z[i]));
    }
}

__global__ __launch_bounds__(256) void gelu_fwd_f32(const float* __restrict__ Z, float* __restrict__ A, int64_t n)
{
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) A[i] = gelu_f(Z[i]);
}

__global__ __launch_bounds__(256) void gelu_bwd_f32(const float* dA, const float* __restrict__ Z,
                                                    float* dZ, int64_t n)   // dZ may alias dA
{
    int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        dZ[i] = dA[i] * gelu_grad_f(Z[i]);
}

// Sums over rows, the bias gradient: partial[blockIdx.y][c] = sum of dY[t][c] over the block's run of rows.
// A pure stream of dY, so what counts is having enough 16-byte loads in flight: VEC consecutive columns
// per thread (16 bytes; 1 where the row length does not allow it), CS_COLS threads side by side and
// 256 / CS_COLS rows at a time, on a grid that cuts the rows as well as the columns.  (One block per 64
// columns walking all rows, as this was, left most compute units idle and each thread with one 2-byte load
// outstanding: 497 us for 8192 x 768, 294 us for 4100 x 4096 in bf16, against about 4 us and 9 us with the sum of
// the partial rows included.)
constexpr int CS_COLS = 32;
template <class T, int VEC>
__global__ __launch_bounds__(256) void column_sums_kernel(const T* __restrict__ dY, float* __restrict__ partial, int64_t Tn, int64_t n,
                                                          int rows_per_block)
{
    constexpr int RL = 256 / CS_COLS;
    __shared__ float part[RL][CS_COLS][VEC + 1];
    const int cl = threadIdx.x % CS_COLS, rl = threadIdx.x / CS_COLS;
    const int64_t col = ((int64_t)blockIdx.x * CS_COLS + cl) * VEC;
    const int64_t t1 = min((int64_t)(blockIdx.y + 1) * rows_per_block, Tn);
    float s[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) s[e] = 0.f;
    if (col < n) {
#pragma unroll 4
        for (int64_t t = (int64_t)blockIdx.y * rows_per_block + rl; t < t1; t += RL) {
            if constexpr (VEC * sizeof(T) == 16) {
                typedef T TV __attribute__((ext_vector_type(VEC)));
                const TV v = *reinterpret_cast<const TV*>(dY + t * n + col);
#pragma unroll
                for (int e = 0; e < VEC; ++e) s[e] += to_f32((T)v[e]);
            } else {
                s[0] += to_f32(dY[t * n + col]);
            }
        }
    }
#pragma unroll
    for (int e = 0; e < VEC; ++e) part[rl][cl][e] = s[e];
    __syncthreads();
    // one thread per column of the block, row lanes in ascending order
    for (int c = threadIdx.x; c < CS_COLS * VEC; c += 256) {
        const int64_t out = (int64_t)blockIdx.x * CS_COLS * VEC + c;
        if (out >= n) break;
        float v = 0.f;
#pragma unroll
        for (int r = 0; r < RL; ++r) v += part[r][c / VEC][c % VEC];
        partial[(int64_t)blockIdx.y * n + out] = v;
    }
}

// The optimizer step of sgd_step_kernel on four consecutive weights whose gradient g has just been
// summed (same arithmetic, so that a step does not depend on where it ran).
struct SgdArgs { float* w; float* m; void* copy; int copy_bf16; float lr, mu, wd; };
__device__ __forceinline__ void sgd_apply4(const SgdArgs& a, int64_t i, f32x4 g)
{
    f32x4 w = *reinterpret_cast<const f32x4*>(a.w + i), m = *reinterpret_cast<const f32x4*>(a.m + i);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        m[e] = fmaf(a.mu, m[e], fmaf(a.wd, w[e], g[e]));
        w[e] = fmaf(-a.lr, m[e], w[e]);
    }
    *reinterpret_cast<f32x4*>(a.m + i) = m;
    *reinterpret_cast<f32x4*>(a.w + i) = w;
    if (a.copy) {
        if (a.copy_bf16) {
            u32x2 pk = {pack_bf16(w[0], w[1]), pack_bf16(w[2], w[3])};
            *reinterpret_cast<u32x2*>(reinterpret_cast<bf16_t*>(a.copy) + i) = pk;
        } else {
            *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(a.copy) + i) = w;
        }
    }
}

// Four consecutive columns of a padded gradient to their place in the cropped one (CropFuse).
struct CropArgs { float* dst; int rows, inner, inner_keep; };
__device__ __forceinline__ void crop_store4(const CropArgs& c, int64_t i, int64_t N, f32x4 v)
{
    typedef f32x4 f32x4u __attribute__((aligned(4)));
    const int m = (int)(i / N), n = (int)(i - (int64_t)m * N);
    const int b = n / c.inner, q = n - b * c.inner, blocks = (int)(N / c.inner);
    if (m >= c.rows) return;
    float* at = c.dst + ((int64_t)m * blocks + b) * c.inner_keep + q;
    if (q + 4 <= c.inner_keep) {
        *reinterpret_cast<f32x4u*>(at) = v;
    } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (q + e < c.inner_keep) at[e] = v[e];
    }
}

enum { SUM_STORE = 0, SUM_SGD = 1, SUM_CROP = 2 };

// C[m][n] = sum_z partial[z][m][n], slices added in ascending z so the result does not depend on
// scheduling.  VEC consecutive columns per thread (N and ldc are multiples of VEC); OutT is the
// result type (fp32 weight gradients, or bf16 activations rounded once from the fp32 sum).
// With SUM_SGD (VEC == 4, fp32, ldc == N) the sum feeds the optimizer step and is not stored, with SUM_CROP
// (VEC == 4, fp32) it goes to its place in a smaller matrix.
template <int VEC, class OutT, int TO = SUM_STORE>
__global__ __launch_bounds__(256) void reduce_partials_kernel(const float* __restrict__ partial, OutT* __restrict__ C,
                                                              int64_t ldc, int64_t M, int64_t N, int splits, SgdArgs sgd = SgdArgs{},
                                                              CropArgs crop = CropArgs{})
{
    const int64_t total = M * N;
    const int64_t groups = total / VEC;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < groups; g += stride) {
        const int64_t i = g * VEC;
        float s[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) s[e] = 0.f;
        for (int z = 0; z < splits; ++z) {
            const float* p = partial + (int64_t)z * total + i;
            if constexpr (VEC % 4 == 0) {
#pragma unroll
                for (int q = 0; q < VEC / 4; ++q) {
                    f32x4 v = *reinterpret_cast<const f32x4*>(p + 4 * q);
                    s[4 * q] += v.x; s[4 * q + 1] += v.y; s[4 * q + 2] += v.z; s[4 * q + 3] += v.w;
                }
            } else {
#pragma unroll
                for (int e = 0; e < VEC; ++e) s[e] += p[e];
            }
        }
        OutT* out = C + (i / N) * ldc + (i % N);
        if constexpr (VEC == 8 && sizeof(OutT) == 2) {
            u32x4 pk = {pack_bf16(s[0], s[1]), pack_bf16(s[2], s[3]), pack_bf16(s[4], s[5]), pack_bf16(s[6], s[7])};
            *reinterpret_cast<u32x4*>(out) = pk;
        } else if constexpr (VEC == 4 && sizeof(OutT) == 4) {
            f32x4 v = {s[0], s[1], s[2], s[3]};
            if constexpr (TO == SUM_SGD) sgd_apply4(sgd, i, v);
            else if constexpr (TO == SUM_CROP) crop_store4(crop, i, N, v);
            else *reinterpret_cast<f32x4*>(out) = v;
        } else {
#pragma unroll
            for (int e = 0; e < VEC; ++e) out[e] = from_f32<OutT>(s[e]);
        }
    }
}

// The same sum for small fp32 results cut into many slices (weight gradients of narrow layers, whose
// reduction runs over all pixels): one thread per output would leave most of the chip idle and walk
// the slices one after the other, so LANES threads share a group of 4 outputs, thread l adds slices
// l, l + LANES, ... in ascending order and the LANES sums are combined by a pairwise tree.  Still a
// fixed order.
template <int LANES, int TO = SUM_STORE>
__global__ __launch_bounds__(256) void reduce_partials_wide_kernel(const float* __restrict__ partial, float* __restrict__ C,
                                                                   int64_t ldc, int64_t M, int64_t N, int splits,
                                                                   SgdArgs sgd = SgdArgs{}, CropArgs crop = CropArgs{})
{
    constexpr int GROUPS = 256 / LANES;       // groups of 4 outputs per block
    __shared__ f32x4 part[LANES][GROUPS + 1];
    const int64_t total = M * N, groups = total / 4;
    const int gl = threadIdx.x % GROUPS, l = threadIdx.x / GROUPS;
    const int64_t g = (int64_t)blockIdx.x * GROUPS + gl;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    if (g < groups)
        for (int z = l; z < splits; z += LANES) s += *reinterpret_cast<const f32x4*>(partial + (int64_t)z * total + g * 4);
    part[l][gl] = s;
    __syncthreads();
    // pairwise tree over the LANES sums (lane l takes in lane l + half): one fixed order again
#pragma unroll
    for (int half = LANES / 2; half >= 1; half /= 2) {
        if (l < half) part[l][gl] += part[l + half][gl];
        __syncthreads();
    }
    if (l == 0 && g < groups) {
        const f32x4 t = part[0][gl];
        const int64_t i = g * 4;
        if constexpr (TO == SUM_SGD) sgd_apply4(sgd, i, t);
        else if constexpr (TO == SUM_CROP) crop_store4(crop, i, N, t);
        else *reinterpret_cast<f32x4*>(C + (i / N) * ldc + (i % N)) = t;
    }
}

// Several of these sums in one launch (SumQueue), each with the lanes that reduce_partials would give it and in the same order.
// Alone they are 3 to 6 us each, half of it the launch: 4100 x 1024 x 4096 layer at rank 257 (dU, dV and the bias gradient) 128 -> 123.6
// us, 8192 x 3072 x 768 with bias and update 85 -> 82.3 us, 64-channel convolution 136 -> 133 us, 512-channel one 159.5 -> 156.6 us.
struct SumArgs {
    struct Task { const float* partial; float* C; int64_t ldc, N, groups; int splits, lanes, to; SgdArgs sgd; CropArgs crop; } task[SumQueue::MOST];
    uint32_t first_block[SumQueue::MOST];
};
__device__ __forceinline__ void finish_sum(const SumArgs::Task& t, int64_t g, f32x4 v)
{
    const int64_t i = g * 4;
    if (t.to == SUM_SGD) sgd_apply4(t.sgd, i, v);
    else if (t.to == SUM_CROP) crop_store4(t.crop, i, t.N, v);
    else *reinterpret_cast<f32x4*>(t.C + (i / t.N) * t.ldc + (i % t.N)) = v;
}
template <int LANES>
__device__ __forceinline__ void wide_sum(const SumArgs::Task& t, uint32_t block, f32x4* part)
{
    constexpr int GROUPS = 256 / LANES;
    const int gl = threadIdx.x % GROUPS, l = threadIdx.x / GROUPS;
    const int64_t g = (int64_t)block * GROUPS + gl, total = t.groups * 4;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    if (g < t.groups)
        for (int z = l; z < t.splits; z += LANES) s += *reinterpret_cast<const f32x4*>(t.partial + (int64_t)z * total + g * 4);
    part[l * (GROUPS + 1) + gl] = s;
    __syncthreads();
#pragma unroll
    for (int half = LANES / 2; half >= 1; half /= 2) {
        if (l < half) part[l * (GROUPS + 1) + gl] += part[(l + half) * (GROUPS + 1) + gl];
        __syncthreads();
    }
    if (l == 0 && g < t.groups) finish_sum(t, g, part[gl]);
}
__global__ __launch_bounds__(256) void sums_kernel(SumArgs a)
{
    __shared__ f32x4 part[64 * 5];      // 16 x 17 or 64 x 5
    int k = 0;
#pragma unroll
    for (int q = 1; q < SumQueue::MOST; ++q) k += blockIdx.x >= a.first_block[q];
    const SumArgs::Task& t = a.task[k];
    const uint32_t block = blockIdx.x - a.first_block[k];
    if (t.lanes == 64) return wide_sum<64>(t, block, part);
    if (t.lanes == 16) return wide_sum<16>(t, block, part);
    const int64_t g = (int64_t)block * 256 + threadIdx.x, total = t.groups * 4;
    if (g >= t.groups) return;
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 4
    for (int z = 0; z < t.splits; ++z) s += *reinterpret_cast<const f32x4*>(t.partial + (int64_t)z * total + g * 4);
    finish_sum(t, g, s);
}

// Zero-padding / cropping copies between dense row-major matrices, up to COPY_JOBS of them in one launch (the
// factors, intermediates and gradients of a raw rank): dst[i][j] = src[i][j] where that exists, else 0.
// Each is a few hundred KB to a few MB: a launch costs more than the bytes of one, so those of a pass share a launch,
// and the loads are 16 bytes wide wherever the row starts (2-byte loads, 16 bytes apart between lanes, took a clock
// per lane).  Forward + backward of a 4100 x 1024 x 4096 layer at rank 257: 39 us of copies as eight launches of a
// kernel with one element and one 64-bit division per thread, 16 us as three of this one, the gradients being
// cropped where their K-slices are summed; the 512-channel 7 x 7 convolution at rank 309: 54 against 20 us.
// A thread writes 16 bytes of the dense destination and finds the row of its first element by one 32-bit division.
struct CopyArgs {
    struct Job { const void* src; void* dst; uint32_t rows_s, cols_s, cols_d, total; int elem_bytes; } job[COPY_JOBS];
    uint32_t first_block[COPY_JOBS];
};
template <class T>
__device__ __forceinline__ void copy_chunk(const CopyArgs::Job& c, uint32_t e)
{
    constexpr uint32_t V = 16 / sizeof(T);
    typedef T TV __attribute__((ext_vector_type(V)));
    typedef TV TU __attribute__((aligned(sizeof(T))));          // a vector at any element
    const T* src = reinterpret_cast<const T*>(c.src);
    T* dst = reinterpret_cast<T*>(c.dst);
    const uint32_t i = e / c.cols_d, j = e - i * c.cols_d, left = c.cols_d - j, total_s = c.rows_s * c.cols_s;
    const uint32_t from = i * c.cols_s + j;                     // the first element; those past the row end (from element
    const uint32_t from2 = from + c.cols_s - c.cols_d;          // `left` on) lie as if the next row began there
    const bool wraps = c.cols_d % V != 0;
    TV v;
    if (c.cols_d >= V && (!wraps || c.cols_s >= c.cols_d) && (wraps ? from2 : from) + V <= total_s) {
        v = *reinterpret_cast<const TU*>(src + from);
        if (wraps) {
            const TV w = *reinterpret_cast<const TU*>(src + from2);
#pragma unroll
            for (uint32_t q = 0; q < V; ++q) v[q] = q < left ? v[q] : w[q];
        } else if (c.cols_s < c.cols_d) {
#pragma unroll
            for (uint32_t q = 0; q < V; ++q) v[q] = j + q < c.cols_s ? v[q] : (T)0.f;
        }
    } else {
        // the last row or two, and rows of less than 16 bytes
        uint32_t ii = i, jj = j;
#pragma unroll
        for (uint32_t q = 0; q < V; ++q) {
            v[q] = ii < c.rows_s && jj < c.cols_s ? src[ii * c.cols_s + jj] : (T)0.f;
            if (++jj == c.cols_d) { jj = 0; ++ii; }
        }
    }
    if (e + V <= c.total) {
        *reinterpret_cast<TV*>(dst + e) = v;
    } else {
#pragma unroll
        for (uint32_t q = 0; q < V; ++q)
            if (e + q < c.total) dst[e + q] = v[q];
    }
}
constexpr uint32_t COPY_RUN = 2;      // 16-byte groups per thread: a block is 8 KB of one destination
__global__ __launch_bounds__(256) void copy2d_kernel(CopyArgs a)
{
    int k = 0;
#pragma unroll
    for (int q = 1; q < COPY_JOBS; ++q) k += blockIdx.x >= a.first_block[q];
    const CopyArgs::Job c = a.job[k];
    const uint32_t g0 = (blockIdx.x - a.first_block[k]) * (256 * COPY_RUN) + threadIdx.x;
#pragma unroll
    for (uint32_t q = 0; q < COPY_RUN; ++q) {
        const uint32_t g = g0 + q * 256;
        if (c.elem_bytes == 2) {
            if (g * 8 < c.total) copy_chunk<bf16_t>(c, g * 8);
        } else {
            if (g * 4 < c.total) copy_chunk<float>(c, g * 4);
        }
    }
}

// w <- w - lr * (m <- mu * m + (g + wd * w)) on fp32 master weights; the compute copy (bf16 or fp32,
// optional) is refreshed from the new master value.
__global__ __launch_bounds__(256) void sgd_step_kernel(float* __restrict__ w, float* __restrict__ m, const float* __restrict__ g,
                                                       void* copy, bool copy_bf16, int64_t n, float lr, float mu, float wd)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
        const float wi = w[i];
        const float mi = fmaf(mu, m[i], fmaf(wd, wi, g[i]));
        const float wn = fmaf(-lr, mi, wi);
        m[i] = mi;
        w[i] = wn;
        if (copy) {
            if (copy_bf16) reinterpret_cast<bf16_t*>(copy)[i] = (bf16_t)wn;
            else reinterpret_cast<float*>(copy)[i] = wn;
        }
    }
}

// wt[i][k*k - 1 - t][o] = w[o][t][i]: the weights with which the data gradient of a stride-1
// convolution is itself a forward convolution (of dY, with padding k - 1 - pad).
__global__ __launch_bounds__(256) void flip_conv_weights_kernel(const bf16_t* __restrict__ w, bf16_t* __restrict__ wt, int O, int I,
                                                                int kk)
{
    const int total = O * kk * I;
    for (int e = blockIdx.x * 256 + threadIdx.x; e < total; e += gridDim.x * 256) {
        const int i = e / (kk * O), rem = e - i * kk * O;
        const int tf = rem / O, o = rem - tf * O;
        wt[e] = w[((int64_t)o * kk + (kk - 1 - tf)) * I + i];
    }
}

inline unsigned blocks_for(int64_t items)
{
    int64_t b = ceil_div(items, 256);
    if (b < 1) b = 1;
    if (b > 256 * 16) b = 256 * 16;
    return (unsigned)b;
}

}  // namespace

hipError_t gelu_fwd(const void* Z, void* A, int64_t n, bool bf16, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    if (bf16) hipLaunchKernelGGL(gelu_fwd_bf16, dim3(blocks_for(n / 8 + 1)), dim3(256), 0, st, (const bf16_t*)Z, (bf16_t*)A, n);
    else hipLaunchKernelGGL(gelu_fwd_f32, dim3(blocks_for(n)), dim3(256), 0, st, (const float*)Z, (float*)A, n);
    return hipGetLastError();
}

hipError_t gelu_bwd(const void* dA, const void* Z, void* dZ, int64_t n, bool bf16, hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    if (bf16) hipLaunchKernelGGL(gelu_bwd_bf16, dim3(blocks_for(n / 8 + 1)), dim3(256), 0, st, (const bf16_t*)dA, (const bf16_t*)Z, (bf16_t*)dZ, n);
    else hipLaunchKernelGGL(gelu_bwd_f32, dim3(blocks_for(n)), dim3(256), 0, st, (const float*)dA, (const float*)Z, (float*)dZ, n);
    return hipGetLastError();
}

namespace {
inline int64_t column_sum_width(const void* dY, int64_t n, bool bf16)
{
    return n % (bf16 ? 8 : 4) == 0 && (reinterpret_cast<uintptr_t>(dY) & 15u) == 0 ? (bf16 ? 8 : 4) : 1;
}
}  // namespace

int64_t column_sum_rows(const void* dY, int64_t T, int64_t n, bool bf16, size_t scratch_bytes, int64_t* partials)
{
    // about 512 blocks of at least 32 rows each, as far as the partial rows fit the scratch (without any, one
    // run of rows goes straight to the result)
    int64_t rb = std::min(ceil_div(512, ceil_div(n, CS_COLS * column_sum_width(dY, n, bf16))), ceil_div(T, 32));
    rb = std::max<int64_t>(1, std::min<int64_t>(rb, (int64_t)(scratch_bytes / ((size_t)n * sizeof(float)))));
    const int64_t rows = ceil_div(T, rb);
    *partials = ceil_div(T, rows);
    return rows;
}

hipError_t column_sums(const void* dY, float* out, int64_t T, int64_t n, bool bf16, void* scratch, size_t scratch_bytes, hipStream_t st, SumQueue* later)
{
    if (n <= 0) return hipSuccess;
    const int64_t vec = column_sum_width(dY, n, bf16), cb = ceil_div(n, CS_COLS * vec);
    int64_t rb;
    const int64_t rows = column_sum_rows(dY, T, n, bf16, scratch ? scratch_bytes : 0, &rb);
    if (rows >= (int64_t(1) << 31) || cb >= (int64_t(1) << 31)) return hipErrorInvalidValue;
    float* partial = rb > 1 ? (float*)scratch : out;
    const dim3 grid((unsigned)cb, (unsigned)rb);
    if (bf16 && vec == 8) hipLaunchKernelGGL((column_sums_kernel<bf16_t, 8>), grid, dim3(256), 0, st, (const bf16_t*)dY, partial, T, n, (int)rows);
    else if (bf16) hipLaunchKernelGGL((column_sums_kernel<bf16_t, 1>), grid, dim3(256), 0, st, (const bf16_t*)dY, partial, T, n, (int)rows);
    else if (vec == 4) hipLaunchKernelGGL((column_sums_kernel<float, 4>), grid, dim3(256), 0, st, (const float*)dY, partial, T, n, (int)rows);
    else hipLaunchKernelGGL((column_sums_kernel<float, 1>), grid, dim3(256), 0, st, (const float*)dY, partial, T, n, (int)rows);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || rb == 1) return e;
    if (put_off(later, partial, out, false, n, 1, n, (int)rb)) return hipSuccess;
    return reduce_partials(partial, out, false, n, 1, n, (int)rb, st);
}

hipError_t copy2d(const CopyJob* jobs, int n, hipStream_t st)
{
    CopyArgs a;
    int used = 0;
    uint32_t blocks = 0;
    auto launch = [&] {
        if (used == 0) return hipSuccess;
        for (int i = used; i < COPY_JOBS; ++i) a.first_block[i] = 0xffffffffu;
        hipLaunchKernelGGL(copy2d_kernel, dim3(blocks), dim3(256), 0, st, a);
        used = 0;
        blocks = 0;
        return hipGetLastError();
    };
    for (int i = 0; i < n; ++i) {
        const CopyJob& j = jobs[i];
        if (j.cols_d <= 0) continue;
        // the kernel counts elements in 32 bits: longer matrices go in runs of rows (whole 16-byte groups each)
        const int64_t run = std::max<int64_t>(8, ((int64_t(1) << 31) / std::max(j.cols_d, j.cols_s)) & ~int64_t(7));
        for (int64_t r0 = 0; r0 < j.rows_d; r0 += run) {
            if (used == COPY_JOBS) {
                const hipError_t e = launch();
                if (e != hipSuccess) return e;
            }
            const int64_t rows_d = std::min(run, j.rows_d - r0), rows_s = std::max<int64_t>(0, std::min(run, j.rows_s - r0));
            a.job[used] = {(const char*)j.src + r0 * j.cols_s * j.elem_bytes, (char*)j.dst + r0 * j.cols_d * j.elem_bytes, (uint32_t)rows_s,
                           (uint32_t)j.cols_s, (uint32_t)j.cols_d, (uint32_t)(rows_d * j.cols_d), j.elem_bytes};
            a.first_block[used++] = blocks;
            blocks += (uint32_t)ceil_div(rows_d * j.cols_d, (int64_t)COPY_RUN * 256 * 16 / j.elem_bytes);
        }
    }
    return launch();
}

hipError_t flip_conv_weights(const void* w, void* wt, int O, int I, int k, hipStream_t st)
{
    const int64_t total = (int64_t)O * k * k * I;
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(flip_conv_weights_kernel, dim3(blocks_for(total)), dim3(256), 0, st, (const bf16_t*)w, (bf16_t*)wt, O, I, k * k);
    return hipGetLastError();
}

hipError_t sgd_step(float* w, float* m, const float* g, void* copy, bool copy_bf16, int64_t n, float lr, float mu, float wd,
                    hipStream_t st)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(sgd_step_kernel, dim3(blocks_for(n)), dim3(256), 0, st, w, m, g, copy, copy_bf16, n, lr, mu, wd);
    return hipGetLastError();
}

namespace {
inline bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
inline bool sgd_fits(const SgdFuse& s, int64_t ldc, int64_t N) { return ldc == N && al16(s.w) && al16(s.m) && al16(s.copy); }
inline bool crop_fits(const CropFuse& c, int64_t M, int64_t N)
{
    return M < (int64_t(1) << 31) && N < (int64_t(1) << 31) && N % c.inner == 0 && c.inner % 4 == 0;
}
// Threads that share a group of 4 outputs, for results of four-wide rows.
inline int sum_lanes(int64_t M, int64_t N, int splits) { return splits >= 64 && M * N / 4 <= 4096 ? 64 : splits >= 16 && M * N / 4 < 256 * 256 ? 16 : 1; }
}  // namespace

bool put_off(SumQueue* q, const float* partial, void* C, bool c_bf16, int64_t ldc, int64_t M, int64_t N, int splits, const SgdFuse* sgd, const CropFuse* crop)
{
    if (!q || q->n == SumQueue::MOST || c_bf16 || !al16(C) || !al16(partial) || N % 4 != 0 || ldc % 4 != 0 || M <= 0 || N <= 0) return false;
    if (sgd && (sgd->done || !sgd_fits(*sgd, ldc, N))) return false;
    if (crop && (crop->done || !crop_fits(*crop, M, N))) return false;
    if (ceil_div(M * N / 4, 4) >= (int64_t(1) << 28)) return false;
    SumTask& t = q->task[q->n++];
    t = {partial, (float*)C, ldc, M, N, splits, sgd ? *sgd : SgdFuse{}, crop ? *crop : CropFuse{}};
    if (sgd) sgd->done = true;
    if (crop) crop->done = true;
    return true;
}

hipError_t run_sums(SumQueue& q, hipStream_t st)
{
    if (q.n == 0) return hipSuccess;
    SumArgs a{};
    uint32_t blocks = 0;
    int64_t results = 0;
    int most = 0;
    for (int i = 0; i < SumQueue::MOST; ++i) {
        a.first_block[i] = i < q.n ? blocks : 0xffffffffu;
        if (i >= q.n) continue;
        const SumTask& s = q.task[i];
        const int lanes = sum_lanes(s.M, s.N, s.splits);
        a.task[i] = {s.partial, s.C, s.ldc, s.N, s.M * s.N / 4, s.splits, lanes, s.sgd.w ? SUM_SGD : s.crop.dst ? SUM_CROP : SUM_STORE,
                     SgdArgs{s.sgd.w, s.sgd.m, s.sgd.copy, s.sgd.copy_bf16 ? 1 : 0, s.sgd.lr, s.sgd.mu, s.sgd.wd},
                     CropArgs{s.crop.dst, (int)s.crop.rows, (int)s.crop.inner, (int)s.crop.inner_keep}};
        blocks += (uint32_t)ceil_div(s.M * s.N / 4, 256 / lanes);
        results += s.M * s.N;
        most = std::max(most, s.splits);
    }
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    const int logged = log_begin(&ev0, &ev1);
    if (logged >= 0) (void)hipEventRecord(ev0, st);
    note_kernel("sums_kernel");
    hipLaunchKernelGGL(sums_kernel, dim3(blocks), dim3(256), 0, st, a);
    const hipError_t e = hipGetLastError();
    if (logged >= 0) {
        (void)hipEventRecord(ev1, st);
        log_end(logged, LRD_ROLE_SUMS, 0, 0, most, results, 1, 1, q.n);
    }
    q.n = 0;
    return e;
}

hipError_t reduce_partials(const float* partial, void* C, bool c_bf16, int64_t ldc, int64_t M, int64_t N, int splits,
                           hipStream_t st, const SgdFuse* sgd, const CropFuse* crop)
{
    if (M <= 0 || N <= 0) return hipSuccess;
    const bool al = al16(C) && al16(partial);
    if (c_bf16) {
        if (al && N % 8 == 0 && ldc % 8 == 0)
            hipLaunchKernelGGL((reduce_partials_kernel<8, bf16_t>), dim3(blocks_for(M * N / 8)), dim3(256), 0, st, partial,
                               (bf16_t*)C, ldc, M, N, splits, SgdArgs{});
        else
            hipLaunchKernelGGL((reduce_partials_kernel<1, bf16_t>), dim3(blocks_for(M * N)), dim3(256), 0, st, partial,
                               (bf16_t*)C, ldc, M, N, splits, SgdArgs{});
        return hipGetLastError();
    }
    const bool vec4 = al && N % 4 == 0 && ldc % 4 == 0;
    const int lanes = vec4 ? sum_lanes(M, N, splits) : 1;
    const bool wide64 = lanes == 64, wide16 = lanes == 16;
    if (sgd && !sgd->done && vec4 && sgd_fits(*sgd, ldc, N)) {
        const SgdArgs a{sgd->w, sgd->m, sgd->copy, sgd->copy_bf16 ? 1 : 0, sgd->lr, sgd->mu, sgd->wd};
        if (wide64)
            hipLaunchKernelGGL((reduce_partials_wide_kernel<64, SUM_SGD>), dim3((unsigned)ceil_div(M * N / 4, 4)), dim3(256), 0, st,
                               partial, (float*)C, ldc, M, N, splits, a);
        else if (wide16)
            hipLaunchKernelGGL((reduce_partials_wide_kernel<16, SUM_SGD>), dim3((unsigned)ceil_div(M * N / 4, 16)), dim3(256), 0, st,
                               partial, (float*)C, ldc, M, N, splits, a);
        else
            hipLaunchKernelGGL((reduce_partials_kernel<4, float, SUM_SGD>), dim3(blocks_for(M * N / 4)), dim3(256), 0, st, partial,
                               (float*)C, ldc, M, N, splits, a);
        sgd->done = true;
        return hipGetLastError();
    }
    if (crop && vec4 && !crop->done && crop_fits(*crop, M, N)) {
        const CropArgs a{crop->dst, (int)crop->rows, (int)crop->inner, (int)crop->inner_keep};
        if (wide64)
            hipLaunchKernelGGL((reduce_partials_wide_kernel<64, SUM_CROP>), dim3((unsigned)ceil_div(M * N / 4, 4)), dim3(256), 0, st,
                               partial, (float*)C, ldc, M, N, splits, SgdArgs{}, a);
        else if (wide16)
            hipLaunchKernelGGL((reduce_partials_wide_kernel<16, SUM_CROP>), dim3((unsigned)ceil_div(M * N / 4, 16)), dim3(256), 0, st,
                               partial, (float*)C, ldc, M, N, splits, SgdArgs{}, a);
        else
            hipLaunchKernelGGL((reduce_partials_kernel<4, float, SUM_CROP>), dim3(blocks_for(M * N / 4)), dim3(256), 0, st, partial,
                               (float*)C, ldc, M, N, splits, SgdArgs{}, a);
        crop->done = true;
        return hipGetLastError();
    }
    if (wide64)
        hipLaunchKernelGGL((reduce_partials_wide_kernel<64>), dim3((unsigned)ceil_div(M * N / 4, 4)), dim3(256), 0, st, partial,
                           (float*)C, ldc, M, N, splits, SgdArgs{});
    else if (wide16)
        hipLaunchKernelGGL((reduce_partials_wide_kernel<16>), dim3((unsigned)ceil_div(M * N / 4, 16)), dim3(256), 0, st, partial,
                           (float*)C, ldc, M, N, splits, SgdArgs{});
    else if (vec4)
        hipLaunchKernelGGL((reduce_partials_kernel<4, float>), dim3(blocks_for(M * N / 4)), dim3(256), 0, st, partial,
                           (float*)C, ldc, M, N, splits, SgdArgs{});
    else
        hipLaunchKernelGGL((reduce_partials_kernel<1, float>), dim3(blocks_for(M * N)), dim3(256), 0, st, partial,
                           (float*)C, ldc, M, N, splits, SgdArgs{});
    return hipGetLastError();
}

}  // namespace lrd
