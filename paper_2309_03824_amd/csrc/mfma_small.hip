// bf16 products of a layer with few tokens, for which the chip is far too large: what counts is how many kernels follow one
// another and how long the chain of dependent loads in each is.
//
// Output tiles of 64 x 64 give such a product a few dozen workgroups that walk K step by step, barrier by barrier (48 x 256
// over 1024: four workgroups of sixteen steps, 5.6 us; 509 x 192 over 3072: four slices and their sum, 9.8 us), and a backward
// pass with bias is seven launches of 3 to 6 us, of which about 2.5 us is the launch.  Here eight waves share a 32-row block
// of the result and cut K among them, every wave loads its own operands into LDS of its own without any barrier, and the waves'
// sums meet in LDS at the end, in wave order.  The products of a backward pass that do
// not wait for one another share a launch: dH = dY.U with dU = dY^T.H and the bias gradient's partial sums, then dX = dH.V with
// dV = dH^T.X and the sum of those.  48 x 1024 -> 4096 at rank 256, forward 9.7 -> 7.3 us, with its backward pass 32 -> 19 us;
// 509 x 768 -> 3072 at rank 192 34.9 -> 26.4 us (times of the kernels one after another in a graph).
#include <algorithm>
#include <cstdio>

#include "lds_load.hpp"
#include "lrd_internal.hpp"

namespace lrd {
namespace {

constexpr int WAVES = 8, THREADS = 64 * WAVES;
constexpr int SLAB = 16384;          // LDS bytes of a wave

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ bf16x8 transposed(const char* lo_at, const char* hi_at)
{
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(lo_at));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(hi_at));
    const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    return __builtin_bit_cast(bf16x8, v);
}

// C[M x N] (bf16) = A . B^T: K and N multiples of 16.
struct ActJob {
    const bf16_t* A;
    const bf16_t* B;
    bf16_t* C;
    bf16_t* aux;
    const float* bias;
    uint32_t lda, ldb, ldc, ldaux;
    int M, N, K, blocks, col_blocks, epilogue;
};
// C[M x N] (fp32) = A^T . B over K rows: M, N multiples of 8.
struct GradJob {
    const bf16_t* A;
    const bf16_t* B;
    float* C;
    uint32_t lda, ldb, ldc;
    int M, N, K, blocks, col_blocks;
};
// Column sums of dY [T x n]: partial rows (into `to` of `slices` rows), or the sum of those.
struct SumJob {
    const bf16_t* dY;
    float* part;
    float* out;
    int T, n, rows, slices, blocks, col_blocks, runs;      // runs: blocks of column_sums that half a workgroup takes in turn
};

// 32 rows x 32 * (8 / KS) columns: KS waves cut the K of each 32 x 32 block.  B k-contiguous [N x K], or (B_KM) k-major [K x N].
// Each wave brings its own operands into its slab, 64 k at a time and two such steps ahead, in whole rows of 128 bytes (64 of
// a k-major B): loads straight in the operand layout, 64 bytes of each of 16 rows, ran at a quarter of the rate.
template <int KS, bool B_KM>
__device__ __forceinline__ void act_tile(const ActJob& g, int block, char* smem, int tid)
{
    constexpr int NB = WAVES / KS, LOADS = 8;
    const int lane = tid & 63, wave = (int)uni(tid >> 6);
    const int ks = wave % KS, nb = wave / KS;
    const int q = lane >> 4, r16 = lane & 15;
    const int m0 = block / g.col_blocks * 32, n0 = block % g.col_blocks * (32 * NB), col = min(n0 + nb * 32, g.N);
    const int per = ((g.K + KS - 1) / KS + 31) & ~31, kbeg = min(ks * per, g.K), kend = min(kbeg + per, g.K);
    const int rows = min(g.M - m0, 32), cols = min(g.N - col, 32);
    const int steps = cols > 0 ? (kend - kbeg + 63) / 64 : 0;
    char* slab = smem + wave * SLAB;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)slab;

    // descriptors end with the wave's last k (k-contiguous: of its last row; other rows are masked in the last step)
    const char* abase = uni_ptr(g.A + (int64_t)m0 * g.lda + kbeg);
    uint32_t aspan = uni((uint32_t)(((int64_t)(rows - 1) * g.lda + kend - kbeg) * 2));
    const char* bbase = uni_ptr(B_KM ? g.B + (int64_t)kbeg * g.ldb + col : g.B + (int64_t)col * g.ldb + kbeg);
    uint32_t bspan = uni(cols > 0 && !B_KM ? (uint32_t)(((int64_t)(cols - 1) * g.ldb + kend - kbeg) * 2) : 0u);
    int64_t bld = (int64_t)uni(g.ldb);
    int krows = (int)uni((uint32_t)(kend - kbeg)), bcols = (int)uni((uint32_t)cols);
    settle(abase, aspan);
    settle(bbase, bspan);
    settle(bbase, bld, krows);
    settle(bbase, bld, bcols);
    uint32_t aoff[4], boff[4];
    int ak[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const int r = p * 8 + (lane >> 3);
        ak[p] = ((lane & 7) ^ kc_swz(r)) * 8;
        aoff[p] = r < rows ? ((uint32_t)r * g.lda + ak[p]) * 2u : BUF_OOB;
        if (B_KM) {
            // [64 k][32 columns], 64 bytes a row; chunks 0, 1 and 2, 3 change places in rows k & 8, so that the rows of one
            // transposing read, k .. k + 3 and those 8 further, fall on different banks
            const int k = p * 16 + (lane >> 2), c = ((lane & 3) ^ (k & 8 ? 2 : 0)) * 8;
            boff[p] = c < cols ? ((uint32_t)k * g.ldb + c) * 2u : BUF_OOB;
        } else {
            boff[p] = r < cols ? ((uint32_t)r * g.ldb + ak[p]) * 2u : BUF_OOB;
        }
    }
    auto load = [&](int t) {
        const int k0 = t * 64, left = krows - k0;
        const uint32_t to = lds0 + (t & 1) * 8192;
#pragma unroll
        for (int p = 0; p < 4; ++p) load_to_lds(to + p * 1024, abase + k0 * 2, aspan - k0 * 2, ak[p] < left ? aoff[p] : BUF_OOB);
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            if constexpr (B_KM) load_to_lds(to + 4096 + p * 1024, bbase + k0 * bld * 2, (uint32_t)((min(left, 64) - 1) * bld + bcols) * 2u, boff[p]);
            else load_to_lds(to + 4096 + p * 1024, bbase + k0 * 2, bspan - k0 * 2, ak[p] < left ? boff[p] : BUF_OOB);
        }
    };
    const uint32_t fk = r16 * 128 + ((q ^ kc_swz(r16)) << 4);      // k-contiguous: block of 16 rows at + 2048, second 32 k at ^ 64
    const uint32_t ft = (q * 8 + (r16 >> 2)) * 64 + (r16 & 3) * 8, fx = (q & 1) * 32;
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (steps > 0) load(0);
    if (steps > 1) load(1);
    for (int t = 0; t < steps; ++t) {
        if (t + 1 < steps) wait_vm<LOADS>();
        else wait_vm<0>();
        const char* at = slab + (t & 1) * 8192;
        bf16x8 a[2][2], b[2][2];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                a[kk][i] = *reinterpret_cast<const bf16x8*>(at + i * 2048 + (kk ? fk ^ 64 : fk));
                if constexpr (B_KM) {
                    const char* p = at + 4096 + kk * 2048 + ft + ((i * 32) ^ fx);
                    b[kk][i] = transposed(p, p + 256);
                } else {
                    b[kk][i] = *reinterpret_cast<const bf16x8*>(at + 4096 + i * 2048 + (kk ? fk ^ 64 : fk));
                }
            }
        if (t + 2 < steps) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // (read before it is overwritten)
            load(t + 2);
        }
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = mfma16(b[kk][j], a[kk][i], acc[i][j]);
    }
    lds_barrier();
    // the waves' sums: [wave][32 rows][32 columns], 16-byte chunks permuted by the row; roles swapped in the products: a lane
    // holds row (l & 15), columns 4 * (l >> 4) + 0..3 of its 16 x 16 block
    float* const sums = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int r = i * 16 + r16, c = j * 4 + q;
            *reinterpret_cast<f32x4*>(sums + wave * 1024 + r * 32 + ((c ^ (r & 7)) << 2)) = acc[i][j];
        }
    __syncthreads();
    for (int e = tid; e < 128 * NB; e += THREADS) {
        const int r = e / (4 * NB), c8 = e % (4 * NB), blk = c8 >> 2, c = (c8 & 3) * 2, m = m0 + r, n = n0 + c8 * 8;
        if (r >= rows || n >= g.N) continue;
        f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = lo;
#pragma unroll
        for (int z = 0; z < KS; ++z) {
            const float* p = sums + (blk * KS + z) * 1024 + r * 32;
            lo += *reinterpret_cast<const f32x4*>(p + ((c ^ (r & 7)) << 2));
            hi += *reinterpret_cast<const f32x4*>(p + (((c + 1) ^ (r & 7)) << 2));
        }
        if (g.bias) {
            lo += *reinterpret_cast<const f32x4*>(g.bias + n);
            hi += *reinterpret_cast<const f32x4*>(g.bias + n + 4);
        }
        u32x4 v = {pack_bf16(lo[0], lo[1]), pack_bf16(lo[2], lo[3]), pack_bf16(hi[0], hi[1]), pack_bf16(hi[2], hi[3])};
        bf16x8 c8v = __builtin_bit_cast(bf16x8, v);
        if (B_KM && g.epilogue == EPI_ACT_GRAD) {
            const bf16x8 z8 = *reinterpret_cast<const bf16x8*>(g.aux + (int64_t)m * g.ldaux + n);
#pragma unroll
            for (int x = 0; x < 8; ++x) c8v[x] = (bf16_t)((float)c8v[x] * gelu_grad_bf16_f((float)z8[x]));
        }
        *reinterpret_cast<bf16x8*>(g.C + (int64_t)m * g.ldc + n) = c8v;
        if (!B_KM && g.epilogue == EPI_ACT_STORE) {
#pragma unroll
            for (int x = 0; x < 8; ++x) c8v[x] = (bf16_t)gelu_bf16_f((float)c8v[x]);
            *reinterpret_cast<bf16x8*>(g.aux + (int64_t)m * g.ldaux + n) = c8v;
        }
    }
}

// 64 x 64 of a weight gradient; every wave takes an eighth of the rows, 64 of them at a time, through its own slab.
__device__ __forceinline__ void grad_tile(const GradJob& g, int block, char* smem, int tid)
{
    const int lane = tid & 63, wave = (int)uni(tid >> 6);
    const int q = lane >> 4, r16 = lane & 15;
    const int m0 = block / g.col_blocks * 64, n0 = block % g.col_blocks * 64;
    const int per = ((g.K + WAVES - 1) / WAVES + 31) & ~31, kbeg = min(wave * per, g.K), kend = min(kbeg + per, g.K);
    char* slab = smem + wave * SLAB;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)slab;
    const char* abase = uni_ptr(g.A + m0);
    const char* bbase = uni_ptr(g.B + n0);
    int64_t lda = (int64_t)uni(g.lda), ldb = (int64_t)uni(g.ldb);
    int acols = (int)uni((uint32_t)min(g.M - m0, 64)), bcols = (int)uni((uint32_t)min(g.N - n0, 64));
    settle(abase, lda, acols);
    settle(bbase, ldb, bcols);
    // a load covers 8 rows of 128 bytes; chunks permuted as for the transposing reads of 64 columns (rows k & 2, k & 8)
    const int lrow = lane >> 3, slot = lane & 7;
    auto voff = [&](int s, uint32_t ld, int cols) {
        const int row = s * 8 + lrow, c = (slot ^ (((row & 2) << 1) | ((row & 8) >> 2))) * 8;
        return c < cols ? ((uint32_t)row * ld + c) * 2u : BUF_OOB;
    };
    const uint32_t f0 = (q * 8 + (r16 >> 2)) * 128 + ((r16 & 2) << 3) + (r16 & 1) * 8, fx = ((r16 >> 2) & 2) << 1 | (q & 1) << 1;
    f32x4 acc[4][4];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int k0 = kbeg; k0 < kend; k0 += 64) {
        const int here = min(kend - k0, 64);
        if (k0 > kbeg) asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        // (rows from `here` on lie past the descriptors: ld >= the tile's columns)
#pragma unroll
        for (int s = 0; s < 8; ++s) load_to_lds(lds0 + s * 1024, abase + (int64_t)k0 * lda * 2, (uint32_t)((here - 1) * lda + acols) * 2u, voff(s, g.lda, acols));
#pragma unroll
        for (int s = 0; s < 8; ++s) load_to_lds(lds0 + 8192 + s * 1024, bbase + (int64_t)k0 * ldb * 2, (uint32_t)((here - 1) * ldb + bcols) * 2u, voff(s, g.ldb, bcols));
        wait_vm<0>();
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            bf16x8 a[4], b[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const char* pa = slab + kk * 4096 + f0 + (((j * 2) ^ fx) << 4);
                a[j] = transposed(pa, pa + 512);
                b[j] = transposed(pa + 8192, pa + 8192 + 512);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = mfma16(b[j], a[i], acc[i][j]);
        }
    }
    lds_barrier();
    float* const sums = reinterpret_cast<float*>(smem);
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = i * 16 + r16, c = j * 4 + q;
            *reinterpret_cast<f32x4*>(sums + wave * 4096 + r * 64 + ((c ^ r16) << 2)) = acc[i][j];
        }
    __syncthreads();
#pragma unroll
    for (int e = tid; e < 1024; e += THREADS) {
        const int r = e >> 4, c = e & 15;
        f32x4 s = *reinterpret_cast<const f32x4*>(sums + r * 64 + ((c ^ (r & 15)) << 2));
#pragma unroll
        for (int z = 1; z < WAVES; ++z) s += *reinterpret_cast<const f32x4*>(sums + z * 4096 + r * 64 + ((c ^ (r & 15)) << 2));
        if (r < g.M - m0 && c * 4 < g.N - n0) *reinterpret_cast<f32x4*>(g.C + (int64_t)(m0 + r) * g.ldc + n0 + c * 4) = s;
    }
}

// The two halves of column_sums (same runs of rows, same order of additions), two of its blocks to a workgroup.
__device__ __forceinline__ void sum_rows(const SumJob& g, int block, char* smem, int tid)
{
    const int half = tid >> 8, t = tid & 255, cl = t & 31, rl = t >> 5;
    float* part = reinterpret_cast<float*>(smem) + half * (8 * 32 * 9);      // [8][32][8 + 1]
    for (int run = 0; run < g.runs; ++run) {
        const int vb = (block * g.runs + run) * 2 + half, cb = vb % g.col_blocks, slice = vb / g.col_blocks;
        const int col = (cb * 32 + cl) * 8, t1 = min((slice + 1) * g.rows, g.T);
        float s[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] = 0.f;
        if (col < g.n && slice < g.slices) {
#pragma unroll 4
            for (int r = slice * g.rows + rl; r < t1; r += 8) {
                const bf16x8 v = *reinterpret_cast<const bf16x8*>(g.dY + (int64_t)r * g.n + col);
#pragma unroll
                for (int e = 0; e < 8; ++e) s[e] += (float)v[e];
            }
        }
        if (run > 0) __syncthreads();
#pragma unroll
        for (int e = 0; e < 8; ++e) part[(rl * 32 + cl) * 9 + e] = s[e];
        __syncthreads();
        const int out = cb * 256 + t;
        if (out < g.n && slice < g.slices) {
            float v = 0.f;
#pragma unroll
            for (int r = 0; r < 8; ++r) v += part[(r * 32 + t / 8) * 9 + t % 8];
            g.part[(int64_t)slice * g.n + out] = v;
        }
    }
}
__device__ __forceinline__ void sum_slices(const SumJob& g, int block, int tid)
{
    const int i = (block * THREADS + tid) * 4;
    if (i >= g.n) return;
    f32x4 p[16];
#pragma unroll
    for (int l = 0; l < 16; ++l) p[l] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int z = 0; z < g.slices; z += 16)
#pragma unroll
        for (int l = 0; l < 16; ++l)
            if (z + l < g.slices) p[l] += *reinterpret_cast<const f32x4*>(g.part + (int64_t)(z + l) * g.n + i);
    if (g.slices < 16) {
#pragma unroll
        for (int l = 1; l < 16; ++l) p[0] += p[l];
    } else {
#pragma unroll
        for (int half = 8; half >= 1; half /= 2)
#pragma unroll
            for (int l = 0; l < half; ++l) p[l] += p[l + half];
    }
    *reinterpret_cast<f32x4*>(g.out + i) = p[0];
}

template <int KS>
__global__ __launch_bounds__(THREADS, 2) void small_fwd_kernel(ActJob g)
{
    extern __shared__ __align__(16) char smem[];
    act_tile<KS, false>(g, blockIdx.x, smem, threadIdx.x);
}

// Jobs of one launch, in the order of their workgroups (those with the longest chains first); a job without blocks is absent.
template <int KS>
__global__ __launch_bounds__(THREADS, 2) void small_bwd_kernel(ActJob d, GradJob w, SumJob s)
{
    extern __shared__ __align__(16) char smem[];
    int block = blockIdx.x;
    if (block < d.blocks) return act_tile<KS, true>(d, block, smem, threadIdx.x);
    block -= d.blocks;
    if (block < w.blocks) return grad_tile(w, block, smem, threadIdx.x);
    block -= w.blocks;
    if (s.dY) sum_rows(s, block, smem, threadIdx.x);
    else sum_slices(s, block, threadIdx.x);
}

template <class Kernel>
hipError_t allow_lds(Kernel kern, int bytes, bool& done)
{
    if (done) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    done = e == hipSuccess;
    return e;
}

constexpr int64_t MOST_TOKENS = 1024;      // above, the tiles are as fast or faster in every shape tried
// How the waves cut a product: its K in eight, or in two with four blocks side by side; the cheaper of the two by rounds of
// workgroups over the chip times the steps of a wave (of 64 k) and about three more for its start and its end.
struct Cut {
    int64_t cols, blocks, steps;
    int64_t cost() const { return ceil_div(blocks, 256) * (steps + 3); }
};
Cut cut(const MatOp& op)
{
    auto by = [&](int64_t ks) {
        const int64_t cols = 32 * WAVES / ks;
        return Cut{cols, ceil_div(op.M, 32) * ceil_div(op.N, cols), ceil_div(op.K, 64 * ks)};
    };
    const Cut eight = by(8), two = by(2);
    return eight.cost() < two.cost() ? eight : two;
}
inline bool in_eight(const Cut& c) { return c.cols == 32; }

ActJob act_job(const MatOp& op, bool b_km)
{
    ActJob g;
    g.A = (const bf16_t*)op.A; g.B = (const bf16_t*)op.B; g.C = (bf16_t*)op.C; g.aux = (bf16_t*)op.aux; g.bias = op.bias;
    g.lda = (uint32_t)op.a_sm; g.ldb = (uint32_t)(b_km ? op.b_sk : op.b_sn); g.ldc = (uint32_t)op.ldc; g.ldaux = (uint32_t)op.ldaux;
    g.M = (int)op.M; g.N = (int)op.N; g.K = (int)op.K; g.epilogue = op.epilogue;
    g.col_blocks = (int)ceil_div(op.N, cut(op).cols);
    g.blocks = (int)ceil_div(op.M, 32) * g.col_blocks;
    return g;
}

bool act_ok(const MatOp& op)
{
    return mfma_gemm2_supported(op) && op.gather == GATHER_NONE && !op.out_f32 && op.batch == 1 && op.a_sk == 1 && op.K % 16 == 0 && op.N % 16 == 0 &&
           op.M <= MOST_TOKENS && op.N < 65536 && op.ldc <= BUF_MAX_LD && op.ldaux <= BUF_MAX_LD &&
           (op.epilogue == EPI_NONE || (op.epilogue == EPI_ACT_GRAD) == (op.b_sk != 1));
}

// A product by itself: one round of workgroups, and few enough steps that the tiles' wider blocks, which bring each operand
// less often, do not win (1024 x 1024 over 4096 cut in two, 32 steps: 34.6 against 28.2 us with the product after it; 1024 x 256
// over 4096 cut in eight, eight steps: even).
bool alone_ok(const MatOp& op)
{
    if (!act_ok(op)) return false;
    const Cut c = cut(op);
    return c.blocks <= 256 && c.steps <= (in_eight(c) ? 8 : 4);
}

}  // namespace

bool mfma_small_fwd_supported(const MatOp& op) { return op.b_sk == 1 && alone_ok(op); }

hipError_t mfma_small_fwd(const MatOp& op, hipStream_t st)
{
    const ActJob g = act_job(op, false);
    constexpr int lds = WAVES * SLAB;
    static bool long_ok = false, short_ok = false;
    const bool eight = in_eight(cut(op));
    const hipError_t e = eight ? allow_lds(small_fwd_kernel<8>, lds, long_ok) : allow_lds(small_fwd_kernel<2>, lds, short_ok);
    if (e != hipSuccess) return e;
    note_kernel(eight ? "small_fwd_kernel<8>" : "small_fwd_kernel<2>");
    if (eight) hipLaunchKernelGGL((small_fwd_kernel<8>), dim3(g.blocks), dim3(THREADS), lds, st, g);
    else hipLaunchKernelGGL((small_fwd_kernel<2>), dim3(g.blocks), dim3(THREADS), lds, st, g);
    return hipGetLastError();
}

bool mfma_small_data_supported(const MatOp& op) { return op.b_sk != 1 && alone_ok(op); }

// The products of a launch of the backward pass: up to 1024 tokens, while all workgroups together are not more than 27 steps a
// unit (a step of a gradient brings twice the bytes, and its workgroups beyond one to a unit count twice).  Below that line the
// launches and sums saved weigh more, above it the tiles' rate: forward + backward with bias of 48 x 1024 x 4096 at rank 256 32 -> 19
// us, 1024 tokens of it 58 -> 54 us, 1536 tokens 67 -> 73 us; 1024 x 3072 x 3072 at rank 384 84 -> 70 us; 509 x 4096 x 4096 at
// rank 512 58 -> 64 us, 256 tokens at rank 1024 63 -> 70 us.
bool mfma_small_bwd_supported(const MatOp* data, const MatOp* grad)
{
    int64_t work = 0;
    if (data) {
        if (data->b_sk == 1 || !act_ok(*data)) return false;
        const Cut c = cut(*data);
        work += c.blocks * (c.steps + 3);
    }
    if (grad) {
        // (neither operand is k-contiguous: any number of tokens, also one)
        MatOp op = *grad;
        op.K = std::max<int64_t>(op.K, 8);
        if (!mfma_gemm2_supported(op) || op.gather != GATHER_NONE || !op.out_f32 || op.batch != 1 || op.a_sk == 1 || op.b_sk == 1 || op.sgd || op.crop ||
            op.K > MOST_TOKENS || op.M >= 65536 || op.N >= 65536 || op.ldc > BUF_MAX_LD)
            return false;
        const int64_t blocks = ceil_div(op.M, 64) * ceil_div(op.N, 64);
        work += (blocks + std::max<int64_t>(0, blocks - 256)) * (2 * ceil_div(op.K, 512) + 3);
    }
    return work <= 27 * 256;
}

hipError_t mfma_small_bwd(const MatOp* data, const MatOp* grad, const SmallSums* sums, hipStream_t st)
{
    ActJob d{};
    GradJob w{};
    SumJob s{};
    if (data) d = act_job(*data, true);
    if (grad) {
        w.A = (const bf16_t*)grad->A; w.B = (const bf16_t*)grad->B; w.C = (float*)grad->C;
        w.lda = (uint32_t)grad->a_sk; w.ldb = (uint32_t)grad->b_sk; w.ldc = (uint32_t)grad->ldc;
        w.M = (int)grad->M; w.N = (int)grad->N; w.K = (int)grad->K;
        w.col_blocks = (int)ceil_div(w.N, 64);
        w.blocks = (int)ceil_div(w.M, 64) * w.col_blocks;
    }
    if (sums) {
        s.dY = (const bf16_t*)sums->dY; s.part = sums->part; s.out = sums->out;
        s.T = (int)sums->T; s.n = (int)sums->n; s.rows = 32; s.slices = (int)ceil_div(sums->T, 32);
        s.col_blocks = (int)ceil_div(sums->n, 256);
        // partial sums on the units that the products leave, or beside them on at least 32
        const int halves = (s.col_blocks * s.slices + 1) / 2;
        s.runs = (int)ceil_div(halves, std::max(32, 256 - d.blocks - w.blocks));
        s.blocks = sums->dY ? (int)ceil_div(halves, s.runs) : (int)ceil_div(sums->n, THREADS * 4);
    }
    const int blocks = d.blocks + w.blocks + s.blocks;
    if (blocks == 0) return hipSuccess;
    constexpr int lds = WAVES * SLAB;
    const bool cut_k = data && in_eight(cut(*data));
    static bool long_ok = false, short_ok = false;
    const hipError_t e = cut_k ? allow_lds(small_bwd_kernel<8>, lds, long_ok) : allow_lds(small_bwd_kernel<2>, lds, short_ok);
    if (e != hipSuccess) return e;
    note_kernel(cut_k ? "small_bwd_kernel<8>" : "small_bwd_kernel<2>");
    if (cut_k) hipLaunchKernelGGL((small_bwd_kernel<8>), dim3(blocks), dim3(THREADS), lds, st, d, w, s);
    else hipLaunchKernelGGL((small_bwd_kernel<2>), dim3(blocks), dim3(THREADS), lds, st, d, w, s);
    return hipGetLastError();
}

}  // namespace lrd
