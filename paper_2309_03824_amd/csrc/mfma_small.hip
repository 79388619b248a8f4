// bf16 products of a layer with few tokens, for which the chip is far too large: what counts is how many kernels follow one
// another and how long the chain of dependent loads in each is.
//
// Output tiles of 64 x 64 give such a product a few dozen workgroups, each with three steps of 64 k under way, and a K-slice or
// a sum more to launch where K is long; a backward pass with bias is seven launches of 3 to 6 us, of which about 2.5 us is the
// launch.  Here a workgroup takes 32 rows and 32, 64 or 128 columns, and as much of K as its LDS holds is on its way at
// once (1024 k of a 32 x 32 block).  The products of a backward pass that do not wait for one another share a launch: dH = dY.U
// with dU = dY^T.H and the bias gradient's partial sums, then dX = dH.V with dV = dH^T.X and the sum of those.  Kernels one after
// another in a graph: 48 x 1024 -> 4096 at rank 256 forward 9.7 -> 7.8 us, its backward pass with bias 24.6 -> 18.9 us; 509 x 768 ->
// 3072 at rank 192 10.6 -> 9.0 and 28.2 -> 17.2 us.
//
// Every result is the chain of additions that the output tiles run, in the slices of K that the product was given, each a chain
// of its own in registers and added in slice order: the same bits whichever kernel a product goes to, so that a layer's results do
// not depend on what else a call wants.  (v_mfma_f32_16x16x32_bf16 adds what two v_mfma_f32_32x32x16_bf16 add, in their order.)
#include <algorithm>
#include <cstdio>

#include "lds_load.hpp"
#include "lrd_internal.hpp"

namespace lrd {
namespace {

constexpr int THREADS = 512;         // waves 0 .. 3 multiply, 4 .. 7 load

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

// C[M x N] (bf16) = A . B^T: K and N multiples of 16.  `slice`: steps of 64 k in a slice of K (1 << 30: unsliced).
struct ActJob {
    const bf16_t* A;
    const bf16_t* B;
    bf16_t* C;
    bf16_t* aux;
    const float* bias;
    uint32_t lda, ldb, ldc, ldaux;
    int M, N, K, blocks, col_blocks, epilogue, slice, ring;
};
// C[M x N] (fp32) = A^T . B over K rows: M, N multiples of 8.
struct GradJob {
    const bf16_t* A;
    const bf16_t* B;
    float* C;
    uint32_t lda, ldb, ldc;
    int M, N, K, blocks, col_blocks, slice, ring;
};
// Column sums of dY [T x n]: partial rows (into `part`, `slices` of them), or the sum of those.
struct SumJob {
    const bf16_t* dY;
    float* part;
    float* out;
    int T, n, rows, slices, blocks, col_blocks, runs;      // runs: blocks of column_sums that half a workgroup takes in turn
};

// K in groups of steps through a ring of `ring` slots in LDS: load(t, slot) starts a loading wave's LOADS loads of group t,
// multiply(slot) reads them.  One barrier to a group, behind which the slot of the group before is filled again.  (One wave to a
// SIMD did both, one after the other, at 160 ns a step of 32 x 32 x 64: address arithmetic and issue took as long as the products.)
template <int MOST, int LOADS, class Load, class Multiply>
__device__ __forceinline__ void stream(bool loads, int groups, int ring, Load load, Multiply multiply)
{
    int slot = 0;
    if (loads) {
        int t = 0;
        auto hand_over = [&](int started) {
            wait_stages<MOST - 1, LOADS>(started - t - 1);
            lds_barrier();
            ++t;
        };
#pragma unroll 1
        for (int n = 0; n < groups; ++n) {
            if (n == ring) hand_over(n);
            if (n >= ring) hand_over(n);      // (everyone is past the group whose slot this is)
            load(n, slot);
            slot = slot + 1 == ring ? 0 : slot + 1;
        }
        while (t < groups) hand_over(groups);
    } else {
#pragma unroll 1
        for (int t = 0; t < groups; ++t) {
            lds_barrier();
            multiply(slot);
            slot = slot + 1 == ring ? 0 : slot + 1;
        }
    }
}

// Chains of a wave's MI x MJ blocks of 16 x 16, one for each K-slice of `slice` steps, added in slice order; or one (not SLICED).
template <int MI, int MJ, bool SLICED>
struct Chains {
    f32x4 acc[MI][MJ], total[SLICED ? MI : 1][SLICED ? MJ : 1];
    int left, slice;
    __device__ __forceinline__ void init(int steps_of_slice)
    {
        left = slice = steps_of_slice;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < MJ; ++j) {
                acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                if constexpr (SLICED) total[i][j] = acc[i][j];
            }
    }
    // one step of 64 k (roles swapped: a lane's four results are consecutive columns of one row)
    __device__ __forceinline__ void step(const bf16x8 (&a)[2][MI], const bf16x8 (&b)[2][MJ])
    {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk)
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < MJ; ++j) acc[i][j] = mfma16(b[kk][j], a[kk][i], acc[i][j]);
    }
    template <int G>
    __device__ __forceinline__ void group(const bf16x8 (&a)[G][2][MI], const bf16x8 (&b)[G][2][MJ])
    {
#pragma unroll
        for (int s = 0; s < G; ++s) {
            step(a[s], b[s]);
            if constexpr (SLICED) {
                if (--left > 0) continue;
                left = slice;
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int j = 0; j < MJ; ++j) {
                        total[i][j] += acc[i][j];
                        acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
                    }
            }
        }
    }
    __device__ __forceinline__ f32x4 result(int i, int j, int steps) const
    {
        if constexpr (SLICED)
            if (slice < steps) return total[i][j] + acc[i][j];
        return acc[i][j];
    }
};

// Blocks of 32 rows x 32 NB columns.
template <int NB>
struct ActShape {
    static_assert(NB == 1 || NB == 2 || NB == 4, "columns in halves, quarters or eighths of 16 to a wave");
    static constexpr int COLS = 32 * NB, STEP = 4096 * (1 + NB), LPS = 1 + NB;
    static constexpr int G = NB == 1 ? 4 : NB == 2 ? 2 : 1, RING = NB == 1 ? 4 : 6;      // steps of a group; most groups under way
    static constexpr int MI = NB == 1 ? 1 : 2, MJ = NB == 4 ? 2 : 1;      // blocks of 16 x 16 of a wave
};
// B k-contiguous [N x K], or (B_KM) k-major [K x N].  Operands come in rows of 128 bytes (64 of a k-major B 32 columns wide): loads
// straight in the operand layout, 64 bytes of each of 16 rows, ran at a quarter of the rate.
template <int NB, bool B_KM>
__device__ __forceinline__ void act_tile(const ActJob& g, int block, char* smem, int tid)
{
    typedef ActShape<NB> S;
    constexpr int COLS = S::COLS, MI = S::MI, MJ = S::MJ, G = S::G;
    const int lane = tid & 63, wave = (int)uni((tid >> 6) & 3);
    const bool loads = uni(tid >> 8) != 0;
    const int q = lane >> 4, r16 = lane & 15, lr = lane >> 3;
    const int m0 = block / g.col_blocks * 32, n0 = block % g.col_blocks * COLS;
    const int rows = min(g.M - m0, 32), cols = min(g.N - n0, COLS), steps = (g.K + 63) / 64;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;

    // descriptors end with the last k (k-contiguous: of the last row; other rows are masked in the last step)
    const char* abase = uni_ptr(g.A + (int64_t)m0 * g.lda);
    uint32_t aspan = uni((uint32_t)(((int64_t)(rows - 1) * g.lda + g.K) * 2));
    const char* bbase = uni_ptr(B_KM ? g.B + n0 : g.B + (int64_t)n0 * g.ldb);
    uint32_t bspan = uni(B_KM ? 0u : (uint32_t)(((int64_t)(cols - 1) * g.ldb + g.K) * 2));
    int64_t bld = (int64_t)uni(g.ldb);
    int K = (int)uni((uint32_t)g.K), bcols = (int)uni((uint32_t)cols);
    settle(abase, aspan);
    settle(bbase, bspan);
    settle(bbase, bld, K);
    settle(bbase, bld, bcols);
    // this wave's loads of a step: 8 rows of A, and of B NB times 8 rows, 32 apart (k-major: chunks permuted so that the rows of one
    // transposing read, k .. k + 3 and those 8 further, fall on different banks; columns in panels of 64)
    const int arow = wave * 8 + lr, ak = ((lane & 7) ^ kc_swz(arow)) * 8;
    const uint32_t aoff = arow < rows ? ((uint32_t)arow * g.lda + ak) * 2u : BUF_OOB;
    uint32_t boff[NB];
#pragma unroll
    for (int p = 0; p < NB; ++p) {
        if constexpr (!B_KM) {
            const int r = p * 32 + arow;
            boff[p] = r < cols ? ((uint32_t)r * g.ldb + ak) * 2u : BUF_OOB;
        } else if constexpr (NB == 1) {
            const int k = wave * 16 + (lane >> 2), c = ((lane & 3) ^ (k & 8 ? 2 : 0)) * 8;
            boff[p] = c < cols ? ((uint32_t)k * g.ldb + c) * 2u : BUF_OOB;
        } else {
            const int b = p * 4 + wave, k = (b & 7) * 8 + lr, c = (b >> 3) * 64 + ((lane & 7) ^ (((k & 2) << 1) | ((k & 8) >> 2))) * 8;
            boff[p] = c < cols ? ((uint32_t)k * g.ldb + c) * 2u : BUF_OOB;
        }
    }
    auto load = [&](int t, int slot) {
        const uint32_t to0 = lds0 + slot * (G * S::STEP) + wave * 1024;
        // (steps past the last k bring zeros)
#pragma unroll
        for (int s = 0; s < G; ++s) {
            const int k0 = (t * G + s) * 64, left = K - k0;
            const uint32_t to = to0 + s * S::STEP;
            load_to_lds(to, abase + k0 * 2, left > 0 ? aspan - k0 * 2 : 0u, ak < left ? aoff : BUF_OOB);
#pragma unroll
            for (int p = 0; p < NB; ++p) {
                if constexpr (B_KM) load_to_lds(to + 4096 + p * 4096, bbase + k0 * bld * 2, left > 0 ? (uint32_t)((min(left, 64) - 1) * bld + bcols) * 2u : 0u, boff[p]);
                else load_to_lds(to + 4096 + p * 4096, bbase + k0 * 2, left > 0 ? bspan - k0 * 2 : 0u, ak < left ? boff[p] : BUF_OOB);
            }
        }
    };

    // what the end needs besides: bias and, for the gradient of GELU, the pre-activations of this thread's 16-byte chunks
    constexpr int CHUNKS = COLS / 8, PER = (32 * CHUNKS + THREADS - 1) / THREADS;
    const int i0 = NB == 1 ? wave >> 1 : 0, j0 = NB == 1 ? wave & 1 : wave * MJ;
    f32x4 bias[MJ];
#pragma unroll
    for (int j = 0; j < MJ; ++j) {
        const int n = n0 + (j0 + j) * 16 + q * 4;
        bias[j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (!B_KM && g.bias && n < g.N) bias[j] = *reinterpret_cast<const f32x4*>(g.bias + n);
    }
    bf16x8 z8[PER];
    if (B_KM && g.epilogue == EPI_ACT_GRAD) {
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const int r = (tid + e * THREADS) / CHUNKS, n = n0 + (tid + e * THREADS) % CHUNKS * 8;
            if (r < rows && n < g.N) z8[e] = *reinterpret_cast<const bf16x8*>(g.aux + (int64_t)(m0 + r) * g.ldaux + n);
        }
    }

    const uint32_t fk = r16 * 128 + ((q ^ kc_swz(r16)) << 4);      // k-contiguous: block of 16 rows at + 2048, second 32 k at ^ 64
    const uint32_t ft = (q * 8 + (r16 >> 2)) * 64 + (r16 & 3) * 8, ftx = (q & 1) * 32;      // k-major, 32 columns wide
    const uint32_t fp = (q * 8 + (r16 >> 2)) * 128 + ((r16 & 2) << 3) + (r16 & 1) * 8, fpx = ((r16 >> 2) & 2) << 1 | (q & 1) << 1;      // 64 wide
    Chains<MI, MJ, NB != 4> c;      // (K of the widest blocks is short)
    c.init(g.slice);
    auto multiply = [&](int ring_slot) {
        bf16x8 a[G][2][MI], b[G][2][MJ];
#pragma unroll
        for (int s = 0; s < G; ++s) {
            const char* at = smem + ring_slot * (G * S::STEP) + s * S::STEP;
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
#pragma unroll
                for (int i = 0; i < MI; ++i) a[s][kk][i] = *reinterpret_cast<const bf16x8*>(at + (i0 + i) * 2048 + (kk ? fk ^ 64 : fk));
#pragma unroll
                for (int j = 0; j < MJ; ++j) {
                    const int jb = j0 + j;
                    if constexpr (!B_KM) {
                        b[s][kk][j] = *reinterpret_cast<const bf16x8*>(at + 4096 + jb * 2048 + (kk ? fk ^ 64 : fk));
                    } else if constexpr (NB == 1) {
                        const char* p = at + 4096 + kk * 2048 + ft + ((jb * 32) ^ ftx);
                        b[s][kk][j] = transposed(p, p + 256);
                    } else {
                        const char* p = at + 4096 + (jb >> 2) * 8192 + kk * 4096 + fp + ((((jb & 3) * 2) ^ fpx) << 4);
                        b[s][kk][j] = transposed(p, p + 512);
                    }
                }
            }
        }
        c.template group<G>(a, b);
    };
    stream<S::RING, G * S::LPS>(loads, (steps + G - 1) / G, g.ring, load, multiply);
    lds_barrier();
    // results as bf16 [32][COLS], 16-byte chunks permuted by the row.  Roles swapped in the products: a lane holds row (l & 15),
    // columns 4 * (l >> 4) + 0..3 of its 16 x 16 block
    auto slot = [&](int r, int ch) { return r * (COLS * 2) + ((ch ^ (NB == 1 ? (r >> 1) & 3 : r & 7)) << 4); };
    if (!loads) {
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < MJ; ++j) {
                f32x4 v = c.result(i, j, steps);
                if (!B_KM && g.bias) v += bias[j];
                const u32x2 pk = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
                *reinterpret_cast<u32x2*>(smem + slot((i0 + i) * 16 + r16, (j0 + j) * 2 + (q >> 1)) + (q & 1) * 8) = pk;
            }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const int r = (tid + e * THREADS) / CHUNKS, ch = (tid + e * THREADS) % CHUNKS, m = m0 + r, n = n0 + ch * 8;
        if (r >= rows || n >= g.N) continue;
        bf16x8 c8 = *reinterpret_cast<const bf16x8*>(smem + slot(r, ch));
        if (B_KM && g.epilogue == EPI_ACT_GRAD) {
#pragma unroll
            for (int x = 0; x < 8; ++x) c8[x] = (bf16_t)((float)c8[x] * gelu_grad_bf16_f((float)z8[e][x]));
        }
        *reinterpret_cast<bf16x8*>(g.C + (int64_t)m * g.ldc + n) = c8;
        if (!B_KM && g.epilogue == EPI_ACT_STORE) {
#pragma unroll
            for (int x = 0; x < 8; ++x) c8[x] = (bf16_t)gelu_bf16_f((float)c8[x]);
            *reinterpret_cast<bf16x8*>(g.aux + (int64_t)m * g.ldaux + n) = c8;
        }
    }
}

// 64 x 64 of a weight gradient, 32 x 32 of it to a wave.
constexpr int GRAD_STEP = 16384, GRAD_G = 1, GRAD_RING = 8;
__device__ __forceinline__ void grad_tile(const GradJob& g, int block, char* smem, int tid)
{
    const int lane = tid & 63, wave = (int)uni((tid >> 6) & 3);
    const bool loads = uni(tid >> 8) != 0;
    const int q = lane >> 4, r16 = lane & 15, lr = lane >> 3;
    const int m0 = block / g.col_blocks * 64, n0 = block % g.col_blocks * 64, steps = (g.K + 63) / 64;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)smem;
    const char* abase = uni_ptr(g.A + m0);
    const char* bbase = uni_ptr(g.B + n0);
    int64_t lda = (int64_t)uni(g.lda), ldb = (int64_t)uni(g.ldb);
    int acols = (int)uni((uint32_t)min(g.M - m0, 64)), bcols = (int)uni((uint32_t)min(g.N - n0, 64));
    settle(abase, lda, acols);
    settle(bbase, ldb, bcols);
    // a load covers 8 rows of 128 bytes; chunks permuted as for the transposing reads of 64 columns (rows k & 2, k & 8)
    uint32_t aoff[2], boff[2];
#pragma unroll
    for (int s = 0; s < 2; ++s) {
        const int row = (s * 4 + wave) * 8 + lr, c = ((lane & 7) ^ (((row & 2) << 1) | ((row & 8) >> 2))) * 8;
        aoff[s] = c < acols ? ((uint32_t)row * g.lda + c) * 2u : BUF_OOB;
        boff[s] = c < bcols ? ((uint32_t)row * g.ldb + c) * 2u : BUF_OOB;
    }
    auto load = [&](int t, int slot) {
#pragma unroll
        for (int s = 0; s < GRAD_G; ++s) {
            // (rows from `here` on lie past the descriptors: ld >= the tile's columns)
            const int k0 = (t * GRAD_G + s) * 64, here = min(g.K - k0, 64);
            const uint32_t to = lds0 + (slot * GRAD_G + s) * GRAD_STEP + wave * 1024;
#pragma unroll
            for (int p = 0; p < 2; ++p) load_to_lds(to + p * 4096, abase + k0 * lda * 2, here > 0 ? (uint32_t)((here - 1) * lda + acols) * 2u : 0u, aoff[p]);
#pragma unroll
            for (int p = 0; p < 2; ++p) load_to_lds(to + 8192 + p * 4096, bbase + k0 * ldb * 2, here > 0 ? (uint32_t)((here - 1) * ldb + bcols) * 2u : 0u, boff[p]);
        }
    };
    const int i0 = (wave >> 1) * 2, j0 = (wave & 1) * 2;
    const uint32_t fp = (q * 8 + (r16 >> 2)) * 128 + ((r16 & 2) << 3) + (r16 & 1) * 8, fpx = ((r16 >> 2) & 2) << 1 | (q & 1) << 1;
    Chains<2, 2, true> c;
    c.init(g.slice);
    auto multiply = [&](int slot) {
        bf16x8 a[GRAD_G][2][2], b[GRAD_G][2][2];
#pragma unroll
        for (int s = 0; s < GRAD_G; ++s)
#pragma unroll
            for (int kk = 0; kk < 2; ++kk)
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const char* at = smem + (slot * GRAD_G + s) * GRAD_STEP + kk * 4096 + fp;
                    const char *pa = at + ((((i0 + i) * 2) ^ fpx) << 4), *pb = at + 8192 + ((((j0 + i) * 2) ^ fpx) << 4);
                    a[s][kk][i] = transposed(pa, pa + 512);
                    b[s][kk][i] = transposed(pb, pb + 512);
                }
        c.group<GRAD_G>(a, b);
    };
    stream<GRAD_RING, GRAD_G * 4>(loads, (steps + GRAD_G - 1) / GRAD_G, g.ring, load, multiply);
    if (loads) return;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int m = m0 + (i0 + i) * 16 + r16, n = n0 + (j0 + j) * 16 + q * 4;
            if (m < g.M && n < g.N) *reinterpret_cast<f32x4*>(g.C + (int64_t)m * g.ldc + n) = c.result(i, j, steps);
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

template <int NB>
__global__ __launch_bounds__(THREADS, 4) void small_fwd_kernel(ActJob g)
{
    extern __shared__ __align__(16) char smem[];
    act_tile<NB, false>(g, blockIdx.x, smem, threadIdx.x);
}

// Jobs of one launch, in the order of their workgroups (those with the longest chains first); a job without blocks is absent.
template <int NB>
__global__ __launch_bounds__(THREADS, 4) void small_bwd_kernel(ActJob d, GradJob w, SumJob s)
{
    extern __shared__ __align__(16) char smem[];
    int block = blockIdx.x;
    if (block < d.blocks) return act_tile<NB, true>(d, block, smem, threadIdx.x);
    block -= d.blocks;
    if (block < w.blocks) return grad_tile(w, block, smem, threadIdx.x);
    block -= w.blocks;
    if (s.dY) sum_rows(s, block, smem, threadIdx.x);
    else sum_slices(s, block, threadIdx.x);
}

constexpr int64_t MOST_TOKENS = 1024;      // above, the tiles are as fast or faster in every shape tried

inline int steps_of(int64_t K) { return (int)ceil_div(K, 64); }
// LDS of a workgroup, for the groups of steps that are under way: as many as there are, up to `most`, and within `limit` bytes
// as far as that leaves two.
inline int ring_of(int64_t K, int group_steps, int most, int step_bytes, int limit)
{
    const int groups = (int)ceil_div(steps_of(K), group_steps);
    return std::min(groups, std::max(std::min(2, most), std::min(most, limit / (group_steps * step_bytes))));
}
// Steps of a K-slice, of the slices that the output tiles would run.
inline int slice_steps(const MatOp& op)
{
    const int64_t splits = op.splits > 1 && op.partial ? op.splits : 1;
    return splits > 1 ? steps_of(ceil_div(op.K, splits)) : 1 << 30;
}

// Width of the blocks of a product that shares its launch with `others` workgroups: the narrowest that give each a unit of its own,
// else 64 columns, and 128 where those alone are more than two rounds (and K is not sliced: the widest keep one chain).  With a
// gradient beside it: 509 x 192 over 3072 17.8 -> 14.6 us in 32 columns, 16.2 in 64; 600 x 1024 over 256 21.6 -> 17.4 us in 64, 19.0
// in 32; 1024 x 4096 over 256 with it 26.4 -> 22.4 us in 128, 24.9 in 64.
struct Cut {
    int nb;
    int64_t blocks;
};
Cut cut(const MatOp& op, int64_t others)
{
    auto by = [&](int nb) { return Cut{nb, ceil_div(op.M, 32) * ceil_div(op.N, 32 * nb)}; };
    if (by(1).blocks + others <= 256) return by(1);
    if (by(2).blocks + others <= 384 || slice_steps(op) < steps_of(op.K)) return by(2);
    return by(4);
}

ActJob act_job(const MatOp& op, bool b_km, const Cut& c)
{
    ActJob g;
    g.A = (const bf16_t*)op.A; g.B = (const bf16_t*)op.B; g.C = (bf16_t*)op.C; g.aux = (bf16_t*)op.aux; g.bias = op.bias;
    g.lda = (uint32_t)op.a_sm; g.ldb = (uint32_t)(b_km ? op.b_sk : op.b_sn); g.ldc = (uint32_t)op.ldc; g.ldaux = (uint32_t)op.ldaux;
    g.M = (int)op.M; g.N = (int)op.N; g.K = (int)op.K; g.epilogue = op.epilogue; g.slice = slice_steps(op);
    g.col_blocks = (int)ceil_div(op.N, 32 * c.nb);
    g.blocks = (int)c.blocks;
    return g;
}

bool act_ok(const MatOp& op)
{
    return mfma_gemm2_supported(op) && op.gather == GATHER_NONE && !op.out_f32 && op.batch == 1 && op.a_sk == 1 && op.K % 16 == 0 && op.N % 16 == 0 &&
           op.M <= MOST_TOKENS && op.N < 65536 && op.ldc <= BUF_MAX_LD && op.ldaux <= BUF_MAX_LD &&
           (op.epilogue == EPI_NONE || (op.epilogue == EPI_ACT_GRAD) == (op.b_sk != 1));
}

// A product by itself: a workgroup to a unit, and a reduction of more than one step (one is no faster than a tile's) up to 2048:
// beyond, a workgroup's chain takes longer than slices over several and their sum (operands not in the caches: 48 x 256 over 1024
// 9.7 -> 8.7 us with the product after it, 48 x 512 over 2048 8.8 -> 7.9 us, 48 x 192 over 3072 8.0 against 9.0, 48 x 256 over 4096 8.7
// against 11.3).  In 64 columns only short ones (509 x 1024 over 256 1.3 us, 600 x 512 over 1024 even).  A k-major operand of 4 MB
// and more comes faster in the tiles' whole lines (1 x 8192 over 512 3.7 against 5.6 us, 2048 x 1008 8.1 -> 7.2 us), and so do more than 512
// rows (1024 x 256 over 1024 5.9 against 6.5 us, 509 of them 6.1 -> 5.7).  Two steps win 0.2 us of 3.2 with operands from memory and lose 0.2 of
// 2.7 with those in the caches; from three on they win 0.5 and are even.
bool alone_ok(const MatOp& op)
{
    if (!act_ok(op) || (op.b_sk != 1 && (op.K * op.N >= (int64_t(1) << 21) || op.M > 512))) return false;
    const Cut c = cut(op, 0);
    const int steps = steps_of(op.K);
    return c.blocks <= 256 && steps > 1 && (c.nb == 1 ? steps <= 32 : c.nb == 2 && steps <= 4);
}

// LDS for each of the workgroups that share a unit (two for up to two rounds of single ones).
inline int lds_limit(int64_t blocks) { return blocks <= 256 ? 160 * 1024 : 80 * 1024; }

template <int NB>
hipError_t launch_fwd(const MatOp& op, const Cut& c, hipStream_t st)
{
    static OncePerDevice allowed;
    typedef ActShape<NB> S;
    const hipError_t e = allow_lds(small_fwd_kernel<NB>, S::RING * S::G * S::STEP, allowed);
    if (e != hipSuccess) return e;
    ActJob g = act_job(op, false, c);
    g.ring = ring_of(op.K, S::G, S::RING, S::STEP, lds_limit(c.blocks));
    note_kernel(NB == 1 ? "small_fwd_kernel<32>" : "small_fwd_kernel<64>");
    hipLaunchKernelGGL((small_fwd_kernel<NB>), dim3((unsigned)c.blocks), dim3(THREADS), g.ring * S::G * S::STEP, st, g);
    return hipGetLastError();
}

template <int NB>
hipError_t launch_bwd(ActJob d, GradJob w, const SumJob& s, hipStream_t st)
{
    typedef ActShape<NB> S;
    constexpr int most = std::max(S::RING * S::G * S::STEP, GRAD_RING * GRAD_G * GRAD_STEP);
    static OncePerDevice allowed;
    const hipError_t e = allow_lds(small_bwd_kernel<NB>, most, allowed);
    if (e != hipSuccess) return e;
    int lds = s.blocks ? 2 * 8 * 32 * 9 * 4 : 0;
    const int limit = lds_limit(d.blocks + w.blocks);
    if (d.blocks) {
        d.ring = ring_of(d.K, S::G, S::RING, S::STEP, limit);
        lds = std::max(lds, d.ring * S::G * S::STEP);
    }
    if (w.blocks) {
        w.ring = ring_of(w.K, GRAD_G, GRAD_RING, GRAD_STEP, limit);
        lds = std::max(lds, w.ring * GRAD_G * GRAD_STEP);
    }
    note_kernel(NB == 1 ? "small_bwd_kernel<32>" : NB == 2 ? "small_bwd_kernel<64>" : "small_bwd_kernel<128>");
    hipLaunchKernelGGL((small_bwd_kernel<NB>), dim3((unsigned)(d.blocks + w.blocks + s.blocks)), dim3(THREADS), lds, st, d, w, s);
    return hipGetLastError();
}

}  // namespace

bool mfma_small_fwd_supported(const MatOp& op) { return op.b_sk == 1 && alone_ok(op); }

hipError_t mfma_small_fwd(const MatOp& op, hipStream_t st)
{
    const Cut c = cut(op, 0);
    return c.nb == 1 ? launch_fwd<1>(op, c, st) : launch_fwd<2>(op, c, st);
}

bool mfma_small_data_supported(const MatOp& op) { return op.b_sk != 1 && alone_ok(op); }

// Two products of the backward pass in one launch.  Below 512 tokens, where the tiles do not cut a gradient's reduction, that saves a
// launch, or two: as long as the workgroups are about two rounds, and the data product's chain is not the longer part (48 x 192 over
// 3072 with its gradient and the product after it 14.6 -> 13.1 us, 48 x 256 over 4096 16.9 against 19.3; 256 x 4096 over 256 17.6 -> 15.3, 509 of
// it 19.0 against 19.3).  Above, it saves the gradient's partial sums as well (600 x 256 over 4096 24.5 -> 20.5, 600 x 4096 over 256 21.6 -> 18.4 us,
// 1024 x 4096 over 1024 42.3 against 44.2).
bool mfma_small_pair_supported(const MatOp& data, const MatOp& grad)
{
    if (data.b_sk == 1 || !act_ok(data)) return false;
    // (neither operand of a gradient is k-contiguous: any number of tokens, also one)
    MatOp op = grad;
    op.K = std::max<int64_t>(op.K, 8);
    if (!mfma_gemm2_supported(op) || op.gather != GATHER_NONE || !op.out_f32 || op.batch != 1 || op.a_sk == 1 || op.b_sk == 1 || op.sgd || op.crop ||
        op.K > MOST_TOKENS || op.M >= 65536 || op.N >= 65536 || op.ldc > BUF_MAX_LD)
        return false;
    const int64_t tiles = ceil_div(op.M, 64) * ceil_div(op.N, 64), all = cut(data, tiles).blocks + tiles;
    return grad.K < 512 ? all <= 512 && steps_of(data.K) <= 48 : all <= 1792 && steps_of(data.K) <= 96;
}

hipError_t mfma_small_bwd(const MatOp* data, const MatOp* grad, const SmallSums* sums, hipStream_t st)
{
    ActJob d{};
    GradJob w{};
    SumJob s{};
    if (grad) {
        w.A = (const bf16_t*)grad->A; w.B = (const bf16_t*)grad->B; w.C = (float*)grad->C;
        w.lda = (uint32_t)grad->a_sk; w.ldb = (uint32_t)grad->b_sk; w.ldc = (uint32_t)grad->ldc;
        w.M = (int)grad->M; w.N = (int)grad->N; w.K = (int)grad->K; w.slice = slice_steps(*grad);
        w.col_blocks = (int)ceil_div(w.N, 64);
        w.blocks = (int)ceil_div(w.M, 64) * w.col_blocks;
    }
    Cut c{1, 0};
    if (data) {
        c = cut(*data, w.blocks);
        d = act_job(*data, true, c);
    }
    if (sums) {
        s.dY = (const bf16_t*)sums->dY; s.part = sums->part; s.out = sums->out;
        s.T = (int)sums->T; s.n = (int)sums->n; s.rows = (int)sums->rows; s.slices = (int)sums->slices;
        s.col_blocks = (int)ceil_div(sums->n, 256);
        // partial sums on the units that the products leave, or beside them on at least 32
        const int halves = (s.col_blocks * s.slices + 1) / 2;
        s.runs = (int)ceil_div(halves, std::max(32, 256 - d.blocks - w.blocks));
        s.blocks = sums->dY ? (int)ceil_div(halves, s.runs) : (int)ceil_div(sums->n, THREADS * 4);
    }
    if (d.blocks + w.blocks + s.blocks == 0) return hipSuccess;
    return c.nb == 1 ? launch_bwd<1>(d, w, s, st) : c.nb == 2 ? launch_bwd<2>(d, w, s, st) : launch_bwd<4>(d, w, s, st);
}

}  // namespace lrd
