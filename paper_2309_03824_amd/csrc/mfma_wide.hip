// bf16 products with a short reduction and a wide result: C[M x N] = A . B^T (+ bias), K <= 512 (the second product of a
// layer pair, K = rank, and its data gradient), with the GELU epilogues.
//
// Such a product is its result leaving: 8192 x 4096 x 256 with GELU writes 134 MB, 26 us at the rate of a kernel that only
// stores, against 9 us of matrix instructions.  In output tiles each workgroup is a chain load -> multiply -> store whose
// ends nothing overlaps, and every tile loads its rows of A again.  Here a wave keeps 32 rows of A in registers, all of K, and a
// workgroup walks along N: B goes by in chunks of 64 columns through two LDS buffers (loads straight into LDS, one chunk
// ahead), and results leave each wave as whole 128-byte lines by way of 4 KB of LDS of its own, without a barrier.  The wait
// before a chunk leaves out the stores of the chunk before: they are younger than the loads it waits for.  (The compiler, which does not see
// that wait, waits for A's registers between the products of every chunk, and with them for those stores and most of the next
// chunk's loads.  Without those waits the kernel is no faster and often slower, as if they kept the workgroups of a unit apart: 8192 x 8192 x 256
// with GELU 62.6 -> 67.6 us, 8192 x 3072 x 192 with its gradient 29.2 -> 28.8, encoder step 4105 -> 4120.)
// v_mfma_f32_16x16x32_bf16 and not 32x32x16: with random operands the shorter form sustains more (16384 x 4096 x 512
// 61 against 67 us).  Multiplying one chunk while the one before leaves, in a second set of accumulators, gave nothing (63 us).
// Against output tiles: 8192 x 4096 x 256 with GELU inside the encoder step 40.4 -> 36.2 us, with its gradient 45.0 -> 38.8
// us; by themselves 16384 x 4096 x 256 53.4 -> 38.4 us, 16384 x 4096 x 512 87.7 -> 60.8 us, inside a layer of that size, where A has
// just been written and the results fill the caches for the next product, 95 -> 75 and 100 -> 80 us (its data gradient).
#include <algorithm>
#include <cstdio>
#include <string>

#include "lds_load.hpp"
#include "lrd_internal.hpp"
#include "wide_plan.hpp"

namespace lrd {
namespace {

constexpr int COLS = 64;             // columns of a chunk: a result row of it is one 128-byte line
constexpr int ROWS = 32;             // rows of a wave
constexpr int SUB = COLS * 64 * 2;   // LDS bytes of 64 k of a chunk
constexpr int AUX_NT = 2;            // non-temporal: results and pre-activations are touched once

struct WideArgs {
    const bf16_t* A;
    const bf16_t* B;
    bf16_t* C;
    bf16_t* aux;
    const float* bias;
    int64_t lda, ldb, ldc, ldaux;
    int64_t a_bs, b_bs, c_bs, aux_bs, bias_bs;
    int M, N, K;
    int inner, outer, chunks;        // a workgroup: 32 rows per wave x `chunks` chunks, the last range of columns with what is left
    int by_columns;                  // row blocks (`inner` of them) of a range follow one another, and not the ranges of a row block
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t descriptor(const char* base, uint32_t span)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(base), 0, (int)span, (int)BUF_FLAGS);
}

// KS = ceil(K / 64).  B k-contiguous [N x K] or (B_KM) k-major [K x N].
template <int KS, int NW, bool B_KM, int EPI>
__global__ __launch_bounds__(64 * NW, 2) void wide_kernel(WideArgs g)
{
    constexpr int CHUNK = KS * SUB, PER = 8 / NW;     // bytes of a chunk, loads per wave of a sub-tile
    constexpr int STORES = EPI == EPI_ACT_STORE ? 8 : 4;     // stores per wave of a chunk
    static_assert(PER * NW == 8, "whole loads");
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63, wave = (int)uni(threadIdx.x >> 6);
    // Workgroups go to the 8 dies in turn: each die takes a run of row blocks, whose column ranges follow one another, so that its
    // L2 fetches a few rows of A and all of B; or, by columns, a few columns of B and all of A.
    const uint32_t total = gridDim.x, f = blockIdx.x, die = f & 7u, per = total >> 3, more = total & 7u;
    uint32_t t = die * per + min(die, more) + (f >> 3);
    // (The order of two loops, chosen on the host: chosen here, the compiler loads the pointers only after these divisions, 0.7 us later.)
    const uint32_t in = t % (uint32_t)g.inner;
    t /= (uint32_t)g.inner;
    const uint32_t out = t % (uint32_t)g.outer;
    const int64_t z = t / (uint32_t)g.outer;
    const int range = (int)(g.by_columns ? out : in);
    const int64_t row0 = (int64_t)(g.by_columns ? in : out) * (ROWS * NW) + wave * ROWS;
    const int rows = (int)max((int64_t)0, min((int64_t)g.M - row0, (int64_t)ROWS));     // of this wave
    const int first = range * g.chunks, n_chunks = min(g.chunks, g.N / COLS - first);

    // B: the chunk moves the base, a sub-tile of 64 k too; a load covers 8 rows of 128 bytes, whose chunks are permuted
    // (kc_swz; k-major: the k rows that one transposing read takes, k .. k + 3 and those 8 further, fall on different banks)
    const uint32_t ldb = uni((uint32_t)g.ldb);
    const char* b0 = uni_ptr(g.B + z * g.b_bs + (int64_t)first * COLS * (B_KM ? 1 : g.ldb));
    const int64_t bstep = COLS * 2 * (B_KM ? (int64_t)1 : (int64_t)ldb);
    const uint32_t K = uni((uint32_t)g.K);
    uint32_t span = B_KM ? (63u * ldb + COLS) * 2u : (63u * ldb + K) * 2u;
    uint32_t span_tail = B_KM ? ((K - (KS - 1) * 64u - 1u) * ldb + COLS) * 2u : span - (KS - 1) * 128u;
    settle(b0, span);
    settle(b0, span_tail);
    uint32_t voff[PER], vtail[PER];
#pragma unroll
    for (int p = 0; p < PER; ++p) {
        const int row = (p * NW + wave) * 8 + (lane >> 3), slot = lane & 7;
        if (B_KM) {
            const int c = slot ^ (((row & 2) << 1) | ((row & 8) >> 2));
            voff[p] = ((uint32_t)row * ldb + c * 8) * 2u;
            vtail[p] = (KS - 1) * 64 + row < g.K ? voff[p] : BUF_OOB;
        } else {
            const int k = (slot ^ kc_swz(row)) * 8;
            voff[p] = ((uint32_t)row * ldb + k) * 2u;
            vtail[p] = (KS - 1) * 64 + k < g.K ? voff[p] : BUF_OOB;
        }
    }
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
    auto load_chunk = [&](int c) {
        const char* at = b0 + c * bstep;
#pragma unroll
        for (int s = 0; s < KS; ++s) {
            const char* sub = at + (B_KM ? (int64_t)s * 128 * ldb : (int64_t)s * 128);
            const uint32_t left = s == KS - 1 ? span_tail : B_KM ? span : span - s * 128u;
#pragma unroll
            for (int p = 0; p < PER; ++p)
                load_to_lds(lds0 + (c & 1) * CHUNK + s * SUB + (p * NW + wave) * 1024, sub, left, s == KS - 1 ? vtail[p] : voff[p]);
        }
    };
    // A in the layout of the MFMA operand: lane l holds row (l & 15), k = 8 * (l >> 4) + 0..7 of each group of 32
    const int q = lane >> 4, r16 = lane & 15;
    bf16x8 a[2][KS * 2];
    {
        const char* base = uni_ptr(g.A + z * g.a_bs + row0 * g.lda);
        const __amdgpu_buffer_rsrc_t ra = descriptor(base, uni(rows > 0 ? (uint32_t)(((rows - 1) * g.lda + g.K) * 2) : 0u));
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int kk = 0; kk < KS * 2; ++kk) {
                const int k = kk * 32 + q * 8, r = i * 16 + r16;
                const uint32_t off = k < g.K && r < rows ? ((uint32_t)r * (uint32_t)g.lda + k) * 2u : BUF_OOB;
                a[i][kk] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(ra, off, 0, 0));
            }
    }

    load_chunk(0);      // (behind A, whose rows the product before has just written: 1 us of 36)

    // fragments of B, in the same layout: column (l & 15) of a block of 16, k = 8 * (l >> 4) + 0..7
    const uint32_t f0 = B_KM ? (q * 8 + (r16 >> 2)) * 128 + ((r16 & 2) << 3) + (r16 & 1) * 8 : r16 * 128 + ((q ^ kc_swz(r16)) << 4);
    const uint32_t fx = B_KM ? (((r16 >> 2) & 2) << 1 | (q & 1) << 1) : 0;
    auto frag = [&](const char* at, int kk, int j) {
        if constexpr (B_KM) {
            typedef short s16x4 __attribute__((ext_vector_type(4)));
            typedef short s16x8 __attribute__((ext_vector_type(8)));
            const char* p = at + kk * 4096 + f0 + (((j * 2) ^ fx) << 4);
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p + 512));
            const s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            return __builtin_bit_cast(bf16x8, v);
        } else {
            return *reinterpret_cast<const bf16x8*>(at + (kk >> 1) * SUB + j * 2048 + ((kk & 1) ? f0 ^ 64 : f0));
        }
    };

    // results: 16 rows at a time go through this wave's staging block, 128 bytes a row with permuted chunks
    char* const stage = reinterpret_cast<char*>(smem) + 2 * CHUNK + wave * 2048;
    const int wr = r16 * 128 + (q & 1) * 8, srow = lane >> 3, scol = lane & 7;
    auto row_span = [&](int64_t ld) { return uni(rows > 0 ? (uint32_t)(((rows - 1) * ld + g.N) * 2) : 0u); };
    const char* const cbase = uni_ptr(g.C + z * g.c_bs + row0 * g.ldc);
    const __amdgpu_buffer_rsrc_t rc = descriptor(cbase, row_span(g.ldc));
    const __amdgpu_buffer_rsrc_t rx = EPI == EPI_NONE ? rc : descriptor(uni_ptr(g.aux + z * g.aux_bs + row0 * g.ldaux), row_span(g.ldaux));
    const float* const bias = g.bias ? g.bias + z * g.bias_bs : nullptr;
    // (rows that do not exist are stored past the descriptor, so that every wave issues the stores its waits count on)
    auto place = [&](int r, int64_t ld, int col0) { return r < rows ? ((uint32_t)r * (uint32_t)ld + col0 + scol * 8) * 2u : BUF_OOB; };

    // Where this loop's 5 KB of code begin counts for 3 % with the gradient of GELU: on a boundary of 128 bytes 8192 x 3072 x 192 takes
    // 29.3 us, 16 or 48 bytes behind one 30.9; x 256 and x 128 take 40.8 and 33.3 there, 40.0 and 32.0 where the compiler puts them.
    if constexpr (EPI == EPI_ACT_GRAD && KS == 3) asm volatile(".p2align 7");
    for (int c = 0; c < n_chunks; ++c) {
        // loads of chunk c: older than the stores of chunk c - 1
        if (c == 0) wait_vm<0>();
        else wait_vm<STORES>();
        lds_barrier();
        const int col0 = (first + c) * COLS;
        u32x4 zs[4];
        if constexpr (EPI == EPI_ACT_GRAD) {
#pragma unroll
            for (int e = 0; e < 4; ++e) zs[e] = __builtin_amdgcn_raw_buffer_load_b128(rx, place(e * 8 + srow, g.ldaux, col0), 0, AUX_NT);
        }
        if (c + 1 < n_chunks) load_chunk(c + 1);
        f32x4 acc[2][4];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        const char* at = reinterpret_cast<const char*>(smem) + (c & 1) * CHUNK;
#pragma unroll
        for (int kk = 0; kk < KS * 2; ++kk) {
            bf16x8 b[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) b[j] = frag(at, kk, j);
            // (operands swapped: a lane's four results are consecutive columns of one row)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i][kk], acc[i][j], 0, 0, 0);
        }
        if (bias) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const f32x4 b4 = *reinterpret_cast<const f32x4*>(bias + col0 + j * 16 + q * 4);
#pragma unroll
                for (int i = 0; i < 2; ++i) acc[i][j] += b4;
            }
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const u32x2 pk = {pack_bf16(acc[i][j][0], acc[i][j][1]), pack_bf16(acc[i][j][2], acc[i][j][3])};
                *reinterpret_cast<u32x2*>(stage + wr + (((j * 2 + (q >> 1)) ^ kc_swz(r16)) << 4)) = pk;
            }
            asm volatile("" ::: "memory");      // (a wave's LDS operations complete in order: its reads see its writes)
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int sr = e * 8 + srow;
                u32x4 v = *reinterpret_cast<const u32x4*>(stage + sr * 128 + ((scol ^ kc_swz(sr)) << 4));
                if constexpr (EPI == EPI_ACT_GRAD) {
                    bf16x8 c8 = __builtin_bit_cast(bf16x8, v), z8 = __builtin_bit_cast(bf16x8, zs[i * 2 + e]);
#pragma unroll
                    for (int x = 0; x < 8; ++x) c8[x] = (bf16_t)((float)c8[x] * gelu_grad_bf16_f((float)z8[x]));
                    v = __builtin_bit_cast(u32x4, c8);
                }
                __builtin_amdgcn_raw_buffer_store_b128(v, rc, place(i * 16 + sr, g.ldc, col0), 0, AUX_NT);
                if constexpr (EPI == EPI_ACT_STORE) {
                    bf16x8 c8 = __builtin_bit_cast(bf16x8, v);
#pragma unroll
                    for (int x = 0; x < 8; ++x) c8[x] = (bf16_t)gelu_bf16_f((float)c8[x]);
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, c8), rx, place(i * 16 + sr, g.ldaux, col0), 0, AUX_NT);
                }
            }
            asm volatile("" ::: "memory");
        }
    }
}

template <int KS, bool B_KM, int EPI>
hipError_t launch(const MatOp& op, hipStream_t st)
{
    // Four waves and two workgroups per compute unit while two of them fit its LDS (K <= 256), else eight waves and one.
    constexpr int NW = KS <= 4 ? 4 : 8, PER_CU = KS <= 4 ? 2 : 1;
    constexpr int lds_bytes = 2 * KS * SUB + NW * 2048;
    static_assert(PER_CU * lds_bytes <= 160 * 1024, "LDS of a compute unit");
    auto kern = wide_kernel<KS, NW, B_KM, EPI>;
    static OncePerDevice lds_allowed;
    const hipError_t e = allow_lds(kern, lds_bytes, lds_allowed);
    if (e != hipSuccess) return e;
    static const std::string tag = [] {
        char b[64];
        snprintf(b, sizeof(b), "wide_kernel<%d,%d,%s%s>", KS * 64, NW, B_KM ? "B_KM" : "B_KC",
                 EPI == EPI_ACT_STORE ? ",gelu" : EPI == EPI_ACT_GRAD ? ",gelu_grad" : "");
        return std::string(b);
    }();
    note_kernel(tag.c_str());
    WideArgs g;
    g.A = (const bf16_t*)op.A; g.B = (const bf16_t*)op.B; g.C = (bf16_t*)op.C; g.aux = (bf16_t*)op.aux; g.bias = op.bias;
    g.lda = op.a_sm; g.ldb = B_KM ? op.b_sk : op.b_sn; g.ldc = op.ldc; g.ldaux = op.ldaux;
    g.a_bs = op.a_bs; g.b_bs = op.b_bs; g.c_bs = op.c_bs; g.aux_bs = op.aux_bs; g.bias_bs = op.bias_bs;
    g.M = (int)op.M; g.N = (int)op.N; g.K = (int)op.K;
    const int row_blocks = (int)ceil_div(op.M, ROWS * NW);
    const int all = (int)(op.N / COLS);
    // By rows each die fetches all of B: slower than tiles once that is the larger part (1024 x 32000 x 256 33.6 us in tiles, 38.9
    // by rows, 27.9 by columns; 4096 x 50304 x 256 171, 139, 119 us).  A square-ish result is the better written by rows, where
    // a die's stores run along them (8192 x 16384 x 320 142 us in tiles, 99 by rows, 134 by columns); at 4 M columns both are even.
    g.by_columns = op.N > 6 * op.M;
    g.chunks = wide_chunks((int64_t)row_blocks * op.batch, all, 256 * PER_CU);
    const int ranges = (int)ceil_div(all, g.chunks);
    g.inner = g.by_columns ? row_blocks : ranges;
    g.outer = g.by_columns ? ranges : row_blocks;
    hipLaunchKernelGGL(kern, dim3((unsigned)((int64_t)row_blocks * ranges * op.batch)), dim3(64 * NW), lds_bytes, st, g);
    return hipGetLastError();
}

template <bool B_KM, int EPI>
hipError_t by_depth(const MatOp& op, hipStream_t st)
{
    switch (ceil_div(op.K, 64)) {
    case 1: return launch<1, B_KM, EPI>(op, st);
    case 2: return launch<2, B_KM, EPI>(op, st);
    case 3: return launch<3, B_KM, EPI>(op, st);
    case 4: return launch<4, B_KM, EPI>(op, st);
    case 5: return launch<5, B_KM, EPI>(op, st);
    case 6: return launch<6, B_KM, EPI>(op, st);
    case 7: return launch<7, B_KM, EPI>(op, st);
    default: return launch<8, B_KM, EPI>(op, st);
    }
}

}  // namespace

// Of the products mfma_gemm2 takes, those in whole chunks of 64 columns whose result is large enough to be what the time goes
// to.  Below 12 M results, or 24 chunks of columns, there are too few chunks per workgroup to pay for its start (8192 x 1024 x
// 256 9.6 us here, 7.9 us in tiles; 2048 x 4096 x 256 9.4 against 8.1 us; three members of 8192 x 1024 over 256 26.2 against
// 24.6 us; 8192 x 1536 x 256 11.2 against 12.3 us); over more than 256 k, where one workgroup fills a unit, below 32 M (8192 x
// 2048 x 512 23.1 against 22.6 us, 4100 x 4096 x 264 22.6 against 19.7 us; 8192 x 4096 x 512 with GELU 47.5 against 52.1 us).
bool mfma_wide_supported(const MatOp& op)
{
    if (!mfma_gemm2_supported(op) || op.gather != GATHER_NONE || op.out_f32 || op.splits > 1 || op.a_sk != 1) return false;
    if (op.N % COLS != 0 || op.N < 24 * COLS || op.K > 512) return false;
    if (op.M * op.N * op.batch < (op.K <= 256 ? 12000000 : 32000000)) return false;
    // Rows of the last row block that do not exist cost what others do: not where they are more than a third of all (300 x 128256 x 320
    // with GELU 55.5 us in tiles, 62.2 here, a block of 256 rows and one of 44; 48 x 262144 x 256 37.0 against 39.8).
    const int64_t block = ROWS * (op.K <= 256 ? 4 : 8);
    if (3 * op.M < 2 * block * ceil_div(op.M, block)) return false;
    // The shortest reductions over the widest results, too, are faster in tiles, which store 256 bytes of a row and not 128 (1024 x
    // 32000 x 64 with GELU 30.8 against 37.6 us, x 128 33.8 against 38.5; 2000 x 32000 x 128 with its gradient 64.1 against 69.9, plain
    // 41.1 -> 37.4 here).
    if (op.N > 24000 && (op.K <= 64 || (op.K <= 128 && (op.M <= 1024 || op.epilogue != EPI_NONE)))) return false;
    if (op.epilogue == EPI_ACT_STORE && op.b_sk != 1) return false;       // no layer pass has these two
    if (op.epilogue == EPI_ACT_GRAD && op.b_sk == 1) return false;
    if (op.M >= (int64_t(1) << 30) || op.ldc > BUF_MAX_LD || (op.epilogue != EPI_NONE && op.ldaux > BUF_MAX_LD)) return false;
    return ceil_div(op.M, 4 * ROWS) * (op.N / COLS) * op.batch < (int64_t(1) << 31);
}

hipError_t mfma_wide(const MatOp& op, hipStream_t st)
{
    if (op.b_sk != 1) return op.epilogue == EPI_ACT_GRAD ? by_depth<true, EPI_ACT_GRAD>(op, st) : by_depth<true, EPI_NONE>(op, st);
    return op.epilogue == EPI_ACT_STORE ? by_depth<false, EPI_ACT_STORE>(op, st) : by_depth<false, EPI_NONE>(op, st);
}

}  // namespace lrd
