// fp32 products on the matrix cores (v_mfma_f32_16x16x4_f32: fp32 operands, fp32 accumulation), any sizes,
// either operand stored K-contiguous or K-major.
//
// The fp32 path runs small products (a few hundred tokens, one layer), so it is bound by latency and by how
// many compute units get work, not by bandwidth: a workgroup takes a small tile of the result, cuts K over its
// waves, and every wave fetches its operand fragments straight from memory (L2) into registers, three or
// seven steps ahead of the matrix instructions; there is no LDS and no barrier before the waves' sums meet at the end.
// [256 x 208] over K = 768: 5.2 us (208 workgroups of 16 x 16 tiles; about 2.5 us of it are the launch)
// against 94 us on 16 workgroups of 64 x 64 FMA tiles with two barriers per 16 k; [2048 x 1024] over K = 1024:
// 62 us = 69 TFLOP/s of about 153.
//
// A step is 16 k.  Lane l belongs to k-group g = l >> 4; matrix instruction c of the step contracts
// k = 4 g + c.  K-contiguous operand: one 16-byte load per 16-row block gives the lane (row l & 15) its four
// values.  K-major operand: for each c one load of T consecutive rows of k gives the lane its value of each of
// the T blocks, block b then being the rows T i + b.
#include <algorithm>

#include "lrd_internal.hpp"

namespace lrd {
namespace {

typedef f32x4 f32x4u __attribute__((aligned(4)));
typedef f32x2 f32x2u __attribute__((aligned(4)));

struct F32Operand {
    const float* p;
    int64_t ld;
    int rows, K;
};

// Fragments of T 16-row blocks for one step.
template <int T, bool KM>
struct F32Frag {
    static_assert(T == 1 || T == 2, "one load per k of a K-major operand");
    float v[T][4];     // [block][c]

    // `row0`: first row of the wave's blocks.  Rows past the end repeat the last one (their results are not
    // stored); TAIL: k from kend on counts as zero.
    template <bool TAIL>
    __device__ __forceinline__ void load(const F32Operand& o, int row0, int k0, int kend, int lane)
    {
        const int i = lane & 15, g = lane >> 4;
        if (KM) {
            const int row = row0 + T * i, from = min(row, o.rows - T);
            const bool last = row == o.rows - 1;        // odd extent: the pair is read one row earlier
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int k = k0 + 4 * g + c;
                if constexpr (T == 1) {
                    const float x = o.p[(int64_t)(TAIL ? min(k, kend - 1) : k) * o.ld + from];
                    v[0][c] = !TAIL || k < kend ? x : 0.f;
                    continue;
                } else {
                const f32x2 x = *reinterpret_cast<const f32x2u*>(o.p + (int64_t)(TAIL ? min(k, kend - 1) : k) * o.ld + from);
                v[0][c] = !TAIL || k < kend ? (last ? x.y : x.x) : 0.f;
                v[1][c] = !TAIL || k < kend ? x.y : 0.f;
                }
            }
        } else {
            const int k = k0 + 4 * g;
#pragma unroll
            for (int b = 0; b < T; ++b) {
                const float* at = o.p + (int64_t)min(row0 + 16 * b + i, o.rows - 1) * o.ld;
                if constexpr (TAIL) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) v[b][c] = k + c < kend ? at[min(k + c, kend - 1)] : 0.f;
                } else {
                    const f32x4 x = *reinterpret_cast<const f32x4u*>(at + k);
#pragma unroll
                    for (int c = 0; c < 4; ++c) v[b][c] = x[c];
                }
            }
        }
    }
};

// Tile of E WM x E WN results, E = 16 T; KS waves share each E x E block, wave s of them taking steps s, s + KS, ...
template <int T, int WM, int WN, int KS, int DEPTH, bool AKM, bool BKM>
__global__ __launch_bounds__(64 * WM * WN * KS) void f32_gemm_kernel(F32Operand A, F32Operand B, float* __restrict__ C, int64_t ldc,
                                                                     const float* __restrict__ bias, float* __restrict__ partial, int M,
                                                                     int N, int k_per_split)
{
    constexpr int E = 16 * T, NT = 64 * WM * WN * KS, LDT = E + 4;
    __shared__ float sums[KS][WM * WN][E * LDT];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ks = wave % KS, blk = wave / KS, wm = blk / WN, wn = blk % WN;
    const int m0 = blockIdx.x * E * WM, n0 = blockIdx.y * E * WN;
    const int mrow = m0 + wm * E, nrow = n0 + wn * E;
    const int kbeg = blockIdx.z * k_per_split, kend = min(A.K, kbeg + k_per_split);

    f32x4 acc[T][T];
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    if (mrow < M && nrow < N) {
        F32Frag<T, AKM> a[DEPTH];
        F32Frag<T, BKM> b[DEPTH];
        auto multiply = [&](int at) {
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int i = 0; i < T; ++i)
#pragma unroll
                    for (int j = 0; j < T; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[at].v[j][c], a[at].v[i][c], acc[i][j], 0, 0, 0);
        };
        const int whole = (kend - kbeg) / 16;                                // steps without a tail
        const int mine = whole > ks ? (whole - ks + KS - 1) / KS : 0;
        auto fetch = [&](int s, int at) {
            const int k = kbeg + 16 * (ks + s * KS);
            a[at].template load<false>(A, mrow, k, kend, lane);
            b[at].template load<false>(B, nrow, k, kend, lane);
        };
#pragma unroll
        for (int d = 0; d < DEPTH - 1; ++d)
            if (d < mine) fetch(d, d);
        int s = 0;
        for (; s + 2 * DEPTH - 1 <= mine; s += DEPTH) {
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                fetch(s + d + DEPTH - 1, (d + DEPTH - 1) % DEPTH);
                multiply(d);
            }
        }
        for (; s < mine; s += DEPTH) {
#pragma unroll
            for (int d = 0; d < DEPTH; ++d) {
                if (s + d + DEPTH - 1 < mine) fetch(s + d + DEPTH - 1, (d + DEPTH - 1) % DEPTH);
                if (s + d < mine) multiply(d);
            }
        }
        if (kbeg + 16 * whole < kend && whole % KS == ks) {
            a[0].template load<true>(A, mrow, kbeg + 16 * whole, kend, lane);
            b[0].template load<true>(B, nrow, kbeg + 16 * whole, kend, lane);
            multiply(0);
        }
    }
    // roles swapped: a lane holds row m = lane & 15 of its block, columns 4 (lane >> 4) + e
    {
        const int i16 = lane & 15, g = lane >> 4;
#pragma unroll
        for (int i = 0; i < T; ++i)
#pragma unroll
            for (int j = 0; j < T; ++j)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int m = AKM ? T * i16 + i : 16 * i + i16;
                    const int n = BKM ? T * (4 * g + e) + j : 16 * j + 4 * g + e;
                    sums[ks][blk][m * LDT + n] = acc[i][j][e];
                }
    }
    __syncthreads();
    float* out = partial ? partial + (int64_t)blockIdx.z * M * N : C;
    const int64_t ldo = partial ? (int64_t)N : ldc;
    constexpr int QR = E / 4, QB = E * QR;      // groups of four columns per row and per block
    for (int q = tid; q < WM * WN * QB; q += NT) {
        const int bk = q / QB, ml = q / QR % E, nl = q % QR * 4;
        f32x4 s = *reinterpret_cast<const f32x4*>(&sums[0][bk][ml * LDT + nl]);
#pragma unroll
        for (int z = 1; z < KS; ++z) s += *reinterpret_cast<const f32x4*>(&sums[z][bk][ml * LDT + nl]);
        const int m = m0 + bk / WN * E + ml, n = n0 + bk % WN * E + nl;
        if (m >= M) continue;
        if (n + 3 < N) {
            if (bias) s += *reinterpret_cast<const f32x4u*>(bias + n);
            *reinterpret_cast<f32x4u*>(out + (int64_t)m * ldo + n) = s;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (n + e < N) out[(int64_t)m * ldo + n + e] = s[e] + (bias ? bias[n + e] : 0.f);
        }
    }
}

template <int T, int WM, int WN, int KS, int DEPTH>
hipError_t launch(const MatOp& op, int splits, hipStream_t st)
{
    const bool akm = op.a_sk != 1, bkm = op.b_sk != 1;
    const F32Operand A{(const float*)op.A, akm ? op.a_sk : op.a_sm, (int)op.M, (int)op.K};
    const F32Operand B{(const float*)op.B, bkm ? op.b_sk : op.b_sn, (int)op.N, (int)op.K};
    const int kps = (int)(ceil_div(ceil_div(op.K, splits), 16) * 16);
    splits = (int)ceil_div(op.K, kps);
    float* partial = splits > 1 ? op.partial : nullptr;
    const float* bias = partial ? nullptr : op.bias;
    const dim3 grid((unsigned)ceil_div(op.M, 16 * T * WM), (unsigned)ceil_div(op.N, 16 * T * WN), (unsigned)splits), block(64 * WM * WN * KS);
#define LRD_F32_LAUNCH(AK, BK_) \
    hipLaunchKernelGGL((f32_gemm_kernel<T, WM, WN, KS, DEPTH, AK, BK_>), grid, block, 0, st, A, B, (float*)op.C, op.ldc, bias, partial, (int)op.M, (int)op.N, kps)
    if (akm) { if (bkm) LRD_F32_LAUNCH(true, true); else LRD_F32_LAUNCH(true, false); }
    else { if (bkm) LRD_F32_LAUNCH(false, true); else LRD_F32_LAUNCH(false, false); }
#undef LRD_F32_LAUNCH
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !partial) return e;
    return reduce_partials(partial, op.C, false, op.ldc, op.M, op.N, splits, st, op.sgd);
}

}  // namespace

bool f32_gemm_supported(const MatOp& op)
{
    if (op.in_bf16 || !op.out_f32 || op.gather != GATHER_NONE || op.batch != 1) return false;
    // A K-major operand is read in pairs of rows: a single token and rank 1 stay with the FMA engine.
    if (op.M < 2 || op.N < 2 || op.K < 1) return false;
    const int64_t lim = int64_t(1) << 30;
    if (op.M >= lim || op.N >= lim || op.K >= lim || ceil_div(op.N, 16) > 65535) return false;
    return (op.a_sk == 1 || op.a_sm == 1) && (op.b_sk == 1 || op.b_sn == 1);
}

hipError_t f32_gemm(const MatOp& op, hipStream_t st)
{
    note_kernel("f32_gemm_kernel");
    const int64_t t32 = ceil_div(op.M, 32) * ceil_div(op.N, 32), t64 = ceil_div(op.M, 64) * ceil_div(op.N, 64);
    // 64 x 64 tiles (each operand value read half as often) from about one workgroup per compute unit on: 2048 x 432
    // over 1024 36.5 us with 32 x 32 tiles, 34.2 us with these; below, 32 x 32, and while those leave half of the
    // chip idle, 16 x 16 ([256 x 208] over 768: 8.2 -> 5.2 us).
    // The waves of a workgroup and the workgroups together cut K into at least as many chains of additions as the
    // caller asked for slices: the error grows with the root of a chain's length (1000 x 1000 over 20000 in 8 chains
    // 9.0e-7, in 2 1.8e-6).
    const int64_t slices = op.partial && !op.bias ? op.splits : 1;
    if (t64 >= 192) return launch<2, 2, 2, 2, 4>(op, (int)ceil_div(slices, 2), st);
    // Beyond that, K is cut over workgroups only where the tiles leave most of the chip idle and the reduction is long
    int64_t splits = op.K < 1024 ? 1 : std::max<int64_t>(1, std::min(slices, 256 / t32));
    splits = std::max(splits, ceil_div(slices, 8));
    if (t32 * splits < 128) return launch<1, 1, 1, 8, 8>(op, (int)splits, st);
    return launch<2, 1, 1, 8, 4>(op, (int)splits, st);
}

}  // namespace lrd
