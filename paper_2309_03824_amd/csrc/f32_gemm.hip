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

// Floats of LDS for the sums of `waves` blocks of 16 T x 16 T.
constexpr int f32_lds(int T, int waves) { return waves * 16 * T * (16 * T + 4); }

// Tile of E WM x E WN results, E = 16 T; KS waves share each E x E block, wave s of them taking steps s, s + KS, ...
template <int T, int WM, int WN, int KS, int DEPTH, bool AKM, bool BKM>
__global__ __launch_bounds__(64 * WM * WN * KS) void f32_gemm_kernel(F32Operand A, F32Operand B, float* __restrict__ C, int64_t ldc,
                                                                     const float* __restrict__ bias, float* __restrict__ partial, int M,
                                                                     int N, int k_per_split)
{
    const unsigned bx = blockIdx.x, by = blockIdx.y, bz = blockIdx.z;
    __shared__ __align__(16) float lds[f32_lds(T, WM * WN * KS)];
#include "f32_tile.inc"
}

struct F32Job {
    F32Operand A, B;
    float* C;
    int64_t ldc;
    const float* bias;
    int M, N, K;
};
// The same tile with all of K, as one of the jobs of a launch.
template <int T, bool AKM>
__device__ __forceinline__ void f32_job_tile(const F32Operand& A, const F32Operand& B, float* C, int64_t ldc, const float* bias, int M, int N, int k_per_split,
                                             unsigned bx, unsigned by, float* lds_of_launch)
{
    constexpr int WM = 1, WN = 1, KS = 8, DEPTH = T == 1 ? 8 : 4;
    constexpr bool BKM = true;
    constexpr unsigned bz = 0;
    constexpr float* partial = nullptr;
    float& lds = *lds_of_launch;
#include "f32_tile.inc"
}

// A data gradient and a weight gradient that do not wait for one another, in one launch: with few tokens neither fills the chip
// and 2.5 us of each is the launch (256 x 768 x 768 layer at rank 208, first factor frozen: a pass 23.2 -> 20.6 us).
// Both tiles sum in one buffer, the larger of the two's: an array of each, side by side, was 72 KB with 32 x 32 blocks of both.
template <int TD, int TW>
__global__ __launch_bounds__(512) void f32_pair_kernel(F32Job d, int d_rows, int d_blocks, F32Job w, int w_rows)
{
    __shared__ __align__(16) float lds[f32_lds(TD > TW ? TD : TW, 8)];
    const int block = blockIdx.x - d_blocks;
    if (block < 0) f32_job_tile<TD, false>(d.A, d.B, d.C, d.ldc, d.bias, d.M, d.N, d.K, blockIdx.x % d_rows, blockIdx.x / d_rows, lds);
    else f32_job_tile<TW, true>(w.A, w.B, w.C, w.ldc, w.bias, w.M, w.N, w.K, block % w_rows, block / w_rows, lds);
}

F32Job f32_job(const MatOp& op)
{
    const bool akm = op.a_sk != 1, bkm = op.b_sk != 1;
    return {{(const float*)op.A, akm ? op.a_sk : op.a_sm, (int)op.M, (int)op.K}, {(const float*)op.B, bkm ? op.b_sk : op.b_sn, (int)op.N, (int)op.K},
            (float*)op.C, op.ldc, op.bias, (int)op.M, (int)op.N, (int)op.K};
}

template <int T, int WM, int WN, int KS, int DEPTH>
hipError_t launch(const MatOp& op, int splits, hipStream_t st)
{
    const bool akm = op.a_sk != 1, bkm = op.b_sk != 1;
    const F32Job g = f32_job(op);
    const int kps = (int)(ceil_div(ceil_div(op.K, splits), 16) * 16);
    splits = (int)ceil_div(op.K, kps);
    float* partial = splits > 1 ? op.partial : nullptr;
    const float* bias = partial ? nullptr : op.bias;
    const dim3 grid((unsigned)ceil_div(op.M, 16 * T * WM), (unsigned)ceil_div(op.N, 16 * T * WN), (unsigned)splits), block(64 * WM * WN * KS);
#define LRD_F32_LAUNCH(AK, BK_) \
    hipLaunchKernelGGL((f32_gemm_kernel<T, WM, WN, KS, DEPTH, AK, BK_>), grid, block, 0, st, g.A, g.B, g.C, g.ldc, bias, partial, g.M, g.N, kps)
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

namespace {
// The tile that f32_gemm gives a product: E = 16 T, or 64 x 64; and the slices of K over workgroups.
struct F32Plan { int t; int64_t splits; };
F32Plan f32_plan(const MatOp& op)
{
    const int64_t t32 = ceil_div(op.M, 32) * ceil_div(op.N, 32), t64 = ceil_div(op.M, 64) * ceil_div(op.N, 64);
    // 64 x 64 tiles (each operand value read half as often) from about one workgroup per compute unit on: 2048 x 432
    // over 1024 36.5 us with 32 x 32 tiles, 34.2 us with these; below, 32 x 32, and while those leave half of the
    // chip idle, 16 x 16 ([256 x 208] over 768: 8.2 -> 5.2 us).
    // The waves of a workgroup and the workgroups together cut K into at least as many chains of additions as the
    // caller asked for slices: the error grows with the root of a chain's length (1000 x 1000 over 20000 in 8 chains
    // 9.0e-7, in 2 1.8e-6).
    const int64_t slices = op.partial && !op.bias ? op.splits : 1;
    if (t64 >= 192) return {4, ceil_div(slices, 2)};
    // Beyond that, K is cut over workgroups only where the tiles leave most of the chip idle and the reduction is long
    int64_t splits = op.K < 1024 ? 1 : std::max<int64_t>(1, std::min(slices, 256 / t32));
    splits = std::max(splits, ceil_div(slices, 8));
    return {t32 * splits < 128 ? 1 : 2, splits};
}
}  // namespace

hipError_t f32_gemm(const MatOp& op, hipStream_t st)
{
    note_kernel("f32_gemm_kernel");
    const F32Plan p = f32_plan(op);
    if (p.t == 4) return launch<2, 2, 2, 2, 4>(op, (int)p.splits, st);
    if (p.t == 1) return launch<1, 1, 1, 8, 8>(op, (int)p.splits, st);
    return launch<2, 1, 1, 8, 4>(op, (int)p.splits, st);
}

// Workgroups of a product in blocks of 16 T x 16 T.
int64_t f32_blocks(const MatOp& op, int t) { return ceil_div(op.M, 16 * t) * ceil_div(op.N, 16 * t); }

// The same tiles as by themselves, in the same order of additions: whatever f32_gemm would run unsliced in 16 x 16 or 32 x 32.  Not
// where the gradient's tiles, the last to start, are the longer chains and more than fit beside the others (two workgroups to a unit):
// they then run on after everything else, 2000 x 768 x 768 at rank 208 with the second factor's gradient 48.4 us apart and 52.4 together,
// 500 x 1000 -> 384 at rank 150 with the first one's 16.8 and 19.5.
bool f32_pair_supported(const MatOp& data, const MatOp& grad)
{
    if (!f32_gemm_supported(data) || !f32_gemm_supported(grad) || data.a_sk != 1 || data.b_sk == 1 || grad.a_sk == 1 || grad.b_sk == 1 || grad.sgd) return false;
    const F32Plan d = f32_plan(data), w = f32_plan(grad);
    if (d.t == 4 || w.t == 4 || d.splits > 1 || w.splits > 1) return false;
    const bool late = d.t == 2 && f32_blocks(data, d.t) + f32_blocks(grad, w.t) > 512 && grad.K > data.K && grad.K >= 256;
    return !late;
}

hipError_t f32_pair(const MatOp& data, const MatOp& grad, hipStream_t st)
{
    const F32Job d = f32_job(data), w = f32_job(grad);
    const int td = f32_plan(data).t, tw = f32_plan(grad).t;
    const int dr = (int)ceil_div(data.M, 16 * td), db = dr * (int)ceil_div(data.N, 16 * td), wr = (int)ceil_div(grad.M, 16 * tw);
    const dim3 grid((unsigned)(db + wr * (int)ceil_div(grad.N, 16 * tw))), block(512);
    note_kernel(td == 1 ? tw == 1 ? "f32_pair_kernel<1,1>" : "f32_pair_kernel<1,2>" : tw == 1 ? "f32_pair_kernel<2,1>" : "f32_pair_kernel<2,2>");
    if (td == 1 && tw == 1) hipLaunchKernelGGL((f32_pair_kernel<1, 1>), grid, block, 0, st, d, dr, db, w, wr);
    else if (td == 1) hipLaunchKernelGGL((f32_pair_kernel<1, 2>), grid, block, 0, st, d, dr, db, w, wr);
    else if (tw == 1) hipLaunchKernelGGL((f32_pair_kernel<2, 1>), grid, block, 0, st, d, dr, db, w, wr);
    else hipLaunchKernelGGL((f32_pair_kernel<2, 2>), grid, block, 0, st, d, dr, db, w, wr);
    return hipGetLastError();
}

}  // namespace lrd
