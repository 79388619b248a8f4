// Engine selection for a single matrix product and the split-K policy.
#include <algorithm>
#include <atomic>
#include <cstdio>
#include <mutex>
#include <vector>

#include "lrd_internal.hpp"
#include "lrd_measure.h"

namespace lrd {

// What a product with a long reduction costs with each output tile: rounds of workgroups over the 256 compute units
// times the K-steps of a workgroup times the time of a step with every unit busy (microseconds, measured: 16384 x 512
// x 4096 takes 62.5 us in 128 x 256 tiles, 75 us in 128 x 128 ones at two workgroups per unit, 82 us in 128 x 128 ones
// at one; 8192 x 256 x 4096 24.5 us in 128 x 64 tiles, 28.4 us in 64 x 64 ones, 52 us in 128 x 256 ones; 16384 x 4096 x
// 4096 470 us in 256 x 256 ones against 485 us in 128 x 256 ones).  Larger tiles move fewer bytes into LDS per
// multiplication, smaller ones fill the chip when the result is small.
namespace {
struct StepTime { float full, one; };      // every unit at its workgroups per unit; at most one per unit
struct TileCost { int bm, bn, per_cu; StepTime step[GEMM_COSTS]; int ends; };
// (COST_WGRAD: 64-column tiles of a k-major operand fetch 128 bytes per row, which costs most when memory is busy: 12 x
// [192 x 3072] over 8192 239 us in 64 x 128 tiles, 215 us in 256 x 256 ones; COST_GATHER: address arithmetic with each
// load, which 64 x 64 tiles with one wave per SIMD cannot hide: 128 x 1152 over 25088 pixels 0.47 us a step.)
constexpr TileCost TILES[GEMM_TILES] = {
    {256, 256, 1, {{1.84f, 1.84f}, {1.84f, 1.84f}, {1e9f, 1e9f}}, 2},     // (no gathers)
    {128, 256, 1, {{0.98f, 0.98f}, {1.00f, 1.00f}, {1.20f, 1.20f}}, 6},
    {128, 128, 1, {{0.62f, 0.62f}, {0.64f, 0.64f}, {0.75f, 0.75f}}, 2},
    {128, 128, 2, {{1.17f, 0.75f}, {1.20f, 0.80f}, {1.20f, 0.90f}}, 2},
    {64, 128, 1, {{0.390f, 0.390f}, {0.55f, 0.44f}, {0.550f, 0.550f}}, 2},
    {128, 64, 1, {{0.395f, 0.395f}, {0.55f, 0.44f}, {0.545f, 0.545f}}, 2},
    {64, 64, 2, {{0.44f, 0.24f}, {0.50f, 0.26f}, {0.65f, 0.47f}}, 1},
};
// Weight gradients, whose slices are given and few steps long: a last round of a few workgroups runs at the rate of one to
// a unit, and a workgroup fills its stages and stores its fp32 tile besides (`ends`, in steps).  312 x 2808 over 6272
// pixels, 8 slices of 13 steps, 47.1 us in the 880 workgroups of 64 x 128 tiles that rounds and steps alone choose, 38.5
// us in 528 of 128 x 128, two to a unit; 1536 x 320 over 3000 tokens, 10 slices of 5 steps, 22.2 us in 128 x 256 tiles,
// 21.0 us in 128 x 128.  (Not from 64 workgroups on: 12 x [192 x 3072] over 8192 would go to 1728 workgroups of 64 x 64,
// 3 % of the FFN stack slower than in 144 of 256 x 256.)
inline float gemm_tile_cost(const TileCost& t, int64_t M, int64_t N, int64_t K, int64_t splits, int64_t batch, GemmCost kind, bool wgrad)
{
    const int64_t wgs = ceil_div(M, t.bm) * ceil_div(N, t.bn) * splits * batch, steps = ceil_div(ceil_div(K, 64), splits);
    const StepTime& step = t.step[kind];
    const int64_t slots = 256 * t.per_cu, left = wgs % slots, few = wgs > slots ? 64 : 256;
    if (!wgrad) return (float)ceil_div(wgs, slots) * (float)steps * (wgs <= 256 ? step.one : step.full);
    return ((float)(wgs / slots) * step.full + (left == 0 ? 0.f : left <= few ? step.one : step.full)) * (float)(steps + t.ends);
}
}  // namespace

GemmTile gemm_best_tile(int64_t M, int64_t N, int64_t K, int64_t splits, int64_t batch, GemmCost kind, bool wgrad)
{
    int best = TILE_64x64;
    float least = 3e38f;
    for (int i = 0; i < GEMM_TILES; ++i) {
        const float c = gemm_tile_cost(TILES[i], M, N, K, splits, batch, kind, wgrad);
        if (c < least) { least = c; best = i; }
    }
    return (GemmTile)best;
}

// Weight-gradient products have a long K (tokens or pixels) and a small output; K is cut into slices so that the
// launch has enough workgroups to fill 256 compute units about twice over in 128 x 128 or 64 x 64 tiles.  The count
// depends only on the shape, is the same for every engine and never falls as K grows, so that workspace queries,
// launches and smaller batches agree.  It also bounds the error: each slice is a chain of fp32 additions, and the
// relative error goes with the root of the chain's length.  Fewer slices (what the tiles of the MFMA engine alone would
// like best: 3072 x 192 over 8192 in 3, 4096 x 256 over 4096 in one) are up to a fifth faster there, 32.8 -> 30.7 us and
// 32.4 -> 26.4 us with the sum, but take the error against 64 bits from 1.7e-7 to 3.2e-7 and from 1.4e-7 to 4.0e-7, and
// leave the engine for unaligned sizes with too few workgroups (1001 x 1003 over 4000 in 8 slices 146 us, in one 772 us).
int choose_splits(int64_t M, int64_t N, int64_t K)
{
    const int64_t t128 = ceil_div(M, 128) * ceil_div(N, 128);
    const int64_t t64 = ceil_div(M, 64) * ceil_div(N, 64);
    int64_t s = t128 >= 24 ? ceil_div(480, t128) : ceil_div(432, t64);
    const int64_t by_k = K / 256;          // keep at least 256 reduction steps per slice
    if (s > by_k) s = by_k;
    if (s > 512) s = 512;
    return s < 2 ? 1 : (int)s;
}

// Products whose result is a [tokens x r] activation (H = X.V^T, dH = dY.U) have few output tiles
// when r is small and a long K when the wide side of the layer is the reduction.  While 64 x 64
// tiles still give every compute unit a workgroup, the unsplit kernel is as fast as any split plus
// its reduce (cold operands: 8192 x 192 over 3072 22.3 us against 26.4 us and more, over 4096 30.0
// against 29.7 us; 4096 x 256 over 4096 22.1 against 22.1 us), so K is cut only below that, down to
// slices of 768.  There it pays with few tokens and a long K (48 x 256 over 4096 16.2 -> 8.7 us in
// 5 slices, 509 x 192 over 3072 13.0 -> 9.5 us in 4, 2048 x 192 over 4096 16.7 -> 14.9 us in 5); with
// more tokens and K = 1536 or 3072 the sum costs what the slices win, or more (4096 x 192 over 3072
// 17.3 against 19.4 us in 3, 2048 x 192 over 1536 8.3 against 10.1 us in 2).
int choose_splits_act(int64_t M, int64_t N, int64_t K, bool in_bf16)
{
    if (!in_bf16 || N % 8 != 0) return 1;           // only the aligned MFMA path reduces into bf16
    const int64_t t64 = ceil_div(M, 64) * ceil_div(N, 64);
    if (t64 >= 256) return 1;
    int64_t s = ceil_div(512, t64);
    const int64_t by_k = K / 768;
    if (s > by_k) s = by_k;
    if (s > 8) s = 8;
    return s < 2 ? 1 : (int)s;
}

// The most rows of partial sums (slices x rows) of choose_splits_act over every number of rows up to M.  Fewer rows are
// cut into more slices, so the product rises and falls; it peaks at the most rows that still get s slices, s = 2 .. 8.
int64_t most_act_rows(int64_t M, int64_t N, int64_t K, bool in_bf16)
{
    auto rows = [&](int64_t m) {
        const int s = choose_splits_act(m, N, K, in_bf16);
        return s > 1 ? s * m : 0;
    };
    int64_t most = rows(M);
    for (int s = 2; s <= 8; ++s) {
        const int64_t tiles = std::min(255, 511 / (s - 1));       // ceil(512 / tiles) >= s, and fewer than 256
        const int64_t m = std::min(M, 64 * (tiles / ceil_div(N, 64)));
        if (m > 0) most = std::max(most, rows(m));
    }
    return most;
}

// Weight gradients of `batch` layers of one shape in one launch: 256 x 256 tiles over all members already give most
// compute units a workgroup when there are a dozen layers; K is sliced only while they do not.  (12 x [1024 x 256] over
// 8192: 88.6 us in 4 slices, error 2.7e-7; 85.8 us in 2, error 4.0e-7.)
int choose_splits_batched(int64_t M, int64_t N, int64_t K, int64_t batch)
{
    const int64_t tiles = ceil_div(M, 256) * ceil_div(N, 256) * batch;
    int64_t s = 224 / tiles;
    const int64_t by_k = K / 512;
    if (s > by_k) s = by_k;
    if (s > 64) s = 64;
    return s < 2 ? 1 : (int)s;
}

namespace {
std::mutex g_log_mutex;
std::atomic<bool> g_log_on{false};
void** g_log_events = nullptr;
int g_log_pairs = 0;
std::vector<lrd_profile_record> g_log;
thread_local const char* t_kernel = "";
}  // namespace

void note_kernel(const char* name) { t_kernel = name; }

int log_begin(hipEvent_t* start, hipEvent_t* stop)
{
    if (!g_log_on.load(std::memory_order_relaxed)) return -1;
    std::lock_guard<std::mutex> lock(g_log_mutex);
    if (!g_log_on.load() || (int)g_log.size() >= g_log_pairs) return -1;
    const int i = (int)g_log.size();
    g_log.push_back(lrd_profile_record{});
    *start = (hipEvent_t)g_log_events[2 * i];
    *stop = (hipEvent_t)g_log_events[2 * i + 1];
    t_kernel = "";
    return i;
}

void log_end(int index, int role, int gather, int epilogue, int splits, int64_t M, int64_t N, int64_t K, int64_t batch, bool shared)
{
    std::lock_guard<std::mutex> lock(g_log_mutex);
    if (index < 0 || index >= (int)g_log.size()) return;
    lrd_profile_record& r = g_log[index];
    r.role = role; r.gather = gather; r.epilogue = epilogue; r.splits = splits;
    r.M = M; r.N = N; r.K = K; r.batch = batch; r.shared = shared;
    snprintf(r.kernel, sizeof(r.kernel), "%s", t_kernel);
}

// The activation epilogue as separate elementwise passes, for engines that do not fuse it.
// C and aux are dense [M x N] here (ldc = ldaux = N), which is all the layer passes produce.
hipError_t apply_epilogue(const MatOp& op, hipStream_t st)
{
    if (op.ldc != op.N || op.ldaux != op.N) return hipErrorInvalidValue;
    const int64_t n = op.M * op.N;
    if (op.epilogue == EPI_ACT_STORE) return gelu_fwd(op.C, op.aux, n, op.in_bf16, st);
    if (op.epilogue == EPI_ACT_GRAD) return gelu_bwd(op.C, op.aux, op.C, n, op.in_bf16, st);
    return hipSuccess;
}

size_t conv_dgrad_flip_bytes(const ConvShape& cs, bool bf16)
{
    if (!bf16 || cs.stride != 1 || cs.k < 2 || cs.pad > cs.k - 1 || cs.I % 8 != 0 || cs.O % 8 != 0) return 0;
    return (size_t)cs.k * cs.k * cs.I * cs.O * 2;
}

namespace {
// The data gradient of a stride-1 convolution as the forward convolution of dY [N][Ho][Wo][O] with
// wt[i][k*k - 1 - t][o] = w[o][t][i] and padding k - 1 - pad.  False if this op is not one of those.
bool conv_dgrad_as_fwd(const MatOp& op, MatOp* fwd)
{
    const ConvShape& cs = op.cs;
    const size_t need = conv_dgrad_flip_bytes(cs, op.in_bf16);
    if (op.gather != GATHER_CONV_DGRAD || op.out_f32 || !need || !op.scratch || op.scratch_bytes < need) return false;
    if (reinterpret_cast<uintptr_t>(op.scratch) & 15u) return false;
    MatOp f = op;
    f.gather = GATHER_CONV_FWD;
    f.cs.H = cs.Ho; f.cs.W = cs.Wo; f.cs.Ho = cs.H; f.cs.Wo = cs.W;
    f.cs.I = cs.O; f.cs.O = cs.I;
    f.cs.pad = cs.k - 1 - cs.pad;
    f.B = op.scratch;
    f.b_sn = (int64_t)cs.k * cs.k * cs.O;
    f.b_sk = 1;
    f.scratch = nullptr;
    f.scratch_bytes = 0;
    if (!mfma_gemm2_supported(f)) return false;
    *fwd = f;
    return true;
}
}  // namespace

hipError_t run_matop(const MatOp& op_in, hipStream_t st)
{
    if (op_in.batch > 1 && !mfma_gemm2_supported(op_in)) {
        // no engine takes this batch in one launch: one product at a time
        const int64_t ein = op_in.in_bf16 ? 2 : 4, eout = op_in.out_f32 ? 4 : ein;
        for (int b = 0; b < op_in.batch; ++b) {
            MatOp one = op_in;
            one.batch = 1;
            one.A = (const char*)op_in.A + b * op_in.a_bs * ein;
            one.B = (const char*)op_in.B + b * op_in.b_bs * ein;
            one.C = (char*)op_in.C + b * op_in.c_bs * eout;
            if (op_in.bias) one.bias = op_in.bias + b * op_in.bias_bs;
            if (op_in.aux) one.aux = (char*)op_in.aux + b * op_in.aux_bs * ein;
            hipError_t e = run_matop(one, st);
            if (e != hipSuccess) return e;
        }
        return hipSuccess;
    }
    MatOp op = op_in;
    if (!op.out_f32 && op.splits > 1 && !mfma_gemm2_supported(op)) {
        op.splits = 1;   // the other engines split K only towards fp32 results
        op.partial = nullptr;
    }
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    const int logged = log_begin(&ev0, &ev1);
    if (logged >= 0) (void)hipEventRecord(ev0, st);
    hipError_t e;
    bool epilogue_done = true;
    MatOp flipped;
    if (conv_direct_supported(op)) e = conv_direct(op, st);
    else if (conv_dgrad_as_fwd(op, &flipped)) {
        e = flip_conv_weights(op.B, op.scratch, op.cs.O, op.cs.I, op.cs.k, st);
        if (e == hipSuccess) e = mfma_gemm2(flipped, st);
    }
    else if (mfma_small_fwd_supported(op)) e = mfma_small_fwd(op, st);
    else if (mfma_small_data_supported(op)) e = mfma_small_bwd(&op, nullptr, nullptr, st);
    else if (mfma_wide_supported(op)) e = mfma_wide(op, st);
    else if (mfma_gemm2_supported(op)) e = mfma_gemm2(op, st);
    else {
        epilogue_done = op.epilogue == EPI_NONE;
        if (f32_gemm_supported(op)) e = f32_gemm(op, st);
        else if (mfma_matop_supported(op)) e = mfma_matop(op, st);
        else e = generic_matop(op, st);
    }
    if (e == hipSuccess && op.sgd && !op.sgd->done) {
        // the engine stored the gradient whole: the step runs on it as a kernel of its own
        if (!op.out_f32 || op.ldc != op.N) e = hipErrorInvalidValue;
        else e = sgd_step(op.sgd->w, op.sgd->m, (const float*)op.C, op.sgd->copy, op.sgd->copy_bf16, op.M * op.N, op.sgd->lr,
                          op.sgd->mu, op.sgd->wd, st);
        op.sgd->done = true;
    }
    if (logged >= 0) {
        (void)hipEventRecord(ev1, st);
        log_end(logged, op.role, op.gather, op.epilogue, op.splits > 1 && op.partial ? op.splits : 1, op.M, op.N, op.K, op.batch);
    }
    if (e != hipSuccess || epilogue_done) return e;
    return apply_epilogue(op, st);
}

bool small_pair_supported(const MatOp& data, const MatOp& grad)
{
    return data.in_bf16 ? mfma_small_pair_supported(data, grad) : f32_pair_supported(data, grad);
}

hipError_t run_small_bwd(const MatOp& data, const MatOp* grad, const SmallSums* sums, hipStream_t st)
{
    const bool f32 = !data.in_bf16;
    // each product has a record of its own, around the launch that they share
    const MatOp* ops[2] = {&data, grad};
    hipEvent_t ev0[2], ev1[2];
    int logged[2] = {-1, -1};
    for (int i = 0; i < 2; ++i)
        if (ops[i] && (logged[i] = log_begin(&ev0[i], &ev1[i])) >= 0) (void)hipEventRecord(ev0[i], st);
    const hipError_t e = f32 ? f32_pair(data, *grad, st) : mfma_small_bwd(&data, grad, sums, st);
    for (int i = 0; i < 2; ++i)
        if (logged[i] >= 0) {
            (void)hipEventRecord(ev1[i], st);
            const MatOp& op = *ops[i];
            log_end(logged[i], op.role, op.gather, op.epilogue, op.splits > 1 && op.partial ? op.splits : 1, op.M, op.N, op.K, 1, i == 1);
        }
    if (e != hipSuccess || !f32 || data.epilogue == EPI_NONE) return e;
    return apply_epilogue(data, st);      // (fp32 engines do not fuse it)
}

}  // namespace lrd

extern "C" {

lrd_status lrd_profile_log_start(void** events, int32_t n_pairs)
{
    if (!events || n_pairs < 1) return LRD_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> lock(lrd::g_log_mutex);
    lrd::g_log.clear();
    lrd::g_log.reserve((size_t)n_pairs);
    lrd::g_log_events = events;
    lrd::g_log_pairs = n_pairs;
    lrd::g_log_on.store(true);
    return LRD_OK;
}

int32_t lrd_profile_log_stop(lrd_profile_record* out, int32_t capacity)
{
    std::lock_guard<std::mutex> lock(lrd::g_log_mutex);
    lrd::g_log_on.store(false);
    const int32_t n = (int32_t)lrd::g_log.size();
    if (out)
        for (int32_t i = 0; i < n && i < capacity; ++i) out[i] = lrd::g_log[i];
    return n;
}

}  // extern "C"
