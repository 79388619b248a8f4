// bf16 MFMA product kernel for 16-byte-aligned operands (the common case: every leading dimension
// a multiple of 8 elements).  One kernel template covers the three operand layouts of a layer:
//   forward / unfused pair      C = A . B^T          A [M x K], B [N x K]   (both k-contiguous)
//   data gradient               C = A . B            A [M x K], B [K x N]   (B k-major)
//   weight gradient (fp32 out)  C = A^T . B          A [K x M], B [K x N]   (both k-major), split-K
//
// Operand tiles go from memory straight into LDS (buffer loads with the LDS bit), STAGES K-steps of them in a
// ring; a wave's loads complete in order, so "all but the newest n" (s_waitcnt vmcnt) plus one barrier per K-step
// hand a stage over, and nothing waits for the loads that are still under way.  The range check of the buffer
// descriptor supplies the zeros: rows, columns and k that do not exist, and the padding of a convolution, get an
// offset no descriptor admits.  K-major operands lie in LDS as in memory and are transposed by the LDS read
// (ds_read_b64_tr_b16) when the MFMA fragments are fetched, so no layout costs a VALU instruction.  A load writes
// 64 consecutive 16-byte chunks of LDS, so rows cannot be padded against bank conflicts: instead each lane picks
// which chunk of its row it loads (kc_swz, km_swz), and the readers apply the same permutation.
// bf16 results leave through LDS so that each lane stores 16 contiguous bytes of an output row.
// Against tiles staged through registers and padded rows (two buffers, loads two steps ahead): 16384 x 512 x 4096
// 99 -> 62 us, 16384 x 4096 x 512 119 -> 80 us, 8192 x 256 x 4096 40 -> 24 us, 8192 x 4096 x 256 32 -> 26 us, weight
// gradient 4096 x 512 x 16384 118 -> 78 us.
//
// Convolutions are the same kernel with gather tiles in place of the plain ones (implicit GEMM:
// forward, data gradient, weight gradient).  The data gradient of a strided convolution runs as one
// product per parity class of the input pixel (class = blockIdx.z), each over the taps that reach
// its pixels, and writes its rows through a row map.
#include <algorithm>
#include <cstdio>
#include <string>
#include <type_traits>

#include "lds_load.hpp"
#include "lrd_internal.hpp"

namespace lrd {
namespace {

constexpr int BK = 64;

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

struct Operand {
    const bf16_t* p;
    int64_t ld;   // elements between rows of the stored matrix
    int rows;     // extent along the tile's row index (M for A, N for B)
};

// A batch of products of one shape in one launch (element strides between consecutive products).
struct BatchArgs {
    int batch = 1, nsplit = 1;
    int64_t a_bs = 0, b_bs = 0, c_bs = 0, aux_bs = 0, bias_bs = 0;
};

// Every tile type: init() once; step(k0) before the loads of a K-step, then one(i) for each of its CH loads.
// Load i of wave w fills the 1024 bytes at (i * NW + w) * 1024 of the tile's part of a stage.

// ---- k-contiguous tile: ROWS x BK, a row is 128 bytes of LDS (its chunks permuted by kc_swz); a load covers 8 rows.
template <int ROWS, int NW>
struct KcTile {
    static_assert(ROWS % (8 * NW) == 0 && NW % 2 == 0, "every load of a lane has the same k offset");
    static constexpr int CH = ROWS / (8 * NW), BYTES = ROWS * BK * 2;
    const char* base;     // first row of the tile, k = 0
    uint32_t span;        // bytes from base to the end of the tile's last existing row
    const char* at;       // base and span at the current K-step
    uint32_t left;
    int kc, k0;
    uint32_t voff[CH];

    __device__ __forceinline__ void init(const Operand& o, int row0, int wave, int lane, const ConvShape&, int K, int)
    {
        base = uni_ptr(o.p + (int64_t)row0 * o.ld);
        const int rows_here = min(o.rows - row0, ROWS);
        span = uni((uint32_t)(((int64_t)(rows_here - 1) * o.ld + K) * 2));
        settle(base, span);
        kc = ((lane & 7) ^ kc_swz(wave * 8 + (lane >> 3))) * 8;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int r = (i * NW + wave) * 8 + (lane >> 3);
            voff[i] = r < rows_here ? (uint32_t)((r * o.ld + kc) * 2) : BUF_OOB;
        }
    }
    __device__ __forceinline__ void step(int k, int)
    {
        k0 = (int)uni((uint32_t)k);
        at = base + k0 * 2;
        left = span - (uint32_t)k0 * 2u;      // k0 < K
    }
    __device__ __forceinline__ void one(int i, uint32_t lds, int kend, int wave)
    {
        load_to_lds(lds + (i * NW + wave) * 1024, at, left, k0 + kc < kend ? voff[i] : BUF_OOB);
    }
};

// ---- k-major tile: BK x COLS, in LDS as in memory ([k][column]); a load covers 512 / COLS rows of k.  Chunk c of
// row k lies in slot c ^ km_swz(k): a transposing read takes 64 bytes from each of four consecutive k, which then
// fall on different quarters of the banks.  km_swz(k) = km_swz(k + 4) = km_swz(k + 8).
template <int COLS>
__device__ __forceinline__ constexpr int km_swz(int k)
{
    return COLS >= 128 ? (k & 3) << 2 : COLS >= 64 ? (k & 2) << 1 : 0;
}
template <int COLS, int NW>
struct KmTile {
    static constexpr int CPK = COLS / 8;                 // 16-byte chunks per k row
    static constexpr int KPI = 64 / CPK;                 // k rows per load
    static constexpr int CH = BK / (KPI * NW), BYTES = COLS * BK * 2;
    static_assert(64 % CPK == 0 && BK % (KPI * NW) == 0, "whole loads");
    const char* base;     // k = 0, first column of the tile
    int64_t ld;
    int cols_here;        // columns that exist from the tile's first one on
    const char* at;
    uint32_t left;
    uint32_t voff[CH];

    __device__ __forceinline__ void init(const Operand& o, int col0, int wave, int lane, const ConvShape&, int, int)
    {
        ld = uni64(o.ld);
        cols_here = (int)uni((uint32_t)(o.rows - col0));
        base = uni_ptr(o.p + col0);
        settle(base, ld, cols_here);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int k = (i * NW + wave) * KPI + lane / CPK;
            const int col = ((lane % CPK) ^ km_swz<COLS>(k)) * 8;
            voff[i] = col < cols_here ? (uint32_t)((k * o.ld + col) * 2) : BUF_OOB;
        }
    }
    __device__ __forceinline__ void step(int k, int kend)
    {
        // bytes from this step's first k row to the last element of its last k row (at most BK rows) in these
        // columns; rows from kend on fall outside because ld >= cols_here
        const int ku = (int)uni((uint32_t)k);
        at = base + (int64_t)ku * ld * 2;
        left = (uint32_t)(min(kend - ku, BK) - 1) * ((uint32_t)ld * 2u) + (uint32_t)cols_here * 2u;
    }
    __device__ __forceinline__ void one(int i, uint32_t lds, int, int wave) { load_to_lds(lds + (i * NW + wave) * 1024, at, left, voff[i]); }
};

// ---- implicit-GEMM operands of a k x k convolution on NHWC data ---------------------------------
// Same LDS layouts as the plain tiles; the offset of a 16-byte chunk comes from the tap geometry, out-of-image
// taps and tails get the offset past the descriptor.  Channel counts are multiples of 8 on this path, so a chunk
// never straddles two taps.  K-steps are loaded strictly in order (k0 = kbeg, kbeg + BK, ...), so the
// decomposition of k into (tap, channel) or (image, y, x) is kept as state and advanced by BK with the loads:
// the only integer divisions are in init().

// floor(t / d) for 0 <= t * d < 65536 by multiplication with ceil(65536 / d): taps by the kernel size
// (d < 32, t <= d * d + 8) and, in the data gradient, pixel coordinates by the stride.  (Unsigned: with d = 1 the product
// reaches 65535 * 65536.)
__device__ __forceinline__ int small_div(int t, int magic) { return (int)(((uint32_t)t * (uint32_t)magic) >> 16); }

// A operand, k-contiguous.  FWD:   row = output pixel, k = (u, v, i), reads X[n, y*s+u-p, x*s+v-p, i].
//                           DGRAD: row = input pixel,  k = (u, v, o), reads dY[n, (a+p-u)/s, (b+p-v)/s, o].
template <int ROWS, int NW, bool DGRAD>
struct ConvRowsTile {
    static_assert(ROWS % (8 * NW) == 0 && NW % 2 == 0, "every load of a lane has the same k offset");
    static constexpr int CH = ROWS / (8 * NW), BYTES = ROWS * BK * 2;
    const char* base;
    uint32_t span;
    ConvShape cs;
    // FWD: image coordinates of tap (0, 0), and the offset of that pixel; DGRAD: those of the input pixel plus pad, and
    // the first row of its image.  A row that does not exist gets coordinates no tap brings into the image.
    int oy[CH], ox[CH], pix[CH];
    int kc, k0, tap, c0;      // this lane's k of the current step, as (tap, channel); same for all its loads
    int ch, q_tap, r_ch, magic, magic_s, u, v;
    int kdiv, u0, v0, ustep;  // tap index -> (u, v): u = u0 + ustep * (tap / kdiv), v = v0 + ustep * (tap % kdiv)

    __device__ __forceinline__ void init(const Operand& o, int row0, int wave, int lane, const ConvShape& shape, int, int kbeg)
    {
        cs = shape;
        ch = DGRAD ? cs.O : cs.I;            // channels of the tensor being gathered
        base = uni_ptr(o.p);
        span = uni((uint32_t)cs.N * (uint32_t)(DGRAD ? cs.Ho * cs.Wo : cs.H * cs.W) * (uint32_t)ch * 2u);
        settle(base, span);
        q_tap = BK / ch;
        r_ch = BK - q_tap * ch;
        const bool cls = DGRAD && cs.cls;
        const ClassTaps tu = class_taps(cs.cy, cs.pad, cs.stride, cs.k), tv = class_taps(cs.cx, cs.pad, cs.stride, cs.k);
        kdiv = cls ? tv.count : cs.k;
        u0 = cls ? tu.first : 0;
        v0 = cls ? tv.first : 0;
        ustep = cls ? cs.stride : 1;
        magic = (65536 + kdiv - 1) / kdiv;
        magic_s = (65536 + cs.stride - 1) / cs.stride;
        kc = ((lane & 7) ^ kc_swz(wave * 8 + (lane >> 3))) * 8;
        tap = (kbeg + kc) / ch - q_tap;          // step() advances to the first K-step
        c0 = (kbeg + kc) % ch - r_ch;
        // rows: output pixels, input pixels, or the input pixels of one parity class
        const int gw = !DGRAD ? cs.Wo : cls ? class_extent(cs.W, cs.cx, cs.stride) : cs.W;
        const int gh = !DGRAD ? cs.Ho : cls ? class_extent(cs.H, cs.cy, cs.stride) : cs.H;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int row = row0 + (i * NW + wave) * 8 + (lane >> 3);
            const int q = row / gw;
            int px = row - q * gw, py = q % gh;
            const int img = q / gh;
            if (cls) {
                px = px * cs.stride + cs.cx;
                py = py * cs.stride + cs.cy;
            }
            oy[i] = DGRAD ? py + cs.pad : py * cs.stride - cs.pad;
            ox[i] = DGRAD ? px + cs.pad : px * cs.stride - cs.pad;
            pix[i] = DGRAD ? img * cs.Ho : (img * cs.H + oy[i]) * cs.W + ox[i];
            if (row >= o.rows) oy[i] = DGRAD ? -1 : cs.H;
        }
    }
    __device__ __forceinline__ void step(int k, int)
    {
        k0 = (int)uni((uint32_t)k);
        c0 += r_ch;
        tap += q_tap;
        if (c0 >= ch) {
            c0 -= ch;
            ++tap;
        }
        const int tq = small_div(tap, magic);
        u = u0 + ustep * tq;
        v = v0 + ustep * (tap - tq * kdiv);
    }
    __device__ __forceinline__ void one(int i, uint32_t lds, int kend, int wave)
    {
        bool ok = k0 + kc < kend;
        int at;
        if (DGRAD) {
            // output pixel (ys, xs) / stride, if that is a whole number inside the output
            const int ys = oy[i] - u, xs = ox[i] - v;
            const int yp = max(ys, 0), xp = max(xs, 0);
            const int yy = small_div(yp, magic_s), xx = small_div(xp, magic_s);
            ok = ok && ys >= 0 && xs >= 0 && yy * cs.stride == yp && xx * cs.stride == xp && yy < cs.Ho && xx < cs.Wo;
            at = (pix[i] + yy) * cs.Wo + xx;
        } else {
            ok = ok && (uint32_t)(oy[i] + u) < (uint32_t)cs.H && (uint32_t)(ox[i] + v) < (uint32_t)cs.W;
            at = pix[i] + u * cs.W + v;
        }
        load_to_lds(lds + (i * NW + wave) * 1024, base, span, ok ? ((uint32_t)at * (uint32_t)ch + (uint32_t)c0) * 2u : BUF_OOB);
    }
};

// B operand, k-major.  DGRAD: column = input channel i, k = (u, v, o), reads W[o][u][v][i].
//                      WGRAD: column = (u, v, i),        k = output pixel, reads X[n, y*s+u-p, x*s+v-p, i].
template <int COLS, int NW, bool WGRAD>
struct ConvKmTile {
    static constexpr int CPK = COLS / 8, KPI = 64 / CPK;
    static constexpr int CH = BK / (KPI * NW), BYTES = COLS * BK * 2;
    static_assert(64 % CPK == 0 && BK % (KPI * NW) == 0, "whole loads");
    static_assert(KPI * NW % 4 == 0, "all loads of a lane have one swizzle, hence one column");
    const char* base;
    uint32_t span;
    ConvShape cs;
    int c0, tu, tv;
    bool colok;
    // k of the next load, per chunk.  DGRAD: (tap, o) in s1, s0.  WGRAD: output pixel as (n, y, x) in s2, s1, s0.
    int s0[CH], s1[CH], s2[CH], kk[CH];
    int d0, d1, d2;           // BK in the same mixed radix
    int ntaps, nv, magic_nv, u0, v0, ustep;   // DGRAD: the taps K runs over (all, or those of a parity class)

    __device__ __forceinline__ void init(const Operand& o, int col0, int wave, int lane, const ConvShape& shape, int, int kbeg)
    {
        base = uni_ptr(o.p);
        cs = shape;
        if (WGRAD) {
            span = uni((uint32_t)cs.N * (uint32_t)(cs.H * cs.W) * (uint32_t)cs.I * 2u);
            d2 = BK / (cs.Ho * cs.Wo);
            int rem = BK - d2 * cs.Ho * cs.Wo;
            d1 = rem / cs.Wo;
            d0 = rem - d1 * cs.Wo;
        } else {
            span = uni((uint32_t)cs.O * (uint32_t)(cs.k * cs.k) * (uint32_t)cs.I * 2u);
            d2 = 0;
            d1 = BK / cs.O;
            d0 = BK - d1 * cs.O;
            const ClassTaps cu = class_taps(cs.cy, cs.pad, cs.stride, cs.k), cv = class_taps(cs.cx, cs.pad, cs.stride, cs.k);
            nv = cs.cls ? cv.count : cs.k;
            ntaps = (cs.cls ? cu.count : cs.k) * nv;
            magic_nv = (65536 + nv - 1) / nv;
            u0 = cs.cls ? cu.first : 0;
            v0 = cs.cls ? cv.first : 0;
            ustep = cs.cls ? cs.stride : 1;
        }
        settle(base, span);
        const int col = col0 + ((lane % CPK) ^ km_swz<COLS>(wave * KPI + lane / CPK)) * 8;
        colok = col < o.rows;
        if (WGRAD) {
            const int tap = col / cs.I;
            c0 = col - tap * cs.I;
            tu = tap / cs.k - cs.pad;
            tv = tap % cs.k - cs.pad;
        } else {
            c0 = col;
            tu = tv = 0;
        }
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int k = kbeg + (i * NW + wave) * KPI + lane / CPK;
            kk[i] = k;
            if (WGRAD) {
                s0[i] = k % cs.Wo;
                int q = k / cs.Wo;
                s1[i] = q % cs.Ho;
                s2[i] = q / cs.Ho;
            } else {
                s1[i] = k / cs.O;
                s0[i] = k - s1[i] * cs.O;
                s2[i] = 0;
            }
        }
    }
    __device__ __forceinline__ void step(int, int) {}
    __device__ __forceinline__ void one(int i, uint32_t lds, int kend, int wave)
    {
        bool ok = colok && kk[i] < kend;
        uint32_t off;
        if (WGRAD) {
            const int yy = s1[i] * cs.stride + tu, xx = s0[i] * cs.stride + tv;
            ok = ok && (uint32_t)yy < (uint32_t)cs.H && (uint32_t)xx < (uint32_t)cs.W;
            off = (uint32_t)((s2[i] * cs.H + yy) * cs.W + xx) * (uint32_t)cs.I + (uint32_t)c0;
        } else {
            const int t = min(s1[i], ntaps - 1);     // (taps past the last one: tail of K)
            const int tq = small_div(t, magic_nv);
            const int tap = (u0 + ustep * tq) * cs.k + v0 + ustep * (t - tq * nv);
            off = (uint32_t)(s0[i] * cs.k * cs.k + tap) * (uint32_t)cs.I + (uint32_t)c0;
        }
        load_to_lds(lds + (i * NW + wave) * 1024, base, span, ok ? off * 2u : BUF_OOB);
        // advance this load's k by BK
        kk[i] += BK;
        s0[i] += d0;
        s1[i] += d1;
        if (WGRAD) {
            if (s0[i] >= cs.Wo) { s0[i] -= cs.Wo; ++s1[i]; }
            s2[i] += d2;
            if (s1[i] >= cs.Ho) { s1[i] -= cs.Ho; ++s2[i]; }
        } else {
            if (s0[i] >= cs.O) { s0[i] -= cs.O; ++s1[i]; }
        }
    }
};

// Tile type by layout (k-major or not) and gather mode (GATHER_* of the product).
template <int ROWS, int NW, bool KM, int G, bool IS_A>
struct TileSel { typedef KcTile<ROWS, NW> type; };
template <int ROWS, int NW, int G, bool IS_A>
struct TileSel<ROWS, NW, true, G, IS_A> { typedef KmTile<ROWS, NW> type; };
template <int ROWS, int NW>
struct TileSel<ROWS, NW, false, GATHER_CONV_FWD, true> { typedef ConvRowsTile<ROWS, NW, false> type; };
template <int ROWS, int NW>
struct TileSel<ROWS, NW, false, GATHER_CONV_DGRAD, true> { typedef ConvRowsTile<ROWS, NW, true> type; };
template <int ROWS, int NW>
struct TileSel<ROWS, NW, true, GATHER_CONV_DGRAD, false> { typedef ConvKmTile<ROWS, NW, false> type; };
template <int ROWS, int NW>
struct TileSel<ROWS, NW, true, GATHER_CONV_WGRAD, false> { typedef ConvKmTile<ROWS, NW, true> type; };

// Operand fragments of the T 32-row blocks of a wave for one 16-wide k step, in the register layout of
// v_mfma_f32_32x32x16_bf16: lane L holds row (L & 31), k = 8 * (L >> 5) + 0..7.  The lane's byte offsets in the
// tile are fixed before the loop.
template <int ROWS, int T, bool KM>
struct Frag {     // k-contiguous tile [row][k]: one 16-byte read
    uint32_t off[BK / 16];
    __device__ __forceinline__ void init(int row0, int lane)
    {
        const int r = row0 + (lane & 31);
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) off[kk] = r * (BK * 2) + (((kk * 2 + (lane >> 5)) ^ kc_swz(r)) << 4);
    }
    __device__ __forceinline__ bf16x8 get(const char* tile, int i, int kk) const
    {
        return *reinterpret_cast<const bf16x8*>(tile + off[kk] + i * 32 * (BK * 2));
    }
};
template <int COLS, int T>
struct Frag<COLS, T, true> {     // k-major tile [k][row]: two transposing reads (see km_frag for their lane layout)
    uint32_t off[T];
    __device__ __forceinline__ void init(int col0, int lane)
    {
        const int blk = lane >> 4, s = lane & 15;
        const int k = 8 * (blk >> 1) + (s >> 2);
#pragma unroll
        for (int i = 0; i < T; ++i) {
            const int col = col0 + i * 32 + 16 * (blk & 1) + 4 * (s & 3);
            off[i] = k * COLS * 2 + (((col >> 3) ^ km_swz<COLS>(k)) << 4) + (col & 7) * 2;
        }
    }
    __device__ __forceinline__ bf16x8 get(const char* tile, int i, int kk) const
    {
        typedef short s16x4 __attribute__((ext_vector_type(4)));
        typedef short s16x8 __attribute__((ext_vector_type(8)));
        const char* p = tile + off[i] + kk * 16 * COLS * 2;
        s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p));
        s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p + 4 * COLS * 2));
        s16x8 v = {lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        return __builtin_bit_cast(bf16x8, v);
    }
};

template <int BM, int BN, int STAGES, class OutT>
constexpr int gemm2_lds_bytes()
{
    int main = STAGES * (BM + BN) * BK * 2;
    int epi = sizeof(OutT) == 2 ? BM * (BN + 8) * 2 : 0;
    return main > epi ? main : epi;
}

// 16 bytes to memory past the caches of this die, kept by the one beside memory.  (The compiler does not see the store's read of
// its data, which a vector instruction may overwrite one state later.)
__device__ __forceinline__ void store_through(void* to, u32x4 v)
{
    asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 0" ::"v"(to), "v"(v) : "memory");
}
// Results up to this many elements (of each member of a batch) are stored that way: they are what the next product reads at once, and
// it finds them there.  Non-temporal stores send them to memory; without these stores the encoder step takes 1.1 % longer (4207
// against 4160 us), the FFN stack 0.9 %, forward of a 1024-wide layer at rank 256 25.4 against 23.5 us for 11648 tokens (3.0 M), 30.2
// against 28.1 for 16000 (4.1 M).  With larger ones the write-backs come due in the next kernel instead: with everything
// stored so a backward pass with nothing frozen takes 12 % longer from 12 M on (46848 tokens 174 against 196 us, at rank 192
// 140 against 156 for 43136), and is even at 6 to 8 M, where forward passes gain up to 10 %.  Per member, because each is what one
// product of the next launch reads: dH of three members of 8192 x 192 with their dX 25.6 -> 24.9 us, 25.7 by the batch's 4.7 M; three of 6144
// x 256 29.1 against 30.2; encoder step 4155 against 4176 us.
constexpr int64_t THROUGH_MOST = int64_t(1) << 22;

// bf16 results of one BM x BN tile: registers -> LDS tile (row-major) -> 16 contiguous bytes per
// lane to global memory, with the optional GELU epilogue.  Large results (and the pre-activation the
// gradient epilogue reads) are streamed with non-temporal accesses: 10 % faster on the wide products.  Every wave must be past its last read
// of the operand tiles in LDS (the staging tile overlays them); ends without a barrier.
template <int BM, int BN, int WGM, int WGN, bool MAPROWS, int EPI, int TM, int TN>
__device__ __forceinline__ void store_bf16_tile(const f32x16 (&acc)[TM][TN], bf16_t* lds, bf16_t* __restrict__ out, int64_t ldc,
                                                const float* __restrict__ bias, int M, int N, int m0, int n0,
                                                bf16_t* __restrict__ aux, int64_t ldaux, int tid, const ConvShape& cs)
{
    constexpr int NT = 64 * WGM * WGN;
    constexpr int WTM = BM / WGM, WTN = BN / WGN;
    static_assert(TM == WTM / 32 && TN == WTN / 32, "accumulator shape");
    constexpr int LDC = BN + 8;
    constexpr int CPR = BN / 8;
    constexpr int PER = BM * CPR / NT;          // 16-byte chunks per thread
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WGN, wn = wave % WGN;
    const int r = lane & 31, h = lane >> 5;
    // The activation-gradient epilogue reads the pre-activation: start those loads now, so they
    // are in flight while the accumulators go through LDS.
    bf16x8 z8[PER];
    if constexpr (EPI == EPI_ACT_GRAD) {
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            int c = tid + q * NT;
            int m = min(m0 + c / CPR, M - 1), n = min(n0 + (c % CPR) * 8, N - 8);
            z8[q] = __builtin_bit_cast(bf16x8, __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(aux + (int64_t)m * ldaux + n)));
        }
    }
    auto stage = [&](auto with_bias) {
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int nl = wn * WTN + j * 32 + 8 * g + 4 * h;
                f32x4 b4 = {0.f, 0.f, 0.f, 0.f};
                if constexpr (with_bias) b4 = *reinterpret_cast<const f32x4*>(bias + min(n0 + nl, N - 4));
#pragma unroll
                for (int i = 0; i < TM; ++i) {
                    f32x4 v = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
                    if constexpr (with_bias) v += b4;
                    const u32x2 pk = {pack_bf16(v.x, v.y), pack_bf16(v.z, v.w)};
                    *reinterpret_cast<u32x2*>(lds + (wm * WTM + i * 32 + r) * LDC + nl) = pk;
                }
            }
    };
    if (bias) stage(std::true_type{});
    else stage(std::false_type{});
    __syncthreads();
    const bool through = (int64_t)M * N <= THROUGH_MOST;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        int c = tid + q * NT;
        int ml = c / CPR, cc = c % CPR;
        int m = m0 + ml, n = n0 + cc * 8;
        const bool ok = m < M && n < N;   // N is a multiple of 8 on this path
        u32x4 v = *reinterpret_cast<const u32x4*>(lds + ml * LDC + cc * 8);
        int64_t mrow = m;
        if (MAPROWS && cs.cls) {
            // row m counts the input pixels of one parity class: its place among all input pixels
            const int gw = class_extent(cs.W, cs.cx, cs.stride), gh = class_extent(cs.H, cs.cy, cs.stride);
            const int mm = min(m, M - 1);
            const int ix = mm % gw, q = mm / gw;
            mrow = ((int64_t)(q / gh) * cs.H + (q % gh) * cs.stride + cs.cy) * cs.W + ix * cs.stride + cs.cx;
        }
        if constexpr (EPI == EPI_ACT_GRAD) {
            bf16x8 c8 = __builtin_bit_cast(bf16x8, v);
#pragma unroll
            for (int e = 0; e < 8; ++e) c8[e] = (bf16_t)((float)c8[e] * gelu_grad_bf16_f((float)z8[q][e]));
            v = __builtin_bit_cast(u32x4, c8);
        }
        if constexpr (EPI == EPI_NONE && !MAPROWS) {
            if (ok && through) store_through(out + mrow * ldc + n, v);
            else if (ok) __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(out + mrow * ldc + n));
        } else {
            if (ok) __builtin_nontemporal_store(v, reinterpret_cast<u32x4*>(out + mrow * ldc + n));
        }
        if constexpr (EPI == EPI_ACT_STORE) {
            bf16x8 c8 = __builtin_bit_cast(bf16x8, v);
#pragma unroll
            for (int e = 0; e < 8; ++e) c8[e] = (bf16_t)gelu_bf16_f((float)c8[e]);
            if (ok) __builtin_nontemporal_store(__builtin_bit_cast(u32x4, c8), reinterpret_cast<u32x4*>(aux + (int64_t)m * ldaux + n));
        }
    }
}

template <int BM, int BN, int WGM, int WGN, int STAGES, bool A_KM, bool B_KM, class OutT, int G, int EPI>
__global__ __launch_bounds__(64 * WGM * WGN, STAGES == 1 ? 6 : 2) void gemm2_kernel(Operand A, Operand B, ConvShape cs, OutT* __restrict__ C, int64_t ldc,
                                                               const float* __restrict__ bias, float* __restrict__ partial,
                                                               int M, int N, int K, int k_per_split,
                                                               bf16_t* __restrict__ aux, int64_t ldaux, BatchArgs bt)
{
    constexpr int NW = WGM * WGN;
    constexpr int WTM = BM / WGM, WTN = BN / WGN;
    constexpr int TM = WTM / 32, TN = WTN / 32;
    typedef typename TileSel<BM, NW, A_KM, G, true>::type TileA;
    typedef typename TileSel<BN, NW, B_KM, G, false>::type TileB;
    constexpr int STAGE = TileA::BYTES + TileB::BYTES, LPS = TileA::CH + TileB::CH;   // bytes and loads per wave of a stage
    extern __shared__ __align__(16) unsigned char smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = (int)uni(tid >> 6);
    const int wm = wave / WGN, wn = wave % WGN;
    // Consecutive workgroups go to the 8 dies in turn, each with an L2 of its own: die x takes a run of consecutive
    // tiles, slice (or batch member) by slice, and within a slice so that the tiles which share rows of the taller
    // operand follow one another: those rows come through one L2 and at one time.
    int tm = blockIdx.x, tn = blockIdx.y, tz = blockIdx.z;
    if constexpr (G != GATHER_CONV_DGRAD) {
        const uint32_t gx = gridDim.x, gy = gridDim.y, tiles = gx * gy, total = tiles * gridDim.z;
        const uint32_t f = (blockIdx.z * gy + blockIdx.y) * gx + blockIdx.x;
        const uint32_t die = f & 7u, per = total >> 3, more = total & 7u;
        uint32_t t = die * per + min(die, more) + (f >> 3);
        tz = (int)(t / tiles);
        t -= (uint32_t)tz * tiles;
        if (M >= N) {
            tm = (int)(t / gy);
            tn = (int)(t - (uint32_t)tm * gy);
        } else {
            tn = (int)(t / gx);
            tm = (int)(t - (uint32_t)tn * gx);
        }
    }
    const int m0 = tm * BM, n0 = tn * BN;
    // z = K-slice, or (batch index, K-slice) for a batch of products of one shape
    int zslice = tz, zbatch = 0;
    if constexpr (G == GATHER_NONE) {
        if (bt.batch > 1) {
            zbatch = tz / bt.nsplit;
            zslice = tz - zbatch * bt.nsplit;
            A.p += zbatch * bt.a_bs;
            B.p += zbatch * bt.b_bs;
            C += zbatch * bt.c_bs;
            if (bias) bias += zbatch * bt.bias_bs;
            if (aux) aux += zbatch * bt.aux_bs;
        }
    }
    int kbeg = zslice * k_per_split;
    if constexpr (G == GATHER_CONV_DGRAD) {
        if (cs.cls) {
            // all parity classes of a strided data gradient in one launch: blockIdx.z is the class,
            // each with its own number of rows and taps; K is not sliced
            cs.cy = blockIdx.z / cs.stride;
            cs.cx = blockIdx.z - cs.cy * cs.stride;
            M = cs.N * class_extent(cs.H, cs.cy, cs.stride) * class_extent(cs.W, cs.cx, cs.stride);
            K = class_taps(cs.cy, cs.pad, cs.stride, cs.k).count * class_taps(cs.cx, cs.pad, cs.stride, cs.k).count * cs.O;
            A.rows = M;
            kbeg = 0;
            k_per_split = K;
            if (m0 >= M) return;
        }
    }
    const int kend = min(K, kbeg + k_per_split);
    const int nk = (kend - kbeg + BK - 1) / BK;

    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    TileA ta;
    TileB tb;
    ta.init(A, m0, wave, lane, cs, K, kbeg);
    tb.init(B, n0, wave, lane, cs, K, kbeg);
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
    auto step = [&](int kt) {
        ta.step(kbeg + kt * BK, kend);
        tb.step(kbeg + kt * BK, kend);
    };
    auto load_one = [&](int d, int stage) {      // load d of the LPS of the step that step() named
        if (d < TileA::CH) ta.one(d, lds0 + stage * STAGE, kend, wave);
        else tb.one(d - TileA::CH, lds0 + stage * STAGE + TileA::BYTES, kend, wave);
    };
#pragma unroll
    for (int s = 0; s < STAGES - 1; ++s)
        if (s < nk) {
            step(s);
#pragma unroll
            for (int d = 0; d < LPS; ++d) load_one(d, s);
        }
    Frag<BM, TM, A_KM> fa;
    Frag<BN, TN, B_KM> fb;
    fa.init(wm * WTM, lane);
    fb.init(wn * WTN, lane);
    bf16x8 a[2][TM], b[2][TN];
    auto fetch = [&](int set, int stage, int kk) {
        const char* at = reinterpret_cast<const char*>(smem) + stage * STAGE;
#pragma unroll
        for (int i = 0; i < TM; ++i) a[set][i] = fa.get(at, i, kk);
#pragma unroll
        for (int j = 0; j < TN; ++j) b[set][j] = fb.get(at + TileA::BYTES, j, kk);
    };
    if constexpr (STAGES == 1) {
        // Three or more workgroups per compute unit, so that nothing needs to overlap inside one (80 registers per lane
        // at most: six waves per SIMD).
        for (int kt = 0; kt < nk; ++kt) {
            if (kt > 0) lds_barrier();
            step(kt);
#pragma unroll
            for (int d = 0; d < LPS; ++d) load_one(d, 0);
            wait_vm<0>();
            lds_barrier();
#pragma unroll
            for (int kk = 0; kk < BK / 16; ++kk) {
                fetch(kk & 1, 0, kk);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[i][j] = mfma32(b[kk & 1][j], a[kk & 1][i], acc[i][j]);
            }
        }
    } else if constexpr (STAGES == 2) {
        // Two or more workgroups per compute unit, which overlap one another: a step waits for its stage, starts the
        // loads of the next one and multiplies.
        for (int kt = 0; kt < nk; ++kt) {
            wait_vm<0>();
            lds_barrier();
            if (kt + 1 < nk) {
                step(kt + 1);
#pragma unroll
                for (int d = 0; d < LPS; ++d) load_one(d, (kt + 1) & 1);
            }
#pragma unroll
            for (int kk = 0; kk < BK / 16; ++kk) {
                fetch(kk & 1, kt & 1, kk);
#pragma unroll
                for (int i = 0; i < TM; ++i)
#pragma unroll
                    for (int j = 0; j < TN; ++j) acc[i][j] = mfma32(b[kk & 1][j], a[kk & 1][i], acc[i][j]);
            }
        }
    } else if (nk > 0) {
        // One workgroup per compute unit: its own waves have to keep the matrix pipes fed.  The fragments of a k-group are
        // read while the one before is multiplied, across the barrier too, and the loads of step +STAGES - 1 are spread
        // between the matrix instructions: issued in one go after the barrier, they held up every wave's fragment reads
        // behind them (128 x 256 tiles, 16384 x 512 x 4096: 71 -> 62 us).
        constexpr int MM = TM * TN, SPREAD = 3 * MM;      // the loads follow the first three k-groups
        auto multiply = [&](int set, int kk, bool loads, int stage) {
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    acc[i][j] = mfma32(b[set][j], a[set][i], acc[i][j]);
                    if (loads) {
#pragma unroll
                        for (int d = 0; d < LPS; ++d)
                            if (d * SPREAD / LPS == kk * MM + i * TN + j) {
                                __builtin_amdgcn_sched_barrier(0);
                                load_one(d, stage);
                                __builtin_amdgcn_sched_barrier(0);
                            }
                    }
                }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto group = [&](int set, int stage, int kk) {
            fetch(set, stage, kk);
            __builtin_amdgcn_sched_barrier(0);
        };
        wait_stages<STAGES - 2, LPS>(nk - 1);
        lds_barrier();
        group(0, 0, 0);
        int cur = 0, freed = STAGES - 1;      // `freed`: the stage read last, which the next loads may overwrite
        auto body = [&](int kt, bool loads) {
            const int nxt = cur + 1 == STAGES ? 0 : cur + 1;
            if (loads) step(kt + STAGES - 1);
            group(1, cur, 1);
            multiply(0, 0, loads, freed);
            group(0, cur, 2);
            multiply(1, 1, loads, freed);
            group(1, cur, 3);
            multiply(0, 2, loads, freed);
            if (loads) wait_vm<(STAGES - 2) * LPS>();
            else wait_stages<STAGES - 2, LPS>(nk - 2 - kt);
            lds_barrier();
            group(0, nxt, 0);
            multiply(1, 3, false, 0);
            freed = cur;
            cur = nxt;
        };
        int kt = 0;
        for (; kt + STAGES - 1 < nk; ++kt) body(kt, true);
        for (; kt + 1 < nk; ++kt) body(kt, false);
        group(1, cur, 1);
        multiply(0, 0, false, 0);
        group(0, cur, 2);
        multiply(1, 1, false, 0);
        group(1, cur, 3);
        multiply(0, 2, false, 0);
        multiply(1, 3, false, 0);
    }

    const int r = lane & 31, h = lane >> 5;
    if constexpr (sizeof(OutT) == 4) {
        // fp32 results (weight gradients or their split-K partials): 16-byte stores straight from registers
        // slices of a batch lie [slice][batch][M][N], so that the sum over slices sees one tall matrix
        float* out = partial ? partial + ((int64_t)zslice * bt.batch + zbatch) * M * N : reinterpret_cast<float*>(C);
        const int64_t ldo = partial ? (int64_t)N : ldc;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            int m = m0 + wm * WTM + i * 32 + r;
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    int n = n0 + wn * WTN + j * 32 + 8 * g + 4 * h;
                    if (m < M && n < N) {   // N is a multiple of 4 on this path
                        f32x4 v = {acc[i][j][4 * g], acc[i][j][4 * g + 1], acc[i][j][4 * g + 2], acc[i][j][4 * g + 3]};
                        *reinterpret_cast<f32x4*>(out + (int64_t)m * ldo + n) = v;
                    }
                }
        }
    } else {
        lds_barrier();      // the staging tile overlays the operand stages
        store_bf16_tile<BM, BN, WGM, WGN, G == GATHER_CONV_DGRAD, EPI>(acc, reinterpret_cast<bf16_t*>(smem), reinterpret_cast<bf16_t*>(C), ldc, bias, M, N, m0, n0,
                                                                  aux, ldaux, tid, cs);
    }
}

// Slices of K a launch really uses (each a whole number of K-steps) and their length.
inline int effective_splits(const MatOp& op, int* k_per_split)
{
    int splits = (op.splits > 1 && op.partial) ? op.splits : 1;
    int kps = (int)(ceil_div(ceil_div(op.K, splits), BK) * BK);
    if (k_per_split) *k_per_split = kps;
    return (int)ceil_div(op.K, kps);
}

template <int BM, int BN, int WGM, int WGN, int STAGES, bool A_KM, bool B_KM, class OutT, int G, int EPI>
hipError_t launch_epi(const MatOp& op, const Operand& A, const Operand& B, hipStream_t st)
{
    constexpr int NT = 64 * WGM * WGN;
    constexpr int lds_bytes = gemm2_lds_bytes<BM, BN, STAGES, OutT>();
    static_assert(lds_bytes <= 160 * 1024, "LDS of a compute unit");
    auto kern = gemm2_kernel<BM, BN, WGM, WGN, STAGES, A_KM, B_KM, OutT, G, EPI>;
    static OncePerDevice lds_allowed;
    hipError_t e = allow_lds(kern, lds_bytes, lds_allowed);
    if (e != hipSuccess) return e;
    static const std::string tag = [] {
        char b[64];
        snprintf(b, sizeof(b), "gemm2_kernel<%d,%d,%d,%d,%d,%s,%s,%s%s%s>", BM, BN, WGM, WGN, STAGES, A_KM ? "A_KM" : "A_KC", B_KM ? "B_KM" : "B_KC",
                 sizeof(OutT) == 2 ? "bf16" : "f32", G == GATHER_NONE ? "" : ",conv",
                 EPI == EPI_ACT_STORE ? ",gelu" : EPI == EPI_ACT_GRAD ? ",gelu_grad" : "");
        return std::string(b);
    }();
    note_kernel(tag.c_str());
    int kps;
    const int splits = effective_splits(op, &kps);
    float* partial = splits > 1 ? op.partial : nullptr;
    if (sizeof(OutT) == 4 && !op.out_f32 && !partial) return hipErrorInvalidValue;   // fp32 tiles need the reduce to reach a bf16 C
    BatchArgs bt;
    bt.batch = G == GATHER_NONE ? op.batch : 1;
    bt.nsplit = splits;
    bt.a_bs = op.a_bs; bt.b_bs = op.b_bs; bt.c_bs = op.c_bs; bt.aux_bs = op.aux_bs; bt.bias_bs = op.bias_bs;
    dim3 grid((unsigned)ceil_div(op.M, BM), (unsigned)ceil_div(op.N, BN), (unsigned)(splits * bt.batch));
    if (G == GATHER_CONV_DGRAD && op.cs.cls) grid.z = (unsigned)(op.cs.stride * op.cs.stride);   // one slab of workgroups per parity class
    hipLaunchKernelGGL(kern, grid, dim3(NT), lds_bytes, st, A, B, op.cs, (OutT*)op.C, op.ldc, op.bias, partial, (int)op.M,
                       (int)op.N, (int)op.K, kps, (bf16_t*)op.aux, op.ldaux, bt);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    // a batch of sliced products is summed as one matrix of batch * M rows (supported() admits only dense results)
    if (splits > 1) {
        const SgdFuse* sgd = op.out_f32 ? op.sgd : nullptr;
        const CropFuse* crop = op.out_f32 ? op.crop : nullptr;
        if (put_off(op.later, op.partial, op.C, !op.out_f32, op.ldc, op.M * bt.batch, op.N, splits, sgd, crop)) return hipSuccess;
        return reduce_partials(op.partial, op.C, !op.out_f32, op.ldc, op.M * bt.batch, op.N, splits, st, sgd, crop);
    }
    return hipSuccess;
}

// The activation epilogues exist for plain bf16 products (the only ones that carry one).
template <int BM, int BN, int WGM, int WGN, int STAGES, bool A_KM, bool B_KM, class OutT, int G = GATHER_NONE>
hipError_t launch(const MatOp& op, const Operand& A, const Operand& B, hipStream_t st)
{
    if constexpr (sizeof(OutT) == 2 && G == GATHER_NONE) {
        if (op.epilogue == EPI_ACT_STORE) return launch_epi<BM, BN, WGM, WGN, STAGES, A_KM, B_KM, OutT, G, EPI_ACT_STORE>(op, A, B, st);
        if (op.epilogue == EPI_ACT_GRAD) return launch_epi<BM, BN, WGM, WGN, STAGES, A_KM, B_KM, OutT, G, EPI_ACT_GRAD>(op, A, B, st);
    }
    return launch_epi<BM, BN, WGM, WGN, STAGES, A_KM, B_KM, OutT, G, EPI_NONE>(op, A, B, st);
}

inline bool al16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Tile choice (see gemm_tile_cost for the figures behind it).
template <bool A_KM, bool B_KM, class OutT, int G = GATHER_NONE>
hipError_t by_tile(const MatOp& op, const Operand& A, const Operand& B, hipStream_t st)
{
    const int64_t splits = effective_splits(op, nullptr), batch = G == GATHER_NONE ? op.batch : 1;
    auto wgs = [&](int bm, int bn) { return ceil_div(op.M, bm) * ceil_div(op.N, bn) * splits * batch; };
    constexpr bool WGRAD = sizeof(OutT) == 4 && A_KM;
    // Results at most 32 columns wide (1x1 and core convolutions at Tucker ranks <= 32): a 128 x 32 tile
    // does a quarter of the MFMA and LDS work of a 128 x 128 one (15 against 23 us at 401408 x 32 x 64).
    if constexpr (sizeof(OutT) == 2 && G != GATHER_CONV_WGRAD) {
        if (op.N <= 32 && wgs(128, 32) >= 256) {
            if (op.K <= BK) return launch<128, 32, 4, 1, 1, A_KM, B_KM, OutT, G>(op, A, B, st);
            if (op.K <= 2 * BK) return launch<128, 32, 4, 1, 2, A_KM, B_KM, OutT, G>(op, A, B, st);
            return launch<128, 32, 4, 1, 4, A_KM, B_KM, OutT, G>(op, A, B, st);
        }
    }
    // Gathers that give a unit many workgroups: two stages of 64 x 64 tiles, five workgroups to a unit, and not four stages
    // or a wider tile, whose two or one cannot cover the address arithmetic of each load.  Results up to 64 columns wide
    // from 3.5 workgroups a unit on (128 images of 56 x 56, 40 -> 40 channels 47.9 -> 35.3 us; 64 -> 64 with stride 2
    // 23.5 -> 17.8 us; at 1.5 a unit over 2304 k 15.5 against 18.5 us), and from 3 on the parity classes of a strided data
    // gradient, whose workgroups run over 1 to 4 taps (128 images of 56 x 56, 64 <- 128 channels 75.5 -> 54.7 us; 64 of
    // 28 x 28, 128 <- 256 36.1 -> 28.3 us; at 1.2 a unit 9.7 against 10.2 us) unless 128 x 128 tiles are the cheaper ones.
    const bool classes = G == GATHER_CONV_DGRAD && op.cs.cls && wgs(64, 64) * op.cs.stride * op.cs.stride >= 3 * 256;
    const bool narrow = G == GATHER_CONV_FWD && op.N <= 64 && 2 * wgs(64, 64) >= 7 * 256;
    // Short reductions (K = rank: second product of a forward pair or of a data gradient) are mostly prologue and
    // epilogue, which only other workgroups on the unit can overlap; eight waves per tile do so better than four.
    if (!WGRAD && op.K <= 8 * BK) {
        if (op.M > 64 && op.N > 64 && (wgs(128, 128) >= 200 || wgs(64, 64) > 2048)) {
            if constexpr (sizeof(OutT) == 2 && G == GATHER_NONE) {
                // (Large results in whole chunks of 64 columns are not here: see mfma_wide_supported.)
                // From three rounds on, 256 x 256 tiles where the multiplication weighs more (with the K x K product
                // before it, 65536 x 1024 x 512: 129 us, 145 us in the next kind, 150 us in the last; 40000 x 1480 x 400
                // 108, 117 and 127); else one stage and three workgroups per unit, against two stages and two of
                // them: 4100 x 4096 x 264 22.6 -> 20.5 us, 32768 x 1024 x 256 with the GELU gradient, with the
                // product before it, 55.5 -> 52.4 us.  Two stages stay faster below three workgroups per unit (8192 x
                // 1024 x 256: 7.9 against 8.2 us) and up to K = 256 without that gradient's second operand to wait
                // for (three members of 1024 columns 24.1 against 26.3 us).
                if (op.K > 6 * BK && op.M > 192 && op.N > 192 && wgs(256, 256) >= 768)
                    return launch<256, 256, 2, 4, 2, A_KM, B_KM, OutT, G>(op, A, B, st);
                if (wgs(128, 128) > 768 && (op.K > 4 * BK || op.epilogue == EPI_ACT_GRAD))
                    return launch<128, 128, 2, 4, 1, A_KM, B_KM, OutT, G>(op, A, B, st);
            }
            return launch<128, 128, 2, 4, 2, A_KM, B_KM, OutT, G>(op, A, B, st);
        }
        // a single K-step needs a single stage: 401408 x 64 x 32 15.1 -> 13.0 us
        if (op.K <= BK) return launch<64, 64, 2, 2, 1, A_KM, B_KM, OutT, G>(op, A, B, st);
        if (op.K <= 4 * BK || classes || narrow) return launch<64, 64, 2, 2, 2, A_KM, B_KM, OutT, G>(op, A, B, st);
        return launch<64, 64, 2, 2, 4, A_KM, B_KM, OutT, G>(op, A, B, st);
    }
    const GemmTile tile = gemm_best_tile(op.M, op.N, op.K, splits, batch, G != GATHER_NONE ? COST_GATHER : WGRAD ? COST_WGRAD : COST_PLAIN, WGRAD);
    if (narrow || (classes && tile >= TILE_64x128)) return launch<64, 64, 2, 2, 2, A_KM, B_KM, OutT, G>(op, A, B, st);
    switch (tile) {
    case TILE_256x256:
        if constexpr (G == GATHER_NONE) return launch<256, 256, 2, 4, 2, A_KM, B_KM, OutT, G>(op, A, B, st);
        [[fallthrough]];
    case TILE_128x256: return launch<128, 256, 2, 4, 3, A_KM, B_KM, OutT, G>(op, A, B, st);
    case TILE_128x128: return launch<128, 128, 2, 4, 4, A_KM, B_KM, OutT, G>(op, A, B, st);
    case TILE_128x128_PAIR: return launch<128, 128, 2, 4, 2, A_KM, B_KM, OutT, G>(op, A, B, st);
    case TILE_64x128: return launch<64, 128, 2, 4, 4, A_KM, B_KM, OutT, G>(op, A, B, st);
    case TILE_128x64: return launch<128, 64, 4, 2, 4, A_KM, B_KM, OutT, G>(op, A, B, st);
    default: return launch<64, 64, 2, 2, 4, A_KM, B_KM, OutT, G>(op, A, B, st);
    }
}

}  // namespace

bool mfma_gemm2_supported(const MatOp& op)
{
    if (!op.in_bf16) return false;
    if (op.M < 1 || op.N < 1 || op.K < 8) return false;
    if (op.M >= (int64_t(1) << 31) || op.N >= (int64_t(1) << 31) || op.K >= (int64_t(1) << 31)) return false;
    if (!al16(op.A) || !al16(op.B) || !al16(op.C)) return false;
    bool akm, bkm;
    if (op.gather == GATHER_NONE) {
        akm = op.a_sk != 1;
        bkm = op.b_sk != 1;
        if (akm && (op.a_sm != 1 || op.a_sk % 8 != 0 || op.M % 8 != 0)) return false;
        if (!akm && op.a_sm % 8 != 0) return false;
        if (bkm && (op.b_sn != 1 || op.b_sk % 8 != 0 || op.N % 8 != 0)) return false;
        if (!bkm && op.b_sn % 8 != 0) return false;
    } else {
        // implicit-GEMM convolution: channel counts must keep every 16-byte chunk inside one tap
        if (op.cs.I % 8 != 0 || op.cs.O % 8 != 0 || op.cs.k < 1 || op.cs.k > 31 || op.cs.stride < 1) return false;
        // byte offsets below BUF_OOB
        const int64_t most = (int64_t(1) << 31) - 16;
        if ((int64_t)op.cs.N * op.cs.H * op.cs.W * op.cs.I >= most || (int64_t)op.cs.N * op.cs.Ho * op.cs.Wo * op.cs.O >= most) return false;
        if ((int64_t)op.cs.O * op.cs.k * op.cs.k * op.cs.I >= most) return false;
        if (op.gather == GATHER_CONV_FWD) {
            akm = false; bkm = false;
            if (op.b_sk != 1 || op.b_sn % 8 != 0) return false;
        } else if (op.gather == GATHER_CONV_DGRAD) {
            akm = false; bkm = true;
            // pixel coordinate / stride is done by multiplication, exact while coordinate * stride < 65536
            if ((int64_t)(std::max(op.cs.H, op.cs.W) + op.cs.pad) * op.cs.stride >= 65536) return false;
        } else {
            akm = true; bkm = true;
            if (op.a_sm != 1 || op.a_sk % 8 != 0 || op.M % 8 != 0) return false;
        }
    }
    if ((!akm || !bkm) && op.K % 8 != 0) return false;    // a k-contiguous operand is read in chunks of 8 k
    if (akm && !bkm) return false;                       // layout not used by any layer pass
    if (op.out_f32) {
        if (!(akm && bkm)) return false;                 // fp32 results are weight gradients
        if (op.N % 4 != 0 || op.ldc % 4 != 0 || op.bias) return false;
    } else {
        if (akm) return false;
        if (op.N % 8 != 0 || op.ldc % 8 != 0) return false;
        // split-K towards a bf16 result: fp32 partials, rounded once by the reduce; plain products only
        if (op.splits > 1 && (op.gather != GATHER_NONE || op.bias || op.epilogue != EPI_NONE)) return false;
        if (op.bias && (op.N < 4 || (reinterpret_cast<uintptr_t>(op.bias) & 15u))) return false;
    }
    if (ceil_div(op.N, 64) > 65535) return false;
    if (op.batch < 1 || op.batch > 1024) return false;
    if (op.batch > 1) {
        if (op.gather != GATHER_NONE || op.sgd) return false;
        if (op.a_bs % 8 != 0 || op.b_bs % 8 != 0 || op.c_bs % 8 != 0 || op.aux_bs % 8 != 0 || op.bias_bs % 4 != 0) return false;
        // sliced reductions of a batch are summed as one tall dense matrix
        if (op.splits > 1 && op.partial && (!op.out_f32 || op.ldc != op.N || op.c_bs != op.M * op.N)) return false;
    }
    if (op.gather == GATHER_NONE && ((akm ? op.a_sk : op.a_sm) > BUF_MAX_LD || (bkm ? op.b_sk : op.b_sn) > BUF_MAX_LD)) return false;
    if (op.epilogue != EPI_NONE && (op.out_f32 || op.gather != GATHER_NONE || !op.aux || !al16(op.aux) || op.ldaux % 8 != 0)) return false;
    return true;
}

hipError_t mfma_gemm2(const MatOp& op, hipStream_t st)
{
    if (op.gather == GATHER_CONV_FWD) {
        Operand A{(const bf16_t*)op.A, 0, (int)op.M};
        Operand B{(const bf16_t*)op.B, op.b_sn, (int)op.N};
        return by_tile<false, false, bf16_t, GATHER_CONV_FWD>(op, A, B, st);
    }
    if (op.gather == GATHER_CONV_DGRAD) {
        Operand B{(const bf16_t*)op.B, 0, (int)op.N};
        const ConvShape& cs = op.cs;
        if (cs.stride > 1 && cs.k >= cs.stride) {
            // Strided: an input pixel hears from an output pixel only through the taps of its parity
            // class, 1 / stride^2 of them on average.  One product per class, over those taps only,
            // written to the class's pixels (as one product over all taps, three quarters of a
            // stride-2 gradient's multiplications are by zeros).
            // The launch is shaped for class (0, 0), which has the most rows; the kernel takes the class
            // from blockIdx.z and works out that class's rows and taps itself.
            MatOp sub = op;
            sub.cs.cls = 1;
            sub.splits = 1;
            sub.M = (int64_t)cs.N * class_extent(cs.H, 0, cs.stride) * class_extent(cs.W, 0, cs.stride);
            int taps = 0;
            for (int c = 0; c < cs.stride; ++c) taps = std::max(taps, class_taps(c, cs.pad, cs.stride, cs.k).count);
            sub.K = (int64_t)taps * taps * cs.O;
            Operand A{(const bf16_t*)op.A, 0, (int)sub.M};
            return by_tile<false, true, bf16_t, GATHER_CONV_DGRAD>(sub, A, B, st);
        }
        Operand A{(const bf16_t*)op.A, 0, (int)op.M};
        return by_tile<false, true, bf16_t, GATHER_CONV_DGRAD>(op, A, B, st);
    }
    if (op.gather == GATHER_CONV_WGRAD) {
        Operand A{(const bf16_t*)op.A, op.a_sk, (int)op.M};
        Operand B{(const bf16_t*)op.B, 0, (int)op.N};
        return by_tile<true, true, float, GATHER_CONV_WGRAD>(op, A, B, st);
    }
    const bool akm = op.a_sk != 1, bkm = op.b_sk != 1;
    Operand A{(const bf16_t*)op.A, akm ? op.a_sk : op.a_sm, (int)op.M};
    Operand B{(const bf16_t*)op.B, bkm ? op.b_sk : op.b_sn, (int)op.N};
    if (op.out_f32) return by_tile<true, true, float>(op, A, B, st);
    if (effective_splits(op, nullptr) > 1)
        return bkm ? by_tile<false, true, float>(op, A, B, st) : by_tile<false, false, float>(op, A, B, st);
    if (bkm) return by_tile<false, true, bf16_t>(op, A, B, st);
    return by_tile<false, false, bf16_t>(op, A, B, st);
}

}  // namespace lrd
