// jk_mixed.hip -- mixed-precision kernels of the CD J/K build.
//
// The bulk products (half-transforms and the exchange contraction) run as
// exact fixed-point slice products on the INT8 matrix cores (slice_core.hpp);
// gamma, J, every cross-chunk sum and the final K accumulation stay FP64.
//
//   slice   rows of an FP64 operand -> NS int8 digit planes + row exponent
//   ht      [X^Q | Y^Q] = slices(B^Q) x slices([C_L | C_R]), recombined in FP64
//   rowmax  exponent of every row (side, k, m) of X/Y over the chunk
//   ex      K_k (+)= slices(X_k) x slices(Y_k) over the chunk, recombined in FP64
#include <algorithm>
#include <mutex>
#include <set>
#include <utility>

#include "jk_batched.hpp"
#include "jk_kernels.hpp"
#include "jk_tiles.hpp"
#include "slice_core.hpp"

namespace jk {

namespace {
constexpr int kNS = kSliceDigits;       // digits per operand (31 bits)
constexpr int kRowPad = 64;             // X/Y planes' rows are padded to this
constexpr int kKPad = kSliceKB;         // plane inner bytes are padded to this
// Workgroup tiles of four 32 x 64 waves, 73.5 KB of LDS, two workgroups per CU
// (the sums of a wave's 32 x 64 outputs take 160 registers).  The
// half-transform and the exchange's vertical tiles are 128 x 64, the
// exchange's horizontal ones 64 x 128.
typedef STileW<128, 64, kNS, 2> TileV;
typedef STileW<64, 128, kNS, 2> TileZ;
constexpr int kLdsBytes = 3 * TileV::STAGE_BYTES;
static_assert(TileV::STAGE_BYTES == TileZ::STAGE_BYTES, "one LDS size");
constexpr int kMhM = 128, kMhN = 64;

inline int cdiv(i64 a, i64 b) { return (int)((a + b - 1) / b); }

// Two doubles at any element: 16-byte loads need 4-byte alignment only.
typedef double d2 __attribute__((ext_vector_type(2), aligned(8)));

__device__ __forceinline__ void write_digits(int8_t *dst, i64 pstride, const int8_t (*d)[kNS])
{
#pragma unroll
    for (int p = 0; p < kNS; p++) {
        const int w = (d[0][p] & 0xff) | ((d[1][p] & 0xff) << 8) | ((d[2][p] & 0xff) << 16) |
                      ((int)(d[3][p] & 0xff) << 24);
        *(int *)(dst + p * pstride) = w;
    }
}
} // namespace

// ------------------------------------------------------------------ slicing
// All slicers read source element (b, m, k) = src[b * bs + m * rs + k * ks]
// for b < nb, m < nr, k < nk and write the digit planes of rows b * rp + m in
// the K-blocked layout of slice_core.hpp; rows m in [nr, rp) and inner bytes
// k in [nk, 32 nkb) get zero digits.

// Generic two-pass slicer (any strides; used for the small [C_L | C_R]
// operand): 8 threads per row (sub = lane & 7), exps[row] = row exponent.
__device__ __forceinline__ void slice_row8(const double *__restrict__ src, i64 bs, i64 rs, i64 ks,
                                           int nr, int nk, int rp, int nkb,
                                           int8_t *__restrict__ out, i64 pstride, i64 kbstride,
                                           int *__restrict__ exps, i64 row, int sub)
{
    const int b = (int)(row / rp), m = (int)(row % rp);
    const bool live = m < nr;
    const double *s = src + (i64)b * bs + (i64)m * rs;
    double mx = 0.0;
    if (live)
        for (int k = sub; k < nk; k += 8)
            mx = fmax(mx, fabs(s[(i64)k * ks]));
    mx = fmax(mx, __shfl_xor(mx, 1));
    mx = fmax(mx, __shfl_xor(mx, 2));
    mx = fmax(mx, __shfl_xor(mx, 4));
    const int e = row_exponent(mx);
    if (sub == 0)
        exps[row] = live ? e : 0;
    int8_t *dst = out + row * kSliceKB + sub * 4;
    for (int kb = 0; kb < nkb; kb++) {
        int8_t d[4][kNS];
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const int k = kb * kSliceKB + sub * 4 + u;
            const double v = (live && k < nk) ? s[(i64)k * ks] : 0.0;
            slice_value(v, e, d[u]);
        }
        write_digits(dst + (i64)kb * kbstride, pstride, d);
    }
}

// 32 rows per workgroup.
__global__ void __launch_bounds__(256) k_slice_rows(const double *__restrict__ src, i64 bs, i64 rs,
                                                    i64 ks, int nb, int nr, int nk, int rp, int nkb,
                                                    int8_t *__restrict__ out, i64 pstride,
                                                    i64 kbstride, int *__restrict__ exps)
{
    const int t = threadIdx.x;
    const i64 row = (i64)blockIdx.x * 32 + (t >> 3);
    if (row >= (i64)nb * rp)        // whole 8-lane row groups leave together
        return;
    slice_row8(src, bs, rs, ks, nr, nk, rp, nkb, out, pstride, kbstride, exps, row, t & 7);
}

// One-pass slicer for unit-stride rows of at most 32 LPR elements: LPR lanes
// hold a row in registers (lane l of the row: elements 4 l + 4 LPR j + u, j < 8),
// reduce its maximum among them, then write the digits.  A wave takes 64 / LPR
// consecutive rows, so that each of its plane writes covers 64 / LPR x 32
// consecutive bytes of LPR / 8 inner blocks.  Bound by memory, 12 bytes per
// element: 5.3 TB/s at nao 300, 4.9 at 250, 5.2 at 500 (one row per wave, in
// 32-byte pieces: 3.8, 3.6 and 4.0).
// ks != 1 (the factors, whose rows are columns of [C_L | C_R]): element loads.
constexpr int kSliceNJ = 8;
template <int LPR, bool UNIT = true>
__device__ __forceinline__ void slice_row_wave(const double *__restrict__ src, i64 bs, i64 rs, i64 ks,
                                               int nr, int nk, int rp, int nkb,
                                               int8_t *__restrict__ out, i64 pstride, i64 kbstride,
                                               int *__restrict__ exps, i64 row)
{
    const int sub = threadIdx.x & (LPR - 1);
    const int b = (int)(row / rp), m = (int)(row % rp);
    const bool live = m < nr;
    const double *s = src + (i64)b * bs + (i64)(live ? m : nr - 1) * rs;
    double v[kSliceNJ][4];
    double mx = 0.0;
#pragma unroll
    for (int j = 0; j < kSliceNJ; j++) {
        if (4 * LPR * j >= nk) {                 // the same for every lane
#pragma unroll
            for (int u = 0; u < 4; u++)
                v[j][u] = 0.0;
            continue;
        }
        const int k0 = 4 * LPR * j + 4 * sub;
        if (UNIT && k0 + 4 <= nk) {
            const d2 lo = *(const d2 *)(s + k0), hi = *(const d2 *)(s + k0 + 2);
            v[j][0] = lo[0];
            v[j][1] = lo[1];
            v[j][2] = hi[0];
            v[j][3] = hi[1];
        } else {
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const double x = s[(UNIT ? 1 : ks) * ((k0 + u) < nk ? k0 + u : nk - 1)];
                v[j][u] = k0 + u < nk ? x : 0.0;
            }
        }
        if (!live)
#pragma unroll
            for (int u = 0; u < 4; u++)
                v[j][u] = 0.0;
    }
#pragma unroll
    for (int j = 0; j < kSliceNJ; j++)
#pragma unroll
        for (int u = 0; u < 4; u++)
            mx = fmax(mx, fabs(v[j][u]));
#pragma unroll
    for (int o = LPR / 2; o >= 1; o >>= 1)
        mx = fmax(mx, __shfl_xor(mx, o));
    const int e = row_exponent(mx);
    if (sub == 0)
        exps[row] = live ? e : 0;
    int8_t *dst = out + row * kSliceKB + 4 * (sub & 7);
#pragma unroll
    for (int j = 0; j < kSliceNJ; j++) {
        const int kb = LPR / 8 * j + (sub >> 3);
        if (kb < nkb) {
            int8_t d[4][kNS];
#pragma unroll
            for (int u = 0; u < 4; u++)
                slice_value(v[j][u], e, d[u]);
            write_digits(dst + (i64)kb * kbstride, pstride, d);
        }
    }
}

template <int LPR>
__global__ void __launch_bounds__(256) k_slice_rows_wave(const double *__restrict__ src, i64 bs,
                                                         i64 rs, int nb, int nr, int nk, int rp,
                                                         int nkb, int8_t *__restrict__ out,
                                                         i64 pstride, i64 kbstride,
                                                         int *__restrict__ exps)
{
    const i64 row = (i64)blockIdx.x * (256 / LPR) + threadIdx.x / LPR;
    if (row >= (i64)nb * rp)        // whole rows of lanes leave together
        return;
    slice_row_wave<LPR>(src, bs, rs, 1, nr, nk, rp, nkb, out, pstride, kbstride, exps, row);
}

// The factors: row c, inner n, element src[n ks + c], one wave per row (few
// rows: 8 lanes per row and two passes took 26 us for 480 columns at nao 300).
__global__ void __launch_bounds__(256) k_slice_cols(const double *__restrict__ src, i64 ks, int nr, int nk,
                                                    int rp, int nkb, int8_t *__restrict__ out,
                                                    i64 pstride, i64 kbstride, int *__restrict__ exps)
{
    const i64 row = (i64)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (row >= rp)
        return;
    slice_row_wave<64, false>(src, 0, 1, ks, nr, nk, rp, nkb, out, pstride, kbstride, exps, row);
}
// Lanes per row for rows of nkb 32-byte inner blocks; 0: longer than 2048.
inline int slice_lanes(int nkb)
{
    return nkb <= 8 ? 8 : nkb <= 16 ? 16 : nkb <= 32 ? 32 : nkb <= 64 ? 64 : 0;
}

// The same for packed symmetric slabs (jk.h JK_B_PACKED).  A workgroup takes
// a band of kBand rows [m0, m0 + kBand) of one slab and first gathers it into
// LDS with coalesced reads: the part n >= m of row m is contiguous in packed
// row m; the part n < m is column m of packed row n, and the band's kBand
// columns of packed row n are contiguous.  Wave w then slices rows w, w + 4
// of the band from LDS exactly as the one-pass slicer does.  nk = nr = nao.
constexpr int kBand = 8;

// Band [m0, m0 + kBand) of packed slab P, plane rows b * rp + m; T holds
// kBand x nao doubles of LDS.
template <int NJ>
__device__ __forceinline__ void slice_band_packed(const double *__restrict__ P, int b, int m0,
                                                  int nao, int rp, int nkb,
                                                  int8_t *__restrict__ out, i64 pstride,
                                                  i64 kbstride, int *__restrict__ exps, double *T)
{
    const int ld = nao;
    const int tid = threadIdx.x;
#pragma unroll 1
    for (int r = 0; r < kBand; r++) {          // n >= m: packed row m
        const int m = m0 + r;
        if (m < nao) {
            const double *row = P + pk_row(m, nao) - m;
            for (int n = m + tid; n < nao; n += 256)
                T[r * ld + n] = row[n];
        }
    }
    const int nlow = (m0 + kBand < nao ? m0 + kBand : nao) * kBand;
    for (int t = tid; t < nlow; t += 256) {    // n < m: column m of packed row n
        const int n = t / kBand, r = t % kBand, m = m0 + r;
        if (n < m && m < nao)
            T[r * ld + n] = P[pk_row(n, nao) + (m - n)];
    }
    __syncthreads();
    const int lane = tid & 63, wave = tid >> 6;
#pragma unroll 1
    for (int r = wave; r < kBand; r += 4) {
        const int m = m0 + r;
        if (m >= rp)
            break;
        const bool live = m < nao;
        const i64 row = (i64)b * rp + m;
        double v[NJ][4];
        double mx = 0.0;
#pragma unroll
        for (int j = 0; j < NJ; j++) {
            const int k0 = 256 * j + 4 * lane;
#pragma unroll
            for (int u = 0; u < 4; u++) {
                const int k = k0 + u;
                v[j][u] = (live && k < nao) ? T[r * ld + k] : 0.0;
                mx = fmax(mx, fabs(v[j][u]));
            }
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1)
            mx = fmax(mx, __shfl_xor(mx, o));
        const int e = row_exponent(mx);
        if (lane == 0)
            exps[row] = live ? e : 0;
        int8_t *dst = out + row * kSliceKB + 4 * (lane & 7);
#pragma unroll
        for (int j = 0; j < NJ; j++) {
            const int kb = 8 * j + (lane >> 3);
            if (kb < nkb) {
                int8_t d[4][kNS];
#pragma unroll
                for (int u = 0; u < 4; u++)
                    slice_value(v[j][u], e, d[u]);
                write_digits(dst + (i64)kb * kbstride, pstride, d);
            }
        }
    }
}

template <int NJ>
__global__ void __launch_bounds__(256) k_slice_band_packed(const double *__restrict__ src, i64 bs,
                                                           int nb, int nao, int rp, int nkb,
                                                           int8_t *__restrict__ out, i64 pstride,
                                                           i64 kbstride, int *__restrict__ exps)
{
    extern __shared__ double T[];              // [kBand][nao]
    const int nband = (rp + kBand - 1) / kBand;
    const int b = blockIdx.x / nband, m0 = (blockIdx.x % nband) * kBand;
    slice_band_packed<NJ>(src + (i64)b * bs, b, m0, nao, rp, nkb, out, pstride, kbstride, exps, T);
}

// Elementwise slicer of the half-transformed factors.  Source XY[ql][m][c]
// (c < nkey r; X_k = columns k*r.., Y_k = columns R + k*r..; nkey = 2 nd, or
// nd when only X is formed), plane row (side * nd + k) * mp + m, inner index
// j = ql * r + i (j < nj).  The row's exponent comes from its nsp partial
// maxima (rowmax below) and is left in exps for the exchange by the threads of
// inner block 0.  32 plane rows x one 32-byte inner block per workgroup (grid:
// row groups x nkb); each plane write of a workgroup is one contiguous
// kilobyte.
__device__ __forceinline__ void slice_xy_block(const double *__restrict__ XY, int nao, int nkey,
                                               int r, int mp, int nj, int8_t *__restrict__ out,
                                               i64 pstride, i64 kbstride,
                                               const uint32_t *__restrict__ mx, int nsp,
                                               int *__restrict__ exps, int row, int sub, int kb)
{
    const int key = row / mp, m = row % mp;
    const bool live = m < nao;
    uint32_t hi = 0;
    if (live)
        for (int u = 0; u < nsp; u++)
            hi = max(hi, mx[(i64)u * nkey * mp + row]);
    const int e = row_exponent_hi(hi);
    if (kb == 0 && sub == 0)
        exps[row] = e;
    const i64 R2 = (i64)nkey * r;     // row length of XY
    // loads are unconditional (clamped addresses), masked afterwards
    const double *s = XY + (i64)(live ? m : nao - 1) * R2 + (i64)key * r;
    const int j0 = kb * kSliceKB + sub * 4;
    double x[4];
    const int q0 = j0 / r, i0 = j0 - q0 * r;
    const double *p0 = s + (i64)q0 * nao * R2 + i0;
    if (j0 + 3 < nj && i0 + 3 < r) {
        const d2 lo = *(const d2 *)p0, hi = *(const d2 *)(p0 + 2);
        x[0] = lo[0];
        x[1] = lo[1];
        x[2] = hi[0];
        x[3] = hi[1];
    } else {
#pragma unroll
        for (int u = 0; u < 4; u++) {
            const int j = (j0 + u) < nj ? (j0 + u) : nj - 1;
            const int ql = j / r, i = j - ql * r;
            x[u] = s[(i64)ql * nao * R2 + i];
        }
    }
    int8_t d[4][kNS];
#pragma unroll
    for (int u = 0; u < 4; u++)
        slice_value((live && j0 + u < nj) ? x[u] : 0.0, e, d[u]);
    write_digits(out + (i64)kb * kbstride + (i64)row * kSliceKB + sub * 4, pstride, d);
}

__global__ void __launch_bounds__(256) k_slice_xy(const double *__restrict__ XY, int nao, int nkey,
                                                  int r, int mp, int nj, int8_t *__restrict__ out,
                                                  i64 pstride, i64 kbstride,
                                                  const uint32_t *__restrict__ mx, int nsp,
                                                  int *__restrict__ exps, int nkb)
{
    const int t = threadIdx.x, sub = t & 7;
    const int row = blockIdx.x * 32 + (t >> 3);
    if (row >= nkey * mp)
        return;
    // inner blocks kb = blockIdx.y, + gridDim.y, ... (grid y is capped at 65535)
    for (int kb = blockIdx.y; kb < nkb; kb += gridDim.y)
        slice_xy_block(XY, nao, nkey, r, mp, nj, out, pstride, kbstride, mx, nsp, exps, row, sub, kb);
}

// ------------------------------------------------------------------ half-transform
// XY[g][c] = 2^(eB + eC - 14) * sum_l S_l 2^(-8 (l - 2)) over the chunk's slabs
// stacked into rows g = ql nao + m (c < R: X = B^Q C_L, c >= R: Y = B^Q C_R),
// so that only the chunk's last tile has rows to spare; A planes: rows g (tiles
// may read up to 127 rows past the chunk), B planes: rows c, cp of them.
//
// The tile also leaves the row maxima the exponents of X and Y need: for each
// of its rows and each key (c / r) its columns meet, the largest |XY| over
// those columns, as the value's high word rounded up (the exponent depends on
// no more), at
//     pm[(cb nslot + key - key0) rows + g]
// (cb = column tile, key0 = its first key, nslot >= the keys a tile meets,
// rows = pm's pitch).  The words go to LDS (the pipeline's buffers, free after
// the products), and one thread per row takes the maxima key by key.  The
// maximum is exact, so the exponents equal those of a pass over XY.
//
// The row and column exponents a lane needs (16 rows, 2 columns) are loaded
// before the products, so that their latency is hidden behind them.
constexpr int kPmLd = kMhN + 1;     // LDS row stride of the |XY| tile (words)
static_assert(kMhM * kPmLd * 4 <= kLdsBytes, "|XY| tile in the pipeline's LDS");

__device__ __forceinline__ void ht_mixed_tile(const int8_t *__restrict__ Bp, i64 bpstride,
                                              i64 bkbstride, const int *__restrict__ eB,
                                              const int8_t *__restrict__ Cp, i64 cpstride,
                                              i64 ckbstride, const int *__restrict__ eC,
                                              double *__restrict__ XY, int nrow, int R2, int cp,
                                              int nkb, int t, char *lds, uint32_t *__restrict__ pm,
                                              int rows, int r, int nslot)
{
    typedef TileV TL;
    const int nct = cp / kMhN;
    const int rb = t / nct, cb = t % nct;
    const int g0 = rb * kMhM, c0 = cb * kMhN;
    // exponents of this lane's rows (element e of either tile) and columns
    int eb[16], ec[TL::TN];
#pragma unroll
    for (int e = 0; e < 16; e++) {
        int row, col;
        stile_coord_wide<TL>(0, e, row, col);
        eb[e] = eB[g0 + row];
    }
#pragma unroll
    for (int tt = 0; tt < TL::TN; tt++) {
        int row, col;
        stile_coord_wide<TL>(tt, 0, row, col);
        ec[tt] = eC[c0 + col] + kSliceProdShift;
    }
    SPlanes a{Bp, bpstride, bkbstride};
    SPlanes b{Cp, cpstride, ckbstride};
    SAccW<TL> acc;
    acc.zero();
    stile_gemm_w4<TL, kNS>(a, b, g0, c0, 1 << 30, cp, 0, nkb, lds, acc);
    uint32_t *tile = (uint32_t *)lds;
    __syncthreads();                          // every wave past its last stage
#pragma unroll
    for (int tt = 0; tt < TL::TN; tt++)
#pragma unroll
        for (int e = 0; e < 16; e++) {
            int row, col;
            stile_coord_wide<TL>(tt, e, row, col);
            const int g = g0 + row, c = c0 + col;
            const double v = ldexp(combine_levels_wide<TL>(acc, tt, e), eb[e] + ec[tt]);
            if (g < nrow && c < R2)
                XY[(i64)g * R2 + c] = v;
            tile[row * kPmLd + col] = high_word_up(v);
        }
    __syncthreads();
    if (threadIdx.x < kMhM) {
        const uint32_t *x = tile + threadIdx.x * kPmLd;
        uint32_t *dst = pm + (i64)cb * nslot * rows + g0 + threadIdx.x;
        const int cend = (c0 + kMhN) < R2 ? kMhN : R2 - c0;
        int left = r - c0 % r;                // columns of the first key
        uint32_t mx = 0;
        for (int cg = 0; cg < cend; cg += 16) {
            uint32_t v[16];
#pragma unroll
            for (int u = 0; u < 16; u++)
                v[u] = x[cg + u];
#pragma unroll
            for (int u = 0; u < 16; u++) {
                mx = max(mx, v[u]);
                if (cg + u < cend && (--left == 0 || cg + u + 1 == cend)) {
                    *dst = mx;
                    dst += rows;
                    left = r;
                    mx = 0;
                }
            }
        }
    }
}

__global__ void __launch_bounds__(256, 2) k_ht_mixed(const int8_t *__restrict__ Bp, i64 bpstride,
                                                     i64 bkbstride, const int *__restrict__ eB,
                                                     const int8_t *__restrict__ Cp, i64 cpstride,
                                                     i64 ckbstride, const int *__restrict__ eC,
                                                     double *__restrict__ XY, int nrow, int R2, int cp,
                                                     int nkb, uint32_t *__restrict__ pm, int rows,
                                                     int r, int nslot)
{
    extern __shared__ char lds[];
    // consecutive tiles (the column tiles of a row panel) on one XCD, sharing its L2
    ht_mixed_tile(Bp, bpstride, bkbstride, eB, Cp, cpstride, ckbstride, eC, XY, nrow, R2, cp, nkb,
                  xcd_swizzle(blockIdx.x, gridDim.x), lds, pm, rows, r, nslot);
}

// Partial-maximum slots per (row, column tile): the keys a column tile of
// kMhN columns can meet.
__host__ __device__ inline int pm_slots(int r, int nkey)
{
    const int n = (kMhN - 1) / r + 2;
    return n < nkey ? n : nkey;
}

// mx[sp nkey mpe + key mpe + m]: the largest of the half-transform's partial
// maxima (pitch rows) over the slabs of split sp of the chunk's nq, and over
// the column tiles that meet key's columns [key r, key r + r), for the 64 rows
// of row block mblk.  Four waves; wave w takes every fourth slab (coalesced
// 256-byte reads); the wave maxima meet in red.
__device__ __forceinline__ void rowmax_pm_block(const uint32_t *__restrict__ pm, int nao, int nq,
                                                int rows, int mpe, int nslot, int nkey, int r,
                                                uint32_t *__restrict__ out, int mblk, int key, int sp,
                                                int nsp, uint32_t (*red)[64])
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int m = mblk * 64 + lane;
    const int mc = m < nao ? m : nao - 1;
    const int cb0 = key * r / kMhN, cb1 = (key * r + r - 1) / kMhN;
    const int len = (nq + nsp - 1) / nsp, q0 = sp * len, q1 = q0 + len < nq ? q0 + len : nq;
    uint32_t mx = 0;
    for (int cb = cb0; cb <= cb1; cb++) {
        const int slot = key - cb * kMhN / r;
        const uint32_t *p = pm + ((i64)cb * nslot + slot) * rows + mc;
        int ql = q0 + w;
        for (; ql + 60 < q1; ql += 64) {         // 16 loads in flight
            uint32_t v[16];
#pragma unroll
            for (int u = 0; u < 16; u++)
                v[u] = p[(i64)(ql + 4 * u) * nao];
#pragma unroll
            for (int u = 0; u < 16; u++)
                mx = max(mx, v[u]);
        }
        for (; ql < q1; ql += 4)
            mx = max(mx, p[(i64)ql * nao]);
    }
    red[w][lane] = mx;
    __syncthreads();
    if (w == 0 && m < nao)
        out[((i64)sp * nkey + key) * mpe + m] = max(max(red[0][lane], red[1][lane]),
                                                   max(red[2][lane], red[3][lane]));
}

// Workgroup: 64 rows of one key, one split of the slabs.
__global__ void __launch_bounds__(256) k_xy_rowmax_pm(const uint32_t *__restrict__ pm, int nao, int nq,
                                                      int rows, int mpe, int nslot, int r,
                                                      uint32_t *__restrict__ out)
{
    __shared__ uint32_t red[4][64];
    rowmax_pm_block(pm, nao, nq, rows, mpe, nslot, gridDim.y, r, out, blockIdx.x, blockIdx.y, blockIdx.z,
                    gridDim.z, red);
}

// ------------------------------------------------------------------ exchange
// Kp[s][k][m][n] (+)= scale 2^(eX + eY - 14) * sum_l S_l 2^(-8 (l - 2)) over the inner
// blocks [s * kbl, (s + 1) * kbl) of split s.  X/Y planes: rows k * mp + m
// from Xp / Yp (same strides); row exponents eX[k * mp + m], eY[k * mp + n].
//
// Tiles: the n x n blocks of 64 x 64 (n = mp / 64) in pairs, side by side along
// each row of blocks, the last column of an odd n on top of each other (general
// densities), so that the padding is that of 64 rows and columns: n = 5 (nao
// 300) takes 13 tiles of 128 x 64 where 128 x 128 ones took 9, twice the size.
// sym (Y = X, the upper triangle): row mb's blocks from mb on in pairs.  The
// exchange of nao 300, naux 1200, 4 densities of rank 30: 278 -> 212 us (93 -> 123
// TFLOP/s of FP64 equivalent); at multiples of 128 the two are even.
__host__ __device__ inline int ex_pairs(int n, int sym)
{
    if (sym)                          // sum over mb of ceil((n - mb) / 2)
        return ((n + 1) / 2) * ((n + 2) / 2);
    return n * (n / 2) + (n & 1 ? (n + 1) / 2 : 0);
}
// Blocks (mb, nb) of pair t; true: on top of each other.
__device__ __forceinline__ bool ex_pair(int t, int n, int sym, int &mb, int &nb)
{
    if (sym) {
        mb = 0;
        while (t >= (n - mb + 1) / 2) {
            t -= (n - mb + 1) / 2;
            mb++;
        }
        nb = mb + 2 * t;
        return false;
    }
    const int h = n / 2;
    if (t < n * h) {
        mb = t / h;
        nb = 2 * (t % h);
        return false;
    }
    mb = 2 * (t - n * h);
    nb = n - 1;
    return true;
}

template <class TL>
__device__ __forceinline__ void ex_mixed_product(const int8_t *__restrict__ Xk,
                                                 const int8_t *__restrict__ Yk, i64 pstride,
                                                 i64 kbstride, const int *__restrict__ eX,
                                                 const int *__restrict__ eY, double *__restrict__ Kk,
                                                 int nao, int mp, int m0, int n0, int kb0, int kb1,
                                                 int accumulate, double scale, char *lds)
{
    SPlanes a{Xk, pstride, kbstride};
    SPlanes b{Yk, pstride, kbstride};
    SAccW<TL> acc;
    acc.zero();
    stile_gemm_w4<TL, kNS>(a, b, m0, n0, mp, mp, kb0, kb1, lds, acc);
    // The lane's row and column exponents, and per tile the partial sums it
    // adds to, each loaded in one batch so that their latencies overlap.
    int ex[16], ey[TL::TN];
#pragma unroll
    for (int e = 0; e < 16; e++) {
        int row, col;
        stile_coord_wide<TL>(0, e, row, col);
        ex[e] = eX[min(m0 + row, mp - 1)];
    }
#pragma unroll
    for (int tt = 0; tt < TL::TN; tt++) {
        int row, col;
        stile_coord_wide<TL>(tt, 0, row, col);
        ey[tt] = eY[min(n0 + col, mp - 1)] + kSliceProdShift;
    }
#pragma unroll
    for (int tt = 0; tt < TL::TN; tt++) {
        double old[16];
#pragma unroll
        for (int e = 0; e < 16; e++) {
            int row, col;
            stile_coord_wide<TL>(tt, e, row, col);
            const int m = m0 + row, n = n0 + col;
            old[e] = (accumulate && m < nao && n < nao) ? Kk[(i64)m * nao + n] : 0.0;
        }
#pragma unroll
        for (int e = 0; e < 16; e++) {
            int row, col;
            stile_coord_wide<TL>(tt, e, row, col);
            const int m = m0 + row, n = n0 + col;
            if (m < nao && n < nao) {
                const double v = scale * ldexp(combine_levels_wide<TL>(acc, tt, e), ex[e] + ey[tt]);
                Kk[(i64)m * nao + n] = accumulate ? old[e] + v : v;
            }
        }
    }
}

__device__ __forceinline__ void ex_mixed_tile(const int8_t *__restrict__ Xp,
                                              const int8_t *__restrict__ Yp, i64 pstride,
                                              i64 kbstride, const int *__restrict__ eX,
                                              const int *__restrict__ eY, double *__restrict__ Kp,
                                              int nao, int nd, int mp, int nkb, int kbl,
                                              int accumulate, int sym, double scale, int t,
                                              char *lds)
{
    const int n = mp / 64, np = ex_pairs(n, sym), per = nd * np;
    const int sp = t / per, rem0 = t % per;
    const int k = rem0 / np;
    int mb, nb;
    const bool vertical = ex_pair(rem0 % np, n, sym, mb, nb);
    const int kb0 = sp * kbl < nkb ? sp * kbl : nkb;
    const int kb1 = (kb0 + kbl) < nkb ? (kb0 + kbl) : nkb;
    const int8_t *Xk = Xp + (i64)k * mp * kSliceKB, *Yk = Yp + (i64)k * mp * kSliceKB;
    const int *eXk = eX + (i64)k * mp, *eYk = eY + (i64)k * mp;
    double *Kk = Kp + ((i64)sp * nd + k) * nao * nao;
    if (vertical)
        ex_mixed_product<TileV>(Xk, Yk, pstride, kbstride, eXk, eYk, Kk, nao, mp, mb * 64, nb * 64, kb0,
                                kb1, accumulate, scale, lds);
    else
        ex_mixed_product<TileZ>(Xk, Yk, pstride, kbstride, eXk, eYk, Kk, nao, mp, mb * 64, nb * 64, kb0,
                                kb1, accumulate, scale, lds);
}

__global__ void __launch_bounds__(256, 2) k_ex_mixed(const int8_t *__restrict__ Xp,
                                                     const int8_t *__restrict__ Yp, i64 pstride,
                                                     i64 kbstride, const int *__restrict__ eX,
                                                     const int *__restrict__ eY,
                                                     double *__restrict__ Kp, int nao, int nd, int mp,
                                                     int nkb, int kbl, int accumulate, int sym,
                                                     double scale)
{
    extern __shared__ char lds[];
    ex_mixed_tile(Xp, Yp, pstride, kbstride, eX, eY, Kp, nao, nd, mp, nkb, kbl, accumulate, sym,
                  scale, xcd_swizzle(blockIdx.x, gridDim.x), lds);
}

// ------------------------------------------------------------------ batched
// The mixed phases over many members (jk_batched.hpp): the launch's table maps
// each workgroup to (member, tile); every member runs its own plan's chunk c
// with single-buffered planes, so a batched member is the same arithmetic as
// a single build of the same plan.

__global__ void __launch_bounds__(256) k_bm_slice_c(const BMember *__restrict__ M,
                                                    const int *__restrict__ tab)
{
    int loc;
    const BMember &m = M[find_member(tab, blockIdx.x, loc)];
    const i64 row = (i64)loc * 4 + (threadIdx.x >> 6);
    if (row >= m.cp)                 // whole waves leave together
        return;
    const int R2 = 2 * m.nd * m.r;
    slice_row_wave<64, false>(m.Cc, 0, 1, R2, R2, m.nao, m.cp, m.kp / kSliceKB, m.Cp, m.cps, m.ckb, m.eC,
                              row);
}

template <int LPR>
__global__ void __launch_bounds__(256) k_bm_slice_b(const BMember *__restrict__ M,
                                                    const int *__restrict__ tab, int c)
{
    int loc;
    const BMember &m = M[find_member(tab, blockIdx.x, loc)];
    int q0, nq;
    chunk_of(m, c, q0, nq);
    const i64 row = (i64)loc * (256 / LPR) + threadIdx.x / LPR;
    if (row >= (i64)nq * m.nao)      // whole rows of lanes leave together
        return;
    slice_row_wave<LPR>(m.B + (i64)q0 * m.npos, m.npos, m.nao, 1, m.nao, m.nao, m.nao, m.kp / kSliceKB,
                        m.Bp, m.bps, m.bkb, m.eB, row);
}

// The chunk's packed slabs (jk.h JK_B_PACKED), bands of kBand rows; the
// dynamic LDS covers the largest member's band.
template <int NJ>
__global__ void __launch_bounds__(256) k_bm_slice_b_packed(const BMember *__restrict__ M,
                                                           const int *__restrict__ tab, int c)
{
    extern __shared__ double T[];
    int loc;
    const BMember &m = M[find_member(tab, blockIdx.x, loc)];
    int q0, nq;
    chunk_of(m, c, q0, nq);
    const int nband = (m.nao + kBand - 1) / kBand;
    const int b = loc / nband, m0 = (loc % nband) * kBand;
    slice_band_packed<NJ>(m.B + (i64)(q0 + b) * m.bslab, b, m0, m.nao, m.nao, m.kp / kSliceKB, m.Bp,
                          m.bps, m.bkb, m.eB, T);
}

__global__ void __launch_bounds__(256, 2) k_bm_ht(const BMember *__restrict__ M,
                                                  const int *__restrict__ tab, int c)
{
    extern __shared__ char lds[];
    int loc;
    const BMember &m = M[find_member(tab, xcd_local(blockIdx.x, gridDim.x), loc)];
    int q0, nq;
    chunk_of(m, c, q0, nq);
    const int nkey = m.sym ? m.nd : 2 * m.nd;
    ht_mixed_tile(m.Bp, m.bps, m.bkb, m.eB, m.Cp, m.cps, m.ckb, m.eC, m.XY, nq * m.nao, nkey * m.r,
                  m.cpx, m.kp / kSliceKB, loc, lds, m.pm, m.rows, m.r, pm_slots(m.r, nkey));
}

// Row maxima from the half-transform's partial ones: tile loc of a
// member is (row block loc % nmb, key loc / nmb), 64 rows, four waves.
__global__ void __launch_bounds__(256) k_bm_rowmax(const BMember *__restrict__ M,
                                                   const int *__restrict__ tab, int c)
{
    __shared__ uint32_t red[4][64];
    int loc;
    const BMember &m = M[find_member(tab, blockIdx.x, loc)];
    int q0, nq;
    chunk_of(m, c, q0, nq);
    const int nkey = m.sym ? m.nd : 2 * m.nd, nmb = (m.nao + 63) / 64;
    rowmax_pm_block(m.pm, m.nao, nq, m.rows, m.mp, pm_slots(m.r, nkey), nkey, m.r, m.mx, loc % nmb,
                    loc / nmb, 0, 1, red);
}

__global__ void __launch_bounds__(256) k_bm_slice_xy(const BMember *__restrict__ M,
                                                     const int *__restrict__ tab, int c)
{
    int loc;
    const BMember &m = M[find_member(tab, blockIdx.x, loc)];
    int q0, nq;
    chunk_of(m, c, q0, nq);
    const int nkey = m.sym ? m.nd : 2 * m.nd;
    const int ngroup = cdiv_i((i64)nkey * m.mp, 32);
    const int row = (loc % ngroup) * 32 + (threadIdx.x >> 3);
    if (row >= nkey * m.mp)
        return;
    slice_xy_block(m.XY, m.nao, nkey, m.r, m.mp, nq * m.r, m.XYp, m.xps, m.xkb, m.mx, 1, m.eXY, row,
                   threadIdx.x & 7, loc / ngroup);
}

__global__ void __launch_bounds__(256, 2) k_bm_ex(const BMember *__restrict__ M,
                                               const int *__restrict__ tab, int c)
{
    extern __shared__ char lds[];
    int loc;
    const BMember &m = M[find_member(tab, xcd_local(blockIdx.x, gridDim.x), loc)];
    int q0, nq;
    chunk_of(m, c, q0, nq);
    const int nkb = cdiv_i((i64)nq * m.r, kSliceKB);
    const int kbl = cdiv_i(nkb, m.nsplit);
    const int8_t *Xp = m.XYp, *Yp = m.sym ? Xp : m.XYp + (i64)m.nd * m.mp * kSliceKB;
    const int *eX = m.eXY, *eY = m.sym ? eX : m.eXY + (i64)m.nd * m.mp;
    ex_mixed_tile(Xp, Yp, m.xps, m.xkb, eX, eY, m.nsplit > 1 ? m.Kp : m.K, m.nao, m.nd, m.mp, nkb,
                  kbl, c > 0, m.sym, 1.0, loc, lds);
}

// ------------------------------------------------------------------ launchers
int mixed_nslice() { return kNS; }
int mixed_row_pad() { return kRowPad; }
i64 mixed_b_rows(i64 nrow) { return (nrow + kMhM - 1) / kMhM * kMhM + kMhM; }
int mixed_col_pad() { return kMhN; }
int mixed_k_pad() { return kKPad; }
int mixed_k_block() { return kSliceKB; }

hipError_t launch_slice_rows(const double *src, i64 bs, i64 rs, i64 ks, int nb, int nr, int nk,
                             int rp, int nkb, int8_t *out, i64 pstride, i64 kbstride, int *exps,
                             hipStream_t s)
{
    {
        ProfScope ps_("slice_rows", s);
        hipLaunchKernelGGL(k_slice_rows, dim3(cdiv((i64)nb * rp, 32)), dim3(256), 0, s, src, bs, rs,
                           ks, nb, nr, nk, rp, nkb, out, pstride, kbstride, exps);
    }
    return hipGetLastError();
}

hipError_t launch_slice_b(const double *src, i64 bs, i64 rs, int nb, int nr, int nk, int rp, int nkb,
                          int8_t *out, i64 pstride, i64 kbstride, int *exps, hipStream_t s)
{
    const int lanes = slice_lanes(nkb);
    if (lanes == 0)     // long rows: generic two-pass slicer
        return launch_slice_rows(src, bs, rs, 1, nb, nr, nk, rp, nkb, out, pstride, kbstride, exps, s);
    const dim3 g(cdiv((i64)nb * rp, 256 / lanes));
    {
        ProfScope ps_("slice_b", s);
        auto go = [&](auto k) {
            hipLaunchKernelGGL(k, g, dim3(256), 0, s, src, bs, rs, nb, nr, nk, rp, nkb, out, pstride,
                               kbstride, exps);
        };
        if (lanes == 8)
            go(k_slice_rows_wave<8>);
        else if (lanes == 16)
            go(k_slice_rows_wave<16>);
        else if (lanes == 32)
            go(k_slice_rows_wave<32>);
        else
            go(k_slice_rows_wave<64>);
    }
    return hipGetLastError();
}
hipError_t launch_slice_c(const double *Cc, int R2, int nao, int cp, int nkb, int8_t *out, i64 pstride,
                          i64 kbstride, int *exps, hipStream_t s)
{
    if (slice_lanes(nkb) == 0)
        return launch_slice_rows(Cc, 0, 1, R2, 1, R2, nao, cp, nkb, out, pstride, kbstride, exps, s);
    {
        ProfScope ps_("slice_rows", s);
        hipLaunchKernelGGL(k_slice_cols, dim3(cdiv(cp, 4)), dim3(256), 0, s, Cc, R2, R2, nao, cp, nkb, out,
                           pstride, kbstride, exps);
    }
    return hipGetLastError();
}
int mixed_slice_lanes(int kp) { return slice_lanes(kp / kSliceKB); }

// Dynamic LDS above 64 KB needs a per-kernel attribute, set once per
// (kernel, device).
static hipError_t set_lds(const void *fn, int bytes)
{
    static std::mutex mu;
    static std::set<std::pair<const void *, int>> done;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess)
        return e;
    std::lock_guard<std::mutex> lk(mu);
    if (done.count({fn, dev}))
        return hipSuccess;
    e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
    if (e == hipSuccess)
        done.insert({fn, dev});
    return e;
}

hipError_t launch_slice_b_packed(const double *src, i64 bs, int nb, int nao, int rp, int nkb,
                                 int8_t *out, i64 pstride, i64 kbstride, int *exps, hipStream_t s)
{
    const int nj = cdiv(nkb, 8);
    if (nj > 8 || nao > rp)
        return hipErrorInvalidValue;        // rows beyond 2048 elements: not supported packed
    const dim3 g((unsigned)((i64)nb * cdiv(rp, kBand)));
    const size_t lds = sizeof(double) * kBand * nao;
    if (lds > 65536) {        // above 64 KB of dynamic LDS: per-kernel attribute
        const void *fn = nj <= 1   ? (const void *)k_slice_band_packed<1>
                         : nj <= 2 ? (const void *)k_slice_band_packed<2>
                         : nj <= 4 ? (const void *)k_slice_band_packed<4>
                                   : (const void *)k_slice_band_packed<8>;
        hipError_t e = set_lds(fn, (int)(sizeof(double) * kBand * 2048));
        if (e != hipSuccess)
            return e;
    }
    {
        ProfScope ps_("slice_b_packed", s);
        if (nj <= 1)
            hipLaunchKernelGGL(k_slice_band_packed<1>, g, dim3(256), lds, s, src, bs, nb, nao, rp,
                               nkb, out, pstride, kbstride, exps);
        else if (nj <= 2)
            hipLaunchKernelGGL(k_slice_band_packed<2>, g, dim3(256), lds, s, src, bs, nb, nao, rp,
                               nkb, out, pstride, kbstride, exps);
        else if (nj <= 4)
            hipLaunchKernelGGL(k_slice_band_packed<4>, g, dim3(256), lds, s, src, bs, nb, nao, rp,
                               nkb, out, pstride, kbstride, exps);
        else
            hipLaunchKernelGGL(k_slice_band_packed<8>, g, dim3(256), lds, s, src, bs, nb, nao, rp,
                               nkb, out, pstride, kbstride, exps);
    }
    return hipGetLastError();
}

// Packed slicer: rows of at most 2048 elements (and a band of 8 rows of
// LDS, 128 KB at that size).
int mixed_packed_ok(int nao, int kp) { return cdiv(kp / kSliceKB, 8) <= 8 && nao <= kp; }

int mixed_rowmax_ok(int R2) { return R2 <= 8192; }

hipError_t launch_slice_xy(const double *XY, int nao, int nkey, int r, int mp, int nj, int nkb,
                           int8_t *out, i64 pstride, i64 kbstride, const uint32_t *mx, int nsp,
                           int *exps, hipStream_t s)
{
    {
        ProfScope ps_("slice_xy", s);
        hipLaunchKernelGGL(k_slice_xy, dim3(cdiv((i64)nkey * mp, 32), nkb < 65535 ? nkb : 65535),
                           dim3(256), 0, s, XY, nao, nkey, r, mp, nj, out, pstride, kbstride, mx, nsp,
                           exps, nkb);
    }
    return hipGetLastError();
}

size_t xy_rowmax_pm_words(i64 rows, int cp, int r, int nkey)
{
    return (size_t)(cp / kMhN) * pm_slots(r, nkey) * rows;
}

hipError_t launch_ht_mixed(const int8_t *Bp, i64 bpstride, i64 bkbstride, const int *eB,
                           const int8_t *Cp, i64 cpstride, i64 ckbstride, const int *eC, double *XY,
                           int nao, int R2, int nq, int cp, int nkb, uint32_t *pm, i64 rows, int r,
                           hipStream_t s)
{
    hipError_t e = set_lds((const void *)k_ht_mixed, kLdsBytes);
    if (e != hipSuccess)
        return e;
    {
        ProfScope ps_("ht_mixed", s);
        hipLaunchKernelGGL(k_ht_mixed, dim3(mixed_ht_tiles(nq * nao, cp)), dim3(TileV::NTHR), kLdsBytes, s,
                           Bp, bpstride, bkbstride, eB, Cp, cpstride, ckbstride, eC, XY, nq * nao, R2, cp,
                           nkb, pm, (int)rows, r, pm_slots(r, R2 / r));
    }
    return hipGetLastError();
}

// Splits of the row maxima's slabs: the row blocks and keys alone leave a
// device of 256 CUs idle.
int xy_rowmax_splits(int nao, int nkey, int nq)
{
    const int n = 512 / (cdiv(nao, 64) * nkey), most = nq / 16;
    return std::max(1, std::min(std::min(n, most), 8));
}

hipError_t launch_xy_rowmax_pm(const uint32_t *pm, int nao, int nq, int nkey, int r, i64 rows, int mpe,
                               uint32_t *mx, int nsp, hipStream_t s)
{
    {
        ProfScope ps_("xy_rowmax_pm", s);
        hipLaunchKernelGGL(k_xy_rowmax_pm, dim3(cdiv(nao, 64), nkey, nsp), dim3(256), 0, s, pm, nao, nq,
                           (int)rows, mpe, pm_slots(r, nkey), r, mx);
    }
    return hipGetLastError();
}

int mixed_max_depth() { return kSliceMaxDepth; }

int ex_mixed_nsplit(int mp, int nd, int nkb, int sym)
{
    const int tiles = nd * ex_pairs(mp / 64, sym);
    int maxs = nkb / 16 > 1 ? nkb / 16 : 1;
    if (maxs > 16)
        maxs = 16;
    const int s = pick_split_slots(tiles, maxs, device_slots());
    // exact int32 level sums: a split of cdiv(nkb, s) inner blocks may hold at
    // most kSliceMaxDepth inner indices
    const int need = cdiv(nkb, kSliceMaxDepth / kSliceKB);
    return s > need ? s : need;
}

hipError_t launch_ex_mixed(const int8_t *Xp, const int8_t *Yp, i64 pstride, i64 kbstride,
                           const int *eX, const int *eY, double *Kp, int nao, int nd, int mp, int nkb,
                           int nsplit, int accumulate, hipStream_t s, int sym, double scale)
{
    hipError_t e = set_lds((const void *)k_ex_mixed, kLdsBytes);
    if (e != hipSuccess)
        return e;
    const int kbl = cdiv(nkb, nsplit);
    {
        ProfScope ps_("ex_mixed", s);
        hipLaunchKernelGGL(k_ex_mixed, dim3(mixed_ex_tiles(mp, nd, nsplit, sym)), dim3(TileV::NTHR),
                           kLdsBytes, s, Xp, Yp, pstride, kbstride, eX, eY, Kp, nao, nd, mp, nkb, kbl,
                           accumulate, sym, scale);
    }
    return hipGetLastError();
}

// Dynamic LDS of the batched mixed kernels above 64 KB, set once per device
// before a launch sequence is captured.
hipError_t prepare_batched_mixed_kernels()
{
    hipError_t e = set_lds((const void *)k_bm_ht, kLdsBytes);
    if (e == hipSuccess)
        e = set_lds((const void *)k_bm_ex, kLdsBytes);
    // the packed slicer's band of the longest rows the packed path takes
    const int band = (int)sizeof(double) * kBand * 2048;
    if (e == hipSuccess)
        e = set_lds((const void *)k_bm_slice_b_packed<1>, band);
    if (e == hipSuccess)
        e = set_lds((const void *)k_bm_slice_b_packed<2>, band);
    if (e == hipSuccess)
        e = set_lds((const void *)k_bm_slice_b_packed<4>, band);
    if (e == hipSuccess)
        e = set_lds((const void *)k_bm_slice_b_packed<8>, band);
    return e;
}

hipError_t launch_batched_mixed_phase(int phase, const BMember *M, const int *tab, int ntiles,
                                      int step, hipStream_t s, int arg)
{
    const dim3 g(ntiles);
    switch (phase) {
    case kPhaseMSliceC: {
        ProfScope ps_("bm_slice_c", s);
        hipLaunchKernelGGL(k_bm_slice_c, g, dim3(256), 0, s, M, tab);
        break;
    }
    case kPhaseMSliceB: {
        ProfScope ps_("bm_slice_b", s);
        if (arg == 8)
            hipLaunchKernelGGL(k_bm_slice_b<8>, g, dim3(256), 0, s, M, tab, step);
        else if (arg == 16)
            hipLaunchKernelGGL(k_bm_slice_b<16>, g, dim3(256), 0, s, M, tab, step);
        else if (arg == 32)
            hipLaunchKernelGGL(k_bm_slice_b<32>, g, dim3(256), 0, s, M, tab, step);
        else if (arg == 64)
            hipLaunchKernelGGL(k_bm_slice_b<64>, g, dim3(256), 0, s, M, tab, step);
        else
            return hipErrorInvalidValue;
        break;
    }
    case kPhaseMSliceBPacked: {
        // arg = 16 x (dynamic LDS bytes) + register blocks
        const int nj = arg & 15;
        const size_t lds = (size_t)(arg >> 4);
        if (lds > sizeof(double) * kBand * 2048)
            return hipErrorInvalidValue;
        ProfScope ps_("bm_slice_b_packed", s);
        if (nj <= 1)
            hipLaunchKernelGGL(k_bm_slice_b_packed<1>, g, dim3(256), lds, s, M, tab, step);
        else if (nj <= 2)
            hipLaunchKernelGGL(k_bm_slice_b_packed<2>, g, dim3(256), lds, s, M, tab, step);
        else if (nj <= 4)
            hipLaunchKernelGGL(k_bm_slice_b_packed<4>, g, dim3(256), lds, s, M, tab, step);
        else if (nj <= 8)
            hipLaunchKernelGGL(k_bm_slice_b_packed<8>, g, dim3(256), lds, s, M, tab, step);
        else
            return hipErrorInvalidValue;
        break;
    }
    case kPhaseMHalf: {
        ProfScope ps_("bm_ht_mixed", s);
        hipLaunchKernelGGL(k_bm_ht, g, dim3(TileV::NTHR), kLdsBytes, s, M, tab, step);
        break;
    }
    case kPhaseMRowmax: {
        ProfScope ps_("bm_xy_rowmax", s);
        hipLaunchKernelGGL(k_bm_rowmax, g, dim3(256), 0, s, M, tab, step);
        break;
    }
    case kPhaseMSliceXY: {
        ProfScope ps_("bm_slice_xy", s);
        hipLaunchKernelGGL(k_bm_slice_xy, g, dim3(256), 0, s, M, tab, step);
        break;
    }
    case kPhaseMExchange: {
        ProfScope ps_("bm_ex_mixed", s);
        hipLaunchKernelGGL(k_bm_ex, g, dim3(TileV::NTHR), kLdsBytes, s, M, tab, step);
        break;
    }
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Tile counts of the batched mixed phases for one member (host).
int mixed_ht_tiles(int nrow, int cpx) { return cdiv(nrow, kMhM) * (cpx / kMhN); }
int mixed_ex_tiles(int mp, int nd, int nsplit, int sym) { return nsplit * nd * ex_pairs(mp / 64, sym); }

} // namespace jk
