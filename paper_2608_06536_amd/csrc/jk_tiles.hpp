// jk_tiles.hpp -- one workgroup's share of each FP64 build phase.
//
// Every phase of the build is a set of independent tiles; these device
// functions compute one tile.  The single-problem kernels (jk_fp64.hip) run
// tile blockIdx.x of one problem; the batched kernels (jk_batched.hip) map
// blockIdx.x to (problem, tile) through a table and run the same function, so
// a member of a batch is computed exactly as it would be alone.
//
// Phases (Sec. 2.3, Eq. (4), half-transform form K = B_V^T B_U):
//   pack          Cc[n][c]       = [C_L | C_R] as one nao x 2R matrix
//   gamma, J      coulomb_upper.hpp
//   reduce        g[k][Q]        = sum of gamma's partials in fixed order
//   half-transform X^Q, Y^Q      = B^Q [C_L | C_R]            (per Q-chunk)
//   exchange      K_k           += sum_{Q in chunk} X^Q_k (Y^Q_k)^T
//   sum splits    K              = sum of the split partials in fixed order
// Chunk workspace: X_ws[k][m][ql*r + i], Y_ws likewise, so each exchange
// operand row is contiguous over the chunk's inner index (Q, i).
#pragma once
#include "f64_core.hpp"
#include "f64_mfma16.hpp"

namespace jk {

// Tile shapes of the 4x4x4 engine: the half-transform uses 128 x 64 workgroup
// tiles of four 64 x 32 wave tiles (two workgroups per CU); the exchange
// product 128 x 64 tiles of eight 64 x 16 wave tiles (four waves per SIMD);
// the density 64 x 64.  Element-wise phases take 1024 elements per tile.
constexpr int kHtM = 128, kHtN = 64;
constexpr int kExM = 128, kExN = 64;
constexpr int kElemTile = 1024;
typedef Tile<kHtM, kHtN, 64, 32, 16> TileHalf;
typedef Tile<kExM, kExN, 64, 16, 16> TileExch;
typedef Tile<64, 64, 32, 32, 16> TileDensity;
// The half-transform's second tile shape (a plan choice, jk_tune.h): 64 x 64,
// four workgroups per CU; wins at small nao where 128-row tiles waste rows.
typedef Tile<64, 64, 32, 32, 16> TileHalf64;
// The half-transform on the 16 x 16 x 4 engine (jk_tune.h tile 4): shape by
// ht_shape over stacked slabs, packed slabs 64 x 64 tiles per slab; narrower
// columns where ht_cols says so.
typedef ShapeTile<kS64x64>::type TileHalf16;

// Shape of the half-transform over stacked slabs (the rows are one matrix, so
// neither shape pads them): 64 x 64, four workgroups per CU, where the inner
// loop of nao indices is too short to cover a workgroup's first loads and
// output with two others (nao 150: 119 us against 132, 208: 313 against 319),
// 128 x 64 beyond, whose wave tiles read less per product (374: 3.08 ms against
// 3.13, 500: 10.1 against 10.3).
inline int ht_shape(int nao) { return nao <= 256 ? kS64x64 : kS128x64; }
// Narrow column tiles, the four waves on top of each other: 128 rows over stacked
// slabs, 64 of a packed slab.
template <int BN>
struct HtNarrow {
    typedef Tile16<128, BN, 32, BN, 16> flat;
    typedef Tile16<64, BN, 16, BN, 16> packed;
};
// Columns of the half-transform's tiles for ncol factor columns: the least padded
// columns over the rate of a width, 64 unless another is 3% better (a wave of a
// narrower tile reads more LDS per product).  us at nao 400, naux 1000, by width
// 64 / 48 / 32 / 16: 16 columns 352 / 300 / 275 / 269 (packed slabs 413 / 329 /
// 241 / 216), 48 columns 362 / 318 / 379 / 375 (431 / 348 / 458 / 459), 96
// columns 657 / 527 / 541 / 620 (823 / 650 / 678 / 837), 112 columns 663 / 751 /
// 721 / 728, 160 columns 973 / 995 / 891 / 1009.
inline int ht_cols(int ncol, bool packed)
{
    const int width[4] = {64, 48, 32, 16};
    const double rate[2][4] = {{1.0, 0.92, 0.9, 0.78}, {1.0, 0.97, 0.91, 0.6}};
    auto cost = [&](int i) { return (ncol + width[i] - 1) / width[i] * width[i] / rate[packed][i]; };
    int best = 0;
    for (int i = 1; i < 4; i++)
        if (cost(i) < 0.97 * cost(0) && cost(i) < cost(best))
            best = i;
    return width[best];
}

__host__ __device__ inline int cdiv_i(i64 a, i64 b) { return (int)((a + b - 1) / b); }

// ------------------------------------------------------------------ packed slabs
// A symmetric slab stored as its upper triangle, row by row: element (m, n),
// m <= n, at pk_row(m) + (n - m), pk_row(m) = m nao - m (m - 1) / 2;
// nao (nao + 1) / 2 doubles per slab.
__host__ __device__ inline i64 pk_size(int nao) { return (i64)nao * (nao + 1) / 2; }
__host__ __device__ inline i64 pk_row(int m, int nao) { return (i64)m * (2 * (i64)nao - m + 1) / 2; }
__host__ __device__ inline i64 pk_index(int m, int n, int nao)
{
    const int a = m < n ? m : n, b = m < n ? n : m;
    return pk_row(a, nao) + (b - a);
}

// element (i, k) of a packed symmetric nao x nao slab, as an A operand of the
// tile engine (both indices clamped for the load, zero outside).  Measured:
// the row-major thread mapping already coalesces below the diagonal (sixteen
// consecutive rows of one column are 128 contiguous bytes), and a per-stage
// column mapping there was no faster.
struct OpPackedSym {
    static constexpr bool kContig = true;
    static constexpr int NRAW = 1;
    const double *p;
    int nao;
    __device__ __forceinline__ void fetch(int i, int k, double *raw) const
    {
        const int ic = i < nao ? i : nao - 1, kc = k < nao ? k : nao - 1;
        raw[0] = p[pk_index(ic, kc, nao)];
    }
    __device__ __forceinline__ double finish(int i, int k, const double *raw) const
    {
        return (i < nao && k < nao) ? raw[0] : 0.0;
    }
};


// ------------------------------------------------------------------ tile counts
__host__ __device__ inline int pack_tiles(int nao, int nd, int r)
{
    return cdiv_i((i64)nao * 2 * nd * r, kElemTile);
}
__host__ __device__ inline int reduce_tiles(int naux, int ndp) { return cdiv_i((i64)naux * ndp, 64); }
__host__ __device__ inline int ht_tiles(int nao, int nd, int r, int nq)
{
    return nq * cdiv_i(nao, kHtM) * cdiv_i(2 * (i64)nd * r, kHtN);
}
__host__ __device__ inline int ht64_tiles(int nao, int nd, int r, int nq)
{
    return nq * cdiv_i(nao, 64) * cdiv_i(2 * (i64)nd * r, 64);
}
// ncol = 2R (X and Y) or R (X only, symmetric densities)
__host__ __device__ inline int ht_tiles_cols(int nao, int ncol, int nq)
{
    return nq * cdiv_i(nao, kHtM) * cdiv_i(ncol, kHtN);
}
// Symmetric exchange (C_L = C_R, K = sum X X^T): only the tiles of bm x bn
// that reach the upper triangle n >= m, row tile mb from column tile
// (mb bm) / bn on.
__host__ __device__ inline int ex_tri_first(int mb, int bm, int bn) { return (mb * bm) / bn; }
__host__ __device__ inline int ex_tri_tiles(int nao, int bm, int bn)
{
    const int nmt = cdiv_i(nao, bm), nnt = cdiv_i(nao, bn);
    int n = 0;
    for (int mb = 0; mb < nmt; mb++) {
        const int f = ex_tri_first(mb, bm, bn);
        n += f < nnt ? nnt - f : 0;
    }
    return n;
}
// tiles of one density's K
__host__ __device__ inline int ex_tiles(int nao, int bm, int bn, int sym)
{
    return sym ? ex_tri_tiles(nao, bm, bn) : cdiv_i(nao, bm) * cdiv_i(nao, bn);
}
__host__ __device__ inline void ex_tri_coords(int t, int nao, int bm, int bn, int &mb, int &nb)
{
    const int nmt = cdiv_i(nao, bm), nnt = cdiv_i(nao, bn);
    for (mb = 0; mb < nmt; mb++) {
        const int f = ex_tri_first(mb, bm, bn);
        const int cnt = f < nnt ? nnt - f : 0;
        if (t < cnt) {
            nb = f + t;
            return;
        }
        t -= cnt;
    }
    mb = nmt - 1;
    nb = nnt - 1;
}
// Elements per workgroup of the split sums: 64, one per lane of each of four
// waves.
constexpr int kSumTile = 64;
__host__ __device__ inline int sum_tiles(i64 n) { return cdiv_i(n, kSumTile); }

// Kk[m][n] = Kk[n][m] for m > n in lower-triangle block b of 32 x 32 (blocks
// (bi, bj), bi >= bj, numbered row by row): fills the lower triangle from the
// upper one through an LDS transpose.  256 threads; t is 32 x 33 doubles.
__device__ __forceinline__ void mirror_tile(double *__restrict__ Kk, int nao, int b,
                                            double (*t)[33])
{
    int bi = 0;
    while (b > bi) {
        b -= bi + 1;
        bi++;
    }
    const int bj = b;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int y = ty; y < 32; y += 8) {
        const int row = bj * 32 + y, col = bi * 32 + tx;       // upper source
        if (row < nao && col < nao)
            t[y][tx] = Kk[(i64)row * nao + col];
    }
    __syncthreads();
    for (int y = ty; y < 32; y += 8) {
        const int m = bi * 32 + y, n = bj * 32 + tx;           // lower target
        if (m < nao && n < nao && m > n)
            Kk[(i64)m * nao + n] = t[tx][y];
    }
    __syncthreads();
}

__host__ __device__ inline int mirror_blocks(int nao)
{
    const int nb = cdiv_i(nao, 32);
    return nb * (nb + 1) / 2;
}

// ------------------------------------------------------------------ pack
__device__ inline void pack_tile(const double *__restrict__ CL, const double *__restrict__ CR,
                                 double *__restrict__ Cc, int nao, int nd, int r, int tile)
{
    const int R = nd * r, R2 = 2 * R;
    const i64 total = (i64)nao * R2;
    for (int u = 0; u < kElemTile / 256; u++) {
        const i64 e = (i64)tile * kElemTile + u * 256 + threadIdx.x;
        if (e < total) {
            const int n = (int)(e / R2), c = (int)(e % R2);
            const double *src = c < R ? CL : CR;
            const int cc = c < R ? c : c - R;
            const int k = cc / r, i = cc % r;
            Cc[e] = src[((i64)k * nao + n) * r + i];
        }
    }
}

// ------------------------------------------------------------------ reduce
// g[k][Q] = sum_{pb} part[pb][Q][k] in a fixed order.  A tile covers 64
// consecutive entries (Q, k) of one partial block; wave w of the four sums
// the blocks pb = w, w + 4, ... (coalesced 512-byte reads), and the four wave
// sums are added in wave order.
// Its share of the partials pb = w, w + 4, ...
__device__ __forceinline__ double reduce_part(const double *__restrict__ src, i64 total, int npb, int w)
{
    double s = 0.0;
    int pb = w;
    for (; pb + 12 < npb; pb += 16) {
        const double v0 = src[(i64)pb * total], v1 = src[(i64)(pb + 4) * total];
        const double v2 = src[(i64)(pb + 8) * total], v3 = src[(i64)(pb + 12) * total];
        s += v0;
        s += v1;
        s += v2;
        s += v3;
    }
    for (; pb < npb; pb += 4)
        s += src[(i64)pb * total];
    return s;
}
__device__ inline void reduce_tile(const double *__restrict__ part, double *__restrict__ g, int naux,
                                   int nd, int ndp, int npb, int tile)
{
    __shared__ double red[4][64];
    const i64 total = (i64)naux * ndp;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const i64 e = (i64)tile * 64 + lane;
    red[w][lane] = e < total ? reduce_part(part + e, total, npb, w) : 0.0;
    __syncthreads();
    if (w == 0 && e < total) {
        const int q = (int)(e / ndp), k = (int)(e % ndp);
        if (k < nd)
            g[(i64)k * naux + q] = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
    }
}

// ------------------------------------------------------------------ half-transform
// For slab Q = q0 + ql (ql < nq): XY[m][c] = sum_n B^Q[m][n] Cc[n][c], written
// as X_ws[k][m][ql*r + i] (c = k*r + i < R) or Y_ws[k][m][ql*r + i] (c - R),
// for the first ncol columns c (2R, or R when only X is needed).
// PACKED: B holds packed slabs (pk_size(nao) doubles each).
template <bool PACKED = false>
__device__ inline void ht_tile(const double *__restrict__ B, const double *__restrict__ Cc,
                               double *__restrict__ Xw, double *__restrict__ Yw, int nao, int nd,
                               int r, int q0, int ldw, int tile, double *lds, int ncol = -1)
{
    typedef TileHalf TL;
    const int R = nd * r, R2 = 2 * R;
    const int nc = ncol < 0 ? R2 : ncol;
    const int nmt = cdiv_i(nao, kHtM), nct = cdiv_i(nc, kHtN);
    const int ql = tile / (nmt * nct), rem = tile % (nmt * nct);
    const int mb = rem / nct, cb = rem % nct;
    const i64 n2 = PACKED ? pk_size(nao) : (i64)nao * nao;
    OpIC b{Cc, R2, nc, nao};
    Acc<TL> acc;
    acc.zero();
    if constexpr (PACKED) {
        OpPackedSym a{B + (i64)(q0 + ql) * n2, nao};
        tile_gemm<TL>(a, b, mb * kHtM, cb * kHtN, 0, nao, lds, acc);
    } else {
        OpKC a{B + (i64)(q0 + ql) * n2, nao, nao, nao};
        tile_gemm<TL>(a, b, mb * kHtM, cb * kHtN, 0, nao, lds, acc);
    }
    tile_foreach(acc, mb * kHtM, cb * kHtN, [&](int m, int c, double v) {
        if (m < nao && c < nc) {
            double *dst = c < R ? Xw : Yw;
            const int cc = c < R ? c : c - R;
            const int k = cc / r, i = cc % r;
            dst[((i64)k * nao + m) * ldw + (i64)ql * r + i] = v;
        }
    });
}

// The half-transform with an arbitrary tile shape TL of the 4x4x4 engine
// (full slabs).
template <class TL>
__device__ inline void ht_tile_tl(const double *__restrict__ B, const double *__restrict__ Cc,
                                  double *__restrict__ Xw, double *__restrict__ Yw, int nao, int nd,
                                  int r, int q0, int ldw, int tile, double *lds, int ncol)
{
    constexpr int BM = TL::BM, BN = TL::BN;
    const int R = nd * r, R2 = 2 * R;
    const int nc = ncol < 0 ? R2 : ncol;
    const int nmt = cdiv_i(nao, BM), nct = cdiv_i(nc, BN);
    const int ql = tile / (nmt * nct), rem = tile % (nmt * nct);
    const int mb = rem / nct, cb = rem % nct;
    const i64 n2 = (i64)nao * nao;
    OpKC a{B + (i64)(q0 + ql) * n2, nao, nao, nao};
    OpIC b{Cc, R2, nc, nao};
    auto out = [&](int m, int c, double v) {
        if (m < nao && c < nc) {
            double *dst = c < R ? Xw : Yw;
            const int cc = c < R ? c : c - R;
            const int k = cc / r, i = cc % r;
            dst[((i64)k * nao + m) * ldw + (i64)ql * r + i] = v;
        }
    };
    Acc<TL> acc;
    acc.zero();
    tile_gemm<TL>(a, b, mb * BM, cb * BN, 0, nao, lds, acc);
    tile_foreach(acc, mb * BM, cb * BN, out);
}

// The half-transform of the chunk's nq slabs as one product: the slabs,
// stacked, are an (nq nao) x nao matrix, so tile rows run across slab
// boundaries and no rows are padded per slab.  Row t of the stack is row
// t % nao of slab q0 + t / nao.  TL is a tile of the 16 x 16 x 4 engine; the
// chunk's slabs must span less than 4 GiB (buf_extent_ok).
template <class TL>
__host__ __device__ inline int ht_flat_tiles(int nao, int ncol, int nq)
{
    return cdiv_i((i64)nq * nao, TL::BM) * cdiv_i(ncol, TL::BN);
}
template <class TL>
__device__ inline void ht_tile_flat(const double *__restrict__ B, const double *__restrict__ Cc,
                                    double *__restrict__ Xw, double *__restrict__ Yw, int nao,
                                    int nd, int r, int q0, int nq, int ldw, int tile, double *lds,
                                    int ncol)
{
    constexpr int BM = TL::BM, BN = TL::BN;
    const int R = nd * r, R2 = 2 * R;
    const int nc = ncol < 0 ? R2 : ncol;
    const int rows = nq * nao;
    const int nct = cdiv_i(nc, BN);
    const int mb = tile / nct, cb = tile % nct;
    BufKC a{B + (i64)q0 * nao * nao, nao, rows, nao};
    BufIC b{Cc, R2, nc, nao};
    Acc16<TL> acc;
    acc.zero();
    // No inner-index masking: past row nao - 1, Cc reads zero (the end of its
    // resource), and the slab rows read there are finite data of the next row.
    if constexpr (TL::BN == 128)
        tile_gemm16<TL, false>(a, b, mb * BM, cb * BN, 0, nao, lds, acc);
    else
        Gemm16Stream<TL, BufKC, BufIC>::run(a, b, mb * BM, cb * BN, nao, lds, acc);
    // Output (t, c) goes to col(c)[row(t)]: col(c) = X_ws or Y_ws at density
    // k = c' / r, column i = c' % r (c' = c or c - R), and row(t) = m ldw +
    // ql r for t = ql nao + m.  A lane holds NB columns and 4 MA rows
    // (16 apart within 4 apart), decoded once each.
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wr = wave / TL::WCOLS, wc = wave % TL::WCOLS;
    const int rb = mb * BM + wr * TL::WM + (lane >> 4);
    const int cb0 = cb * BN + wc * TL::WN + (lane & 15);
    double *col[TL::NB];
    bool col_ok[TL::NB];
#pragma unroll
    for (int j = 0; j < TL::NB; j++) {
        const int c = cb0 + 16 * j;
        col_ok[j] = c < nc;
        const int cc = c < R ? c : c - R;
        const int k = cc / r, i = cc - k * r;
        col[j] = (c < R ? Xw : Yw) + (i64)k * nao * ldw + i;
    }
    const int ql0 = rb / nao, m0 = rb - ql0 * nao;
#pragma unroll
    for (int i = 0; i < TL::MA; i++)
#pragma unroll
        for (int v = 0; v < 4; v++) {
            const int d = 16 * i + 4 * v;
            if (rb + d < rows) {
                int m = m0 + d, ql = ql0;
                while (m >= nao) {
                    m -= nao;
                    ql++;
                }
                const i64 off = (i64)m * ldw + (i64)ql * r;
#pragma unroll
                for (int j = 0; j < TL::NB; j++)
                    if (col_ok[j])
                        col[j][off] = acc.c[i][j][v];
            }
        }
}

// The half-transform of packed slabs (jk.h JK_B_PACKED) on the 16 x 16 x 4
// engine: tiles per slab, the packed operand read in the form each stage
// allows (above, below or on the diagonal).  No inner-index mask: past row
// nao - 1, Cc reads zero and the packed reads are finite data or zero.
template <class TL>
__device__ inline void ht_tile16_packed(const double *__restrict__ B, const double *__restrict__ Cc,
                                        double *__restrict__ Xw, double *__restrict__ Yw, int nao,
                                        int nd, int r, int q0, int ldw, int tile, double *lds,
                                        int ncol)
{
    constexpr int BM = TL::BM, BN = TL::BN;
    const int R = nd * r, R2 = 2 * R;
    const int nc = ncol < 0 ? R2 : ncol;
    const int nmt = cdiv_i(nao, BM), nct = cdiv_i(nc, BN);
    const int ql = tile / (nmt * nct), rem = tile % (nmt * nct);
    const int mb = rem / nct, cb = rem % nct;
    BufPackedSym a{B + (i64)(q0 + ql) * pk_size(nao), nao};
    BufIC b{Cc, R2, nc, nao};
    Acc16<TL> acc;
    acc.zero();
    Gemm16Stream<TL, BufPackedSym, BufIC>::run(a, b, mb * BM, cb * BN, nao, lds, acc);
    tile_foreach16(acc, mb * BM, cb * BN, [&](int m, int c, double v) {
        if (m < nao && c < nc) {
            double *dst = c < R ? Xw : Yw;
            const int cc = c < R ? c : c - R;
            const int k = cc / r, i = cc - k * r;
            dst[((i64)k * nao + m) * ldw + (i64)ql * r + i] = v;
        }
    });
}

// ------------------------------------------------------------------ exchange
// Kp[s][k][m][n] (+)= sum_{j in split s} X_ws[k][m][j] Y_ws[k][n][j]; the
// inner range [0, nj) is cut into nsplit contiguous pieces of jlen.
// With sym != 0 (Yw = Xw) only the tiles reaching n >= m are computed; the
// rest of K is filled by mirroring afterwards.
// Kp[split][k] (+)= scale * (the chunk's X Y^T over the split's inner range).
template <class TL = TileExch, bool MASK = true>
__device__ inline void ex_tile(const double *__restrict__ Xw, const double *__restrict__ Yw,
                               double *__restrict__ Kp, int nao, int nd, int nj, int ldw, int jlen,
                               int accumulate, int tile, double *lds, int sym = 0,
                               double scale = 1.0)
{
    constexpr int BM = TL::BM, BN = TL::BN;
    const int nnt = cdiv_i(nao, BN);
    const int pk = ex_tiles(nao, BM, BN, sym);
    const int per = nd * pk;
    const int sp = tile / per;
    const int t = tile % per;
    const int k = t / pk, rem = t % pk;
    int mb, nb;
    if (sym) {
        ex_tri_coords(rem, nao, BM, BN, mb, nb);
    } else {
        mb = rem / nnt;
        nb = rem % nnt;
    }
    const int j0 = sp * jlen, j1 = (j0 + jlen) < nj ? (j0 + jlen) : nj;
    double *Kk = Kp + ((i64)sp * nd + k) * nao * nao;
    auto out = [&](int m, int n, double v) {
        if (m < nao && n < nao) {
            const i64 o = (i64)m * nao + n;
            Kk[o] = accumulate ? Kk[o] + scale * v : scale * v;
        }
    };
    if constexpr (TL::kMfma16) {
        // Resources end at column j1 of the last row.  MASK: inner indices
        // past j1 are zeroed in the last stage (needed unless every split
        // ends on a 16-deep stage boundary).
        BufKC a{Xw + (i64)k * nao * ldw, ldw, nao, j1};
        BufKC b{Yw + (i64)k * nao * ldw, ldw, nao, j1};
        Acc16<TL> acc;
        acc.zero();
        tile_gemm16<TL, MASK>(a, b, mb * BM, nb * BN, j0, j1, lds, acc);
        tile_update16(acc, mb * BM, nb * BN, Kk, nao, nao, nao, accumulate, scale);
    } else {
        OpKC a{Xw + (i64)k * nao * ldw, ldw, nao, j1};
        OpKC b{Yw + (i64)k * nao * ldw, ldw, nao, j1};
        Acc<TL> acc;
        acc.zero();
        tile_gemm<TL>(a, b, mb * BM, nb * BN, j0, j1, lds, acc);
        tile_foreach(acc, mb * BM, nb * BN, out);
    }
}

// The sum over the splits of one element, in four interleaved partial sums
// (splits w, w + 4, ... for w < 4) added in order: the same arithmetic whether
// one thread or four form them.
__device__ __forceinline__ double sum_part(const double *__restrict__ p, i64 n, int nsplit, int w)
{
    double s = 0.0;
    int sp = w;
    for (; sp + 12 < nsplit; sp += 16) {
        const double v0 = p[(i64)sp * n], v1 = p[(i64)(sp + 4) * n];
        const double v2 = p[(i64)(sp + 8) * n], v3 = p[(i64)(sp + 12) * n];
        s += v0;
        s += v1;
        s += v2;
        s += v3;
    }
    for (; sp < nsplit; sp += 4)
        s += p[(i64)sp * n];
    return s;
}

// out[e] = sum_{s < nsplit} part[s * n + e] for the 64 elements of one tile,
// wave w of the four taking the splits w, w + 4, ...
__device__ inline void sum_tile(const double *__restrict__ part, double *__restrict__ out, i64 n,
                                int nsplit, int tile)
{
    __shared__ double red[4][kSumTile];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const i64 e = (i64)tile * kSumTile + lane;
    red[w][lane] = e < n ? sum_part(part + e, n, nsplit, w) : 0.0;
    __syncthreads();
    if (w == 0 && e < n)
        out[e] = ((red[0][lane] + red[1][lane]) + red[2][lane]) + red[3][lane];
}

// The same for symmetric K_k whose partials hold the upper triangle only:
// block b of 16 x 16 (blocks (bi, bj), bi <= bj, numbered row by row from the
// diagonal) is summed and written at (m, n) and (n, m).
constexpr int kSymBlk = 16;
__host__ __device__ inline int sum_sym_blocks(int nao)
{
    const int nb = cdiv_i(nao, kSymBlk);
    return nb * (nb + 1) / 2;
}
__device__ inline void sum_sym_tile(const double *__restrict__ part, double *__restrict__ out,
                                    int nao, i64 n, int nsplit, int b)
{
    __shared__ double T[kSymBlk][kSymBlk + 1];
    const int nb = cdiv_i(nao, kSymBlk);
    int bi = 0;
    while (b >= nb - bi) {
        b -= nb - bi;
        bi++;
    }
    const int bj = bi + b;
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int m = bi * kSymBlk + ty, c = bj * kSymBlk + tx;
    if (m < nao && c < nao && m <= c) {
        const double *p = part + (i64)m * nao + c;
        double s[4];
#pragma unroll
        for (int w = 0; w < 4; w++)
            s[w] = sum_part(p, n, nsplit, w);
        const double v = ((s[0] + s[1]) + s[2]) + s[3];
        out[(i64)m * nao + c] = v;
        T[ty][tx] = v;
    }
    __syncthreads();
    const int r = bj * kSymBlk + ty, q = bi * kSymBlk + tx;      // (r, q) = the mirror of (q, r)
    if (r < nao && q < nao && r > q)
        out[(i64)r * nao + q] = T[tx][ty];
}

} // namespace jk
