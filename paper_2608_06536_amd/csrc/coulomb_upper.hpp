// coulomb_upper.hpp -- the HBM streams over B (gamma, omega and J) on the
// upper triangles of the slabs, full squares and packed slabs alike.
//
// Every slab B^Q is symmetric (a precondition), so both passes run over the
// npk = nao (nao + 1) / 2 positions p of the upper triangle, numbered row by
// row (the packed order); a position is B^Q[m][n] in a full square and
// element p of a packed slab:
//
//     gamma_kQ = <B^Q, D_k> = sum_p B^Q[p] S_k[p],
//         S_k[p] = D_k[m][n] + D_k[n][m] (m < n), D_k[m][m]
//     J_k[m][n] = J_k[n][m] = sum_Q gamma_kQ B^Q[p]
//
// Both are bound by HBM (half the bytes of full squares): one element of B
// takes one multiply-add per density, on the vector units (a matrix instruction
// would spend 16 columns on nd densities).  Every sum has a fixed order that
// depends on nao and naux only.
//
// Measured, triangle bytes over time (a large copy moves 4.7 TB/s): gamma at
// nao 500, naux 2000, 8 densities 378 us, 5.3 TB/s; nao 300, naux 1200, 4: 84
// us, 5.1 TB/s (150 with partial sums per 256 slabs on the matrix cores); nao
// 48: 7 us (9).  J: 410 us, 4.9 TB/s; 108 us (140 with one workgroup per 256
// positions over all slabs); nao 48: 5.5 us (14).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "jk_tiles.hpp"

namespace jk {

// Row m and column n of position p.
__device__ __forceinline__ void pk_coords(i64 p, int nao, int &m, int &n)
{
    const double f = 2.0 * nao + 1.0;
    m = (int)((f - sqrt(f * f - 8.0 * (double)p)) * 0.5);
    m = m < 0 ? 0 : m >= nao ? nao - 1 : m;
    while (m + 1 < nao && pk_row(m + 1, nao) <= p)
        m++;
    while (pk_row(m, nao) > p)
        m--;
    n = m + (int)(p - pk_row(m, nao));
}

// ------------------------------------------------------------------ S = fold(D)
// S_k on one upper 64 x 64 tile, formed from the factors: D_k[m][n] +
// D_k[n][m] = sum_i CL[m][i] CR[n][i] + CR[m][i] CL[n][i] (halved on the
// diagonal), two products into one accumulator.
__host__ __device__ inline int fold_tiles(int nao, int nd)
{
    const int nt = cdiv_i(nao, 64);
    return nd * (nt * (nt + 1) / 2);
}
__device__ inline void fold_density_tile(const double *__restrict__ CL, const double *__restrict__ CR,
                                         double *__restrict__ S, int nao, int r, int tile, double *lds)
{
    typedef TileDensity TL;
    const int nt = cdiv_i(nao, 64), per = nt * (nt + 1) / 2;
    const int k = tile / per;
    int rem = tile % per, mb = 0;
    while (rem >= nt - mb) {
        rem -= nt - mb;
        mb++;
    }
    const int nb = mb + rem;
    OpKC l{CL + (i64)k * nao * r, r, nao, r};
    OpKC q{CR + (i64)k * nao * r, r, nao, r};
    Acc<TL> acc;
    acc.zero();
    tile_gemm<TL>(l, q, mb * 64, nb * 64, 0, r, lds, acc);
    tile_gemm<TL>(q, l, mb * 64, nb * 64, 0, r, lds, acc);
    double *Sk = S + (i64)k * pk_size(nao);
    tile_foreach(acc, mb * 64, nb * 64, [&](int m, int n, double v) {
        if (m <= n && n < nao)
            Sk[pk_row(m, nao) + (n - m)] = m == n ? 0.5 * v : v;
    });
}

// E[k][a][b] = D_k[a][b] - 2 D_k[b][a], D_k = CL_k CR_k^T (the derivative's affine
// term): two products per 64 x 64 tile, sum_i CL[a][i] CR[b][i] - 2 sum_i
// CR[a][i] CL[b][i].
__device__ inline void e_matrix_tile(const double *__restrict__ CL, const double *__restrict__ CR,
                                     double *__restrict__ E, int nao, int r, int tile, double *lds)
{
    typedef TileDensity TL;
    const int nt = cdiv_i(nao, 64);
    const int k = tile / (nt * nt), rem = tile % (nt * nt);
    const int mb = rem / nt, nb = rem % nt;
    OpKC l{CL + (i64)k * nao * r, r, nao, r};
    OpKC q{CR + (i64)k * nao * r, r, nao, r};
    Acc<TL> d, dt;
    d.zero();
    dt.zero();
    tile_gemm<TL>(l, q, mb * 64, nb * 64, 0, r, lds, d);
    tile_gemm<TL>(q, l, mb * 64, nb * 64, 0, r, lds, dt);
#pragma unroll
    for (int i = 0; i < TL::MA; i++)
#pragma unroll
        for (int j = 0; j < TL::NB; j++)
            d.c[i][j] -= 2.0 * dt.c[i][j];
    double *Ek = E + (i64)k * nao * nao;
    tile_foreach(d, mb * 64, nb * 64, [&](int m, int n, double v) {
        if (m < nao && n < nao)
            Ek[(i64)m * nao + n] = v;
    });
}

// S_k from a given matrix A_k (a cotangent, or D_k): one 32 x 32 tile pair
// (bi <= bj) through LDS, so that the tile and its mirror image are both read
// as rows.  256 threads; T is 32 x 33 doubles.
__host__ __device__ inline int sym_pack_tiles(int nao)
{
    const int nb = cdiv_i(nao, 32);
    return nb * (nb + 1) / 2;
}
__device__ inline void sym_pack_tile(const double *__restrict__ A, double *__restrict__ S, int nao,
                                     int k, int b, double (*T)[33])
{
    const int nb = cdiv_i(nao, 32);
    int bi = 0;
    while (b >= nb - bi) {
        b -= nb - bi;
        bi++;
    }
    const int bj = bi + b;
    const double *Ak = A + (i64)k * nao * nao;
    double *Sk = S + (i64)k * pk_size(nao);
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int y = ty; y < 32; y += 8) {
        const int row = bj * 32 + y, col = bi * 32 + tx;
        if (row < nao && col < nao)
            T[y][tx] = Ak[(i64)row * nao + col];
    }
    __syncthreads();
    for (int y = ty; y < 32; y += 8) {
        const int m = bi * 32 + y, n = bj * 32 + tx;
        if (m <= n && n < nao)
            Sk[pk_row(m, nao) + (n - m)] =
                m == n ? T[y][tx] : Ak[(i64)m * nao + n] + T[tx][y];
    }
}

// ------------------------------------------------------------------ gamma
// Matrices per pass over B: up to 8 in a group of the next power of two, more
// in groups of 16.
__host__ __device__ inline int pj_width(int nd)
{
    return nd > 8 ? 16 : nd > 4 ? 8 : nd > 2 ? 4 : nd;
}
__host__ __device__ inline int pj_groups(int nd) { return cdiv_i(nd, pj_width(nd)); }
// A workgroup streams blocks of 1024 positions (four per thread), summing the
// lanes slab by slab and the waves every 16 slabs; the sums of up to 128 slabs
// stay in LDS over its blocks.
constexpr int kPjPos = 1024, kPjQ = 16, kPjMaxQ = 128;
inline int pj_all_blocks(int nao) { return cdiv_i(pk_size(nao), kPjPos); }
// Blocks per workgroup: partial sums of at most 64 groups of blocks, and of at
// most 32 MB at 16 columns (one group beyond), whatever the matrices.
inline int pj_per_wg(int nao, int naux)
{
    i64 nb = ((i64)32 << 20) / ((i64)naux * 16 * 8);
    nb = nb < 1 ? 1 : nb > 64 ? 64 : nb;
    return cdiv_i(pj_all_blocks(nao), nb);
}
inline int pj_blocks(int nao, int naux)
{
    return cdiv_i(pj_all_blocks(nao), pj_per_wg(nao, naux));
}
// Slabs per workgroup, a multiple of kPjQ: about wgs workgroups, more than the
// chip holds at once but not many more, as each reads its S again.
constexpr int kPjWgs = 1536;
inline int pj_qlen(int nao, int naux, int nd, int wgs)
{
    const int nb = pj_blocks(nao, naux) * pj_groups(nd);
    const int slices = wgs / nb < 1 ? 1 : wgs / nb;
    const int len = cdiv_i(cdiv_i(naux, slices), kPjQ) * kPjQ;
    return len < kPjMaxQ ? len : kPjMaxQ;
}
// The split of one pass, worked out on the host.
struct PjGeom {
    int nbg, per, nall, nkg, qlen;
};
inline PjGeom pj_geom(int nao, int naux, int nd, int wgs = kPjWgs)
{
    return {pj_blocks(nao, naux), pj_per_wg(nao, naux), pj_all_blocks(nao), pj_groups(nd),
            pj_qlen(nao, naux, nd, wgs)};
}
inline int pj_tiles(const PjGeom &g, int naux)
{
    return g.nbg * g.nkg * cdiv_i(naux, g.qlen);
}

// x of the lane paired at step O (32, 16: the lane O away; below, the lane
// pairing within 16 that one data-parallel-primitive move gives: 8 away, mirror
// image in 8, 2 away, 1 away), so no step goes through LDS.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double x)
{
    const i64 v = __builtin_bit_cast(i64, x);
    const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(v >> 32), CTRL, 0xf, 0xf, true);
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <int O>
__device__ __forceinline__ double lane_pair_sum(double a, double b)
{
    // lanes with bit O clear: a summed over the pair, the others: b
    if constexpr (O >= 16) {
        const uint64_t x = __builtin_bit_cast(uint64_t, a), y = __builtin_bit_cast(uint64_t, b);
        unsigned l0, l1, h0, h1;
        if constexpr (O == 32) {
            const auto l = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
            const auto h = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
            l0 = l[0], l1 = l[1], h0 = h[0], h1 = h[1];
        } else {
            const auto l = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
            const auto h = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
            l0 = l[0], l1 = l[1], h0 = h[0], h1 = h[1];
        }
        return __builtin_bit_cast(double, ((uint64_t)h0 << 32) | l0) +
               __builtin_bit_cast(double, ((uint64_t)h1 << 32) | l1);
    } else {
        constexpr int ctrl = O == 8 ? 0x128 : O == 4 ? 0x141 : O == 2 ? 0x4e : 0xb1;
        const bool up = (threadIdx.x & O) != 0;
        const double keep = up ? b : a, give = up ? a : b;
        return keep + dpp_move<ctrl>(give);
    }
}
// Sums v[0 .. N) over the 64 lanes: at each step a lane adds its pair's share
// and keeps half of its values while it has several.  Lane l ends with the sum
// of value pj_owner(l) (the same tree for every N).
template <int N, int O = 32>
__device__ __forceinline__ double lane_sum(const double (&v)[N])
{
    if constexpr (O == 0) {
        return v[0];
    } else if constexpr (N == 1) {
        const double w[1] = {lane_pair_sum<O>(v[0], v[0])};
        return lane_sum<1, O / 2>(w);
    } else {
        double w[N / 2];
#pragma unroll
        for (int i = 0; i < N / 2; i++)
            w[i] = lane_pair_sum<O>(v[i], v[N / 2 + i]);
        return lane_sum<N / 2, O / 2>(w);
    }
}
template <int NK>
__device__ __forceinline__ int pj_owner(int lane)
{
    int k = 0;
#pragma unroll
    for (int o = 32, n = NK; n > 1; o >>= 1, n /= 2)
        k = k * 2 + ((lane & o) != 0 ? 1 : 0);
    return k;
}

// part[pb][Q][kg NK + k] = sum over the positions of block group pb of B^Q S_k
// for the slabs of one range: each thread keeps S_k of its four positions (256
// apart, so a wave's load is 512 contiguous bytes) in registers and streams B,
// four slabs' loads in flight; the lanes are summed per slab, the four waves
// every 16 slabs through LDS.  pj_groups(nd) x NK columns per slab.
// red: 2 x 4 x kPjQ x NK doubles, sum: kPjMaxQ x NK.
template <int NK>
__device__ __forceinline__ void project_tile(const double *__restrict__ B, const double *__restrict__ S,
                                    double *__restrict__ part, int nao, int naux, int nd, int packed,
                                    const PjGeom &geo, int tile, double (*red)[4][kPjQ][NK],
                                    double (*sum)[NK])
{
    const int nbg = geo.nbg, per = geo.per, nall = geo.nall, nkg = geo.nkg, qlen = geo.qlen;
    const int pb = tile % nbg, rest = tile / nbg;
    const int kg = rest % nkg, q0 = (rest / nkg) * qlen;
    const int q1 = (q0 + qlen) < naux ? (q0 + qlen) : naux;
    const int k0 = kg * NK;
    const i64 npk = pk_size(nao), slab = packed ? npk : (i64)nao * nao;
    const int t = threadIdx.x, wave = t >> 6, lane = t & 63;
    const int own = pj_owner<NK>(lane);
    int buf = 0;
    for (int b0 = pb * per; b0 < (pb + 1) * per && b0 < nall; b0++) {
        double s[4][NK];
        i64 off[4];
#pragma unroll
        for (int j = 0; j < 4; j++) {
            const i64 p = (i64)b0 * kPjPos + j * 256 + t;
            const bool live = p < npk;
            const i64 pc = live ? p : npk - 1;       // idle lanes: a valid address, zero weight
            if (packed) {
                off[j] = pc;
            } else {
                int m, n;
                pk_coords(pc, nao, m, n);
                off[j] = (i64)m * nao + n;
            }
#pragma unroll
            for (int k = 0; k < NK; k++)
            {                                        // columns beyond nd: a copy, not read
                const double x = S[(i64)(k0 + k < nd ? k0 + k : nd - 1) * npk + pc];
                s[j][k] = live ? x : 0.0;
            }
        }
        for (int qb = q0; qb < q1; qb += kPjQ) {
#pragma unroll 1
            for (int u0 = 0; u0 < kPjQ && qb + u0 < q1; u0 += 4) {
                double v[4][4];
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    const int q = (qb + u0 + u) < q1 ? qb + u0 + u : q1 - 1;
                    const double *b = B + (i64)q * slab;
#pragma unroll
                    for (int j = 0; j < 4; j++)
                        v[u][j] = __builtin_nontemporal_load(b + off[j]);
                }
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    double a[NK];
#pragma unroll
                    for (int k = 0; k < NK; k++) {
                        a[k] = s[0][k] * v[u][0];
#pragma unroll
                        for (int j = 1; j < 4; j++)
                            a[k] = fma(s[j][k], v[u][j], a[k]);
                    }
                    const double x = lane_sum<NK>(a);
                    if ((lane & (64 / NK - 1)) == 0)
                        red[buf][wave][u0 + u][own] = x;
                }
            }
            __syncthreads();
            // thread e always holds the same (slab, matrix) of a 16-slab block
            for (int e = t; e < kPjQ * NK; e += 256) {
                const int u = e / NK, k = e % NK;
                if (qb + u < q1) {
                    const double x =
                        ((red[buf][0][u][k] + red[buf][1][u][k]) + red[buf][2][u][k]) + red[buf][3][u][k];
                    double *d = &sum[qb - q0 + u][k];
                    *d = b0 == pb * per ? x : *d + x;
                }
            }
            buf ^= 1;                                // the next block's writes go to the other half
        }
    }
    for (int qb = q0; qb < q1; qb += kPjQ)
        for (int e = t; e < kPjQ * NK; e += 256) {
            const int u = e / NK, k = e % NK, q = qb + u;
            if (q < q1)
                part[((i64)pb * naux + q) * (nkg * NK) + k0 + k] = sum[q - q0][k];
        }
}

// ------------------------------------------------------------------ J
// A wave takes cu_runs runs of 64 positions.  Slab slices of one position, as
// a power of two: each position's slabs lie in contiguous ranges summed through
// LDS in slice order.
// From 65536 positions (nao 362) on, four runs: a wave reads 2 KB of a slab at
// a time, which the memory system takes better (nao 1000, 16 densities: 478 us
// against 542 with one run, 3.7 -> 4.2 TB/s; nao 500, 8: 217 against 236 us);
// below, one run and 8 slices, or the chip is not filled (nao 236: 42 against
// 57 us; nao 48: 7.5 against 13).
__host__ __device__ inline int cu_runs(int nao) { return pk_size(nao) > 65536 ? 4 : 1; }
__host__ __device__ inline int cu_slices_log2(int nao)
{
    if (cu_runs(nao) == 1)
        return 3;
    const i64 nb = (pk_size(nao) + 255) >> 8;        // about 3000 waves
    return nb < 563 ? 3 : nb < 1125 ? 2 : nb < 2250 ? 1 : 0;
}
// workgroups of 512 threads: 512 runs / slices positions each, groups of NK
// densities
inline int cu_tiles(int nao, int nd, int NK, int runs)
{
    const int P = 512 * runs >> cu_slices_log2(nao);
    return cdiv_i(nd, NK) * cdiv_i(pk_size(nao), P);
}

// J_k (+)= scale * sum_Q g[k][Q] B^Q at the positions of one workgroup for the
// NK densities of group kg: wave w takes 64 NP positions and the slabs of one
// slice, 16 loads in flight per lane; the slices' sums meet in LDS (red: 8
// x NK x 64 doubles, a run of 64 positions at a time) and each is written at
// (m, n) and (n, m).  g's first row is density kfirst.
template <int NK, int NP>
__device__ __forceinline__ void coulomb_tile(const double *__restrict__ B, const double *__restrict__ g,
                                    double *__restrict__ J, int nao, int naux, int nd, int packed,
                                    int tile, double *red, double scale = 1.0, int accumulate = 0,
                                    int kfirst = 0)
{
    constexpr int U = 16 / NP;
    const int lg = cu_slices_log2(nao), SL = 1 << lg, P = (512 >> lg) * NP;
    const i64 npk = pk_size(nao), npos = (i64)nao * nao, slab = packed ? npk : npos;
    const int nt = (int)((npk + P - 1) / P);
    const int kg = tile / nt, pb = tile - kg * nt;
    const int k0 = kg * NK;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int sl = wave & (SL - 1), pw = wave >> lg; // slice, block of positions
    const i64 p0 = (i64)pb * P + pw * (64 * NP) + lane;
    const double *b[NP];
#pragma unroll
    for (int j = 0; j < NP; j++) {
        const i64 pc = p0 + j * 64 < npk ? p0 + j * 64 : npk - 1;
        i64 off = pc;
        if (!packed) {
            int m, n;
            pk_coords(pc, nao, m, n);
            off = (i64)m * nao + n;
        }
        b[j] = B + off;
    }
    const int qlen = (naux + SL - 1) >> lg;
    const int q0 = sl * qlen < naux ? sl * qlen : naux;
    const int q1 = (q0 + qlen) < naux ? (q0 + qlen) : naux;
    const double *gk[NK];
#pragma unroll
    for (int k = 0; k < NK; k++)
        gk[k] = g + (i64)((k0 + k < nd ? k0 + k : nd - 1) - kfirst) * naux;
    double a[NP][NK];
#pragma unroll
    for (int j = 0; j < NP; j++)
#pragma unroll
        for (int k = 0; k < NK; k++)
            a[j][k] = 0.0;
    int q = q0;
    for (; q + U <= q1; q += U) {
        double v[U][NP];
#pragma unroll
        for (int u = 0; u < U; u++)
#pragma unroll
            for (int j = 0; j < NP; j++)
                v[u][j] = __builtin_nontemporal_load(b[j] + (i64)(q + u) * slab);
#pragma unroll
        for (int u = 0; u < U; u++)
#pragma unroll
            for (int k = 0; k < NK; k++) {
                const double gq = gk[k][q + u];
#pragma unroll
                for (int j = 0; j < NP; j++)
                    a[j][k] = fma(gq, v[u][j], a[j][k]);
            }
    }
    for (; q < q1; q++) {
#pragma unroll
        for (int j = 0; j < NP; j++) {
            const double v = b[j][(i64)q * slab];
#pragma unroll
            for (int k = 0; k < NK; k++)
                a[j][k] = fma(gk[k][q], v, a[j][k]);
        }
    }
#pragma unroll
    for (int j = 0; j < NP; j++) {
        if (j > 0)
            __syncthreads();
#pragma unroll
        for (int k = 0; k < NK; k++)
            red[(wave * NK + k) * 64 + lane] = a[j][k];
        __syncthreads();
        // one run of 64 positions of each block: (512 / SL) x NK sums
        for (int e = threadIdx.x; e < (512 >> lg) * NK; e += 512) {
            const int k = e >> (9 - lg), pos = e & ((512 >> lg) - 1);
            const i64 pp = (i64)pb * P + (pos >> 6) * (64 * NP) + j * 64 + (pos & 63);
            if (k0 + k < nd && pp < npk) {
                const double *x = red + ((pos >> 6) * SL * NK + k) * 64 + (pos & 63);
                double v = 0.0;
                for (int w = 0; w < SL; w++)
                    v += x[w * NK * 64];
                int mm, nn;
                pk_coords(pp, nao, mm, nn);
                double *Jk = J + (i64)(k0 + k) * npos;
                const i64 o = (i64)mm * nao + nn, tr = (i64)nn * nao + mm;
                Jk[o] = accumulate ? Jk[o] + scale * v : scale * v;
                if (mm != nn)
                    Jk[tr] = accumulate ? Jk[tr] + scale * v : scale * v;
            }
        }
    }
}

// Runs f for the group width w (1, 2, 4, 8 or 16) up to MAX.
template <int MAX, class F>
__host__ __device__ __forceinline__ void width_dispatch(int w, F &&f)
{
    if constexpr (MAX >= 16)
        if (w == 16)
            return f(std::integral_constant<int, 16>());
    if (w == 8)
        f(std::integral_constant<int, 8>());
    else if (w == 4)
        f(std::integral_constant<int, 4>());
    else if (w == 2)
        f(std::integral_constant<int, 2>());
    else
        f(std::integral_constant<int, 1>());
}

} // namespace jk
