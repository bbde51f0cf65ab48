// jk_batched.hip -- many J/K problems of uneven size per launch.
//
// A batched build runs the phases of the FP64 build (jk_tiles.hpp) once for
// the whole batch: each launch covers the tiles of every member that takes
// part in that phase, in one grid.  blockIdx.x is mapped to (member, tile)
// through a table of prefix sums; members are listed in decreasing order of
// per-tile cost so the longest tiles start first.  Each member runs the
// single-build plan for a chunk budget of 256 MB (members own their chunk
// buffers, so the budget is smaller than a single build's 1 GB); where both
// budgets give the same chunking -- every problem whose slabs fit one 256 MB
// chunk -- its outputs are bit-for-bit those of a single jk_build.
//
// The member descriptors and the tables live in the caller's workspace; the
// host writes them with one asynchronous copy per call.  Kernel arguments are
// only workspace pointers, so a captured graph of the launch sequence can be
// replayed for any batch of the same shapes in the same workspace.
#include "jk_batched.hpp"
#include "jk_kernels.hpp"
#include "jk_tiles.hpp"
#include "coulomb_upper.hpp"

namespace jk {

__global__ void __launch_bounds__(256) k_b_pack(const BMember *__restrict__ M, const int *__restrict__ tab)
{
    int loc;
    const BMember &m = M[find_member(tab, blockIdx.x, loc)];
    pack_tile(m.CL, m.CR, m.Cc, m.nao, m.nd, m.r, loc);
}

__global__ void __launch_bounds__(256) k_b_density(const BMember *__restrict__ M,
                                                   const int *__restrict__ tab)
{
    __shared__ double lds[TileDensity::LDS_DOUBLES];
    int loc;
    const BMember &m = M[find_member(tab, blockIdx.x, loc)];
    fold_density_tile(m.CL, m.CR, m.S, m.nao, m.r, loc, lds);
}

// Group widths up to MAX: 16 takes all; batches of at most 8 densities run with
// the registers of the narrower passes (8).
template <int MAX>
__global__ void __launch_bounds__(256, MAX == 16 ? 2 : 3)
    k_b_project(const BMember *__restrict__ M, const int *__restrict__ tab)
{
    __shared__ double lds[(2 * 4 * kPjQ + kPjMaxQ) * MAX];
    int loc;
    const BMember &m = M[find_member(tab, blockIdx.x, loc)];
    width_dispatch<MAX>(pj_width(m.nd), [&](auto nk) {
        constexpr int NK = decltype(nk)::value;
        project_tile<NK>(m.B, m.S, m.part, m.nao, m.naux, m.nd, m.packed, m.pj, loc,
                         (double (*)[4][kPjQ][NK])lds, (double (*)[NK])(lds + 2 * 4 * kPjQ * NK));
    });
}

__global__ void __launch_bounds__(256) k_b_reduce(const BMember *__restrict__ M,
                                                  const int *__restrict__ tab)
{
    int loc;
    const BMember &m = M[find_member(tab, blockIdx.x, loc)];
    reduce_tile(m.part, m.g, m.naux, m.nd, m.pj.nkg * pj_width(m.nd), m.pj.nbg, loc);
}

// ws: the workspace start (where M lies), as doubles; g is read at ws + goff.
// kBatchRuns runs of positions per wave for every member: the same sums (the
// slices are the member's own).
template <int MAX>
__global__ void __launch_bounds__(512) k_b_coulomb(const BMember *__restrict__ M,
                                                   const int *__restrict__ tab,
                                                   const double *__restrict__ ws)
{
    __shared__ double red[8 * MAX * 64];
    int loc;
    const BMember &m = M[find_member(tab, blockIdx.x, loc)];
    const double *g = ws + m.goff;
    width_dispatch<MAX>(pj_width(m.nd), [&](auto nk) {
        coulomb_tile<decltype(nk)::value, kBatchRuns>(m.B, g, m.J, m.nao, m.naux, m.nd, m.packed, loc, red);
    });
}

__global__ void __launch_bounds__(256, 3) k_b_half_transform(const BMember *__restrict__ M,
                                                             const int *__restrict__ tab, int c)
{
    __shared__ double lds[TileHalf::LDS_DOUBLES];
    int loc;
    const BMember &m = M[find_member(tab, xcd_local(blockIdx.x, gridDim.x), loc)];
    int q0, nq;
    chunk_of(m, c, q0, nq);
    ht_tile(m.B, m.Cc, m.Xw, m.Yw, m.nao, m.nd, m.r, q0, m.ldw, loc, lds);
}

__global__ void __launch_bounds__(256, 4) k_b_half_transform64(const BMember *__restrict__ M,
                                                               const int *__restrict__ tab, int c)
{
    __shared__ double lds[TileHalf64::LDS_DOUBLES];
    int loc;
    const BMember &m = M[find_member(tab, xcd_local(blockIdx.x, gridDim.x), loc)];
    int q0, nq;
    chunk_of(m, c, q0, nq);
    ht_tile_tl<TileHalf64>(m.B, m.Cc, m.Xw, m.Yw, m.nao, m.nd, m.r, q0, m.ldw, loc, lds, -1);
}

// Stacked-slab half-transform on the 16 x 16 x 4 engine (the plan's tile 3
// or 4; the schedule keeps members whose chunk of slabs spans 4 GiB or more
// on the 4x4x4 tile), one launch per shape.
typedef TileHalf16 TileB16;
template <int SHAPE>
__global__ void __launch_bounds__(256, shape_wgs(SHAPE))
    k_b_half_transform16(const BMember *__restrict__ M, const int *__restrict__ tab, int c)
{
    extern __shared__ double lds[];
    int loc;
    const BMember &m = M[find_member(tab, xcd_local(blockIdx.x, gridDim.x), loc)];
    int q0, nq;
    chunk_of(m, c, q0, nq);
    ht_tile_flat<typename ShapeTile<SHAPE>::type>(m.B, m.Cc, m.Xw, m.Yw, m.nao, m.nd, m.r, q0, nq,
                                                  m.ldw, loc, lds, m.sym ? m.nd * m.r : -1);
}

// Packed slabs on the 16 x 16 x 4 engine: 64 x 64 tiles per slab.
__global__ void __launch_bounds__(256, 4) k_b_half_transform16_packed(const BMember *__restrict__ M,
                                                                      const int *__restrict__ tab,
                                                                      int c)
{
    extern __shared__ double lds[];
    int loc;
    const BMember &m = M[find_member(tab, xcd_local(blockIdx.x, gridDim.x), loc)];
    int q0, nq;
    chunk_of(m, c, q0, nq);
    ht_tile16_packed<TileB16>(m.B, m.Cc, m.Xw, m.Yw, m.nao, m.nd, m.r, q0, m.ldw, loc, lds,
                              m.sym ? m.nd * m.r : -1);
}

// The exchange on the 16 x 16 x 4 engine (member chunk workspaces are capped
// at 256 MB, so X and Y of a density stay within a buffer resource's reach).
__global__ void __launch_bounds__(256, 3) k_b_exchange(const BMember *__restrict__ M,
                                                       const int *__restrict__ tab, int c)
{
    extern __shared__ double lds[];
    int loc;
    const BMember &m = M[find_member(tab, xcd_local(blockIdx.x, gridDim.x), loc)];
    int q0, nq;
    chunk_of(m, c, q0, nq);
    const int nj = nq * m.r;
    int jlen = cdiv_i(nj, m.nsplit);
    jlen = ((jlen + 15) / 16) * 16;
    const double *Y = m.sym ? m.Xw : m.Yw;
    double *K = m.nsplit > 1 ? m.Kp : m.K;
    // the member's tile shape; the workgroups of one member are consecutive,
    // so a CU's residents mostly share one
    switch (m.exs) {
    case kS128x64:
        ex_tile<ShapeTile<kS128x64>::type>(m.Xw, Y, K, m.nao, m.nd, nj, m.ldw, jlen, c > 0, loc, lds, m.sym);
        break;
    case kS96x64:
        ex_tile<ShapeTile<kS96x64>::type>(m.Xw, Y, K, m.nao, m.nd, nj, m.ldw, jlen, c > 0, loc, lds, m.sym);
        break;
    case kS80x64:
        ex_tile<ShapeTile<kS80x64>::type>(m.Xw, Y, K, m.nao, m.nd, nj, m.ldw, jlen, c > 0, loc, lds, m.sym);
        break;
    default:
        ex_tile<ShapeTile<kS64x64>::type>(m.Xw, Y, K, m.nao, m.nd, nj, m.ldw, jlen, c > 0, loc, lds, m.sym);
    }
}

__global__ void __launch_bounds__(256) k_b_mirror(const BMember *__restrict__ M,
                                                  const int *__restrict__ tab)
{
    __shared__ double t[32][33];
    int loc;
    const BMember &m = M[find_member(tab, blockIdx.x, loc)];
    const int nb = mirror_blocks(m.nao);
    mirror_tile(m.K + (i64)(loc / nb) * m.npos, m.nao, loc % nb, t);
}

__global__ void __launch_bounds__(256) k_b_sum_splits(const BMember *__restrict__ M,
                                                      const int *__restrict__ tab)
{
    int loc;
    const BMember &m = M[find_member(tab, blockIdx.x, loc)];
    sum_tile(m.Kp, m.K, (i64)m.nd * m.npos, m.nsplit, loc);
}

// ------------------------------------------------------------------ launch
static constexpr int kLds16 = (int)sizeof(double) * TileB16::LDS_DOUBLES;
template <int SHAPE>
static constexpr int shape_lds() { return (int)sizeof(double) * ShapeTile<SHAPE>::type::LDS_DOUBLES; }
// the exchange kernel holds every shape: the largest one's LDS
static constexpr int kLdsEx = shape_lds<kS128x64>();

hipError_t prepare_batched_kernels()
{
    hipError_t e = set_dynamic_lds((const void *)k_b_half_transform16<kS128x64>, shape_lds<kS128x64>());
    if (e == hipSuccess)
        e = set_dynamic_lds((const void *)k_b_half_transform16<kS64x64>, shape_lds<kS64x64>());
    if (e == hipSuccess)
        e = set_dynamic_lds((const void *)k_b_half_transform16_packed, kLds16);
    if (e == hipSuccess)
        e = set_dynamic_lds((const void *)k_b_exchange, kLdsEx);
    return e;
}

hipError_t launch_batched_phase(int phase, const BMember *M, const int *tab, int ntiles, int step,
                                hipStream_t s, int arg)
{
    if (ntiles <= 0)
        return hipSuccess;
    if (phase >= kPhaseMSliceC)
        return launch_batched_mixed_phase(phase, M, tab, ntiles, step, s, arg);
    const dim3 g(ntiles);
    switch (phase) {
    case kPhaseMirror: {
        ProfScope ps_("b_mirror", s);
        hipLaunchKernelGGL(k_b_mirror, g, dim3(256), 0, s, M, tab);
        break;
    }
    case kPhasePack: {
        ProfScope ps_("b_pack", s);
        hipLaunchKernelGGL(k_b_pack, g, dim3(256), 0, s, M, tab);
        break;
    }
    case kPhaseDensity: {
        ProfScope ps_("b_density", s);
        hipLaunchKernelGGL(k_b_density, g, dim3(256), 0, s, M, tab);
        break;
    }
    case kPhaseProject: {
        ProfScope ps_("b_project", s);
        hipLaunchKernelGGL(arg > 8 ? k_b_project<16> : k_b_project<8>, g, dim3(256), 0, s, M, tab);
        break;
    }
    case kPhaseReduce: {
        ProfScope ps_("b_reduce", s);
        hipLaunchKernelGGL(k_b_reduce, g, dim3(256), 0, s, M, tab);
        break;
    }
    case kPhaseCoulomb: {
        ProfScope ps_("b_coulomb", s);
        hipLaunchKernelGGL(arg > 8 ? k_b_coulomb<16> : k_b_coulomb<8>, g, dim3(512), 0, s, M, tab,
                           (const double *)M);
        break;
    }
    case kPhaseHalf: {
        ProfScope ps_("b_half_transform", s);
        hipLaunchKernelGGL(k_b_half_transform, g, dim3(256), 0, s, M, tab, step);
        break;
    }
    case kPhaseHalf64: {
        ProfScope ps_("b_half_transform", s);
        hipLaunchKernelGGL(k_b_half_transform64, g, dim3(256), 0, s, M, tab, step);
        break;
    }
    case kPhaseHalf16: {
        ProfScope ps_("b_half_transform", s);
        hipLaunchKernelGGL(k_b_half_transform16<kS128x64>, g, dim3(256), shape_lds<kS128x64>(), s, M, tab,
                           step);
        break;
    }
    case kPhaseHalf16S: {
        ProfScope ps_("b_half_transform", s);
        hipLaunchKernelGGL(k_b_half_transform16<kS64x64>, g, dim3(256), shape_lds<kS64x64>(), s, M, tab,
                           step);
        break;
    }
    case kPhaseHalf16Packed: {
        ProfScope ps_("b_half_transform", s);
        hipLaunchKernelGGL(k_b_half_transform16_packed, g, dim3(TileB16::NTHR), kLds16, s, M, tab,
                           step);
        break;
    }
    case kPhaseExchange: {
        ProfScope ps_("b_exchange", s);
        hipLaunchKernelGGL(k_b_exchange, g, dim3(256), kLdsEx, s, M, tab, step);
        break;
    }
    case kPhaseSum: {
        ProfScope ps_("b_sum_splits", s);
        hipLaunchKernelGGL(k_b_sum_splits, g, dim3(256), 0, s, M, tab);
        break;
    }
    default:
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

} // namespace jk
