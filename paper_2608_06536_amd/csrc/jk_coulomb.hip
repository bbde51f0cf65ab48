// jk_coulomb.hip -- gamma and the Coulomb matrix from the upper triangles of
// symmetric slabs, full or packed (coulomb_upper.hpp).
#include "coulomb_upper.hpp"
#include "jk_kernels.hpp"

namespace jk {

__global__ void __launch_bounds__(256) k_fold_density(const double *__restrict__ CL,
                                                      const double *__restrict__ CR,
                                                      double *__restrict__ S, int nao, int r)
{
    __shared__ double lds[TileDensity::LDS_DOUBLES];
    fold_density_tile(CL, CR, S, nao, r, blockIdx.x, lds);
}

__global__ void __launch_bounds__(256) k_sym_pack(const double *__restrict__ A,
                                                  double *__restrict__ S, int nao)
{
    __shared__ double T[32][33];
    const int nt = sym_pack_tiles(nao);
    sym_pack_tile(A, S, nao, blockIdx.x / nt, blockIdx.x % nt, T);
}

template <int NK>
__global__ void __launch_bounds__(256, NK == 16 ? 2 : 3)
    k_project(const double *__restrict__ B, const double *__restrict__ S, double *__restrict__ part,
              int nao, int naux, int nd, int packed, PjGeom geo)
{
    __shared__ double red[2][4][kPjQ][NK], sum[kPjMaxQ][NK];
    project_tile<NK>(B, S, part, nao, naux, nd, packed, geo, blockIdx.x, red, sum);
}

__global__ void __launch_bounds__(256) k_project_reduce(const double *__restrict__ part,
                                                        double *__restrict__ g, int naux, int nd,
                                                        int ndp, int npb)
{
    reduce_tile(part, g, naux, nd, ndp, npb, blockIdx.x);
}

template <int NK, int NP>
__global__ void __launch_bounds__(512) k_coulomb(const double *__restrict__ B,
                                                 const double *__restrict__ g, double *__restrict__ J,
                                                 int nao, int naux, int nd, int packed, double scale,
                                                 int accumulate)
{
    __shared__ double red[8 * NK * 64];
    coulomb_tile<NK, NP>(B, g, J, nao, naux, nd, packed, blockIdx.x, red, scale, accumulate);
}

hipError_t launch_fold_density(const double *CL, const double *CR, double *S, int nao, int nd, int r,
                               hipStream_t s)
{
    {
        ProfScope ps_("density", s);
        hipLaunchKernelGGL(k_fold_density, dim3(fold_tiles(nao, nd)), dim3(256), 0, s, CL, CR, S, nao, r);
    }
    return hipGetLastError();
}

hipError_t launch_sym_pack(const double *A, double *S, int nao, int nmat, hipStream_t s)
{
    {
        ProfScope ps_("sym_pack", s);
        hipLaunchKernelGGL(k_sym_pack, dim3(nmat * sym_pack_tiles(nao)), dim3(256), 0, s, A, S, nao);
    }
    return hipGetLastError();
}

size_t project_part_doubles(int nao, int naux, int nd)
{
    return (size_t)pj_blocks(nao, naux) * naux * pj_groups(nd) * pj_width(nd);
}

hipError_t launch_project(const double *B, const double *S, double *part, double *g, int nao, int naux,
                          int nd, int packed, hipStream_t s)
{
    {
        ProfScope ps_(nd > 8 ? "project16" : "project", s);
        const PjGeom geo = pj_geom(nao, naux, nd);
        const dim3 grid(pj_tiles(geo, naux));
        auto go = [&](auto nk) {
            hipLaunchKernelGGL(k_project<decltype(nk)::value>, grid, dim3(256), 0, s, B, S, part, nao,
                               naux, nd, packed, geo);
        };
        width_dispatch<16>(pj_width(nd), go);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return e;
    {
        ProfScope ps_("project_reduce", s);
        const int ndp = pj_groups(nd) * pj_width(nd);
        hipLaunchKernelGGL(k_project_reduce, dim3(reduce_tiles(naux, ndp)), dim3(256), 0, s, part, g, naux,
                           nd, ndp, pj_blocks(nao, naux));
    }
    return hipGetLastError();
}

hipError_t launch_coulomb(const double *B, const double *g, double *J, int nao, int naux, int nd,
                          int packed, hipStream_t s, double scale, int accumulate)
{
    {
        ProfScope ps_("coulomb", s);
        const int runs = cu_runs(nao), w = pj_width(nd);
        const dim3 grid(cu_tiles(nao, nd, w, runs));
        auto go = [&](auto nk) {
            if (runs == 1)
                hipLaunchKernelGGL((k_coulomb<decltype(nk)::value, 1>), grid, dim3(512), 0, s, B, g, J,
                                   nao, naux, nd, packed, scale, accumulate);
            else
                hipLaunchKernelGGL((k_coulomb<decltype(nk)::value, 4>), grid, dim3(512), 0, s, B, g, J,
                                   nao, naux, nd, packed, scale, accumulate);
        };
        width_dispatch<16>(w, go);
    }
    return hipGetLastError();
}

} // namespace jk
