// jk_coulomb.hip -- gamma and the Coulomb matrix from the upper triangles of
// symmetric slabs, full or packed (coulomb_upper.hpp).
#include "coulomb_upper.hpp"
#include "jk_kernels.hpp"

namespace jk {

constexpr int kFuseGamma = 4096;

// What a build needs before it reads B, independent of each other, as one
// launch: ranges of workgroups for the derivative's E, the folded densities, the
// folded cotangent and [C_L | C_R].  Each takes a few microseconds, as does a
// launch: nao 48 38.0 -> 34.5 us for a build, with gamma's last sum in the J pass.
__global__ void __launch_bounds__(256) k_prep(PrepArgs a, int ne, int nf, int ns)
{
    __shared__ double lds[TileDensity::LDS_DOUBLES];
    static_assert(TileDensity::LDS_DOUBLES >= 32 * 33, "sym_pack_tile");
    int b = blockIdx.x;
    if (b < ne) {
        e_matrix_tile(a.CL, a.CR, a.E, a.nao, a.r, b, lds);
    } else if ((b -= ne) < nf) {
        fold_density_tile(a.CL, a.CR, a.S, a.nao, a.r, b, lds);
    } else if ((b -= nf) < ns) {
        const int nt = sym_pack_tiles(a.nao);
        sym_pack_tile(a.W, a.SW, a.nao, b / nt, b % nt, (double (*)[33])lds);
    } else {
        pack_tile(a.CL, a.CR, a.Cc, a.nao, a.nd, a.r, b - ns);
    }
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

// The same with gamma's partial sums added up here, by every workgroup for the
// slabs and densities it reads (kFuseGamma numbers of LDS at most).
template <int NK>
__global__ void __launch_bounds__(512) k_coulomb_sum(const double *__restrict__ B,
                                                     const double *__restrict__ part,
                                                     double *__restrict__ J, int nao, int naux, int nd,
                                                     int packed, int ndp, int npb, double scale,
                                                     int accumulate)
{
    __shared__ double red[8 * NK * 64], g[kFuseGamma];
    const int nt = cdiv_i(pk_size(nao), 64);         // 64 positions per workgroup
    const int k0 = (int)blockIdx.x / nt * NK;
    for (int e = threadIdx.x; e < naux * NK; e += 512) {
        const int q = e / NK, k = e % NK;
        double w[4];
#pragma unroll
        for (int u = 0; u < 4; u++)
            w[u] = reduce_part(part + (i64)q * ndp + k0 + k, (i64)naux * ndp, npb, u);
        g[k * naux + q] = ((w[0] + w[1]) + w[2]) + w[3];
    }
    __syncthreads();
    coulomb_tile<NK, 1>(B, g, J, nao, naux, nd, packed, blockIdx.x, red, scale, accumulate, k0);
}

hipError_t launch_prep(const PrepArgs &a, hipStream_t s)
{
    const int nt = cdiv_i(a.nao, 64);
    const int ne = a.E ? a.nd * nt * nt : 0, nf = a.S ? fold_tiles(a.nao, a.nd) : 0;
    const int ns = a.W ? a.nd * sym_pack_tiles(a.nao) : 0, nc = a.Cc ? pack_tiles(a.nao, a.nd, a.r) : 0;
    if (ne + nf + ns + nc == 0)
        return hipSuccess;
    {
        ProfScope ps_("prep", s);
        hipLaunchKernelGGL(k_prep, dim3(ne + nf + ns + nc), dim3(256), 0, s, a, ne, nf, ns);
    }
    return hipGetLastError();
}

size_t project_part_doubles(int nao, int naux, int nd)
{
    return (size_t)pj_blocks(nao, naux) * naux * pj_width(nd);
}

hipError_t launch_project(const double *B, const double *S, double *part, double *g, int nao, int naux,
                          int nd, int packed, hipStream_t s, bool reduce)
{
    // one group of columns at a time, each through the same partial sums
    for (int k0 = 0; k0 < nd; k0 += 16) {
        const int n = nd - k0 < 16 ? nd - k0 : 16;
        const double *Sk = S + (i64)k0 * pk_size(nao);
        const PjGeom geo = pj_geom(nao, naux, n);
        {
            ProfScope ps_(nd > 8 ? "project16" : "project", s);
            width_dispatch<16>(pj_width(n), [&](auto nk) {
                hipLaunchKernelGGL(k_project<decltype(nk)::value>, dim3(pj_tiles(geo, naux)), dim3(256), 0, s,
                                   B, Sk, part, nao, naux, n, packed, geo);
            });
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            return e;
        if (!reduce)
            continue;
        {
            ProfScope ps_("project_reduce", s);
            hipLaunchKernelGGL(k_project_reduce, dim3(reduce_tiles(naux, pj_width(n))), dim3(256), 0, s, part,
                               g + (i64)k0 * naux, naux, n, pj_width(n), geo.nbg);
        }
        e = hipGetLastError();
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
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

// At most 8 partial sums (nao 127), one group of columns and kFuseGamma numbers:
// larger builds keep the sum in a launch of its own, where every number is
// summed once.
bool coulomb_sums_gamma(int nao, int naux, int nd)
{
    return nd <= 16 && pj_blocks(nao, naux) <= 8 && (i64)naux * pj_width(nd) <= kFuseGamma && cu_runs(nao) == 1 &&
           cu_slices_log2(nao) == 3;
}

hipError_t launch_coulomb_sum(const double *B, const double *part, double *J, int nao, int naux, int nd,
                              int packed, hipStream_t s, double scale, int accumulate)
{
    {
        ProfScope ps_("coulomb", s);
        const int w = pj_width(nd);
        width_dispatch<16>(w, [&](auto nk) {
            hipLaunchKernelGGL(k_coulomb_sum<decltype(nk)::value>, dim3(cu_tiles(nao, nd, w, 1)), dim3(512),
                               0, s, B, part, J, nao, naux, nd, packed, w,
                               pj_blocks(nao, naux), scale, accumulate);
        });
    }
    return hipGetLastError();
}

} // namespace jk
