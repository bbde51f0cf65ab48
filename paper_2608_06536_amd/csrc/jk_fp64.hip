// jk_fp64.hip -- single-problem FP64 kernels of the Cholesky-decomposed J/K
// build: each kernel runs tile blockIdx.x of one phase (jk_tiles.hpp).
#include "jk_kernels.hpp"
#include "jk_tiles.hpp"

#include <cmath>
#include <mutex>
#include <set>
#include <utility>

namespace jk {

__global__ void __launch_bounds__(256, 3) k_half_transform(const double *__restrict__ B,
                                                           const double *__restrict__ Cc,
                                                           double *__restrict__ Xw,
                                                           double *__restrict__ Yw, int nao, int nd,
                                                           int r, int q0, int nq, int ldw, int ncol)
{
    __shared__ double lds[TileHalf::LDS_DOUBLES];
    const int n = ht_tiles_cols(nao, ncol, nq);
    ht_tile(B, Cc, Xw, Yw, nao, nd, r, q0, ldw, xcd_swizzle(blockIdx.x, n), lds, ncol);
}

// The half-transform with 64 x 64 tiles (four workgroups per CU): a plan
// choice (jk_tune.h) for shapes where the 128-row tiles waste rows.
__global__ void __launch_bounds__(256, 4) k_half_transform64(const double *__restrict__ B,
                                                             const double *__restrict__ Cc,
                                                             double *__restrict__ Xw,
                                                             double *__restrict__ Yw, int nao,
                                                             int nd, int r, int q0, int nq, int ldw,
                                                             int ncol)
{
    __shared__ double lds[TileHalf64::LDS_DOUBLES];
    const int n = nq * cdiv_i(nao, 64) * cdiv_i(ncol, 64);
    ht_tile_tl<TileHalf64>(B, Cc, Xw, Yw, nao, nd, r, q0, ldw, xcd_swizzle(blockIdx.x, n), lds,
                           ncol);
}

// The half-transform with the 128 x 64 tile split over eight 64 x 16 wave
// tiles (110 VGPRs, four waves per SIMD): more waves to hide the fragment
// reads and barriers of each stage (measured 49.7 against 47.3 TF at nao 500).
typedef Tile<128, 64, 64, 16, 16> TileHalfW8;
__global__ void __launch_bounds__(512, 2) k_half_transform_w8(const double *__restrict__ B,
                                                              const double *__restrict__ Cc,
                                                              double *__restrict__ Xw,
                                                              double *__restrict__ Yw, int nao,
                                                              int nd, int r, int q0, int nq,
                                                              int ldw, int ncol)
{
    __shared__ double lds[TileHalfW8::LDS_DOUBLES];
    const int n = ht_tiles_cols(nao, ncol, nq);
    ht_tile_tl<TileHalfW8>(B, Cc, Xw, Yw, nao, nd, r, q0, ldw, xcd_swizzle(blockIdx.x, n), lds,
                           ncol);
}

// The half-transform on the 16 x 16 x 4 engine, over the chunk's stacked
// slabs.  The 128 x 128 tile has a kernel of its own name (plan tile 3 asks
// for it alone; tile 4 takes ht_shape's choice).
template <int SHAPE>
__global__ void __launch_bounds__(256, shape_wgs(SHAPE))
    k_half_transform16(const double *__restrict__ B, const double *__restrict__ Cc,
                       double *__restrict__ Xw, double *__restrict__ Yw, int nao, int nd, int r,
                       int q0, int nq, int ldw, int ncol)
{
    typedef typename ShapeTile<SHAPE>::type TL;
    extern __shared__ double lds_dyn[];
    const int n = ht_flat_tiles<TL>(nao, ncol, nq);
    ht_tile_flat<TL>(B, Cc, Xw, Yw, nao, nd, r, q0, nq, ldw, xcd_swizzle(blockIdx.x, n), lds_dyn,
                     ncol);
}
__global__ void __launch_bounds__(256, shape_wgs(kS128x128))
    k_half_transform16a(const double *__restrict__ B, const double *__restrict__ Cc,
                        double *__restrict__ Xw, double *__restrict__ Yw, int nao, int nd, int r,
                        int q0, int nq, int ldw, int ncol)
{
    typedef ShapeTile<kS128x128>::type TL;
    extern __shared__ double lds_dyn[];
    const int n = ht_flat_tiles<TL>(nao, ncol, nq);
    ht_tile_flat<TL>(B, Cc, Xw, Yw, nao, nd, r, q0, nq, ldw, xcd_swizzle(blockIdx.x, n), lds_dyn,
                     ncol);
}

template <int BN>
__global__ void __launch_bounds__(256, 4)
    k_half_transform16n(const double *__restrict__ B, const double *__restrict__ Cc,
                        double *__restrict__ Xw, double *__restrict__ Yw, int nao, int nd, int r,
                        int q0, int nq, int ldw, int ncol)
{
    typedef typename HtNarrow<BN>::flat TL;
    extern __shared__ double lds_dyn[];
    const int n = ht_flat_tiles<TL>(nao, ncol, nq);
    ht_tile_flat<TL>(B, Cc, Xw, Yw, nao, nd, r, q0, nq, ldw, xcd_swizzle(blockIdx.x, n), lds_dyn,
                     ncol);
}

// Packed slabs on the 16 x 16 x 4 engine (plan tiles 3 and 4): tiles of 64 rows
// per slab, four workgroups per CU.
template <class TL>
__global__ void __launch_bounds__(256, 4)
    k_half_transform16_packed(const double *__restrict__ B, const double *__restrict__ Cc,
                              double *__restrict__ Xw, double *__restrict__ Yw, int nao, int nd, int r,
                              int q0, int nq, int ldw, int ncol)
{
    extern __shared__ double lds_dyn[];
    const int n = nq * cdiv_i(nao, TL::BM) * cdiv_i(ncol, TL::BN);
    ht_tile16_packed<TL>(B, Cc, Xw, Yw, nao, nd, r, q0, ldw, xcd_swizzle(blockIdx.x, n), lds_dyn, ncol);
}

// The same on packed slabs (jk.h JK_B_PACKED).
__global__ void __launch_bounds__(256, 3) k_half_transform_packed(const double *__restrict__ B,
                                                                  const double *__restrict__ Cc,
                                                                  double *__restrict__ Xw,
                                                                  double *__restrict__ Yw, int nao,
                                                                  int nd, int r, int q0, int nq,
                                                                  int ldw, int ncol)
{
    __shared__ double lds[TileHalf::LDS_DOUBLES];
    const int n = ht_tiles_cols(nao, ncol, nq);
    ht_tile<true>(B, Cc, Xw, Yw, nao, nd, r, q0, ldw, xcd_swizzle(blockIdx.x, n), lds, ncol);
}

// The exchange product on the 16 x 16 x 4 engine, tile shape by pick_shape:
// two to four workgroups per CU, 35 to 70 KB of dynamic LDS.
template <int SHAPE, bool MASK>
__global__ void __launch_bounds__(256, shape_wgs(SHAPE))
    k_exchange16(const double *__restrict__ Xw, const double *__restrict__ Yw,
                 double *__restrict__ Kp, int nao, int nd, int nj, int ldw, int nsplit, int jlen,
                 int accumulate, int sym, double scale)
{
    typedef typename ShapeTile<SHAPE>::type TL;
    extern __shared__ double lds_dyn[];
    const int n = nsplit * nd * ex_tiles(nao, TL::BM, TL::BN, sym);
    ex_tile<TL, MASK>(Xw, Yw, Kp, nao, nd, nj, ldw, jlen, accumulate, xcd_swizzle(blockIdx.x, n),
                      lds_dyn, sym, scale);
}

__global__ void __launch_bounds__(512, 4) k_exchange(const double *__restrict__ Xw,
                                                     const double *__restrict__ Yw,
                                                     double *__restrict__ Kp, int nao, int nd, int nj,
                                                     int ldw, int nsplit, int jlen, int accumulate,
                                                     int sym, double scale)
{
    __shared__ double lds[TileExch::LDS_DOUBLES];
    const int n = nsplit * nd * ex_tiles(nao, kExM, kExN, sym);
    ex_tile(Xw, Yw, Kp, nao, nd, nj, ldw, jlen, accumulate, xcd_swizzle(blockIdx.x, n), lds, sym,
            scale);
}

__global__ void __launch_bounds__(256) k_mirror_upper(double *__restrict__ K, int nao, int nd)
{
    __shared__ double t[32][33];
    // densities k = blockIdx.y, + gridDim.y, ... (grid y is capped at 65535)
    for (int k = blockIdx.y; k < nd; k += gridDim.y)
        mirror_tile(K + (i64)k * nao * nao, nao, blockIdx.x, t);
}

__global__ void __launch_bounds__(256) k_sum_splits(const double *__restrict__ part,
                                                    double *__restrict__ out, i64 n, int nsplit)
{
    sum_tile(part, out, n, nsplit, blockIdx.x);
}

__global__ void __launch_bounds__(256) k_sum_splits_sym(const double *__restrict__ part,
                                                        double *__restrict__ K, int nao, int nd,
                                                        int nsplit)
{
    const i64 npos = (i64)nao * nao;
    // densities k = blockIdx.y, + gridDim.y, ... (grid y is capped at 65535)
    for (int k = blockIdx.y; k < nd; k += gridDim.y) {
        sum_sym_tile(part + k * npos, K + k * npos, nao, nd * npos, nsplit, blockIdx.x);
        __syncthreads();
    }
}

// ------------------------------------------------------------------ launchers

static inline int cdiv(i64 a, i64 b) { return (int)((a + b - 1) / b); }

int device_slots()
{
    static int slots = 0;
    if (slots == 0) {
        int dev = 0, ncu = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            ncu <= 0)
            ncu = 256;
        slots = 2 * ncu;
    }
    return slots;
}

int pick_split(int tiles, int smax) { return pick_split_slots(tiles, smax, device_slots()); }

int pick_split_slots(int tiles, int smax, int slots)
{
    if (smax < 1)
        smax = 1;
    int best = 1;
    double best_eff = -1.0;
    for (int s = 1; s <= smax; s++) {
        const i64 w = (i64)tiles * s;
        const i64 rounds = (w + slots - 1) / slots;
        const double eff = (double)w / (double)(rounds * slots);
        if (w >= slots && eff >= 0.9)
            return s;
        if (eff > best_eff + 1e-9) {
            best_eff = eff;
            best = s;
        }
    }
    return best;
}

// Dynamic LDS above 64 KB needs a per-kernel attribute, set once per
// (kernel, device).
hipError_t set_dynamic_lds(const void *fn, int bytes)
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

namespace {
typedef void (*HtKernel)(const double *, const double *, double *, double *, int, int, int, int, int,
                         int, int);
template <class TL>
hipError_t launch_ht16(HtKernel k, int ntiles, const double *B, const double *Cc, double *Xw,
                       double *Yw, int nao, int nd, int r, int q0, int nq, int ldw, int ncol,
                       hipStream_t s, const char *prof)
{
    const int lds = (int)sizeof(double) * TL::LDS_DOUBLES;
    hipError_t e = set_dynamic_lds((const void *)k, lds);
    if (e != hipSuccess)
        return e;
    ProfScope ps_(prof, s);
    hipLaunchKernelGGL(k, dim3(ntiles), dim3(TL::NTHR), lds, s, B, Cc, Xw, Yw,
                       nao, nd, r, q0, nq, ldw, ncol);
    return hipSuccess;
}
} // namespace

hipError_t launch_half_transform(const double *B, const double *Cc, double *Xw, double *Yw,
                                 int nao, int nd, int r, int q0, int nq, int ldw, hipStream_t s,
                                 int ncol, int packed, int tile, const char *prof)
{
    if (ncol < 0)
        ncol = 2 * nd * r;
    // packed slabs: one buffer resource per slab
    if (!packed && tile >= 3 && !buf_extent_ok((i64)nq * nao * nao))
        tile = 2;                                 // chunk beyond the buffer loads' 4 GiB reach
    auto flat = [&](auto tl, HtKernel k) {
        typedef decltype(tl) TL;
        return launch_ht16<TL>(k, ht_flat_tiles<TL>(nao, ncol, nq), B, Cc, Xw, Yw, nao, nd, r, q0, nq, ldw,
                               ncol, s, prof);
    };
    auto slabs = [&](auto tl) {
        typedef decltype(tl) TL;
        return launch_ht16<TL>(k_half_transform16_packed<TL>, nq * cdiv(nao, TL::BM) * cdiv(ncol, TL::BN), B,
                               Cc, Xw, Yw, nao, nd, r, q0, nq, ldw, ncol, s, "half_transform_packed");
    };
    if (packed && tile >= 3) {
        hipError_t e;
        switch (ht_cols(ncol, true)) {
        case 16: e = slabs(HtNarrow<16>::packed()); break;
        case 32: e = slabs(HtNarrow<32>::packed()); break;
        case 48: e = slabs(HtNarrow<48>::packed()); break;
        default: e = slabs(TileHalf16());
        }
        if (e != hipSuccess)
            return e;
    } else if (packed) {
        ProfScope ps_("half_transform_packed", s);
        hipLaunchKernelGGL(k_half_transform_packed, dim3(ht_tiles_cols(nao, ncol, nq)), dim3(256), 0,
                           s, B, Cc, Xw, Yw, nao, nd, r, q0, nq, ldw, ncol);
    } else if (tile == 3 || tile == 4) {
        hipError_t e;
        const int bn = tile == 3 ? 128 : ht_cols(ncol, false);
        if (bn == 128)
            e = flat(ShapeTile<kS128x128>::type(), k_half_transform16a);
        else if (bn == 16)
            e = flat(HtNarrow<16>::flat(), k_half_transform16n<16>);
        else if (bn == 32)
            e = flat(HtNarrow<32>::flat(), k_half_transform16n<32>);
        else if (bn == 48)
            e = flat(HtNarrow<48>::flat(), k_half_transform16n<48>);
        else if (ht_shape(nao) == kS128x64)
            e = flat(ShapeTile<kS128x64>::type(), k_half_transform16<kS128x64>);
        else
            e = flat(ShapeTile<kS64x64>::type(), k_half_transform16<kS64x64>);
        if (e != hipSuccess)
            return e;
    } else if (tile == 2) {
        ProfScope ps_(prof, s);
        hipLaunchKernelGGL(k_half_transform_w8, dim3(ht_tiles_cols(nao, ncol, nq)), dim3(512), 0, s, B,
                           Cc, Xw, Yw, nao, nd, r, q0, nq, ldw, ncol);
    } else if (tile == 1) {
        ProfScope ps_(prof, s);
        hipLaunchKernelGGL(k_half_transform64, dim3(nq * cdiv(nao, 64) * cdiv(ncol, 64)), dim3(256), 0,
                           s, B, Cc, Xw, Yw, nao, nd, r, q0, nq, ldw, ncol);
    } else {
        ProfScope ps_(prof, s);
        hipLaunchKernelGGL(k_half_transform, dim3(ht_tiles_cols(nao, ncol, nq)), dim3(256), 0, s, B, Cc,
                           Xw, Yw, nao, nd, r, q0, nq, ldw, ncol);
    }
    return hipGetLastError();
}

hipError_t launch_mirror_upper(double *K, int nao, int nd, hipStream_t s)
{
    const int nb = cdiv(nao, 32);
    {
        ProfScope ps_("mirror", s);
        hipLaunchKernelGGL(k_mirror_upper, dim3(nb * (nb + 1) / 2, nd < 65535 ? nd : 65535), dim3(256),
                           0, s, K, nao, nd);
    }
    return hipGetLastError();
}

// One or two 128 x 128 tiles a side leave few workgroups per split (nao 100:
// 30 us against 24 with 128 x 64; 208: 204 against 198), four or more keep the
// power down (500: 904 us a chunk against 930).
int exchange_shape(int nao) { return pick_shape(nao, nao, nao <= 256 ? kS128x64 : kS128x128); }

// Splits of the exchange's inner range: the count with the least estimated
// time.  A CU runs ceil(workgroups / CUs) workgroups one after the other at
// the rate of the matrix cores (fewer residents cover fewer of the stage
// barriers: 0.77, 0.86 and 0.9 of the peak with one, two and three); every
// round of residents pays about 3 us of first loads and output; the partial
// sums are written and read back (nao^2 per density and split) at about 4
// TB/s.  Each split keeps at least 32 inner indices, and the partials stay
// within kp_cap bytes.  At most 16 splits of at least 256 indices, the rule
// before, left one symmetric density of nao 236 and rank 48 (depth 45312, 6
// tiles) on 96 workgroups: 220 us, now 83; nao 48, depth 1536: 25 us, now 8.
int exchange_nsplit(int nao, int nd, int nj, int sym, size_t kp_cap)
{
    const int shape = exchange_shape(nao);
    const double tiles = (double)nd * ex_tiles(nao, shape_bm(shape), shape_bn(shape), sym);
    const double kbytes = 8.0 * nd * nao * (double)nao;
    const int ncu = device_slots() / 2, occ = shape_wgs(shape);
    int smax = nj / 32;
    if (smax > 512)
        smax = 512;
    if (smax * kbytes > (double)kp_cap)
        smax = (int)(kp_cap / kbytes);
    auto cost = [&](int s) {
        const double n = ceil(tiles * s / ncu);                   // workgroups of a CU
        const double depth = 16.0 * cdiv(cdiv(nj, s), 16);
        const double per = 2.0 * shape_bm(shape) * shape_bn(shape) * depth / (77e12 / 256);
        const double eff = n >= 3 ? 0.9 : n == 2 ? 0.86 : 0.77;
        double t = n * per / eff + 3e-6 * ceil(n / occ);
        if (s > 1)
            t += 3e-6 + 2.0 * s * kbytes / 4e12;
        return t;
    };
    // candidates: one split, and the most splits that give a CU n workgroups
    int best = 1;
    double tbest = cost(1);
    for (int n = 1; n <= 4 * occ; n++) {
        const double sn = floor(n * ncu / tiles);
        const int s = sn < smax ? (int)sn : smax;
        if (s <= 1)
            continue;
        const double t = cost(s);
        if (t < tbest) {
            best = s;
            tbest = t;
        }
        if (s == smax)
            break;
    }
    return best;
}

namespace {
struct ExArgs {
    const double *Xw, *Yw;
    double *Kp;
    int nao, nd, nj, ldw, nsplit, jlen, accumulate, sym;
    double scale;
};
template <int SHAPE, bool MASK>
hipError_t launch_exchange16(const ExArgs &a, hipStream_t s)
{
    typedef typename ShapeTile<SHAPE>::type TL;
    const int lds = (int)sizeof(double) * TL::LDS_DOUBLES;
    hipError_t e = set_dynamic_lds((const void *)k_exchange16<SHAPE, MASK>, lds);
    if (e != hipSuccess)
        return e;
    ProfScope ps_("exchange", s);
    hipLaunchKernelGGL((k_exchange16<SHAPE, MASK>), dim3(a.nsplit * a.nd * ex_tiles(a.nao, TL::BM, TL::BN, a.sym)),
                       dim3(TL::NTHR), lds, s, a.Xw, a.Yw, a.Kp, a.nao, a.nd, a.nj, a.ldw, a.nsplit,
                       a.jlen, a.accumulate, a.sym, a.scale);
    return hipSuccess;
}
template <int SHAPE>
hipError_t launch_exchange16_m(const ExArgs &a, hipStream_t s)
{
    // splits end on 16-deep stage boundaries (jlen is a multiple of 16), so
    // only a depth nj off that grid leaves a stage to mask
    return a.nj % 16 != 0 ? launch_exchange16<SHAPE, true>(a, s) : launch_exchange16<SHAPE, false>(a, s);
}
} // namespace

hipError_t launch_exchange(const double *Xw, const double *Yw, double *Kp, int nao, int nd, int nj,
                           int ldw, int nsplit, int accumulate, hipStream_t s, int sym, double scale)
{
    int jlen = cdiv(nj, nsplit);
    jlen = ((jlen + 15) / 16) * 16;
    if (buf_extent_ok((i64)nao * ldw)) {
        const ExArgs a{Xw, Yw, Kp, nao, nd, nj, ldw, nsplit, jlen, accumulate, sym, scale};
        hipError_t e = hipErrorInvalidValue;
        switch (exchange_shape(nao)) {
        case kS128x128: e = launch_exchange16_m<kS128x128>(a, s); break;
        case kS128x64: e = launch_exchange16_m<kS128x64>(a, s); break;
        case kS96x64: e = launch_exchange16_m<kS96x64>(a, s); break;
        case kS80x64: e = launch_exchange16_m<kS80x64>(a, s); break;
        case kS64x64: e = launch_exchange16_m<kS64x64>(a, s); break;
        }
        if (e != hipSuccess)
            return e;
    } else {
        ProfScope ps_("exchange", s);
        hipLaunchKernelGGL(k_exchange, dim3(nsplit * nd * ex_tiles(nao, kExM, kExN, sym)), dim3(TileExch::NTHR),
                           0, s, Xw, Yw, Kp, nao, nd, nj, ldw, nsplit, jlen, accumulate, sym, scale);
    }
    return hipGetLastError();
}

hipError_t launch_sum_splits_sym(const double *part, double *K, int nao, int nd, int nsplit,
                                 hipStream_t s)
{
    {
        ProfScope ps_("sum_splits", s);
        hipLaunchKernelGGL(k_sum_splits_sym, dim3(sum_sym_blocks(nao), nd < 65535 ? nd : 65535),
                           dim3(256), 0, s, part, K, nao, nd, nsplit);
    }
    return hipGetLastError();
}

hipError_t launch_sum_splits(const double *part, double *out, i64 n, int nsplit, hipStream_t s)
{
    {
        ProfScope ps_("sum_splits", s);
        hipLaunchKernelGGL(k_sum_splits, dim3(sum_tiles(n)), dim3(256), 0, s, part, out, n, nsplit);
    }
    return hipGetLastError();
}

} // namespace jk
