// jk_batched.hpp -- device descriptor of one member of a batched build.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "coulomb_upper.hpp"

namespace jk {

// One problem of a batch: its inputs, outputs, the workspace pointers of its
// own single-build plan, and that plan's chunk and split parameters.
struct BMember {
    const double *B, *CL, *CR;
    double *J, *K;
    double *Cc, *S, *part, *g, *Xw, *Yw, *Kp;   // S: densities folded onto the packed positions
    long long npos;
    // g as an offset in doubles from the start of the workspace (the batch's
    // descriptors): the Coulomb pass reads g through a kernel argument, whose
    // read-only, unaliased loads the compiler makes scalar (one load per
    // wave, not per lane)
    long long goff;
    int nao, naux, nd, r;
    int qc, ldw, nsplit;
    PjGeom pj;          // gamma's split
    int exs;            // FP64: the exchange's tile shape (Shape16)
    int sym;            // C_L and C_R are one buffer: X only, K on the upper triangle
    // JK_MIXED members: digit planes (single-buffered), their row exponents
    // and strides (slice_core.hpp layout), the FP64 half-transform chunk XY
    int8_t *Bp, *Cp, *XYp;
    int *eB, *eC, *eXY;
    double *XY;
    uint32_t *pm, *mx;  // the half-transform's partial row maxima of X/Y, and their maxima
    long long bkb, bps, ckb, cps, xkb, xps;
    int mp, kp, cp, cpx;    // padded rows / inner bytes; cpx: [C_L | C_R] rows the products use
    int rows;               // rows of B's planes (slabs x nao and spare)
    // doubles per slab of B: npos for full squares, packed-triangular slabs
    // (jk.h JK_B_PACKED) otherwise
    long long bslab;
    int packed;
};

// Runs of 64 positions per wave of the Coulomb pass (coulomb_upper.hpp): four
// whatever the size, as the members together fill the chip (24 members of nao
// 100-250: 544 us, 604 with one run; 12 of 100-500: 1.50 ms, 1.72).
constexpr int kBatchRuns = 4;

// Table layout: tab[0] = n entries, tab[1 .. n+1] = start offsets (n+1
// values), tab[n+2 .. 2n+2) = member indices.  Returns the member of tile t
// and its tile index within the member.
__device__ __forceinline__ int find_member(const int *__restrict__ tab, int t, int &local)
{
    const int n = tab[0];
    const int *start = tab + 1;
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (start[mid] <= t)
            lo = mid;
        else
            hi = mid - 1;
    }
    local = t - start[lo];
    return tab[n + 2 + lo];
}

// Workgroup index remapped so that runs of kXcdRun consecutive table tiles
// (the column tiles of one row panel, the tiles of one exchange row) land on
// one XCD and share its L2, while the table's order (larger tiles first)
// holds at the scale of 8 kXcdRun tiles.  Within each full block of
// 8 kXcdRun indices, logical = block start + (hw % 8) kXcdRun + (hw / 8) %
// kXcdRun (the hardware deals workgroups round-robin over the 8 XCDs); the
// indices of a last, partial block keep their place.
constexpr int kXcdRun = 16;
template <int RUN = kXcdRun>
__device__ __forceinline__ int xcd_local(int hw, int n)
{
    constexpr int blk = 8 * RUN;
    const int b0 = hw - hw % blk;
    if (b0 + blk > n)
        return hw;
    const int r = hw - b0;
    return b0 + (r & 7) * RUN + (r >> 3);
}

// Chunk of member m at step c: first slab and slab count.
__device__ __forceinline__ void chunk_of(const BMember &m, int c, int &q0, int &nq)
{
    q0 = c * m.qc;
    nq = (m.naux - q0) < m.qc ? (m.naux - q0) : m.qc;
}

enum {
    kPhasePack = 0,
    kPhaseDensity = 1,   // the folded densities
    kPhaseProject = 2,
    kPhaseReduce = 3,
    kPhaseCoulomb = 4,
    kPhaseHalf = 5,
    kPhaseExchange = 6,
    kPhaseSum = 7,
    kPhaseHalf64 = 8,    // the half-transform with 64 x 64 tiles (members whose plan chose them)
    kPhaseHalf16 = 9,    // the half-transform on the 16 x 16 x 4 engine over stacked slabs, 128 x 64 tiles
    kPhaseHalf16S = 15,  // the same with 64 x 64 tiles (ht_shape)
    kPhaseMirror = 10,   // lower triangle of K from the upper (symmetric members)
    kPhaseHalf16Packed = 13,  // packed B: the 16 x 16 x 4 half-transform, tiles per slab
    // JK_MIXED phases (jk_mixed.hip)
    kPhaseMSliceC = 20,  // digit planes of [C_L | C_R]
    kPhaseMSliceB = 21,  // digit planes of the chunk's slabs of B
    kPhaseMHalf = 22,    // INT8 half-transform of the chunk
    kPhaseMRowmax = 23,  // row exponents of the chunk's X and Y
    kPhaseMSliceXY = 24, // digit planes of the chunk's X and Y
    kPhaseMExchange = 25, // INT8 exchange of the chunk
    kPhaseMSliceBPacked = 26  // digit planes of the chunk's packed slabs
};

// Sets the dynamic LDS size of the batched kernels that need it on the
// current device (before a launch sequence is captured).
hipError_t prepare_batched_kernels();

// One launch of a phase over the members listed in tab (device pointer):
// ntiles workgroups, step = chunk index for the chunked phases.  arg: the
// slicer's register blocks (kPhaseMSliceB), or 16 x the dynamic LDS bytes
// plus the register blocks (kPhaseMSliceBPacked).
hipError_t launch_batched_phase(int phase, const BMember *M, const int *tab, int ntiles, int step,
                                hipStream_t s, int arg = 0);
hipError_t launch_batched_mixed_phase(int phase, const BMember *M, const int *tab, int ntiles,
                                      int step, hipStream_t s, int arg);
hipError_t prepare_batched_mixed_kernels();

} // namespace jk
