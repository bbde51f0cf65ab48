// slice_core.hpp -- fixed-point slice products on gfx950 INT8 matrix cores.
//
// Split-precision scheme of the mixed J/K path.  Every FP64 row a[0..n) of an
// operand gets one power-of-two scale 2^e with max|a| <= 2^e * 127/128, and
// each element is rounded to the 31-bit integer N = rint(a 2^(31 - e)),
// |N| <= 127 * 2^24, written as NS = 4 balanced base-256 digits
//     N = d1 2^24 + d2 2^16 + d3 2^8 + d4,   d2..d4 in [-128, 127],
// taken from the bottom (d4 = ((N + 128) mod 256) - 128, then N -> (N - d4)/256,
// ...); the leading digit is what remains, |d1| <= 127.  So
//     a = 2^(e - 7) * sum_{i=1..4} d_i 2^(-8 (i - 1)) + rest,  |rest| <= 2^(e - 32).
// A product of two rows is
//     sum_k a_k b_k = 2^(ea + eb - 14) * sum_{l=2..L} 2^(-8 (l - 2)) * S_l,
//     S_l = sum_{i+j=l} sum_k d_i(a_k) d_j(b_k),
// keeping the 13 digit pairs with i + j <= L = 6.  Each S_l is an exact
// integer: the matrix cores multiply int8 digits and accumulate in int32; a
// level holds at most 4 pairs of |d_i d_j| <= 2^14 per inner index, so
// |S_l| <= 2^16 n < 2^31 for n <= kSliceMaxDepth = 32767 inner indices per
// accumulation (enforced by the planner).  The levels are combined in FP64
// with power-of-two weights, so the only approximations are the rounding of
// N (relative 2^-32 of the row scale), the three dropped pairs, and FP64
// rounding of the combination.
//
// Instruction: V_MFMA_I32_32X32X32_I8.  Lane layout (measured on the device):
// lane l holds A[row l % 32][k 16*(l/32) .. +15] and B[k 16*(l/32) .. +15][col
// l % 32] as 16 bytes each, and output element j (0..15) is
// C[8*(j/4) + 4*(l/32) + j%4][l % 32].
//
// Digit planes live in global memory K-blocked (see SPlanes) with rows and
// inner bytes padded by zero digits, so the GEMM loaders copy 16-byte chunks
// without bounds checks.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace jk {

typedef int64_t i64;
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));

constexpr int kSliceDigits = 4;        // digits per value (planes per operand)
constexpr int kSliceLevel = 6;         // products d_i d_j with i + j <= 6 are kept
constexpr int kSliceKB = 32;           // inner block: bytes per row per block
constexpr int kSliceProdShift = -14;   // a row product is 2^(ea + eb - 14) * sum_l ...
// Most inner indices one int32 level sum may take (see above): at most 4
// digit pairs of |d_i d_j| <= 2^14 per index, so n indices give
// |S_l| <= 2^16 n, below 2^31 for n <= 32767.  Every plan splits its
// contractions so that no accumulation exceeds this depth.
constexpr int kSliceMaxDepth = 32767;

__device__ __forceinline__ v16i mfma_i8(v4i a, v4i b, v16i c)
{
    return __builtin_amdgcn_mfma_i32_32x32x32_i8(a, b, c, 0, 0, 0);
}

// Scale exponent of a row: the smallest e with maxabs <= 2^e * 127/128 (0 for
// an all-zero row).  Both comparisons are exact in FP64.
__device__ __forceinline__ int row_exponent(double maxabs)
{
    if (!(maxabs > 0.0))
        return 0;
    int e = ilogb(maxabs) + 1;                       // 2^(e-1) <= maxabs < 2^e
    if (maxabs * 128.0 > ldexp(127.0, e))
        e++;
    return e;
}

// The same from the high word of maxabs, rounded up if its low word is not
// zero (high_word_up): the threshold's low word is zero, so both comparisons
// have the same outcome.
__device__ __forceinline__ uint32_t high_word_up(double x)
{
    const uint64_t v = __builtin_bit_cast(uint64_t, x);
    return ((uint32_t)(v >> 32) & 0x7fffffffu) + ((uint32_t)v != 0);
}
__device__ __forceinline__ int row_exponent_hi(uint32_t hi)
{
    return row_exponent(__builtin_bit_cast(double, (uint64_t)hi << 32));
}

// The four digits of a, given the row exponent e (|a| <= 2^e * 127/128):
// d[0] is the leading digit.
__device__ __forceinline__ void slice_value(double a, int e, int8_t *d)
{
    int n = (int)rint(ldexp(a, 31 - e));             // |n| <= 127 * 2^24
#pragma unroll
    for (int i = kSliceDigits - 1; i > 0; i--) {
        const int t = ((n + 128) & 255) - 128;
        d[i] = (int8_t)t;
        n = (n - t) >> 8;                            // exact: n - t is a multiple of 256
    }
    d[0] = (int8_t)n;
}

// ---------------------------------------------------------------- planes
// Digit planes in global memory are K-blocked: plane p, row i, inner byte k
// lives at base[p * pstride + (k / 32) * kbstride + i * 32 + k % 32], with
// kbstride = (rows of the array) * 32.  A tile of rows x 32 inner bytes of one
// plane is therefore one contiguous block; rows and inner bytes are padded
// with zero digits, so tile loads need no bounds checks.
struct SPlanes {
    const int8_t *base;   // already offset to the first row of the operand
    i64 pstride;          // bytes between planes
    i64 kbstride;         // bytes between inner blocks
};

// Byte offset of (row, 16-byte half) inside a plane of an LDS stage.  The two
// 16-byte halves of a row swap places on every other group of 8 rows, so the
// 64 lanes of a fragment read (rows r..r+31, half l/32) spread evenly over
// the LDS banks.
__device__ __forceinline__ int slds_off(int row, int half)
{
    return row * kSliceKB + ((half ^ ((row >> 3) & 1)) << 4);
}

// 16 bytes per lane from global memory straight into LDS at dst + 16 * lane
// (dst is the same for the whole wave).  The builtin exists only in the
// device compilation.
__device__ __forceinline__ void global_to_lds16(const int8_t *src, char *dst)
{
#if defined(__HIP_DEVICE_COMPILE__)
    __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void *)dst, 16, 0, 0);
#endif
}

// ---------------------------------------------------------------- tiles
// Workgroup tile BM x BN; each wave owns 32 x (32 WTN) outputs (WTN MFMA
// tiles side by side), so one A fragment feeds WTN tiles.  Waves (BM/32) x
// (BN/(32 WTN)).  One pipeline stage is one 32-byte inner block of NS planes
// of both operands.
template <int BM, int BN, int NS, int WTN>
struct STileW {
    static constexpr int WROWS = BM / 32, WCOLS = BN / (32 * WTN);
    static constexpr int NWAVE = WROWS * WCOLS;
    static constexpr int NTHR = NWAVE * 64;
    static constexpr int NLEV = kSliceLevel - 1;       // levels 2..kSliceLevel
    static constexpr int TN = WTN;
    static constexpr int A_BYTES = NS * BM * kSliceKB, B_BYTES = NS * BN * kSliceKB;
    static constexpr int STAGE_BYTES = A_BYTES + B_BYTES;
};

template <class TL>
struct SAccW {
    v16i c[TL::TN][TL::NLEV];
    __device__ __forceinline__ void zero()
    {
#pragma unroll
        for (int t = 0; t < TL::TN; t++)
#pragma unroll
            for (int l = 0; l < TL::NLEV; l++)
#pragma unroll
                for (int e = 0; e < 16; e++)
                    c[t][l][e] = 0;
    }
};

// s_waitcnt with vmcnt <= n and the other counters unconstrained (gfx9
// encoding: vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8).
template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    __builtin_amdgcn_s_waitcnt((N & 0xF) | ((N >> 4) << 14) | (0x7 << 4) | (0xF << 8));
}

// s_waitcnt vmcnt(n * PER) for a run-time n in [0, NMAX].
template <int PER, int NMAX>
__device__ __forceinline__ void wait_vm_stages(int n)
{
    if (NMAX >= 3 && n >= 3)
        wait_vmcnt<3 * PER>();
    else if (NMAX >= 2 && n == 2)
        wait_vmcnt<2 * PER>();
    else if (NMAX >= 1 && n == 1)
        wait_vmcnt<PER>();
    else
        wait_vmcnt<0>();
}


// A pointer that is the same for every lane of the wave, kept in scalar
// registers.
__device__ __forceinline__ const int8_t *uniform_ptr(const int8_t *p)
{
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const int8_t *)(((uint64_t)hi << 32) | lo);
}

// Workgroup barrier without the memory fence of __syncthreads(): that fence
// waits for every outstanding global load (vmcnt 0), which would drain the
// copies of later stages.  The waits each phase needs are explicit.  The
// empty asm statements keep memory accesses on their side of it, and the
// scheduling barriers keep every other instruction there too (the compiler
// would otherwise hoist matrix products into the other group's phase).
__device__ __forceinline__ void wg_barrier()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}

// ---------------------------------------------------------------- GEMM
// acc_l += sum over inner blocks [kb_begin, kb_end) of the kept digit pairs of
// level l, for one tile of four waves of 32 x 64 outputs (two workgroups per
// CU).  m_rows, n_rows: plane rows of the operands (multiples of 32): blocks of
// 32 rows beyond them repeat the last one (their outputs are not stored).
//
// Three LDS stage buffers, one stage = one 32-byte inner block.  A stage's 26
// products use 12 fragments (4 of A, 8 of B); a wave reads the next stage's
// while it multiplies, each into the registers of a fragment that has had its
// last use, in an order of the pairs in which every fragment is free at least
// six pairs (12 products) before it is needed again, so a stage never starts
// with a wait on LDS (A digit, B digit):
//   (1,4) (2,4) (1,3) (2,3) (3,3)
//   barrier: every wave holds this stage in registers, the next is in LDS;
//            this stage's buffer takes the copies of the one three ahead
//   reads B4 B3   (1,2) (1,1)   A1   (2,2) (2,1)   A2   (3,2) (3,1)   A3
//                 (4,2)   B2   (4,1)   A4 B1
// Bound by power: with the matrix cores half busy the clock falls from 2.1 to
// 1.97 GHz, so what a tile costs beyond its products (padding, LDS reads) counts
// more than stalls.  As the half-transform: nao 250 450 -> 386 us, nao 1000 159
// -> 176 TFLOP/s of FP64 equivalent against reading a stage's fragments before
// its products.
template <class TL, int NS>
__device__ __forceinline__ void stile_gemm_w4(const SPlanes &A, const SPlanes &B, int m0, int n0,
                                              int m_rows, int n_rows, int kb_begin, int kb_end,
                                              char *lds, SAccW<TL> &acc)
{
    static_assert(TL::NWAVE == 4 && NS == 4 && TL::TN == 2, "four waves, 13 digit pairs");
    constexpr int BM = TL::WROWS * 32, BN = TL::WCOLS * 32 * TL::TN, WTN = TL::TN;
    constexpr int NBUF = 3;
    constexpr int NBA = NS * (BM / 32), NB = NBA + NS * (BN / 32);
    constexpr int NW = TL::NWAVE, PER = (NB + NW - 1) / NW;
    static_assert(NB % NW == 0, "whole blocks per wave");
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave / TL::WCOLS, wc = wave % TL::WCOLS;
    const int nst = kb_end - kb_begin;
    if (nst <= 0)
        return;
    // Block copies: a block is 32 rows x 32 bytes of one plane (1 KB, one
    // wave instruction).  The block's global start and LDS slot are the same
    // for the whole wave; lane l copies row l / 2, half (l & 1) swizzled to
    // the LDS layout of slds_off.
    const uint32_t lane_off = (lane >> 1) * kSliceKB + (((lane & 1) ^ ((lane >> 4) & 1)) << 4);
    const int8_t *ub[PER];
    int loff[PER];
#pragma unroll
    for (int u = 0; u < PER; u++) {
        const int b = wave + u * NW;
        const bool isA = b < NBA;
        const int bl = isA ? b : b - NBA;
        const int T = isA ? BM : BN;
        const int p = bl / (T / 32), rh = bl % (T / 32);
        const SPlanes &op = isA ? A : B;
        const int row = (isA ? m0 : n0) + rh * 32, last = (isA ? m_rows : n_rows) - 32;
        ub[u] = uniform_ptr(op.base + p * op.pstride + (i64)(row < last ? row : last) * kSliceKB);
        loff[u] = (isA ? 0 : TL::A_BYTES) + p * T * kSliceKB + rh * 32 * kSliceKB;
    }
    const i64 akbs = A.kbstride, bkbs = B.kbstride;
    auto issue = [&](int kb, int buf) {
#pragma unroll
        for (int u = 0; u < PER; u++)
            global_to_lds16(ub[u] + (i64)kb * (wave + u * NW < NBA ? akbs : bkbs) + lane_off,
                            lds + buf * TL::STAGE_BYTES + loff[u]);
    };
    const int aoff = slds_off(wr * 32 + (lane & 31), lane >> 5);
    int boff[WTN];
#pragma unroll
    for (int t = 0; t < WTN; t++)
        boff[t] = TL::A_BYTES + slds_off((wc * WTN + t) * 32 + (lane & 31), lane >> 5);
    v4i fa[NS], fb[WTN][NS];
    auto read_a = [&](const char *st, int p) { return *(const v4i *)(st + p * BM * kSliceKB + aoff); };
    auto read_b = [&](const char *st, int p) {
#pragma unroll
        for (int t = 0; t < WTN; t++)
            fb[t][p] = *(const v4i *)(st + p * BN * kSliceKB + boff[t]);
    };
    auto mult = [&](int i, int j) {
#pragma unroll
        for (int t = 0; t < WTN; t++)
            acc.c[t][i + j] = mfma_i8(fa[i], fb[t][j], acc.c[t][i + j]);
    };
    for (int s0 = 0; s0 < NBUF; s0++)
        if (s0 < nst)
            issue(kb_begin + s0, s0);
    wait_vm_stages<PER, NBUF - 1>(min(nst - 1, NBUF - 1));
    wg_barrier();
    read_b(lds, 3);
    read_b(lds, 2);
    fa[0] = read_a(lds, 0);
    fa[1] = read_a(lds, 1);
    fa[2] = read_a(lds, 2);
    read_b(lds, 1);
    fa[3] = read_a(lds, 3);
    read_b(lds, 0);
    auto head = [&]() {
        mult(0, 3);
        mult(1, 3);
        mult(0, 2);
        mult(1, 2);
        mult(2, 2);
        __builtin_amdgcn_sched_barrier(0);
    };
    head();
    int cur = 0;
#pragma clang loop unroll(disable)
    for (int st = 0; st + 1 < nst; st++) {
        __builtin_amdgcn_s_waitcnt(0xC07F);          // lgkmcnt(0): this stage is in registers
        wait_vm_stages<PER, 1>(min(nst - st - 2, 1));        // stage st + 1 has landed
        wg_barrier();
        if (st + NBUF < nst)
            issue(kb_begin + st + NBUF, cur);
        cur = cur == NBUF - 1 ? 0 : cur + 1;
        const char *nx = lds + cur * TL::STAGE_BYTES;
        read_b(nx, 3);
        read_b(nx, 2);
        __builtin_amdgcn_sched_barrier(0);
        mult(0, 1);
        mult(0, 0);
        __builtin_amdgcn_sched_barrier(0);
        fa[0] = read_a(nx, 0);
        mult(1, 1);
        mult(1, 0);
        __builtin_amdgcn_sched_barrier(0);
        fa[1] = read_a(nx, 1);
        mult(2, 1);
        mult(2, 0);
        __builtin_amdgcn_sched_barrier(0);
        fa[2] = read_a(nx, 2);
        mult(3, 1);
        __builtin_amdgcn_sched_barrier(0);
        read_b(nx, 1);
        mult(3, 0);
        __builtin_amdgcn_sched_barrier(0);
        fa[3] = read_a(nx, 3);
        read_b(nx, 0);
        __builtin_amdgcn_sched_barrier(0);
        head();
    }
    mult(0, 1);
    mult(0, 0);
    mult(1, 1);
    mult(1, 0);
    mult(2, 1);
    mult(2, 0);
    mult(3, 1);
    mult(3, 0);
}

// Output coordinates of element e of tile t of this lane.
template <class TL>
__device__ __forceinline__ void stile_coord_wide(int t, int e, int &row, int &col)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wr = wave / TL::WCOLS, wc = wave % TL::WCOLS;
    row = wr * 32 + 8 * (e >> 2) + 4 * (lane >> 5) + (e & 3);
    col = (wc * TL::TN + t) * 32 + (lane & 31);
}

// FP64 value of output element e of tile t of this lane:
// sum_l S_l 2^(-8 (l - 2)), before the 2^(ea + eb + kSliceProdShift) row and
// column scale.  Every step is exact (power-of-two weights) unless the sum
// needs more than 53 bits.
template <class TL>
__device__ __forceinline__ double combine_levels_wide(const SAccW<TL> &acc, int t, int e)
{
    double v = (double)acc.c[t][TL::NLEV - 1][e];
#pragma unroll
    for (int l = TL::NLEV - 2; l >= 0; l--)
        v = fma(v, 0x1p-8, (double)acc.c[t][l][e]);
    return v;
}

} // namespace jk
