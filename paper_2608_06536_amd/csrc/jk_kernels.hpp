// jk_kernels.hpp -- launchers of the device kernels (internal to the library).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace jk {

typedef int64_t i64;

// Brackets one kernel launch with timing events when jk_prof_enable is on
// (include/jk_prof.h); does nothing otherwise.
class ProfScope {
  public:
    ProfScope(const char *name, hipStream_t s);
    ~ProfScope();
    // While a stream is being captured into a graph no events are recorded.
    static void set_capturing(bool on);
    ProfScope(const ProfScope &) = delete;
    ProfScope &operator=(const ProfScope &) = delete;

  private:
    hipStream_t stream_;
    int pair_;
};

// Workgroup slots of the current device for two resident workgroups per CU.
int device_slots();
// Split count s in [1, smax] for a grid of tiles * s workgroups: the smallest s
// whose last round of workgroups is at least 90% full with at least one full
// round, else the s with the fullest rounds.
int pick_split(int tiles, int smax);
// Allows `bytes` of dynamic LDS for kernel fn on the current device (once per
// kernel and device).
hipError_t set_dynamic_lds(const void *fn, int bytes);
// Same with an explicit number of concurrent workgroup slots.
int pick_split_slots(int tiles, int smax, int slots);

// gamma and J on the upper triangles of the slabs (coulomb_upper.hpp), full
// squares or packed slabs.  S_k: matrices folded onto the packed positions
// (A[m][n] + A[n][m] above the diagonal), from the factors or from given
// matrices (nmat of them).  project: g[k][Q] = sum_p B^Q[p] S_k[p], all nd
// matrices, in groups of 16 that share part (project_part_doubles doubles).  coulomb: J (+)= scale *
// sum_Q g B^Q in full; accumulate adds to what J holds.
// What a build needs before it reads B; null pointers are left out.
struct PrepArgs {
    const double *CL, *CR;
    double *Cc;             // [C_L | C_R] as one nao x 2 nd r matrix
    double *S;              // folded densities
    const double *W;        // cotangent, folded into SW
    double *SW;
    double *E;              // D - 2 D^T
    int nao, nd, r;
};
hipError_t launch_prep(const PrepArgs &a, hipStream_t s);
size_t project_part_doubles(int nao, int naux, int nd);
hipError_t launch_project(const double *B, const double *S, double *part, double *g, int nao, int naux,
                          int nd, int packed, hipStream_t s, bool reduce = true);
hipError_t launch_coulomb(const double *B, const double *g, double *J, int nao, int naux, int nd,
                          int packed, hipStream_t s, double scale = 1.0, int accumulate = 0);
// J from the partial sums of a projection with reduce = false, where
// coulomb_sums_gamma says so: the same numbers.
bool coulomb_sums_gamma(int nao, int naux, int nd);
hipError_t launch_coulomb_sum(const double *B, const double *part, double *J, int nao, int naux, int nd,
                              int packed, hipStream_t s, double scale = 1.0, int accumulate = 0);
// packed: B holds packed upper-triangle slabs (nao (nao + 1) / 2 doubles).
// tile (full slabs only; jk_tune.h): 0 = 128 x 64 workgroup tiles of four
// waves, 1 = 64 x 64, 2 = 128 x 64 of eight waves (4x4x4 engine); 3 = 128 x 128,
// 4 = 128 x 64 over stacked slabs (16x16x4 engine).  prof: the name the
// launch is timed under.
hipError_t launch_half_transform(const double *B, const double *Cc, double *Xw, double *Yw,
                                 int nao, int nd, int r, int q0, int nq, int ldw, hipStream_t s,
                                 int ncol = -1, int packed = 0, int tile = 0,
                                 const char *prof = "half_transform");
// Lower triangle of every K_k from its upper triangle.
hipError_t launch_mirror_upper(double *K, int nao, int nd, hipStream_t s);
// Tile shape (Shape16) and splits of the exchange of one chunk; the partial
// sums of all splits stay within kp_cap bytes.
int exchange_shape(int nao);
int exchange_nsplit(int nao, int nd, int nj, int sym, size_t kp_cap);
// Every chunk's contribution is multiplied by scale before it is stored or
// added (scale 1 leaves it unchanged bit for bit).
hipError_t launch_exchange(const double *Xw, const double *Yw, double *Kp, int nao, int nd, int nj,
                           int ldw, int nsplit, int accumulate, hipStream_t s, int sym = 0,
                           double scale = 1.0);
hipError_t launch_sum_splits(const double *part, double *out, i64 n, int nsplit, hipStream_t s);
// The same for symmetric K_k whose partials hold the upper triangle (both
// triangles of K are written).
hipError_t launch_sum_splits_sym(const double *part, double *K, int nao, int nd, int nsplit,
                                 hipStream_t s);

// derivative (jk_vjp.hip)
// both of stage B's products; omega in om[k][Q]
hipError_t launch_vjp_stage_b(const double *V, const double *Xw, const double *Yw, const double *Cc,
                              const double *om, double *L, int nao, int nd, int r, int naux, int q0,
                              int nj, int ldw, int has_v, int has_w, hipStream_t s);
int vjp_stage_c_nsplit(int nao, int R, int qc);
hipError_t launch_vjp_stage_c(const double *B, const double *L, double *dCp, int nao, int R,
                              int q0, int nq, int nsplit, int accumulate, hipStream_t s);
hipError_t launch_vjp_dc_finish(const double *dCp, double *dCL, double *dCR, int nao, int nd,
                                int r, int nsplit, hipStream_t s);
hipError_t launch_vjp_stage_d(const double *L, const double *Cc, double *dB, int nao, int R,
                              int q0, int nq, hipStream_t s);
// Packed B (jk.h JK_B_PACKED): full squares of slabs q0 .. q0 + nq - 1 into
// out[nq][nao][nao]; stage D writing the packed gradient of those slabs
// (dB[a][b] + dB[b][a] for a < b, dB[a][a] on the diagonal).
hipError_t launch_unpack_slabs(const double *Bp, double *out, int nao, int q0, int nq,
                               hipStream_t s);
hipError_t launch_vjp_stage_d_packed(const double *L, const double *Cc, double *dB, int nao, int R,
                                     int q0, int nq, hipStream_t s);
// dB^Q += sum_k gam W + esign om E
hipError_t launch_vjp_db_affine(const double *gam, const double *om, const double *W,
                                const double *E, double esign, double *dB, int nd, int naux,
                                i64 npos, int q0, int nq, hipStream_t s);

// mixed precision (jk_mixed.hip)
int mixed_nslice();
int mixed_row_pad();
// rows of B's digit planes for nrow = slabs x nao stacked rows (with the rows a
// half-transform tile may read past them), and the padding of [C_L | C_R]'s
i64 mixed_b_rows(i64 nrow);
int mixed_col_pad();
int mixed_k_pad();
int mixed_k_block();
hipError_t launch_slice_rows(const double *src, i64 bs, i64 rs, i64 ks, int nb, int nr, int nk,
                             int rp, int nkb, int8_t *out, i64 pstride, i64 kbstride, int *exps,
                             hipStream_t s);
// digits of [C_L | C_R]: row c, inner n, element Cc[n][c]
hipError_t launch_slice_c(const double *Cc, int R2, int nao, int cp, int nkb, int8_t *out, i64 pstride,
                          i64 kbstride, int *exps, hipStream_t s);
hipError_t launch_slice_b(const double *src, i64 bs, i64 rs, int nb, int nr, int nk, int rp, int nkb,
                          int8_t *out, i64 pstride, i64 kbstride, int *exps, hipStream_t s);
// lanes of the one-pass slicer per row of kp inner bytes (0: rows too long for it)
int mixed_slice_lanes(int kp);
// widths 2 nd r of X/Y the mixed path takes
int mixed_rowmax_ok(int R2);
// XY's digit planes; the row exponents (left in exps) from nsp partial maxima.
hipError_t launch_slice_xy(const double *XY, int nao, int nkey, int r, int mp, int nj, int nkb,
                           int8_t *out, i64 pstride, i64 kbstride, const uint32_t *mx, int nsp,
                           int *exps, hipStream_t s);
// pm: the row maxima of the chunk's X and Y per tile, pitch rows
// (xy_rowmax_pm_words words), reduced to nsp partial maxima per row of the X/Y
// planes, mx[sp nkey mpe + key mpe + m], by launch_xy_rowmax_pm.
hipError_t launch_ht_mixed(const int8_t *Bp, i64 bpstride, i64 bkbstride, const int *eB,
                           const int8_t *Cp, i64 cpstride, i64 ckbstride, const int *eC, double *XY,
                           int nao, int R2, int nq, int cp, int nkb, uint32_t *pm, i64 rows, int r,
                           hipStream_t s);
size_t xy_rowmax_pm_words(i64 rows, int cp, int r, int nkey);
int xy_rowmax_splits(int nao, int nkey, int nq);
hipError_t launch_xy_rowmax_pm(const uint32_t *pm, int nao, int nq, int nkey, int r, i64 rows, int mpe,
                               uint32_t *mx, int nsp, hipStream_t s);
// Exchange splits of a chunk of nkb inner blocks: chosen for occupancy, and
// never fewer than keep each split's int32 sums exact (mixed_max_depth()
// inner indices at most).
int ex_mixed_nsplit(int mp, int nd, int nkb, int sym = 0);
int mixed_max_depth();
// Workgroups of the mixed half-transform of nrow stacked rows (cpx padded
// factor columns) and of the mixed exchange with nsplit splits.
int mixed_ht_tiles(int nrow, int cpx);
int mixed_ex_tiles(int mp, int nd, int nsplit, int sym);
// B digit planes from packed slabs (slab stride bs = nao (nao + 1) / 2);
// mixed_packed_ok tells whether the packed slicer covers rows of kp inner
// elements (kp <= 2048).
hipError_t launch_slice_b_packed(const double *src, i64 bs, int nb, int nao, int rp, int nkb,
                                 int8_t *out, i64 pstride, i64 kbstride, int *exps, hipStream_t s);
int mixed_packed_ok(int nao, int kp);
hipError_t launch_ex_mixed(const int8_t *Xp, const int8_t *Yp, i64 pstride, i64 kbstride,
                           const int *eX, const int *eY, double *Kp, int nao, int nd, int mp, int nkb,
                           int nsplit, int accumulate, hipStream_t s, int sym = 0,
                           double scale = 1.0);

} // namespace jk
