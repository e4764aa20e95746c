// Kernel launch wrappers of the FBC library (all enqueue on `st`, no synchronisation).
#pragma once
#include "common.h"

struct BondTable {
    int n[12][3];        // primitive-basis offsets of the 12 nearest-neighbour bonds
    double p[12][6];     // k * Rhat Rhat^T in symmetric order xx yy zz xy xz yz
};

// ---- assembly (Appendix B, discrete Brillouin-zone sum) ----
void launch_dinv(hipStream_t st, double2* pk, int m0, int nmc, int nz, int m1, int m2,
                 int logL, const double* sn, const BondTable& bt);
void launch_fft_rows(hipStream_t st, double2* data, int64_t nrows, int logn, const double2* tw,
                     bool inverse);
void launch_transpose_c(hipStream_t st, const double2* in, double2* out, int batches, int rows,
                        int cols);
void launch_gather_table(hipStream_t st, const double2* t, double2* tab, int nmc, int m1, int m2,
                         int64_t n_off, const int32_t* off_d1, const int32_t* off_d2,
                         int64_t tab_mode_stride, double scale);
// Table modes are on the finest line grid of the context: cell mode m reads table mode
// m * mode_mult.
void launch_rowmean(hipStream_t st, const double2* tab, double2* rowmean, int nm, int mode_mult,
                    int64_t n_off, int n_b, int n_i, const int32_t* cols_b, const int32_t* cols_i,
                    const int32_t* lut, int d1min, int d2min, int w2);
// Per table mode: largest magnitude (amax) and the distance beyond which every block is
// below tau * amax (rhocut); both as bit patterns of non-negative doubles.
void launch_tab_rhocut(hipStream_t st, const double2* tab, int T, int64_t n_off, const int32_t* d1,
                       const int32_t* d2, double tau, unsigned long long* amax,
                       unsigned long long* rhocut);
// Compact dense store of one cell (chunk-tiles of the negligible-block windows; see
// k_build_dense): reg_pre [nm * n_tiles + 1] (prefix sums of the window lengths, in
// chunk-tiles) and win_start [nm * n_tiles] on the device; n_ct = reg_pre[last].
void launch_build_dense(hipStream_t st, int form, void* store, const double2* tab,
                        const double2* rowmean, const int64_t* reg_pre, const int32_t* win_start,
                        int nm, int n_tiles, int n_chunks, int tile_rows, int64_t n_ct, int mode_mult,
                        int64_t n_off, int n_b, int n_i, const int32_t* cols_b, const int32_t* cols_i,
                        const int32_t* lut, int d1min, int d2min, int w2, unsigned long long* amax);

// Table of the reduced forms (RTabView): records of every table mode; amax: largest magnitude per
// table mode (split FP16: its scale).
void launch_build_rtab(hipStream_t st, int form, const double2* tab, int T, int64_t n_off, const int32_t* d1,
                       const int32_t* d2, const RBox& box, const unsigned long long* amax, char* rtab);
void launch_tab_absmax(hipStream_t st, const double2* tab, int T, int64_t n_off, unsigned long long* amax);

// ---- apply (Section 2.3.2 update in line-mode form) ----
// Per-layer sums sums[r][n0][6] (net force, absolute force), cell totals tot[r][3] with
// the net-force check, and (shat != NULL) the line transform of the per-layer net force.
// Relaxation: the step factors of this step from f_{k+1} and f_k (fprev, then f_{k+1} for the next
// step; NULL: no relaxation), part [R][nz][3]; the step bound from the maxima of |w|.
struct RelaxIn {
    double *fprev, *part, *alpha, *finf;
    const int* kdev;
    int relax;
    double alpha_min;
};
struct RelaxClamp {
    const double* wmax_part;
    int n_part;
    double *alpha, *stepinf;
    double du_max;
    const int* kdev;
    int relax;
};
// launch_forward: these (if `statistics`; bexp: also the operand scale of split FP16), then the
// transforms of f into the product's B fragments (place: CellPlan::place_i, offset-table forms).
void launch_forward(hipStream_t st, int form, const double* f, double* sums, double* tot, double2* shat, int* shat_on,
                    bool statistics, double tol, int check, int project, void* bfrag, int R, int nz, int n_i, int kp,
                    int ct, const double2* tw, int* bexp, int* status, const int32_t* place, const RelaxIn& rx);
// Reduced forms.  variant: one of gemm_variants(form, jt) kernel instantiations (bitwise the
// same result); q != NULL: persistent work-queue kernel on these lists.
void launch_gemm(hipStream_t st, int form, const GemmJob* jobs, int njobs, int jt, const void* a,
                 const RTabView& tv, const void* b, double* c, const CellDev* cells, const PqLists* q, int variant);
void gemm_kernels_init(int form, int jt);
int gemm_groups_per_cu(int form, int jt);
int gemm_variants(int form, int jt);
std::string gemm_shape(int form, int jt, int variant);
// Offset-table forms (gemm_table.hip): one job per wave, 16 pad columns over a window of
// interface columns.  q != NULL: persistent work-queue kernel; mixed: jobs carry their precision;
// variant 1: work groups of four waves instead of one (bitwise the same result).
#define TAB_COLS 16
void launch_gemm_dtab(hipStream_t st, const GemmJob* jobs, int njobs, int ct, const TabView& tv, const double* b,
                      double* c, const CellDev* cells, const PqLists* q, int mixed, int variant);
// H-matrix product step (hmat.hip): B fragments of one FP64 cell in, product records out
void hmat_enqueue_pipeline(fbc_hmat* h, const double* bfrag, int64_t bf_mode, int kp, const int32_t* place, double* rec,
                           int mp, int nm, int ct, hipStream_t st);
const fbc_ctx* hmat_context(const fbc_hmat* h);
void irfft_shape(int nz, int* tr, int* pp);
void launch_line_irfft(hipStream_t st, const double* c, double* w, double* wmax_part, int R,
                       int nz, int mp, int M, int ct, int ct_grid, const double2* tw, int nsplit,
                       int64_t split_stride, const double2* rowmean, const double2* shat,
                       const int* shat_on, const unsigned long long* amax, const int* bexp,
                       int* n_part_out);
// Raises the dynamic-LDS limit of the 1024-thread line-transform kernels on the current
// device (once per device; call outside stream capture, e.g. at context creation).
void apply_kernels_init();
// The mean that an update removes, mu[r][3] (mu NULL: none).  nbr > 0: the kernel that updates u
// still has to form it, from nbr <= MEAN_INLINE partial sums per RHS, and to write it.
#define MEAN_INLINE 32
struct MeanIn {
    double* mu;
    const double* part;
    int nbr;
    double inv_n;
};
// u <- u - alpha_r w - mu_r (mu optional) through a tiled transpose
void launch_axpy(hipStream_t st, const double* w, double* u, int R, int nz, int M, double alpha,
                 const double* alpha_d, const int* status, const MeanIn& mean);
// fused inverse transform + update (fbc_apply, fbc_green_apply, the relaxation step without
// a step bound), and the mean it removes; update_shape is false where the line is too long
// for the fused kernel.  alpha_d: per-RHS step factors on the device (else alpha);
// wmax_part: per RHS and row group (ceil(M / tr) of them) the largest |w|, or NULL.
bool update_shape(int nz, int* tr);
void launch_irfft_update(hipStream_t st, const double* c, double* u, int R, int nz, int mp, int M,
                         int ct_grid, const double2* tw, int nsplit, int64_t split_stride,
                         const double2* rowmean, const double2* shat, const int* shat_on,
                         const unsigned long long* amax, const int* bexp, double alpha,
                         const MeanIn& mean, int read_u, const int* status,
                         const double* alpha_d = nullptr, double* wmax_part = nullptr);
int mean_blocks(int64_t per_rhs);
MeanIn launch_update_mean(hipStream_t st, const double* u, const double* c, double* part, int R, int nz,
                        int mp, int M, int nsplit, int64_t split_stride, const double2* rowmean,
                        const double2* shat, const int* shat_on, const unsigned long long* amax,
                        const int* bexp, double alpha, double* mu, const int* status,
                        const double* alpha_d = nullptr, const RelaxClamp* clamp = nullptr);

// ---- relax (Section 2.3.3, Algorithm 2); kdev: the iteration index on the device ----
void launch_relax_clamp(hipStream_t st, const RelaxClamp& a, int R);
// relaxation output and the index advance
void launch_relax_finish(hipStream_t st, const double* alpha_d, const double* finf_d, const double* stepinf_d,
                         const double* mean_d, fbc_relax_out* out, int R, int* kdev, double tol_f);
// kdev <- v (v >= 0) or kdev + 1 (v < 0)
void launch_relax_index(hipStream_t st, int* kdev, int v);
void launch_fill(hipStream_t st, double* p, int64_t n, double v);
