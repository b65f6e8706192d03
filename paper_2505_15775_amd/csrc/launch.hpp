// Host-side declarations of the kernel launchers (defined in the .hip files).
#pragma once

#include "kernels.hpp"

namespace almbm {

// Hub-row neighbour sums of C X into out (no-op when C has no hubs).
// lb: the L-BFGS rings (empty: gradient descent).  With rings, the row kernels
// step along the ring's current direction E instead of G and the gradient
// passes write y_k = G_new - G_old (ring type RingT<T>); the line-search
// product (instantiated for the ring type) multiplies E.
template <typename T>
void launch_hub_rows(const Cost<typename Acc<T>::type>& C, int r, int variant, const T* X,
                     typename Acc<T>::type* out, const DevScalars* sc, int refresh_every, hipStream_t st,
                     const LbfgsRing<T>& lb = LbfgsRing<T>{});
template <typename T>
void launch_objgrad_diag(const Cost<typename Acc<T>::type>& C, int r, int variant, const T* R, const double* y,
                         const double* b, double sigma, T* G, double* Av, double* part, const DevScalars* sc,
                         int refresh_every, const BlockTab& tab, int nblk, hipStream_t st,
                         const LbfgsRing<RingT<T>>& lb = LbfgsRing<RingT<T>>{});
template <typename T>
void launch_quadq_diag(const Cost<typename Acc<T>::type>& C, int r, int variant, const T* G,
                       typename Acc<T>::type* Q, double* part, const DevScalars* sc, const BlockTab& tab, int nblk,
                       hipStream_t st, const LbfgsRing<T>& lb = LbfgsRing<T>{}, const SideFin& side = SideFin{});
template <typename T>
void launch_upd_eval_diag(long n, int r, int variant, T* R, T* G, const typename Acc<T>::type* Q, const double* y,
                          const double* b, double sigma, double* Av, double* part, const DevScalars* sc,
                          int refresh_every, const BlockTab& tab, int nblk, hipStream_t st,
                          const LbfgsRing<RingT<T>>& lb = LbfgsRing<RingT<T>>{});
// L-BFGS steps (lbfgs_kernels.hip).  Reset at the start of a subproblem.
// Empty memories of m pairs for `count` instances (states s[0..count)).
void launch_lbfgs_reset(LbfgsState* s, int m, hipStream_t st, int count = 1);
// Inner products of the new gradient G and of y_k with the stored vectors of a
// memory of m pairs (len = n*r elements each without a table; with one, the
// rows of each block at width r), lbfgs_dot_slots of them per block of at most
// nb blocks; returns the blocks launched.
template <typename T>
int launch_lbfgs_dots(long len, int r, int m, const T* G, const LbfgsRing<RingT<T>>& lb, double* part, int nb,
                      const DevScalars* sc, hipStream_t st, const BlockTab& tab = BlockTab{},
                      const SideFin& side = SideFin{});
// Pair update and the coefficients of the next direction (one block per
// instance) from the partials of nb blocks.
void launch_fin_lbfgs(const double* part, int nb, int m, const DevScalars* sc, LbfgsState* s, hipStream_t st,
                      const BlockTab& tab = BlockTab{}, int count = 1);
// E = cg G + sum (ce E_a + cy y_a) into the current slot, and the quartic's
// direction-dependent partial sums along -E (NUM_P per block).
template <typename T>
void launch_lbfgs_combine(long n, int r, int variant, const T* R, const T* G, const double* y, const double* b,
                          double sigma, const double* Av, const LbfgsRing<RingT<T>>& lb, double* part,
                          const DevScalars* sc, int nblk, hipStream_t st, const BlockTab& tab = BlockTab{});
// Direction-dependent totals of the quartic from the combine partials (one block per instance).
void launch_fin_lsdir(const double* part, int nb, DevScalars* sc, LbfgsState* s, hipStream_t st,
                      const BlockTab& tab = BlockTab{}, int count = 1);
// Rows that a block of the row kernels takes at a time at rank r.
template <typename T> int diag_rows_per_trip(int r, int variant);
// Grid of a single evaluation or line search where nb is the default grid for n rows.
template <typename T> int diag_call_blocks(long n, int r, int variant, int nb);
template <typename T>
void launch_quad_diag(const Cost<typename Acc<T>::type>& C, int r, int variant, const T* G, double* part,
                      const DevScalars* sc, int nblk, hipStream_t st);
template <typename T>
void launch_ls_diag(const Cost<typename Acc<T>::type>& C, int r, int variant, const T* R, const T* G,
                    const double* y, const double* b, double* part, int nblk, hipStream_t st);

// Objective and gradient of the edge family at R (passes 1 and 2 and their
// finalizers).  With G_in the direction is read instead of computed and G is
// not written (line-search API).  mode and f_out as for launch_fin_objgrad.  With
// defer the last finalizer is left to launch_edges_p3.
template <typename T>
void launch_edges_eval(const Cost<typename Acc<T>::type>& C, const EdgeAdj& A, long n, int r, int variant, const T* R,
                       const double* y, const double* b, double sigma, double c_tr, double j_coef, double rho,
                       double* Av, double* wE, const T* G_in, T* G, double* part, DevScalars* sc, int nblk, int mode,
                       double* f_out, hipStream_t st, EdgeFin* defer = nullptr);
// side: a deferred finalizer, run by a block of pass 3.  Returns the table that pass 3
// leaves its partial sums in.
template <typename T>
double* launch_edges_p3(const Cost<typename Acc<T>::type>& C, const EdgeAdj& A, int r, int variant, const T* R,
                        const T* G, const double* y, const double* b, const double* Av, double* part,
                        const DevScalars* sc, int nblk, hipStream_t st, double rho = 1.0,
                        const EdgeFin& side = EdgeFin{});
void launch_fin_edges3(const double* part, int nb, int r, DevScalars* sc, const double* y, const double* b,
                       double sigma, double c_tr, double j_coef, int mode, double* coeffs_out, double* t_out,
                       hipStream_t st);

void launch_fin_objgrad(const double* part, int nb, DevScalars* sc, double sigma, int mode, double* f_out,
                        hipStream_t st, const BlockTab& tab = BlockTab{}, int count = 1);
void launch_fin_step(const double* part_c2, int nb, DevScalars* sc, double sigma, int mode, double* coeffs_out,
                     double* t_out, hipStream_t st, const BlockTab& tab = BlockTab{}, int count = 1);
void launch_dual_batch(long m, const double* Av, const double* b, const double* y_in, double* y_out, double sigma,
                       double* part, DevScalars* sc, const double* bnorms, const BlockTab& tab, int nb, int count,
                       hipStream_t st);
void launch_inner_reset_batch(DevScalars* sc, int count, const double* tols, const int32_t* active, int max_inner,
                              int step_rule, double eta, hipStream_t st);
void launch_copy_active(long m, const double* src, double* dst, const int32_t* active, const BlockTab& tab, int nb,
                        hipStream_t st);
template <typename T>
void launch_fill_column(long n, int rs, T* R, const double* v, const int32_t* col, const double* scale,
                        const BlockTab& tab, int nb, hipStream_t st);
void launch_fin_ls(const double* part, int nb, DevScalars* sc, double sigma, double* coeffs_out, double* t_out,
                   hipStream_t st);
template <typename T>
void launch_update(long len, T* R, const T* G, const DevScalars* sc, int use_flag, hipStream_t st);
int dual_blocks(long m);
// y_out = y_in - sigma (Av - b) on row 0 and - sigma_tail (Av - b) on the other
// rows (sigma_tail <= 0: sigma everywhere).
void launch_dual(long m, const double* Av, const double* b, const double* y_in, double* y_out, double sigma,
                 double* part, DevScalars* sc, double bnorm, double* pinf_out, hipStream_t st,
                 double sigma_tail = 0.0);
void launch_inner_reset(DevScalars* sc, double tol, int max_inner, int step_rule, double eta, hipStream_t st);
template <typename T>
void launch_set_column(long n, int rs, int c, T* R, const double* v, double scale, hipStream_t st);
template <typename T>
void launch_restride_batch(const BlockTab& tab, int nb, const T* src, T* dst, const int64_t* ob, const int32_t* os,
                           const int64_t* nbase, const int32_t* ns, const int32_t* nc, hipStream_t st);
template <typename T>
void launch_relayout(long n, int ss, int nc, int rd, const T* src, T* dst, const double* v, double scale,
                     hipStream_t st);
template <typename S, typename D>
void launch_convert(long len, const S* src, D* dst, hipStream_t st);

int vec_blocks(long n, bool ordered = false);
// out = Z(y) x; qsum: 1^T x where the cost has a -J term.
void launch_slack_mv(const Cost<double>& C, int cons_kind, const EdgeAdj& A, const double* y, double c_tr,
                     double j_coef, const double* qsum, const double* x, double* out, hipStream_t st);
void launch_slack_mv_tab(const Cost<double>& C, const double* y, const double* x, double* out, int nb, hipStream_t st,
                         const VecBatch& vb);
// A step of the Lanczos recurrence.  The vector kernels leave partial sums per
// block at part[c * pld + slot]; up to kLzFewBlocks of them are added by the
// kernel that needs the total instead of by a finalizer of their own (single
// instances: at 64 blocks, n = 16384, every block adds 64 values per column;
// beyond, a finalizer costs less than the repeated sums).
constexpr int kLzFewBlocks = 64;
struct LzStep {
  int j;               // column of this step
  const double* part;  // partial sums of ||w||^2 and of w (launch_gs2's part_n)
  int nb;
  int pld;
  const double* h1;    // projections of step j - 1
  const double* h2;
  double* alpha;       // tridiagonal entries
  double* beta;
  bool sums;           // step j - 1 ended without launch_fin_ab
};
// out = Z(y) q_j with q_j = w / beta_{j-1} stored at qcol; for j = 0 w is q_0.
// qsum: 1^T q_j where the cost has a -J term (launch_fin_ab's, or q_0's).
void launch_lz_mv(const Cost<double>& C, int cons_kind, const EdgeAdj& A, const double* y, double c_tr, double j_coef,
                  const double* qsum, const LzStep& s, const double* w, double* qcol, double* out, int nb,
                  hipStream_t st, const VecBatch& vb = VecBatch{});
// h = Q^T w (first ncol columns).
void launch_dots(long n, int ncol, const double* Q, long ldq, double* w, double* part, int pld, int nb, double* h,
                 hipStream_t st, const VecBatch& vb = VecBatch{});
// Two classical Gram-Schmidt passes of w against the first ncol columns:
// coefficients h1, h2; partial sums of ||w||^2 and of w in part_n (2 x pld).
// part, part_b: ncol x pld.
void launch_gs2(long n, int ncol, const double* Q, long ldq, double* w, double* part, double* part_b, double* part_n,
                int pld, int nb, double* h1, double* h2, hipStream_t st, const VecBatch& vb = VecBatch{});
// launch_gs2 with sums whose order follows from n and nb alone (single
// instances), for alm_bm_lanczos_min_eig and for costs with hub rows.  A pass
// restarted from a Ritz vector brings the rounding of the one before, in the
// directions that it has found already, back to size one, so that another order
// of sums gives another vector (Poisson degrees, n = 1e6, two passes: 1.7e-8
// apart) or, on power-law costs, another residual (R-MAT 2^13, four passes: 5 %).
void launch_gs2_ordered(long n, int ncol, const double* Q, long ldq, double* w, double* part, double* part_n, int pld,
                        int nb, double* h1, double* h2, hipStream_t st);
void launch_fin_ab(const double* part, int nb, int pld, const double* h1, const double* h2, int j, double* alpha,
                   double* beta, double* qsum, hipStream_t st, const VecBatch& vb = VecBatch{});
void launch_scale(long n, const double* w, const double* beta, double* q, double* part, int nb, double* qsum,
                  hipStream_t st, const VecBatch& vb = VecBatch{}, int bstride = 0);
void launch_gather_flags(const DevScalars* sc, int count, int32_t* out, hipStream_t st);
void launch_fin_sum(const double* part, int nb, double* out, int do_sqrt, hipStream_t st,
                    const VecBatch& vb = VecBatch{}, int ostride = 0);
void launch_rand(long n, uint64_t seed, double* x, double* part, int nb, hipStream_t st,
                 const VecBatch& vb = VecBatch{});
// x <- v + eps x / ||x|| per instance (norms[inst * nstride]), partial ||x||^2.
void launch_mix(long n, double eps, const double* v, double* x, const double* norms, int nstride, double* part,
                int nb, hipStream_t st, const VecBatch& vb = VecBatch{});
// Fourth moments of q <= 8 directions (V n x q column-major) per block of the
// nb-block grid: part[b * ne + e], ne = np (np + 1) / 2, np = q (q + 1) / 2.
void launch_gram4(long n, int q, const double* V, double* part, int nb, hipStream_t st);
// The edge-row moments of the trace + edge family (edges ei[e] < ej[e], E of them).
void launch_gram4_edges(long E, long n, int q, const int32_t* ei, const int32_t* ej, const double* V, double* part,
                        int nb, hipStream_t st);
// v = sum_{c < ncol} Q[:, c] s[c] (per instance s + inst * hstride; with
// ncols, at most ncols[inst] columns), partial ||v||^2.
void launch_combine(long n, int ncol, const double* Q, long ldq, const double* s, double* v, double* part, int nb,
                    hipStream_t st, const VecBatch& vb = VecBatch{}, const int32_t* ncols = nullptr);
void launch_resid(long n, const double* z, const double* v, double theta, const double* thetas, double* part, int nb,
                  hipStream_t st, const VecBatch& vb = VecBatch{});
void launch_quartic_norm(long n, int cons_kind, const EdgeAdj& A, const double* x, double* part, int nb,
                         hipStream_t st, const VecBatch& vb = VecBatch{});

// pair: n float2 of scratch.
void launch_ws_features(const Cost<double>& C, float* F, float2* pair, hipStream_t st);
int ws_param_count(int nin, int h);
bool launch_ws_forward(const float* P, int nin, int h, const float* mu, const float* isd, long n, const float* X,
                       double* out, hipStream_t st);
void launch_ws_pool(const float* F, long n, double* part, int nb, double* out, hipStream_t st);
bool launch_ws_backward(const float* P, int nin, int h, const float* mu, const float* isd, long n, const float* X,
                        const float* T, float* gpart, double* lpart, int nb, float* grad, double* loss,
                        hipStream_t st);
void launch_ws_adam(float* P, const float* g, float* m, float* v, int np, float lr, float b1, float b2, float eps,
                    int step, hipStream_t st);

}  // namespace almbm
