// Lanczos for lambda_min of the dual slack Z(y) = C - A*(y) (Sec. 1.2), used
// by the KKT measure of Sec. 6 and the rank test of Alg. 1.  Everything in FP64:
// the matrix-free product, dot products and the full reorthogonalisation
// (classical Gram-Schmidt applied twice) against the stored basis Q
// (column-major, n x (k+1), leading dimension ldq).
#include "launch.hpp"

namespace almbm {

constexpr int kSpmvLpr = 4;  // lanes per row in the slack product (avg degree ~ 8)

// ---- Lanczos step ------------------------------------------------------------------
//
// One step on column j: k_lz_mv (q_j = w / beta and w' = Z q_j), then two
// classical Gram-Schmidt passes: dots of w' with the basis, w' -= Q h together
// with the dots of the second pass (one read of the basis for both), w' -= Q h
// again with ||w'||^2.  Three reads of the basis per step, the two passes'
// definition being the same as with four.  Partial sums per block at
// part[c * pld + slot] (column-major, so that a column's finalizer reads
// contiguously).

// Projection coefficients of a column block: either reduced (h + inst * hstride)
// or, when few blocks hold them, the partial sums themselves (part, nb of them
// per column), which every block then adds in the same order, saving the
// finalizer's launch; block 0 leaves the totals at out.
struct LzCoef {
  const double* h = nullptr;
  int hstride = 0;
  const double* part = nullptr;
  int nb = 0;
  int pld = 0;
  double* out = nullptr;
};

__device__ __forceinline__ double sum_strided4(const double* __restrict__ p, int nb) {
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  int b = 0;
  for (; b + 4 <= nb; b += 4) {
    a0 += p[b];
    a1 += p[b + 1];
    a2 += p[b + 2];
    a3 += p[b + 3];
  }
  for (; b < nb; ++b) a0 += p[b];
  return (a0 + a1) + (a2 + a3);
}

// hs[c] (shared) for c < ncol, zero up to the next multiple of 16.
__device__ __forceinline__ void load_coef(const LzCoef& hc, int inst, int ncol, double* __restrict__ hs) {
  for (int c = threadIdx.x; c < (ncol + 15) / 16 * 16; c += kBlock) {
    double x = 0.0;
    if (c < ncol) {
      x = hc.part ? sum_strided4(hc.part + (long)c * hc.pld, hc.nb) : hc.h[(long)inst * hc.hstride + c];
      if (hc.part && blockIdx.x == 0) hc.out[c] = x;
    }
    hs[c] = x;
  }
  __syncthreads();
}

// Per-block partial sums of q_c . w into part; SUB: of the w left by w -= Q h.  A thread
// owns a row and holds its entries of all ncol <= NC columns at once, so a wave
// has ncol 512-byte loads in flight; the columns' dots are summed over the wave
// by halving, which leaves column l / (64 / NC) in lane l.  Bound by HBM: over a
// 56-column pass at n = 1e6 the dots run at 5.2 TB/s and with SUB at 4.7
// TB/s, where column-per-wave dots and row-per-thread subtraction on 248 blocks
// ran at 3.0 and 3.5 TB/s and read the basis once more.
template <int NC, bool SUB>
__global__ void __launch_bounds__(kBlock)
k_lz_proj(long n, int ncol, const double* __restrict__ Q, long ldq, LzCoef hc, double* __restrict__ w,
          double* __restrict__ part, int pld, BlockTab tab) {
  const Rows ch = rows_of(n, tab);
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  __shared__ double hs[SUB ? NC : 1];
  if constexpr (SUB) load_coef(hc, ch.inst, ncol, hs);
  double acc = 0.0;
  for (long base = ch.lo; base < ch.hi; base += kBlock) {
    const long i = base + threadIdx.x;
    const bool in = i < ch.hi;
    double q[NC];
    double v = in ? w[i] : 0.0;
#pragma unroll
    for (int g = 0; g < NC; g += 8) {
#pragma unroll
      for (int c = g; c < g + 8; ++c) q[c] = 0.0;
      if (g < ncol && in) {
#pragma unroll
        for (int c = g; c < g + 8; ++c) q[c] = Q[(long)(c < ncol ? c : ncol - 1) * ldq + i];
      }
    }
    if constexpr (SUB) {
      double s[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int g = 0; g < NC; g += 8) {
        if (g < ncol) {
#pragma unroll
          for (int c = g; c < g + 8; ++c) s[c % 4] += q[c] * hs[c];
        }
        __builtin_amdgcn_sched_barrier(0);  // eight coefficients from LDS at a time, not NC of them in registers
      }
      v -= (s[0] + s[1]) + (s[2] + s[3]);
      if (in) w[i] = v;
      if (!in) v = 0.0;
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) q[c] *= v;
    acc += wave_sum_many<NC>(q, lane);
  }
  __shared__ double red[kBlock / kWave][NC];
  constexpr int W = kWave / NC;
  if (lane % W == 0) red[wave][lane / W] = acc;
  __syncthreads();
  for (int c = threadIdx.x; c < ncol; c += kBlock) {
    double t = 0.0;
#pragma unroll
    for (int k = 0; k < kBlock / kWave; ++k) t += red[k][c];
    part[(long)c * pld + part_slot(tab)] = t;
  }
}

// The same for more than 64 columns (DOTS), and for any number without the dots, with
// partial sums of ||w||^2 and of w in part[slot] and part[pld + slot] instead: the
// columns go by in chunks of CH, and SUB + DOTS reads them twice (the second time the
// block's tile is in L2 or the Infinity Cache).
template <bool SUB, bool DOTS>
__global__ void __launch_bounds__(kBlock)
k_lz_proj_wide(long n, int ncol, const double* __restrict__ Q, long ldq, LzCoef hc, double* __restrict__ w,
               double* __restrict__ part, int pld, BlockTab tab) {
  constexpr int CH = 32, CS = 16;  // columns in flight per thread: dots, subtraction
  constexpr int MAXC = 512 + CS;
  const Rows ch = rows_of(n, tab);
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  __shared__ double hs[SUB ? MAXC : 1];
  __shared__ double red[DOTS ? kBlock / kWave : 1][DOTS ? MAXC + CH : 1];
  if constexpr (SUB) load_coef(hc, ch.inst, ncol, hs);
  if constexpr (DOTS) {
    for (int c = lane; c < MAXC + CH; c += kWave) red[wave][c] = 0.0;
  }
  double nrm = 0.0, sum = 0.0;
  for (long base = ch.lo; base < ch.hi; base += kBlock) {
    const long i = base + threadIdx.x;
    const bool in = i < ch.hi;
    double v = in ? w[i] : 0.0;
    if constexpr (SUB) {
      double s[4] = {0.0, 0.0, 0.0, 0.0};
      if (in) {
        for (int c0 = 0; c0 < ncol; c0 += CS) {
          double q[CS];
#pragma unroll
          for (int c = 0; c < CS; ++c) q[c] = Q[(long)(c0 + c < ncol ? c0 + c : ncol - 1) * ldq + i];
#pragma unroll
          for (int c = 0; c < CS; ++c) s[c % 4] += q[c] * hs[c0 + c];
        }
        v -= (s[0] + s[1]) + (s[2] + s[3]);
        w[i] = v;
      }
    }
    if constexpr (DOTS) {
      for (int c0 = 0; c0 < ncol; c0 += CH) {
        double q[CH];
#pragma unroll
        for (int c = 0; c < CH; ++c) q[c] = in ? Q[(long)(c0 + c < ncol ? c0 + c : ncol - 1) * ldq + i] * v : 0.0;
        const double x = wave_sum_many<CH>(q, lane);
        if (lane % (kWave / CH) == 0) red[wave][c0 + lane / (kWave / CH)] += x;
      }
    } else {
      nrm += v * v;
      sum += v;
    }
  }
  if constexpr (DOTS) {
    __syncthreads();
    for (int c = threadIdx.x; c < ncol; c += kBlock) {
      double t = 0.0;
#pragma unroll
      for (int k = 0; k < kBlock / kWave; ++k) t += red[k][c];
      part[(long)c * pld + part_slot(tab)] = t;
    }
  } else {
    double two[2] = {nrm, sum};
    __shared__ double out[2];
    block_sum_store<2>(two, out);
    __syncthreads();
    if (threadIdx.x < 2) part[(long)threadIdx.x * pld + part_slot(tab)] = out[threadIdx.x];
  }
}

// The same projections with every sum in an order of the row count alone
// (launch_gs2_ordered): a wave per column and row chunk, four running sums
// per lane; the subtraction column by column; the norm over row chunks.
__global__ void __launch_bounds__(kBlock)
k_dots_ordered(long n, int ncol, const double* __restrict__ Q, long ldq, const double* __restrict__ w,
               double* __restrict__ part, int pld) {
  const RowChunk ch = row_chunk(n);
  const int lane = threadIdx.x % kWave;
  const int c = blockIdx.y * (kBlock / kWave) + threadIdx.x / kWave;
  if (c >= ncol) return;
  const double* q = Q + (long)c * ldq;
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  long i = ch.lo + lane;
#pragma unroll 4
  for (; i + 3 * kWave < ch.hi; i += 4 * kWave) {
    a0 += q[i] * w[i];
    a1 += q[i + kWave] * w[i + kWave];
    a2 += q[i + 2 * kWave] * w[i + 2 * kWave];
    a3 += q[i + 3 * kWave] * w[i + 3 * kWave];
  }
  for (; i < ch.hi; i += kWave) a0 += q[i] * w[i];
  const double a = wave_sum((a0 + a1) + (a2 + a3));
  if (lane == 0) part[(long)c * pld + blockIdx.x] = a;
}

__global__ void __launch_bounds__(kBlock)
k_sub_ordered(long n, int ncol, const double* __restrict__ Q, long ldq, const double* __restrict__ h,
              double* __restrict__ w) {
  constexpr int CS = 16;
  __shared__ double hs[512 + CS];
  LzCoef hc;
  hc.h = h;
  load_coef(hc, 0, ncol, hs);
  const long i = (long)blockIdx.x * kBlock + threadIdx.x;
  if (i >= n) return;
  double v = w[i];
  for (int c0 = 0; c0 < ncol; c0 += CS) {
    double q[CS];
#pragma unroll
    for (int c = 0; c < CS; ++c) q[c] = Q[(long)(c0 + c < ncol ? c0 + c : ncol - 1) * ldq + i];
#pragma unroll
    for (int c = 0; c < CS; ++c) v -= q[c] * hs[c0 + c];
  }
  w[i] = v;
}

// k_sub_ordered and the k_dots_ordered after it with one read of the basis, for up
// to NC columns, bit for bit: a thread owns a row of each 256-row trip, so that wave
// k's threads hold what the lanes' running sums a_k of k_dots_ordered hold, and the
// rows of a last, partial trip go to a_0 in their order as there.  A thread keeps its
// row's NC entries and NC sums in registers (one wave per SIMD for NC = 64, with all
// loads of a trip in flight).  Bound by HBM: n = 1e6, 33 to 56 columns, 88 us (4.2
// TB/s) against 58 + 85 us as two kernels.  One block per row chunk cannot fill the
// chip with fewer than 128 of them (n = 5.2e5), where the two kernels stay.
template <int NC>
__global__ void __launch_bounds__(kBlock)
k_sub_dots_ordered(long n, int ncol, const double* __restrict__ Q, long ldq, const double* __restrict__ h,
                   double* __restrict__ w, double* __restrict__ part, int pld) {
  constexpr int G = 16;  // columns added up together at the end
  __shared__ double hs[NC];
  __shared__ double vs[kBlock];
  __shared__ double sm[kBlock / kWave][G][kWave];
  LzCoef hc;
  hc.h = h;
  load_coef(hc, 0, ncol, hs);
  const RowChunk ch = row_chunk(n);
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  double acc[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) acc[c] = 0.0;
  for (long base = ch.lo; base < ch.hi; base += kBlock) {
    const long i = base + threadIdx.x;
    const bool in = i < ch.hi;
    double q[NC];
    double v = in ? w[i] : 0.0;
#pragma unroll
    for (int g = 0; g < NC; g += 8) {
#pragma unroll
      for (int c = g; c < g + 8; ++c) q[c] = 0.0;
      if (g < ncol && in) {
#pragma unroll
        for (int c = g; c < g + 8; ++c) q[c] = Q[(long)(c < ncol ? c : ncol - 1) * ldq + i];
      }
    }
#pragma unroll
    for (int g = 0; g < NC; g += 8) {
      if (g < ncol) {
#pragma unroll
        for (int c = g; c < g + 8; ++c) v -= q[c] * hs[c];
      }
      __builtin_amdgcn_sched_barrier(0);  // eight coefficients from LDS at a time
    }
    if (in) w[i] = v;
    if (base + lane + (kBlock - kWave) < ch.hi) {
#pragma unroll
      for (int c = 0; c < NC; ++c) acc[c] += q[c] * v;
    }
    if (base + kBlock > ch.hi) {  // the last, partial trip
      vs[threadIdx.x] = v;
      __syncthreads();
      if (wave == 0 && base + lane + (kBlock - kWave) >= ch.hi) {
        for (int k = 0; k < kBlock / kWave - 1; ++k) {
          const long row = base + lane + k * kWave;
          if (row >= ch.hi) break;
          const double x = vs[lane + k * kWave];
#pragma unroll
          for (int c = 0; c < NC; ++c) acc[c] += Q[(long)(c < ncol ? c : ncol - 1) * ldq + row] * x;
        }
      }
    }
  }
#pragma unroll
  for (int c0 = 0; c0 < NC; c0 += G) {
    if (c0 >= ncol) break;
#pragma unroll
    for (int c = 0; c < G; ++c) sm[wave][c][lane] = acc[c0 + c];
    __syncthreads();
#pragma unroll
    for (int k = 0; k < G / (kBlock / kWave); ++k) {
      const int c = wave * (G / (kBlock / kWave)) + k;
      const double a = wave_sum((sm[0][c][lane] + sm[1][c][lane]) + (sm[2][c][lane] + sm[3][c][lane]));
      if (lane == 0 && c0 + c < ncol) part[(long)(c0 + c) * pld + blockIdx.x] = a;
    }
    __syncthreads();
  }
}

__global__ void __launch_bounds__(kBlock)
k_norm_ordered(long n, const double* __restrict__ w, double* __restrict__ part, int pld) {
  const RowChunk ch = row_chunk(n);
  double acc[1] = {0.0};
  for (long i = ch.lo + threadIdx.x; i < ch.hi; i += kBlock) {
    const double v = w[i];
    acc[0] += v * v;
  }
  block_sum_store<1>(acc, part + blockIdx.x);
  if (threadIdx.x == 0) part[(long)pld + blockIdx.x] = 0.0;  // the sum of w is for -J terms only
}

// h[q][c] = sum of the block partials of column c over instance q's blocks
// (grid: columns x instances, fixed order).
__global__ void __launch_bounds__(kBlock)
k_fin_dots(const double* __restrict__ part, int nb, int pld, int ncol, double* __restrict__ h, int hstride,
           BlockTab tab) {
  const int c = blockIdx.x, q = blockIdx.y;
  if (c >= ncol) return;
  int b0, b1;
  inst_blocks(tab, q, nb, b0, b1);
  double acc[1] = {0.0};
  for (int b = b0 + threadIdx.x; b < b1; b += kBlock) acc[0] += part[(long)c * pld + b];
  block_sum_store<1>(acc, h + (long)q * hstride + c);
}

// Tridiagonal entries after the two projections: alpha_j = h1[j] + h2[j],
// beta_j = ||w||; qsum (nullable): 1^T w / beta_j, the sum of the next column.
__global__ void __launch_bounds__(kBlock)
k_fin_ab(const double* __restrict__ part, int nb, int pld, const double* __restrict__ h1,
         const double* __restrict__ h2, int hstride, int j, double* __restrict__ alpha, double* __restrict__ beta,
         int astride, double* __restrict__ qsum, BlockTab tab) {
  const int q = blockIdx.x;
  int b0, b1;
  inst_blocks(tab, q, nb, b0, b1);
  h1 += (long)q * hstride;
  h2 += (long)q * hstride;
  alpha += (long)q * astride;
  beta += (long)q * astride;
  double acc[2] = {0.0, 0.0};
  for (int b = b0 + threadIdx.x; b < b1; b += kBlock) {
    acc[0] += part[b];
    acc[1] += part[(long)pld + b];
  }
  __shared__ double tot[2];
  block_sum_store<2>(acc, tot);
  __syncthreads();
  if (threadIdx.x == 0) {
    alpha[j] = h1[j] + h2[j];
    const double bj = sqrt(tot[0]);
    beta[j] = bj;
    if (qsum) *qsum = bj > 0.0 ? tot[1] / bj : 0.0;
  }
}

// Scaling of the incoming vector of k_lz_mv: none (part and beta null: w is q_j
// already and qsum its sum), beta at beta + inst * bstride with qsum given, or
// from nb partial sums of ||w||^2 and of w, which every block adds alike; block
// 0 then also writes the tridiagonal entries of step j - 1.
struct LzScale {
  const double* beta = nullptr;
  int bstride = 0;
  const double* part = nullptr;
  int nb = 0;
  int pld = 0;
  const double* h1 = nullptr;
  const double* h2 = nullptr;
  double* alpha_out = nullptr;  // entry j - 1
  double* beta_out = nullptr;
  int jm1 = 0;
};

// q = w / beta stored (when scaled), out = Z(y) q, gathering w and scaling each
// entry as it comes (the same product as from q):
// DIAG: (d_i - y_i) q_i + sum_k S_ik q_k.
// TRACE_EDGES: (S q)_i + d_i q_i - j (1^T q) - c_tr y_0 q_i - 1/2 sum_{k~i} y_{1+e(ik)} q_k.
// L lanes per row, U entries of the row in flight per lane, so that a row of up
// to 16 entries costs one trip through the index and gather latencies.  Bound
// by the gathers: n = 1e6, 8e6 entries (8 MB vector, two L2 slices' worth): 109
// us one entry at a time, 101 us with four (79e9 gathers/s); non-temporal index
// and value loads made it 125 us (they no longer come from the Infinity Cache).
// A batch of 24 instances, n = 275 113 together, 5.0e6 entries (vectors of 320 KB at
// most, from the L2): 43 us with 256 rows a block, 34 us with 64.
__global__ void __launch_bounds__(kBlock)
k_lz_mv(Cost<double> C, int cons_kind, EdgeAdj A, const double* __restrict__ y, double c_tr, double j_coef,
        const double* __restrict__ qsum_in, LzScale sc, const double* __restrict__ w, double* __restrict__ qcol,
        double* __restrict__ out, BlockTab tab) {
  constexpr int L = kSpmvLpr;
  constexpr int U = 4;
  constexpr int RPB = kBlock / L;
  const Rows ch = rows_of(C.n, tab, C.skewed);
  const int lane = threadIdx.x % L;
  double inv = 1.0, qsum = (j_coef != 0.0 && qsum_in) ? *qsum_in : 0.0;
  const bool scaled = sc.part || sc.beta;
  if (sc.part) {
    const double b2 = sum_strided4(sc.part, sc.nb);
    const double beta = sqrt(b2);
    inv = beta > 0.0 ? 1.0 / beta : 0.0;
    if (j_coef != 0.0) qsum = beta > 0.0 ? sum_strided4(sc.part + sc.pld, sc.nb) / beta : 0.0;
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) {
      *sc.alpha_out = sc.h1[sc.jm1] + sc.h2[sc.jm1];
      *sc.beta_out = beta;
    }
  } else if (sc.beta) {
    const double beta = sc.beta[(long)ch.inst * sc.bstride];
    inv = beta > 0.0 ? 1.0 / beta : 0.0;
  }
  for (long base = ch.lo + (long)blockIdx.y * RPB; base < ch.hi; base += (long)gridDim.y * RPB) {
    const long i = base + threadIdx.x / L;
    const bool in = i < ch.hi;
    double acc = 0.0;
    if (in) {
      long k0 = 0, k1 = 0;
      if (C.ell > 0) {
        k0 = i * (long)C.ell;
        k1 = k0 + C.ell;
      } else if (C.rp) {
        k0 = C.rp[i];
        k1 = C.rp[i + 1];
      }
      if (C.nh > 0 && k1 - k0 > C.hthr) {  // hub row: sum of the unscaled vector precomputed by k_hub_rows
        if (lane == 0) acc = C.hsum[hub_index(C, i)] * inv;
      } else {
        for (long k = k0 + lane; k < k1; k += L * U) {
          int j[U];
          double c[U], x[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const long kk = k + u * L;
            j[u] = kk < k1 ? C.ci[kk] : (int)i;
            c[u] = kk < k1 ? C.cv[kk] : 0.0;
          }
#pragma unroll
          for (int u = 0; u < U; ++u) x[u] = w[j[u]];
#pragma unroll
          for (int u = 0; u < U; ++u)
            if (k + u * L < k1) acc += c[u] * (x[u] * inv);
        }
      }
      if (cons_kind == 1) {
        const int a0 = A.rp[i], a1 = A.rp[i + 1];
        for (int k = a0 + lane; k < a1; k += L) acc -= 0.5 * y[1 + A.eid[k]] * (w[A.ci[k]] * inv);
      }
    }
    acc = group_sum<L>(acc);
    if (in && lane == 0) {
      const double xi = w[i] * inv;
      if (scaled) qcol[i] = xi;
      double d = C.dg ? C.dg[i] : 0.0;
      if (cons_kind == 0) d -= y[i];
      else d -= c_tr * y[0];
      double v = acc + d * xi;
      if (j_coef != 0.0) v -= j_coef * qsum;
      out[i] = v;
    }
  }
}

// q = w / beta (beta > 0), partial sums of q for the -jJ term.
__global__ void __launch_bounds__(kBlock)
k_scale(long n, const double* __restrict__ w, const double* __restrict__ beta_ptr, int bstride, double* __restrict__ q,
        double* __restrict__ part, BlockTab tab) {
  const Rows ch = rows_of(n, tab);
  const double beta = beta_ptr[(long)ch.inst * bstride];
  const double inv = beta > 0.0 ? 1.0 / beta : 0.0;
  double acc[1] = {0.0};
  for (long i = ch.lo + threadIdx.x; i < ch.hi; i += kBlock) {
    const double v = w[i] * inv;
    q[i] = v;
    acc[0] += v;
  }
  block_sum_store<1>(acc, part + part_slot(tab));
}

__global__ void __launch_bounds__(kBlock)
k_fin_sum(const double* __restrict__ part, int nb, double* __restrict__ out, int ostride, int do_sqrt, BlockTab tab) {
  const int q = blockIdx.x;
  int b0, b1;
  inst_blocks(tab, q, nb, b0, b1);
  out += (long)q * ostride;
  __shared__ double red[kBlock / kWave];
  double a = 0.0;
  for (int b = b0 + threadIdx.x; b < b1; b += kBlock) a += part[b];
  a = wave_sum(a);
  if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = a;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < kBlock / kWave; ++w) t += red[w];
    *out = do_sqrt ? sqrt(t) : t;
  }
}

// Start vector: counter-based uniform entries, partial ||x||^2.
__global__ void __launch_bounds__(kBlock)
k_rand(long n, uint64_t seed, double* __restrict__ x, double* __restrict__ part, BlockTab tab) {
  const Rows ch = rows_of(n, tab);
  double acc[1] = {0.0};
  for (long i = ch.lo + threadIdx.x; i < ch.hi; i += kBlock) {
    const double v = counter_uniform(seed, (uint64_t)i);
    x[i] = v;
    acc[0] += v * v;
  }
  block_sum_store<1>(acc, part + part_slot(tab));
}

// Warm start of a Lanczos pass: x = v + eps x / ||x|| per instance (x holds a
// random vector whose per-instance norm is at norms[inst * nstride], v the
// previous unit Ritz vector); partial ||x||^2.  The random share keeps every
// eigenvector in the start, so a bottom eigenvector that moved away from v is
// still found.
__global__ void __launch_bounds__(kBlock)
k_mix(long n, double eps, const double* __restrict__ v, double* __restrict__ x, const double* __restrict__ norms,
      int nstride, double* __restrict__ part, BlockTab tab) {
  const Rows ch = rows_of(n, tab);
  const double a = eps / fmax(norms[(long)ch.inst * nstride], 1e-300);
  double acc[1] = {0.0};
  for (long i = ch.lo + threadIdx.x; i < ch.hi; i += kBlock) {
    const double t = v[i] + a * x[i];
    x[i] = t;
    acc[0] += t * t;
  }
  block_sum_store<1>(acc, part + part_slot(tab));
}

// v = sum_c Q[c] s[c]; partial ||v||^2.
__global__ void __launch_bounds__(kBlock)
k_combine(long n, int ncol, const double* __restrict__ Q, long ldq, const double* __restrict__ s, int sstride,
          double* __restrict__ v, double* __restrict__ part, BlockTab tab, const int32_t* __restrict__ ncols) {
  const Rows ch = rows_of(n, tab);
  // per-instance basis sizes: columns past an instance's own count were not
  // written for its rows in this pass
  if (ncols && ncols[ch.inst] < ncol) ncol = ncols[ch.inst];
  __shared__ double ss[512 + 1];
  for (int c = threadIdx.x; c < ncol; c += kBlock) ss[c] = s[(long)ch.inst * sstride + c];
  __syncthreads();
  double acc[1] = {0.0};
  for (long i = ch.lo + threadIdx.x; i < ch.hi; i += kBlock) {
    double a = 0.0;
    for (int c = 0; c < ncol; ++c) a += Q[(long)c * ldq + i] * ss[c];
    v[i] = a;
    acc[0] += a * a;
  }
  block_sum_store<1>(acc, part + part_slot(tab));
}

// partial ||z - theta v||^2 (residual of the Ritz pair).
__global__ void __launch_bounds__(kBlock)
k_resid(long n, const double* __restrict__ z, const double* __restrict__ v, double theta,
        const double* __restrict__ thetas, double* __restrict__ part, BlockTab tab) {
  const Rows ch = rows_of(n, tab);
  if (thetas) theta = thetas[ch.inst];
  double acc[1] = {0.0};
  for (long i = ch.lo + threadIdx.x; i < ch.hi; i += kBlock) {
    const double d = z[i] - theta * v[i];
    acc[0] += d * d;
  }
  block_sum_store<1>(acc, part + part_slot(tab));
}

// sum_i x_i^4 (DIAG) or sum over edges of (x_i x_j)^2 (TRACE_EDGES): the
// curvature ||A(v v^T)||^2 of the rank-one step, without the trace row.
__global__ void __launch_bounds__(kBlock)
k_quartic_norm(long n, int cons_kind, EdgeAdj A, const double* __restrict__ x, double* __restrict__ part,
               BlockTab tab) {
  const Rows ch = rows_of(n, tab);
  double acc[1] = {0.0};
  for (long i = ch.lo + threadIdx.x; i < ch.hi; i += kBlock) {
    const double xi = x[i];
    if (cons_kind == 0) {
      acc[0] += xi * xi * xi * xi;
    } else {
      for (int k = A.urp[i]; k < A.urp[i + 1]; ++k) {
        const double p = xi * x[A.uci[k]];
        acc[0] += p * p;
      }
    }
  }
  block_sum_store<1>(acc, part + part_slot(tab));
}

// Fourth moments of q directions over the rows (DIAG family), for the block
// rank step: with the pairs (a <= b) numbered in row-major order and the
// pairs of pairs (P1 <= P2) likewise, entry e of block b is
//   part[b * ne + e] = sum over the block's rows i of V_ia V_ib V_ic V_id,
// ne = np (np + 1) / 2, np = q (q + 1) / 2.  V is n x q column-major.  The
// block's rows go through LDS kBlock at a time; thread t owns the entries
// t, t + kBlock, ... (at most kGramPerThread of them for q <= kMaxBlockDir).
constexpr int kMaxBlockDir = 8;
constexpr int kGramPerThread = 3;
__device__ __forceinline__ void pair_of(int pidx, int q, int& a, int& b) {
  a = 0;
  while (pidx >= q - a) {
    pidx -= q - a;
    ++a;
  }
  b = a + pidx;
}
__global__ void __launch_bounds__(kBlock)
k_gram4(long n, int q, const double* __restrict__ V, double* __restrict__ part) {
  __shared__ double tile[kBlock][kMaxBlockDir];
  const int np = q * (q + 1) / 2;
  const int ne = np * (np + 1) / 2;
  int ia[kGramPerThread], ib[kGramPerThread], ic[kGramPerThread], id[kGramPerThread];
  int cnt = 0;
  for (int e = threadIdx.x; e < ne && cnt < kGramPerThread; e += kBlock) {
    int p1 = 0, rem = e;
    while (rem >= np - p1) {
      rem -= np - p1;
      ++p1;
    }
    pair_of(p1, q, ia[cnt], ib[cnt]);
    pair_of(p1 + rem, q, ic[cnt], id[cnt]);
    ++cnt;
  }
  double acc[kGramPerThread] = {0.0, 0.0, 0.0};
  const long per = (n + gridDim.x - 1) / gridDim.x;
  const long lo = (long)blockIdx.x * per < n ? (long)blockIdx.x * per : n;
  const long hi = lo + per < n ? lo + per : n;
  for (long base = lo; base < hi; base += kBlock) {
    const long i = base + threadIdx.x;
    for (int k = 0; k < q; ++k) tile[threadIdx.x][k] = (i < hi) ? V[(long)k * n + i] : 0.0;
    __syncthreads();
    const int rows = hi - base < kBlock ? (int)(hi - base) : kBlock;
    for (int t = 0; t < cnt; ++t) {
      double s = 0.0;
      for (int rr = 0; rr < rows; ++rr) {
        const double* v = tile[rr];
        s += v[ia[t]] * v[ib[t]] * v[ic[t]] * v[id[t]];
      }
      acc[t] += s;
    }
    __syncthreads();
  }
  for (int t = 0; t < cnt; ++t) part[(long)blockIdx.x * ne + threadIdx.x + t * kBlock] = acc[t];
}

// The same moments for the edge rows of the trace + edge family: with
// K_e(ab) = (V_ia V_jb + V_ja V_ib) / 2 for edge e = (i, j) (the edge row of
// A(v_a v_b^T)), part[b * ne + e'] = sum over the block's edges of
// K_e(P1) K_e(P2) for the pair of pairs e' = (P1, P2).  Edges go through LDS
// kEdgeChunk at a time.
constexpr int kEdgeChunk = 128;
__global__ void __launch_bounds__(kBlock)
k_gram4_edges(long E, long n, int q, const int32_t* __restrict__ ei, const int32_t* __restrict__ ej,
              const double* __restrict__ V, double* __restrict__ part) {
  __shared__ double tile[kEdgeChunk][kMaxBlockDir * (kMaxBlockDir + 1) / 2];
  const int np = q * (q + 1) / 2;
  const int ne = np * (np + 1) / 2;
  int p1s[kGramPerThread], p2s[kGramPerThread];
  int cnt = 0;
  for (int e = threadIdx.x; e < ne && cnt < kGramPerThread; e += kBlock) {
    int p1 = 0, rem = e;
    while (rem >= np - p1) {
      rem -= np - p1;
      ++p1;
    }
    p1s[cnt] = p1;
    p2s[cnt] = p1 + rem;
    ++cnt;
  }
  double acc[kGramPerThread] = {0.0, 0.0, 0.0};
  const long per = (E + gridDim.x - 1) / gridDim.x;
  const long lo = (long)blockIdx.x * per < E ? (long)blockIdx.x * per : E;
  const long hi = lo + per < E ? lo + per : E;
  for (long base = lo; base < hi; base += kEdgeChunk) {
    const int rows = hi - base < kEdgeChunk ? (int)(hi - base) : kEdgeChunk;
    for (int idx = threadIdx.x; idx < rows * np; idx += kBlock) {
      const int el = idx / np, pp = idx % np;
      int a, b;
      pair_of(pp, q, a, b);
      const long i = ei[base + el], j = ej[base + el];
      tile[el][pp] = 0.5 * (V[(long)a * n + i] * V[(long)b * n + j] + V[(long)a * n + j] * V[(long)b * n + i]);
    }
    __syncthreads();
    for (int t = 0; t < cnt; ++t) {
      double s = 0.0;
      for (int rr = 0; rr < rows; ++rr) s += tile[rr][p1s[t]] * tile[rr][p2s[t]];
      acc[t] += s;
    }
    __syncthreads();
  }
  for (int t = 0; t < cnt; ++t) part[(long)blockIdx.x * ne + threadIdx.x + t * kBlock] = acc[t];
}

// ---- launchers (single instance: empty table, count 1, strides 0) ---------------

void launch_gram4_edges(long E, long n, int q, const int32_t* ei, const int32_t* ej, const double* V, double* part,
                        int nb, hipStream_t st) {
  hipLaunchKernelGGL(k_gram4_edges, dim3(nb), dim3(kBlock), 0, st, E, n, q, ei, ej, V, part);
}

void launch_gram4(long n, int q, const double* V, double* part, int nb, hipStream_t st) {
  hipLaunchKernelGGL(k_gram4, dim3(nb), dim3(kBlock), 0, st, n, q, V, part);
}

// Blocks of the vector kernels: 256 rows each for small n (so that the columns of
// a step are loaded in one trip), 1024 rows beyond, at most 1024.  For the
// ordered steps chunks of 4096 rows, at least 8.
int vec_blocks(long n, bool ordered) {
  if (ordered) {
    long nb = (n + kBlock * 16 - 1) / (kBlock * 16);
    nb = nb < 8 ? 8 : (nb > 1024 ? 1024 : nb);
    return (int)((nb + 7) / 8 * 8);
  }
  long nb = n <= 65536 ? (n + kBlock - 1) / kBlock : (n + kBlock * 4 - 1) / (kBlock * 4);
  if (nb < 8) nb = 8;
  if (nb > 1024) nb = 1024;
  return (int)((nb + 7) / 8 * 8);
}

template <bool SUB, bool DOTS>
static void launch_proj(long n, int ncol, const double* Q, long ldq, const LzCoef& hc, double* w, double* part,
                        int pld, int nb, hipStream_t st, const BlockTab& tab) {
#define ALMBM_PROJ(K) hipLaunchKernelGGL((K), dim3(nb), dim3(kBlock), 0, st, n, ncol, Q, ldq, hc, w, part, pld, tab)
  if constexpr (!DOTS) {  // nothing to keep from the subtraction
    ALMBM_PROJ((k_lz_proj_wide<SUB, false>));
  } else {
    if (ncol <= 16) ALMBM_PROJ((k_lz_proj<16, SUB>));
    else if (ncol <= 32) ALMBM_PROJ((k_lz_proj<32, SUB>));
    else if (ncol <= 64) ALMBM_PROJ((k_lz_proj<64, SUB>));
    else ALMBM_PROJ((k_lz_proj_wide<SUB, true>));
  }
#undef ALMBM_PROJ
}

// Partial sums of few blocks are left to the next kernel, which adds them itself.
static bool lz_consumer_sums(const VecBatch& vb, int nb) { return !vb.tab.inst && nb <= kLzFewBlocks; }

static LzCoef lz_coef(double* h, const double* part, int pld, int nb, const VecBatch& vb) {
  LzCoef hc;
  if (lz_consumer_sums(vb, nb)) {
    hc.part = part;
    hc.nb = nb;
    hc.pld = pld;
    hc.out = h;
  } else {
    hc.h = h;
    hc.hstride = vb.hstride;
  }
  return hc;
}

static void fin_dots(int ncol, const double* part, int pld, int nb, double* h, hipStream_t st, const VecBatch& vb) {
  hipLaunchKernelGGL(k_fin_dots, dim3(ncol, vb.count), dim3(kBlock), 0, st, part, nb, pld, ncol, h, vb.hstride,
                     vb.tab);
}

void launch_dots(long n, int ncol, const double* Q, long ldq, double* w, double* part, int pld, int nb, double* h,
                 hipStream_t st, const VecBatch& vb) {
  launch_proj<false, true>(n, ncol, Q, ldq, LzCoef{}, w, part, pld, nb, st, vb.tab);
  fin_dots(ncol, part, pld, nb, h, st, vb);
}

void launch_gs2(long n, int ncol, const double* Q, long ldq, double* w, double* part, double* part_b, double* part_n,
                int pld, int nb, double* h1, double* h2, hipStream_t st, const VecBatch& vb) {
  const bool few = lz_consumer_sums(vb, nb);
  launch_proj<false, true>(n, ncol, Q, ldq, LzCoef{}, w, part, pld, nb, st, vb.tab);
  if (!few) fin_dots(ncol, part, pld, nb, h1, st, vb);
  launch_proj<true, true>(n, ncol, Q, ldq, lz_coef(h1, part, pld, nb, vb), w, part_b, pld, nb, st, vb.tab);
  if (!few) fin_dots(ncol, part_b, pld, nb, h2, st, vb);
  launch_proj<true, false>(n, ncol, Q, ldq, lz_coef(h2, part_b, pld, nb, vb), w, part_n, pld, nb, st, vb.tab);
}

void launch_gs2_ordered(long n, int ncol, const double* Q, long ldq, double* w, double* part, double* part_n, int pld,
                        int nb, double* h1, double* h2, hipStream_t st) {
  const dim3 cols(nb, (ncol + kBlock / kWave - 1) / (kBlock / kWave));
  const int rows = (int)((n + kBlock - 1) / kBlock);
  const bool fused = nb >= 128 && ncol <= 64;  // see k_sub_dots_ordered
  hipLaunchKernelGGL(k_dots_ordered, cols, dim3(kBlock), 0, st, n, ncol, Q, ldq, w, part, pld);
  fin_dots(ncol, part, pld, nb, h1, st, VecBatch{});
  if (fused) {
    if (ncol <= 16)
      hipLaunchKernelGGL(k_sub_dots_ordered<16>, dim3(nb), dim3(kBlock), 0, st, n, ncol, Q, ldq, h1, w, part, pld);
    else if (ncol <= 32)
      hipLaunchKernelGGL(k_sub_dots_ordered<32>, dim3(nb), dim3(kBlock), 0, st, n, ncol, Q, ldq, h1, w, part, pld);
    else
      hipLaunchKernelGGL(k_sub_dots_ordered<64>, dim3(nb), dim3(kBlock), 0, st, n, ncol, Q, ldq, h1, w, part, pld);
  } else {
    hipLaunchKernelGGL(k_sub_ordered, dim3(rows), dim3(kBlock), 0, st, n, ncol, Q, ldq, h1, w);
    hipLaunchKernelGGL(k_dots_ordered, cols, dim3(kBlock), 0, st, n, ncol, Q, ldq, w, part, pld);
  }
  fin_dots(ncol, part, pld, nb, h2, st, VecBatch{});
  hipLaunchKernelGGL(k_sub_ordered, dim3(rows), dim3(kBlock), 0, st, n, ncol, Q, ldq, h2, w);
  hipLaunchKernelGGL(k_norm_ordered, dim3(nb), dim3(kBlock), 0, st, n, w, part_n, pld);
}

void launch_fin_ab(const double* part, int nb, int pld, const double* h1, const double* h2, int j, double* alpha,
                   double* beta, double* qsum, hipStream_t st, const VecBatch& vb) {
  hipLaunchKernelGGL(k_fin_ab, dim3(vb.count), dim3(kBlock), 0, st, part, nb, pld, h1, h2, vb.hstride, j, alpha, beta,
                     vb.astride, qsum, vb.tab);
}

void launch_lz_mv(const Cost<double>& C, int cons_kind, const EdgeAdj& A, const double* y, double c_tr, double j_coef,
                  const double* qsum, const LzStep& s, const double* w, double* qcol, double* out, int nb,
                  hipStream_t st, const VecBatch& vb) {
  if (C.nh > 0) launch_hub_rows<double>(C, 1, 0, w, C.hsum, nullptr, 0, st);
  LzScale sc;  // s.j = 0: w is the column itself
  if (s.j > 0 && s.sums && lz_consumer_sums(vb, s.nb)) {
    sc.part = s.part;
    sc.nb = s.nb;
    sc.pld = s.pld;
    sc.h1 = s.h1;
    sc.h2 = s.h2;
    sc.alpha_out = s.alpha + s.j - 1;
    sc.beta_out = s.beta + s.j - 1;
    sc.jm1 = s.j - 1;
  } else if (s.j > 0) {
    sc.beta = s.beta + s.j - 1;
    sc.bstride = vb.astride;
  }
  // one trip of the rows per block; with a table, whose blocks have many more rows,
  // by sharing each of its entries among grid.y blocks (no partial sums depend on it)
  constexpr long kRows = kBlock / kSpmvLpr;
  int ny = 1;
  if (!vb.tab.inst) {
    long g = (C.n + kRows - 1) / kRows;
    g = g < 8 ? 8 : (g > 8192 ? 8192 : g);
    nb = (int)((g + 7) / 8 * 8);
  } else {
    const long g = (C.n + nb * kRows - 1) / (nb * kRows);
    ny = (int)(g < 1 ? 1 : (g > 8 ? 8 : g));
  }
  hipLaunchKernelGGL(k_lz_mv, dim3(nb, ny), dim3(kBlock), 0, st, C, cons_kind, A, y, c_tr, j_coef, qsum, sc, w, qcol, out,
                     vb.tab);
}
void launch_slack_mv(const Cost<double>& C, int cons_kind, const EdgeAdj& A, const double* y, double c_tr,
                     double j_coef, const double* qsum, const double* x, double* out, hipStream_t st) {
  launch_lz_mv(C, cons_kind, A, y, c_tr, j_coef, qsum, LzStep{}, x, nullptr, out, 0, st);
}
void launch_slack_mv_tab(const Cost<double>& C, const double* y, const double* x, double* out, int nb, hipStream_t st,
                         const VecBatch& vb) {
  launch_lz_mv(C, 0, EdgeAdj{}, y, 0.0, 0.0, nullptr, LzStep{}, x, nullptr, out, nb, st, vb);
}
void launch_scale(long n, const double* w, const double* beta, double* q, double* part, int nb, double* qsum,
                  hipStream_t st, const VecBatch& vb, int bstride) {
  hipLaunchKernelGGL(k_scale, dim3(nb), dim3(kBlock), 0, st, n, w, beta, bstride, q, part, vb.tab);
  if (qsum) hipLaunchKernelGGL(k_fin_sum, dim3(vb.count), dim3(kBlock), 0, st, part, nb, qsum, 0, 0, vb.tab);
}
void launch_fin_sum(const double* part, int nb, double* out, int do_sqrt, hipStream_t st, const VecBatch& vb,
                    int ostride) {
  hipLaunchKernelGGL(k_fin_sum, dim3(vb.count), dim3(kBlock), 0, st, part, nb, out, ostride, do_sqrt, vb.tab);
}
void launch_mix(long n, double eps, const double* v, double* x, const double* norms, int nstride, double* part,
                int nb, hipStream_t st, const VecBatch& vb) {
  hipLaunchKernelGGL(k_mix, dim3(nb), dim3(kBlock), 0, st, n, eps, v, x, norms, nstride, part, vb.tab);
}
void launch_rand(long n, uint64_t seed, double* x, double* part, int nb, hipStream_t st, const VecBatch& vb) {
  hipLaunchKernelGGL(k_rand, dim3(nb), dim3(kBlock), 0, st, n, seed, x, part, vb.tab);
}
void launch_combine(long n, int ncol, const double* Q, long ldq, const double* s, double* v, double* part, int nb,
                    hipStream_t st, const VecBatch& vb, const int32_t* ncols) {
  hipLaunchKernelGGL(k_combine, dim3(nb), dim3(kBlock), 0, st, n, ncol, Q, ldq, s, vb.hstride, v, part, vb.tab,
                     ncols);
}
void launch_resid(long n, const double* z, const double* v, double theta, const double* thetas, double* part, int nb,
                  hipStream_t st, const VecBatch& vb) {
  hipLaunchKernelGGL(k_resid, dim3(nb), dim3(kBlock), 0, st, n, z, v, theta, thetas, part, vb.tab);
}
void launch_quartic_norm(long n, int cons_kind, const EdgeAdj& A, const double* x, double* part, int nb,
                         hipStream_t st, const VecBatch& vb) {
  hipLaunchKernelGGL(k_quartic_norm, dim3(nb), dim3(kBlock), 0, st, n, cons_kind, A, x, part, vb.tab);
}

// flags[q] = sc[q].flag, iters[q] = sc[q].iter (compact copy for the host).
__global__ void k_gather_flags(const DevScalars* __restrict__ sc, int count, int32_t* __restrict__ out) {
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= count) return;
  out[2 * q] = sc[q].flag;
  out[2 * q + 1] = sc[q].iter;
}

void launch_gather_flags(const DevScalars* sc, int count, int32_t* out, hipStream_t st) {
  hipLaunchKernelGGL(k_gather_flags, dim3((count + 63) / 64), dim3(64), 0, st, sc, count, out);
}

}  // namespace almbm
