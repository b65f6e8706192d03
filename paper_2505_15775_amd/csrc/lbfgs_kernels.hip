// L-BFGS subproblem solver of the inner loop (DIAG family): the direction
// E = H G of the limited-memory BFGS inverse-Hessian estimate built from the
// last m pairs (s, y), taken with the same exact quartic line search as
// gradient descent (R <- R - t E).  SDPLR, the ALM-BM solver Sec. 2 names,
// solves its subproblems this way.
//
// Per step, after the gradient pass (which also writes y_k = G_new - G_old):
//   k_lbfgs_dots      inner products of G and y_k with the stored vectors
//   k_fin_lbfgs       takes the pair (s_k, y_k) if s_k^T y_k > 0 (relative
//                     to ||s|| ||y||), updates the small Gram matrices and
//                     runs the two-loop recursion on coefficients
//   k_lbfgs_combine   E = cg G + sum_a (ce_a E_a + cy_a y_a) and the
//                     quartic's direction-dependent partial sums
//   k_fin_lsdir       their totals
// then the line-search product C E and the step rule as for gradient descent.
// Pure streaming kernels: no gathers, no MFMA.
#include <algorithm>

#include "finalize.hpp"
#include "spmm_row.hpp"

namespace almbm {

// ---- reset -----------------------------------------------------------------------

// One block per instance (state s + blockIdx.x).
__global__ void k_lbfgs_reset(LbfgsState* s, int m) {
  if (threadIdx.x != 0) return;
  s += blockIdx.x;
  s->m = m;
  s->cnt = 0;
  s->cur = 0;
  s->have = 0;
  s->resets = 0;
  s->accepted = 0;
  s->ee = 0.0;
  s->cg = 1.0;
  for (int a = 0; a < kMaxLbfgs; ++a) {
    s->ord[a] = 0;
    s->ce[a] = 0.0;
    s->cy[a] = 0.0;
  }
  for (int a = 0; a < kLbfgsSlots; ++a) s->tp[a] = 0.0;
}

// ---- inner products ------------------------------------------------------------
//
// Partial slots per block, M + 1 each (M the template bound on the pairs held):
// G . E_a, G . y_a, y_k . E_a, y_k . y_a for the held pairs a < cnt in set order
// at positions a and for the current direction (E_k, y_k) at position M; then
// E_k . y_a (a < cnt).  The y_k and E_k products only when a direction was
// taken (have).

template <typename T> struct FlatVec { static constexpr int N = 16 / sizeof(T); };

template <typename T, int N>
__device__ __forceinline__ void load_flat(const T* __restrict__ p, typename Acc<T>::type (&out)[N]) {
  if constexpr (N == 1) {
    out[0] = to_acc<T>(p[0]);
  } else {
    using W = typename VecWord<N * sizeof(T)>::type;
    W w = *reinterpret_cast<const W*>(p);
    const T* e = reinterpret_cast<const T*>(&w);
#pragma unroll
    for (int v = 0; v < N; ++v) out[v] = to_acc<T>(e[v]);
  }
}

template <typename V, int M> struct DotAcc {
  V gE[M + 1], gY[M + 1], kE[M + 1], kY[M + 1], eY[M];
};

// NV consecutive elements at idx of every vector.
template <typename T, int NV, int M, typename S = RingT<T>>
__device__ __forceinline__ void dots_chunk(DotAcc<typename Acc<T>::type, M>& A, long idx, const T* __restrict__ G,
                                           const S* __restrict__ yk, const S* __restrict__ ek,
                                           const S* const (&ea)[M], const S* const (&ya)[M], int cnt, bool have) {
  using V = typename Acc<T>::type;
  V g[NV], y_k[NV], e_k[NV];
  load_flat<T, NV>(G + idx, g);
  if (have) {
    load_flat<S, NV>(yk + idx, y_k);
    load_flat<S, NV>(ek + idx, e_k);
  }
#pragma unroll
  for (int a = 0; a < M; ++a) {
    if (a < cnt) {
      V ev[NV], yv[NV];
      load_flat<S, NV>(ea[a] + idx, ev);
      load_flat<S, NV>(ya[a] + idx, yv);
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        A.gE[a] += g[v] * ev[v];
        A.gY[a] += g[v] * yv[v];
      }
      if (have) {
#pragma unroll
        for (int v = 0; v < NV; ++v) {
          A.kE[a] += y_k[v] * ev[v];
          A.kY[a] += y_k[v] * yv[v];
          A.eY[a] += e_k[v] * yv[v];
        }
      }
    }
  }
  if (have) {
#pragma unroll
    for (int v = 0; v < NV; ++v) {
      A.gE[M] += g[v] * e_k[v];
      A.gY[M] += g[v] * y_k[v];
      A.kE[M] += y_k[v] * e_k[v];
      A.kY[M] += y_k[v] * y_k[v];
    }
  }
}

// Without a table the vectors are shared out to vgrid virtual blocks (element
// chunk q to thread q mod (vgrid kBlock)) and each block runs the virtual blocks
// blockIdx.x, blockIdx.x + gridDim.x, ....  A virtual thread sums its chunks in
// the arithmetic type and its sums are added in FP64, so that the rounding of
// float sums depends on vgrid, a function of n, and not on the blocks launched.
// With a table each block takes the elements of its rows, [xbase + lo r,
// xbase + hi r) of its instance (stored at width r), with the instance's own
// state and stop flag.
//
// Bound by HBM streaming (2 M + 3 vectors).  M bounds the pairs at compile
// time: with the memory of 3 that solves use by default 19 accumulators remain
// of the 44 of memory 8, and the block's sums take 32 shuffles instead of 270.
// n = 193 176, r = 16, FP64, memory 3 (222 MB): 88 us with 44
// accumulators on one block per 64 rows, 36 us (6.2 TB/s) now.
template <typename T, int M>
__global__ void __launch_bounds__(kBlock)
k_lbfgs_dots(long len, int r, const T* __restrict__ G, LbfgsRing<RingT<T>> lb, double* __restrict__ part,
             const DevScalars* sc_base, BlockTab tab, int vgrid, SideFin side) {
  if (run_side_fin(side)) return;
  using V = typename Acc<T>::type;
  using R = RingT<T>;
  constexpr int N = FlatVec<T>::N;
  long a = 0, e = len;
  int inst = 0, vb0 = blockIdx.x, vstep = gridDim.x - (side.part ? 1 : 0);
  if (tab.inst) {
    inst = tab.inst[blockIdx.x];
    const long xb = row_base(tab, inst);
    a = xb + (long)tab.lo[blockIdx.x] * r;
    e = xb + (long)tab.hi[blockIdx.x] * r;
    vb0 = 0;
    vgrid = 1;
    vstep = 1;
  }
  if (block_stopped(sc_base + inst)) return;
  const LbfgsState* S = lb.s + inst;
  const int cnt = S->cnt;
  const bool have = S->have != 0;
  const R* yk = lb.y + (long)S->cur * lb.stride;
  const R* ek = lb.e + (long)S->cur * lb.stride;
  const R* ea[M];
  const R* ya[M];
#pragma unroll
  for (int a = 0; a < M; ++a) {
    const int sl = a < cnt ? S->ord[a] : 0;
    ea[a] = lb.e + (long)sl * lb.stride;
    ya[a] = lb.y + (long)sl * lb.stride;
  }
  constexpr int ND = lbfgs_dot_slots(M);
  double acc[ND];
#pragma unroll
  for (int k = 0; k < ND; ++k) acc[k] = 0.0;
  // element-wise head up to N-element alignment, N-element chunks, element-wise tail
  const long pad = (N - a % N) % N;
  const long a_al = a + pad < e ? a + pad : e;
  const long nvec = (e - a_al) / N;
  const long tstride = (long)vgrid * kBlock;
  for (int vb = vb0; vb < vgrid; vb += vstep) {
    const long t0 = (long)vb * kBlock + threadIdx.x;
    DotAcc<V, M> A;
#pragma unroll
    for (int k = 0; k <= M; ++k) A.gE[k] = A.gY[k] = A.kE[k] = A.kY[k] = V(0);
#pragma unroll
    for (int k = 0; k < M; ++k) A.eY[k] = V(0);
    for (long idx = a + t0; idx < a_al; idx += tstride) dots_chunk<T, 1, M>(A, idx, G, yk, ek, ea, ya, cnt, have);
    for (long q = t0; q < nvec; q += tstride) dots_chunk<T, N, M>(A, a_al + q * N, G, yk, ek, ea, ya, cnt, have);
    for (long idx = a_al + nvec * N + t0; idx < e; idx += tstride)
      dots_chunk<T, 1, M>(A, idx, G, yk, ek, ea, ya, cnt, have);
#pragma unroll
    for (int k = 0; k <= M; ++k) {
      acc[k] += (double)A.gE[k];
      acc[M + 1 + k] += (double)A.gY[k];
      acc[2 * (M + 1) + k] += (double)A.kE[k];
      acc[3 * (M + 1) + k] += (double)A.kY[k];
      if (k < M) acc[4 * (M + 1) + k] += (double)A.eY[k];
    }
  }
  block_sum_many<ND>(acc, part + part_slot(tab) * ND);
}

// ---- pair update and the two-loop recursion on coefficients ----------------------

// One block per instance (blockIdx.x; a single instance without a table).  M as
// in k_lbfgs_dots: every loop over the pairs is unrolled to M and guarded, so
// that thread 0's small matrices stay in registers (indexed by a run-time count
// they would live in scratch memory).  Bound by latency; n = 193 176, r = 16,
// memory 3: 51 us before, 10 us now (with the rows of fewer blocks to add).
template <int M>
__global__ void __launch_bounds__(kFin)
k_fin_lbfgs(const double* __restrict__ part, int nb, const DevScalars* __restrict__ sc_base,
            LbfgsState* __restrict__ S_base, BlockTab tab) {
  const DevScalars* sc = sc_base + blockIdx.x;
  LbfgsState* S = S_base + blockIdx.x;
  if (sc->flag) return;
  int b0, b1;
  inst_blocks(tab, blockIdx.x, nb, b0, b1);
  constexpr int ND = lbfgs_dot_slots(M);
  __shared__ double tot[ND];
  fin_rows<ND>(part + (long)b0 * ND, b1 - b0, tot);
  if (threadIdx.x != 0) return;
  const double* gE = tot;
  const double* gY = tot + (M + 1);
  const double* kE = tot + 2 * (M + 1);
  const double* kY = tot + 3 * (M + 1);
  const double* eY = tot + 4 * (M + 1);
  const int m = S->m;
  int c = S->cnt;
  const int cur = S->cur;
  const double t = sc->t;  // the step just taken along E_k
  // the held pairs in set order: slots, steps, Gram matrices, products with G
  int ord[M];
  double tp[M], SY[M][M], YY[M][M], gsE[M], gsY[M];
#pragma unroll
  for (int a = 0; a < M; ++a) {
    const bool in = a < c;
    ord[a] = in ? S->ord[a] : 0;
    tp[a] = in ? S->tp[ord[a]] : 0.0;
    gsE[a] = gE[a];
    gsY[a] = gY[a];
#pragma unroll
    for (int b = 0; b < M; ++b) {
      SY[a][b] = in && b < c ? S->SY[a][b] : 0.0;
      YY[a][b] = in && b < c ? S->YY[a][b] : 0.0;
    }
  }
  int next = cur;
  bool taken = false;
  if (S->have) {
    if (!(t > 0.0)) {
      // a zero step: clear the memory, the next direction is the gradient
      c = 0;
      S->resets += 1;
    } else {
      const double sy = -t * kE[M];  // s_k . y_k with s_k = -t E_k
      const double ss = t * t * S->ee;
      const double yy = kY[M];
      if (sy > 1e-12 * sqrt(ss) * sqrt(yy)) {
        double col[M], row[M], yrow[M];
#pragma unroll
        for (int a = 0; a < M; ++a) {
          col[a] = -tp[a] * kE[a];  // s_a . y_k
          row[a] = -t * eY[a];      // s_k . y_a
          yrow[a] = kY[a];          // y_k . y_a
        }
        if (c == m) {  // drop the oldest pair
          next = ord[0];
#pragma unroll
          for (int a = 0; a + 1 < M; ++a) {
            ord[a] = ord[a + 1];
            tp[a] = tp[a + 1];
            gsE[a] = gsE[a + 1];
            gsY[a] = gsY[a + 1];
            col[a] = col[a + 1];
            row[a] = row[a + 1];
            yrow[a] = yrow[a + 1];
#pragma unroll
            for (int b = 0; b + 1 < M; ++b) {
              SY[a][b] = SY[a + 1][b + 1];
              YY[a][b] = YY[a + 1][b + 1];
            }
          }
          c -= 1;
        } else {
          // first slot held by no pair and not the current one
          for (int sl = 0; sl < kLbfgsSlots; ++sl) {
            bool used = sl == cur;
#pragma unroll
            for (int a = 0; a < M; ++a) used = used || (a < c && ord[a] == sl);
            if (!used) {
              next = sl;
              break;
            }
          }
        }
#pragma unroll
        for (int d = 0; d < M; ++d) {
          if (d != c) continue;  // the new pair's position
          ord[d] = cur;
          tp[d] = t;
          gsE[d] = gE[M];
          gsY[d] = gY[M];
#pragma unroll
          for (int a = 0; a < M; ++a) {
            if (a >= c) continue;
            SY[a][d] = col[a];
            SY[d][a] = row[a];
            YY[a][d] = YY[d][a] = yrow[a];
          }
          SY[d][d] = sy;
          YY[d][d] = yy;
        }
        S->tp[cur] = t;
        c += 1;
        S->accepted += 1;
        taken = true;
      }
    }
  }
  if (taken) {
#pragma unroll
    for (int a = 0; a < M; ++a) {
      if (a >= c) continue;
      S->ord[a] = ord[a];
#pragma unroll
      for (int b = 0; b < M; ++b) {
        if (b >= c) continue;
        S->SY[a][b] = SY[a][b];
        S->YY[a][b] = YY[a][b];
      }
    }
  }
  // two-loop recursion on the coefficients of q = H G in {G, y_a, s_a}
  double gs[M], rho[M], alpha[M], qy[M], rs[M];
  double gam = 1.0;
#pragma unroll
  for (int a = 0; a < M; ++a) {
    const bool in = a < c;
    gs[a] = in ? -tp[a] * gsE[a] : 0.0;
    rho[a] = in ? 1.0 / SY[a][a] : 0.0;
    qy[a] = rs[a] = alpha[a] = 0.0;
    if (a == c - 1) gam = SY[a][a] / YY[a][a];
  }
#pragma unroll
  for (int a = M - 1; a >= 0; --a) {
    if (a >= c) continue;
    double sq = gs[a];
#pragma unroll
    for (int b = 0; b < M; ++b)
      if (b < c) sq += qy[b] * SY[a][b];
    alpha[a] = rho[a] * sq;
    qy[a] -= alpha[a];
  }
  const double rg = gam;
#pragma unroll
  for (int b = 0; b < M; ++b) qy[b] *= gam;
#pragma unroll
  for (int a = 0; a < M; ++a) {
    if (a >= c) continue;
    double yr = rg * gsY[a];
#pragma unroll
    for (int b = 0; b < M; ++b)
      if (b < c) yr += qy[b] * YY[a][b] + rs[b] * SY[b][a];
    const double beta = rho[a] * yr;
    rs[a] += alpha[a] - beta;
  }
  // descent test E . G > 0 from the same products
  double eg = rg * sc->tot[P_GG];
#pragma unroll
  for (int a = 0; a < M; ++a)
    if (a < c) eg += qy[a] * gsY[a] + rs[a] * gs[a];
  if (c > 0 && !(eg > 0.0)) {
    c = 0;
    S->resets += 1;
  }
  S->cg = c == 0 ? 1.0 : rg;
#pragma unroll
  for (int a = 0; a < M; ++a) {
    if (a >= c) continue;
    S->cy[a] = qy[a];
    S->ce[a] = -tp[a] * rs[a];
  }
  S->cnt = c;
  S->cur = next;
  S->have = 1;
}

// ---- the direction and its line-search partials ----------------------------------

template <typename T, int LPR, int VEC, bool FULL>
__global__ void __launch_bounds__(kBlock)
k_lbfgs_combine(long n, int r, const T* __restrict__ R, const T* __restrict__ G, const double* __restrict__ y,
                const double* __restrict__ b, double sigma, const double* __restrict__ Av, LbfgsRing<RingT<T>> lb,
                double* __restrict__ part, const DevScalars* __restrict__ sc_base, BlockTab tab) {
  using V = typename Acc<T>::type;
  using RS = RingT<T>;
  const Rows ch = rows_of(n, tab);
  if (sc_base[ch.inst].flag) return;
  const LbfgsState* S = lb.s + ch.inst;
  const int c = S->cnt;
  const V cg = static_cast<V>(S->cg);
  const long xb = row_base(tab, ch.inst);
  R += xb;
  G += xb;
  RS* __restrict__ E = lb.e + (long)S->cur * lb.stride + xb;
  constexpr int RPB = kBlock / LPR;
  const int lane = threadIdx.x % LPR;
  const int slot = threadIdx.x / LPR;
  SplitAcc<NUM_P, LPR> acc;
  acc.zero();
  for (long base = ch.lo; base < ch.hi; base += RPB) {
    const long i = base + slot;
    if (i >= ch.hi) break;
    V ri[VEC], gi[VEC], e[VEC];
    load_frag<T, VEC, FULL>(R + i * r, lane, r, ri);
    load_frag<T, VEC, FULL>(G + i * r, lane, r, gi);
#pragma unroll
    for (int v = 0; v < VEC; ++v) e[v] = cg * gi[v];
    for (int a = 0; a < c; ++a) {
      const long off = (long)S->ord[a] * lb.stride + xb + i * r;
      const V ca = static_cast<V>(S->ce[a]), cb = static_cast<V>(S->cy[a]);
      V ev[VEC], yv[VEC];
      load_frag<RS, VEC, FULL>(lb.e + off, lane, r, ev);
      load_frag<RS, VEC, FULL>(lb.y + off, lane, r, yv);
#pragma unroll
      for (int v = 0; v < VEC; ++v) e[v] += ca * ev[v] + cb * yv[v];
    }
#pragma unroll
    for (int v = 0; v < VEC; ++v) e[v] = round_st<RS>(e[v]);  // the direction as stored
    store_frag<RS, VEC, FULL>(E + i * r, lane, r, e);
    // C R = G/2 + w R at the current point
    const double yi = y[i], ai = Av[i], ei = ai - b[i];
    const V wv = static_cast<V>(yi - sigma * ei);
    V ee = 0, ep = 0, re = 0;
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      const V p = V(0.5) * gi[v] + wv * ri[v];
      ee += e[v] * e[v];
      ep += e[v] * p;
      re += ri[v] * e[v];
    }
    ee = group_sum<LPR>(ee);
    ep = group_sum<LPR>(ep);
    re = group_sum<LPR>(re);
    const double a1 = 2.0 * (double)re, a2 = (double)ee;
    acc.add(lane, P_GG, a2);
    acc.add(lane, P_GP, (double)ep);
    acc.add(lane, P_YA1, yi * a1);
    acc.add(lane, P_YA2, yi * a2);
    acc.add(lane, P_EA1, ei * a1);
    acc.add(lane, P_EA2, ei * a2);
    acc.add(lane, P_A1A1, a1 * a1);
    acc.add(lane, P_A1A2, a1 * a2);
    acc.add(lane, P_A2A2, a2 * a2);
    acc.add(lane, P_RG, (double)re);
  }
  acc.block_store(part + part_slot(tab) * NUM_P);
}

__global__ void __launch_bounds__(kFin)
k_fin_lsdir(const double* __restrict__ part, int nb, DevScalars* __restrict__ sc_base, LbfgsState* __restrict__ S_base,
            BlockTab tab) {
  DevScalars* sc = sc_base + blockIdx.x;
  LbfgsState* S = S_base + blockIdx.x;
  if (sc->flag) return;
  int b0, b1;
  inst_blocks(tab, blockIdx.x, nb, b0, b1);
  __shared__ double tot[NUM_P];
  fin_rows<NUM_P>(part + (long)b0 * NUM_P, b1 - b0, tot);
  if (threadIdx.x == 0) finish_lsdir(tot, sc, S);
}

// ---- launchers ---------------------------------------------------------------------

void launch_lbfgs_reset(LbfgsState* s, int m, hipStream_t st, int count) {
  hipLaunchKernelGGL(k_lbfgs_reset, dim3(count), dim3(64), 0, st, s, m);
}

// Without a table: one virtual block per 64 rows, up to 4096, on blocks of at
// least four vector chunks per thread and at most nb of them (the row kernels' grid, 1024
// by default), so that the block sums and the finalizer's rows stay few.
template <typename T>
int launch_lbfgs_dots(long len, int r, int m, const T* G, const LbfgsRing<RingT<T>>& lb, double* part, int nb,
                      const DevScalars* sc, hipStream_t st, const BlockTab& tab, const SideFin& side) {
  int vgrid = 1;
  if (!tab.inst) {
    const long v = std::min<long>(4096, std::max<long>(8, (len / r + 63) / 64));
    vgrid = (int)((v + 7) / 8 * 8);
    const long b = (len / FlatVec<T>::N + 4 * kBlock - 1) / (4 * kBlock);
    nb = (int)std::min<long>({(long)nb, (long)vgrid, std::max<long>(8, b)});
    if (sizeof(typename Acc<T>::type) == 8) vgrid = nb;  // FP64 sums need no virtual blocks
  }
  const dim3 grid(nb + (side.part ? 1 : 0));
  if (m <= 3)
    hipLaunchKernelGGL((k_lbfgs_dots<T, 3>), grid, dim3(kBlock), 0, st, len, r, G, lb, part, sc, tab, vgrid, side);
  else
    hipLaunchKernelGGL((k_lbfgs_dots<T, kMaxLbfgs>), grid, dim3(kBlock), 0, st, len, r, G, lb, part, sc, tab, vgrid,
                       side);
  return nb;
}

void launch_fin_lbfgs(const double* part, int nb, int m, const DevScalars* sc, LbfgsState* s, hipStream_t st,
                      const BlockTab& tab, int count) {
  if (m <= 3)
    hipLaunchKernelGGL(k_fin_lbfgs<3>, dim3(count), dim3(kFin), 0, st, part, nb, sc, s, tab);
  else
    hipLaunchKernelGGL(k_fin_lbfgs<kMaxLbfgs>, dim3(count), dim3(kFin), 0, st, part, nb, sc, s, tab);
}

template <typename T, int LPR, int VEC>
static void launch_combine_cfg(long n, int r, const T* R, const T* G, const double* y, const double* b, double sigma,
                               const double* Av, const LbfgsRing<RingT<T>>& lb, double* part,
                               const DevScalars* sc, int nblk, hipStream_t st, const BlockTab& tab) {
  if (r == LPR * VEC)
    hipLaunchKernelGGL((k_lbfgs_combine<T, LPR, VEC, true>), dim3(nblk), dim3(kBlock), 0, st, n, r, R, G, y, b,
                       sigma, Av, lb, part, sc, tab);
  else
    hipLaunchKernelGGL((k_lbfgs_combine<T, LPR, VEC, false>), dim3(nblk), dim3(kBlock), 0, st, n, r, R, G, y, b,
                       sigma, Av, lb, part, sc, tab);
}

template <typename T>
void launch_lbfgs_combine(long n, int r, int variant, const T* R, const T* G, const double* y, const double* b,
                          double sigma, const double* Av, const LbfgsRing<RingT<T>>& lb, double* part,
                          const DevScalars* sc, int nblk, hipStream_t st, const BlockTab& tab) {
  ALMBM_DISPATCH_DIAG(T, launch_combine_cfg, n, r, R, G, y, b, sigma, Av, lb, part, sc, nblk, st, tab);
}

void launch_fin_lsdir(const double* part, int nb, DevScalars* sc, LbfgsState* s, hipStream_t st,
                      const BlockTab& tab, int count) {
  hipLaunchKernelGGL(k_fin_lsdir, dim3(count), dim3(kFin), 0, st, part, nb, sc, s, tab);
}

#define ALMBM_LBFGS_INST(T)                                                                               \
  template int launch_lbfgs_dots<T>(long, int, int, const T*, const LbfgsRing<RingT<T>>&, double*, int,    \
                                    const DevScalars*, hipStream_t, const BlockTab&, const SideFin&);      \
  template void launch_lbfgs_combine<T>(long, int, int, const T*, const T*, const double*, const double*,   \
                                        double, const double*, const LbfgsRing<RingT<T>>&, double*,          \
                                        const DevScalars*, int, hipStream_t, const BlockTab&);

ALMBM_LBFGS_INST(double)
ALMBM_LBFGS_INST(float)
ALMBM_LBFGS_INST(bf16)

}  // namespace almbm
