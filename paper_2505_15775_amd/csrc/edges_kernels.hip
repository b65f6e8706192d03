// Kernels for the TRACE_EDGES constraint family: A_0 = c_tr I and, per
// edge e = {i, j}, A_{1+e} = (e_i e_j^T + e_j e_i^T)/2 (entry constraints as in
// the examples of Sec. 3.3 / Sec. 4.3; with C = -J they give the Lovasz-theta
// SDP).  Cost C = S + Diag(d) - j J.
//
// Pass 1 (SDDMM): a_{1+e} = <R_i, R_j> for every edge, w_e = y_e - sigma
//   (a_e - b_e), plus column sums 1^T R and ||R||^2 for the trace row and J.
// Pass 2 (SpMM): G_i = 2 (P_i - c_tr w_0 R_i - 1/2 sum_{j~i} w_{e(ij)} R_j) with
//   P_i = (S R)_i + d_i R_i - j (1^T R); the symmetric pattern carries edge ids.
// Pass 3 (line search): a1_e = <R_i,G_j> + <G_i,R_j>, a2_e = <G_i,G_j> over the
//   edges and <G, (S + D) G>.
// The edge rows may carry their own penalty rho * sigma (the trace row keeps
// sigma): pass 1 forms w_e with it and weights the edge residual sums by rho,
// pass 3 weights the edge terms of the quartic by rho, so the finalizers'
// common factor sigma yields sigma on the trace row and rho sigma on the edges.
//
// Passes 1 and 3 walk the edges, not the rows: the edges of a sorted list all
// belong to their smaller end, so rows own very uneven shares of them (in matrix
// completion the first half of the rows owns every edge and the second none).
// Each block takes an equal run of edges, one group of LPR lanes per edge,
// several edges in flight; consecutive groups read consecutive entries of the
// edge arrays, and R_i of consecutive edges is mostly the same row and comes
// from L1.  Pass 2 walks rows of the symmetric pattern.
#include "finalize.hpp"
#include "quartic.hpp"
#include "spmm_row.hpp"

namespace almbm {

// Partial slots of pass 1, pass 2 and pass 3 (then, when the cost has a -J
// term, the r column sums of R and of G after those of passes 1 and 2).
enum { E1_YBMA = 0, E1_EE, E1_RR, E1_N };
enum { E2_C0 = 0, E2_GG, E2_GP, E2_RG, E2_N };
enum { E3_C2 = 0, E3_YA1, E3_YA2, E3_EA1, E3_EA2, E3_A1A1, E3_A1A2, E3_A2A2, E3_N };

// Sum over the lanes of a block that share the same lane-in-row index (i.e.
// over row groups) of a VEC-wide fragment, in fixed order, into the first r of
// LPR * VEC columns of out.
template <int LPR, int VEC>
__device__ __forceinline__ void block_colsum_store(double (&cs)[VEC], int r, double* __restrict__ out) {
  __shared__ double red[kBlock / kWave][LPR * VEC];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
#pragma unroll
  for (int v = 0; v < VEC; ++v) {
    double x = cs[v];
    for (int o = kWave / 2; o >= LPR; o >>= 1) x += __shfl_xor(x, o, kWave);
    cs[v] = x;
  }
  if (lane < LPR) {
#pragma unroll
    for (int v = 0; v < VEC; ++v) red[wave][lane * VEC + v] = cs[v];
  }
  __syncthreads();
  for (int c = threadIdx.x; c < r; c += kBlock) {
    double t = 0.0;
    for (int w = 0; w < kBlock / kWave; ++w) t += red[w][c];
    out[c] = t;
  }
}

// The U edges base + u * step (u < U, those below hi) of a group of LPR lanes.
// Lane q keeps the edge data of edge q, one load for all of them, and passes the
// row numbers to the group; the FP64 work of an edge is then done by one lane
// instead of all LPR.  A lane alone (LPR = 1) keeps all U edges (M of them).
// Rows of absent edges are row 0.
template <int U, int LPR> struct EdgeLanes {
  static_assert(LPR == 1 || U <= LPR, "a lane per edge");
  static constexpr int M = LPR == 1 ? U : 1;
  long e[M];
  bool in[M];
  int i[M], j[M];
  int lane;
  __device__ __forceinline__ EdgeLanes(const EdgeAdj& A, long base, int step, long hi, int lane_) : lane(lane_) {
#pragma unroll
    for (int q = 0; q < M; ++q) {
      const int u = LPR == 1 ? q : lane;
      e[q] = base + (long)u * step;
      in[q] = u < U && e[q] < hi;
      i[q] = in[q] ? A.ui[e[q]] : 0;
      j[q] = in[q] ? A.uci[e[q]] : 0;
    }
  }
  __device__ __forceinline__ long row_i(int u) const { return LPR == 1 ? i[u % M] : __shfl(i[0], u, LPR); }
  __device__ __forceinline__ long row_j(int u) const { return LPR == 1 ? j[u % M] : __shfl(j[0], u, LPR); }
  // of U values known to the whole group, the one of the lane's edge q
  template <typename V> __device__ __forceinline__ V mine(const V (&s)[U], int q) const {
    if constexpr (LPR == 1) return s[q];
    V x = s[0];
#pragma unroll
    for (int u = 1; u < U; ++u) x = lane == u ? s[u] : x;
    return x;
  }
};

// Bound by the gathers of R_j (and, at small r, by the 44 bytes of edge data).
// Lovasz n = 1e5, 1e6 edges, r = 32, FP32: 90 us walking rows, 40 us here
// (25e9 rows/s); completion n = 2e4, 1.8e6 edges, r = 3, FP64: 69 us with 4
// lanes per edge and half of the rows idle, 20 us (3.9 TB/s) here.
template <typename T, int LPR, int VEC, bool FULL>
__global__ void __launch_bounds__(kBlock)
k_edges_p1(EdgeAdj A, long n, int r, const T* __restrict__ R, const double* __restrict__ y,
           const double* __restrict__ b, double sigma, double* __restrict__ Av, double* __restrict__ wE,
           double* __restrict__ part, const DevScalars* __restrict__ sc, double rho, int ncs) {
  using V = typename Acc<T>::type;
  if (sc && sc->flag) return;
  constexpr int RPB = kBlock / LPR;
  constexpr int U = LPR >= 4 ? kUnroll : 2;
  const int lane = threadIdx.x % LPR;
  const int slot = threadIdx.x / LPR;
  SplitAcc<E1_N, 1> acc;  // every lane its own sums
  acc.zero();
  const RowChunk ce = row_chunk(A.E);
  for (long base = ce.lo + slot; base < ce.hi; base += RPB * U) {
    EdgeLanes<U, LPR> ed(A, base, RPB, ce.hi, lane);
    double be[ed.M], ye[ed.M];
#pragma unroll
    for (int q = 0; q < ed.M; ++q) {
      be[q] = ed.in[q] ? b[1 + ed.e[q]] : 0.0;
      ye[q] = ed.in[q] ? y[1 + ed.e[q]] : 0.0;
    }
    V ri[U][VEC], rj[U][VEC];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      load_frag<T, VEC, FULL>(R + ed.row_i(u) * r, lane, r, ri[u]);
      load_frag<T, VEC, FULL>(R + ed.row_j(u) * r, lane, r, rj[u]);
    }
    V s[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      s[u] = 0;
#pragma unroll
      for (int v = 0; v < VEC; ++v) s[u] += ri[u][v] * rj[u][v];
      s[u] = group_sum<LPR>(s[u]);
    }
#pragma unroll
    for (int q = 0; q < ed.M; ++q) {
      if (!ed.in[q]) continue;
      const double a = ed.mine(s, q);
      const double res = a - be[q];
      if (Av) Av[1 + ed.e[q]] = a;
      wE[ed.e[q]] = ye[q] - rho * sigma * res;
      acc.a[E1_YBMA] += ye[q] * (be[q] - a);
      acc.a[E1_EE] += rho * res * res;
    }
  }
  double cs[VEC];
#pragma unroll
  for (int v = 0; v < VEC; ++v) cs[v] = 0.0;
  const RowChunk ch = row_chunk(n);
  for (long i = ch.lo + slot; i < ch.hi; i += RPB) {
    V ri[VEC];
    load_frag<T, VEC, FULL>(R + i * r, lane, r, ri);
    V rr = 0;
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      rr += ri[v] * ri[v];
      cs[v] += (double)ri[v];
    }
    rr = group_sum<LPR>(rr);
    if (lane == 0) acc.a[E1_RR] += (double)rr;
  }
  double* out = part + (long)blockIdx.x * (E1_N + ncs);
  acc.block_store(out);
  if (ncs) block_colsum_store<LPR, VEC>(cs, r, out + E1_N);
}

// Pass 2: P = C R, gradient and its partials.  If G_in is given, the direction
// is read instead of computed (line-search API) and nothing is written.  Rows
// with many neighbours are split over the S = 64 / LPR groups of a wave, U
// neighbours in flight per group; the groups' shares are added in a fixed
// order.  Bound by the row gathers and the random wE of the lower half.
// Completion n = 2e4, r = 3, FP64: 62 us with 4 lanes per neighbour and one in
// flight, 47 us; Lovasz n = 1e5, r = 32, FP32: 92 us, 61 us (33e9 rows/s).
// HASS: the cost has stored entries (the two workloads above have none; without
// the product's gathers the FP64 kernel for r <= 4 needs 78 registers, not 126).
template <typename T, int LPR, int VEC, bool FULL, int S, bool HASS>
__global__ void __launch_bounds__(kBlock)
k_edges_p2(Cost<typename Acc<T>::type> C, EdgeAdj A, int r, const T* __restrict__ R,
           const double* __restrict__ wE, double c_tr, double j_coef, const T* __restrict__ G_in,
           T* __restrict__ G, double* __restrict__ part, const DevScalars* __restrict__ sc, int ncs) {
  using V = typename Acc<T>::type;
  if (sc->flag) return;
  constexpr int RPB = kBlock / (LPR * S);
  constexpr int U = LPR == 1 ? 2 : (LPR >= 8 && sizeof(V) * VEC <= 16 ? 8 : 4);
  const int lane = threadIdx.x % LPR;
  const int grp = (threadIdx.x / LPR) % S;
  const int slot = threadIdx.x / (LPR * S);
  SplitAcc<E2_N, LPR> acc;
  acc.zero();
  double gcs[VEC];
  V jcs[VEC];
#pragma unroll
  for (int v = 0; v < VEC; ++v) {
    gcs[v] = 0.0;
    const int c = lane * VEC + v;
    jcs[v] = (c < r && ncs) ? static_cast<V>(j_coef * sc->colsum[c]) : V(0);
  }
  const V cw0 = c_tr != 0.0 ? static_cast<V>(c_tr * sc->w0) : V(0);
  const RowChunk ch = row_chunk(C.n);
  for (long base = ch.lo; base < ch.hi; base += RPB) {
    const long i = base + slot;
    if (i >= ch.hi) break;
    const int k0 = A.rp[i], k1 = A.rp[i + 1];
    V ad[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) ad[v] = V(0);
    if constexpr (LPR >= 4) {
      // lane q of the group loads the column, edge id and weight of neighbour
      // k + q, the next U columns and ids while the rows are on their way
      const int q = lane % U;
      int k = k0 + grp * U;
      int jq = k + q < k1 ? A.ci[k + q] : (int)i;
      int iq = k + q < k1 ? A.eid[k + q] : -1;
      for (; k < k1; k += S * U) {
        V rj[U][VEC];
        const V wq = iq >= 0 ? static_cast<V>(0.5 * wE[iq]) : V(0);
#pragma unroll
        for (int u = 0; u < U; ++u)
          load_frag<T, VEC, FULL>(R + (long)__shfl(jq, u, LPR) * r, lane, r, rj[u]);
        const int kn = k + S * U + q;
        jq = kn < k1 ? A.ci[kn] : (int)i;
        iq = kn < k1 ? A.eid[kn] : -1;
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const V we = __shfl(wq, u, LPR);
          if (k + u < k1) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) ad[v] += we * rj[u][v];
          }
        }
      }
    } else {
      for (int k = k0 + grp; k < k1; k += S * U) {
        int jj[U], id[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int kk = k + u * S;
          jj[u] = kk < k1 ? A.ci[kk] : (int)i;
          id[u] = kk < k1 ? A.eid[kk] : -1;
        }
        V we[U], rj[U][VEC];
#pragma unroll
        for (int u = 0; u < U; ++u) {
          we[u] = id[u] >= 0 ? static_cast<V>(0.5 * wE[id[u]]) : V(0);
          load_frag<T, VEC, FULL>(R + (long)jj[u] * r, lane, r, rj[u]);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
          if (id[u] >= 0) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) ad[v] += we[u] * rj[u][v];
          }
      }
    }
    if constexpr (S > 1 && VEC <= S) {
      // halving leaves column (l, v) in lanes v (64 / VEC) + l; every lane takes it from there
      const int wl = threadIdx.x % kWave;
      const V x = wave_sum_many<VEC, LPR>(ad, wl);
#pragma unroll
      for (int v = 0; v < VEC; ++v) ad[v] = __shfl(x, v * (kWave / VEC) + lane, kWave);
    } else {
#pragma unroll
      for (int o = LPR; o < LPR * S; o <<= 1)
#pragma unroll
        for (int v = 0; v < VEC; ++v) ad[v] += __shfl_xor(ad[v], o, kWave);
    }
    if (grp == 0) {  // the row's own terms, once
      V ri[VEC], p[VEC], g[VEC];
      load_frag<T, VEC, FULL>(R + i * r, lane, r, ri);
      if constexpr (HASS) {
        spmm_row<T, LPR, VEC, FULL>(C, i, lane, r, R, ri, p);
      } else {
        const V di = C.dg ? C.dg[i] : V(0);
#pragma unroll
        for (int v = 0; v < VEC; ++v) p[v] = di * ri[v];
      }
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
        p[v] -= jcs[v];
        ad[v] += cw0 * ri[v];
      }
      if (G_in) {
        load_frag<T, VEC, FULL>(G_in + i * r, lane, r, g);
      } else {
#pragma unroll
        for (int v = 0; v < VEC; ++v) g[v] = round_st<T>(V(2) * (p[v] - ad[v]));
        if (G) store_frag<T, VEC, FULL>(G + i * r, lane, r, g);
      }
      V rp = 0, gg = 0, gp = 0, rg = 0;
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
        rp += ri[v] * p[v];
        gg += g[v] * g[v];
        gp += g[v] * p[v];
        rg += ri[v] * g[v];
        gcs[v] += (double)g[v];
      }
      rp = group_sum<LPR>(rp);
      gg = group_sum<LPR>(gg);
      gp = group_sum<LPR>(gp);
      rg = group_sum<LPR>(rg);
      acc.add(lane, E2_C0, (double)rp);
      acc.add(lane, E2_GG, (double)gg);
      acc.add(lane, E2_GP, (double)gp);
      acc.add(lane, E2_RG, (double)rg);
    }
  }
  double* out = part + (long)blockIdx.x * (E2_N + ncs);
  acc.block_store(out);
  if (ncs) block_colsum_store<LPR, VEC>(gcs, r, out + E2_N);
}

// Finalize of passes 1 and 2, either one or both (a null table skips its half).
// Pass 1: trace row, w_0, column sums; writes Av[0].  Pass 2: objective and
// (mode 1) the inner stop test.
template <int THREADS>
__device__ __forceinline__ void finish_edges12(const EdgeFin& F) {
  DevScalars* sc = F.sc;
  const int nb = F.nb, ncs = F.ncs;
  const double *y = F.y, *b = F.b;
  const double sigma = F.sigma, c_tr = F.c_tr;
  double *Av = F.Av, *f_out = F.f_out;
  const int mode = F.mode;
  __shared__ double t1[E1_N + kMaxR], t2[E2_N + kMaxR];
  if (F.part1) {
    fin_table<THREADS>(F.part1, nb, E1_N + ncs, t1);
    if (threadIdx.x < ncs) sc->colsum[threadIdx.x] = t1[E1_N + threadIdx.x];
    if (threadIdx.x == 0) {
      const double rr = t1[E1_RR];
      const double a0 = c_tr * rr;
      const double e0 = a0 - b[0];
      sc->a0 = a0;
      sc->w0 = y[0] - sigma * e0;
      if (Av) Av[0] = a0;
      sc->tot[P_YBMA] = t1[E1_YBMA] + y[0] * (b[0] - a0);
      sc->tot[P_EE] = t1[E1_EE] + e0 * e0;
      sc->tot[P_RR] = rr;
    }
  }
  if (!F.part2) return;
  fin_table<THREADS>(F.part2, nb, E2_N + ncs, t2);
  if (threadIdx.x < ncs) sc->gcolsum[threadIdx.x] = t2[E2_N + threadIdx.x];
  if (threadIdx.x != 0) return;
  sc->tot[P_C0] = t2[E2_C0];
  sc->tot[P_GG] = t2[E2_GG];
  sc->tot[P_GP] = t2[E2_GP];
  sc->tot[P_RG] = t2[E2_RG];
  const double f = t2[E2_C0] + sc->tot[P_YBMA] + 0.5 * sigma * sc->tot[P_EE];
  sc->f = f;
  if (!isfinite(f) || !isfinite(t2[E2_GG])) sc->numeric_error = 1;
  if (f_out) *f_out = f;
  if (mode == 1) {
    const double lhs = sqrt(t2[E2_GG]) * sqrt(sc->tot[P_RR]);
    if (sc->iter >= sc->max_inner) sc->flag = 2;
    else if (lhs <= sc->tol * (1.0 + fabs(t2[E2_C0])) || !isfinite(lhs)) sc->flag = 1;
    else sc->iter += 1;
  }
}
__global__ void __launch_bounds__(kFin) k_fin_edges12(EdgeFin F) {
  if (F.sc->flag) return;
  finish_edges12<kFin>(F);
}

// Pass 3: line-search partials over the edges and <G, (S + D) G>.  As pass 1,
// with two rows (R_j, G_j) gathered per edge.  Completion n = 2e4, r = 3, FP64:
// 64 us walking rows, 33 us here.
template <typename T, int LPR, int VEC, bool FULL>
__global__ void __launch_bounds__(kBlock)
k_edges_p3(Cost<typename Acc<T>::type> C, EdgeAdj A, int r, const T* __restrict__ R, const T* __restrict__ G,
           const double* __restrict__ y, const double* __restrict__ b, const double* __restrict__ Av,
           double* __restrict__ part, const DevScalars* sc, double rho, EdgeFin side) {
  using V = typename Acc<T>::type;
  if (block_stopped(sc)) return;
  const int nblk = gridDim.x - (side.part2 ? 1 : 0);
  if ((int)blockIdx.x == nblk) {  // the finalizer of passes 1 and 2
    finish_edges12<kBlock>(side);
    return;
  }
  constexpr int RPB = kBlock / LPR;
  constexpr int U = 2;
  const int lane = threadIdx.x % LPR;
  const int slot = threadIdx.x / LPR;
  SplitAcc<E3_N, 1> acc;  // every lane its own sums
  acc.zero();
  const RowChunk ce = row_chunk(A.E, false, nblk);
  for (long base = ce.lo + slot; base < ce.hi; base += RPB * U) {
    EdgeLanes<U, LPR> ed(A, base, RPB, ce.hi, lane);
    double res[ed.M], ye[ed.M];
#pragma unroll
    for (int q = 0; q < ed.M; ++q) {
      res[q] = ed.in[q] ? Av[1 + ed.e[q]] - b[1 + ed.e[q]] : 0.0;
      ye[q] = ed.in[q] ? y[1 + ed.e[q]] : 0.0;
    }
    V a1[U], a2[U];
    {
      V ri[U][VEC], gi[U][VEC], rj[U][VEC], gj[U][VEC];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const long i = ed.row_i(u), j = ed.row_j(u);
        load_frag<T, VEC, FULL>(R + j * r, lane, r, rj[u]);
        load_frag<T, VEC, FULL>(G + j * r, lane, r, gj[u]);
        load_frag<T, VEC, FULL>(R + i * r, lane, r, ri[u]);
        load_frag<T, VEC, FULL>(G + i * r, lane, r, gi[u]);
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        a1[u] = a2[u] = 0;
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
          a1[u] += ri[u][v] * gj[u][v] + gi[u][v] * rj[u][v];
          a2[u] += gi[u][v] * gj[u][v];
        }
        a1[u] = group_sum<LPR>(a1[u]);
        a2[u] = group_sum<LPR>(a2[u]);
      }
    }
#pragma unroll
    for (int q = 0; q < ed.M; ++q) {
      if (!ed.in[q]) continue;
      const double d1 = ed.mine(a1, q), d2 = ed.mine(a2, q);
      acc.a[E3_YA1] += ye[q] * d1;
      acc.a[E3_YA2] += ye[q] * d2;
      acc.a[E3_EA1] += rho * res[q] * d1;
      acc.a[E3_EA2] += rho * res[q] * d2;
      acc.a[E3_A1A1] += rho * d1 * d1;
      acc.a[E3_A1A2] += rho * d1 * d2;
      acc.a[E3_A2A2] += rho * d2 * d2;
    }
  }
  if (C.rp || C.ell > 0 || C.dg) {
    const RowChunk ch = row_chunk(C.n, false, nblk);
    for (long i = ch.lo + slot; i < ch.hi; i += RPB) {
      V gi[VEC], q[VEC];
      load_frag<T, VEC, FULL>(G + i * r, lane, r, gi);
      spmm_row<T, LPR, VEC, FULL>(C, i, lane, r, G, gi, q);
      V gq = 0;
#pragma unroll
      for (int v = 0; v < VEC; ++v) gq += gi[v] * q[v];
      gq = group_sum<LPR>(gq);
      if (lane == 0) acc.a[E3_C2] += (double)gq;
    }
  }
  acc.block_store(part + (long)blockIdx.x * E3_N);
}

// Finalize of pass 3: add the trace row and the -jJ terms, then the step.
__global__ void __launch_bounds__(kFin)
k_fin_edges3(const double* __restrict__ part, int nb, int r, DevScalars* __restrict__ sc, const double* __restrict__ y,
             const double* __restrict__ b, double sigma, double c_tr, double j_coef, int mode,
             double* __restrict__ coeffs_out, double* __restrict__ t_out) {
  if (mode == 1 && sc->flag) return;
  __shared__ double t3[E3_N];
  fin_rows<E3_N>(part, nb, t3);
  if (threadIdx.x != 0) return;
  double gj2 = 0.0;
  if (j_coef != 0.0)
    for (int c = 0; c < r; ++c) gj2 += sc->gcolsum[c] * sc->gcolsum[c];
  const double a1_0 = 2.0 * c_tr * sc->tot[P_RG];
  const double a2_0 = c_tr * sc->tot[P_GG];
  const double e0 = sc->a0 - b[0];
  double* tot = sc->tot;
  tot[P_C2] = t3[E3_C2] - j_coef * gj2;
  tot[P_YA1] = t3[E3_YA1] + y[0] * a1_0;
  tot[P_YA2] = t3[E3_YA2] + y[0] * a2_0;
  tot[P_EA1] = t3[E3_EA1] + e0 * a1_0;
  tot[P_EA2] = t3[E3_EA2] + e0 * a2_0;
  tot[P_A1A1] = t3[E3_A1A1] + a1_0 * a1_0;
  tot[P_A1A2] = t3[E3_A1A2] + a1_0 * a2_0;
  tot[P_A2A2] = t3[E3_A2A2] + a2_0 * a2_0;
  double k[5];
  quartic_coeffs(tot, sigma, k);
  for (int s = 0; s < 5; ++s) sc->coeffs[s] = k[s];
  double t = (mode == 1 && sc->step_rule == 1) ? sc->eta_fixed : quartic_argmin(k);
  if (!isfinite(t)) {
    t = 0.0;
    sc->numeric_error = 1;
  }
  sc->t = t;
  if (coeffs_out)
    for (int s = 0; s < 5; ++s) coeffs_out[s] = k[s];
  if (t_out) *t_out = t;
}

// ---- launchers -----------------------------------------------------------------

// Tile (lanes, columns per lane) for a rank r.  In FP64, up to r = 8 one or two
// lanes hold a whole row: an edge or a neighbour per lane keeps the edge arrays'
// loads dense and needs (almost) no shuffles.  The float types keep more lanes
// per row, whose sums of few products round like a tree rather than a chain.
#define ALMBM_DISPATCH_EDGES(T, FN, ...)                                \
  do {                                                                  \
    if constexpr (sizeof(T) == 8) {                                     \
      if (r <= 4) FN<T, 1, 4>(__VA_ARGS__);                             \
      else if (r <= 8) FN<T, 2, 4>(__VA_ARGS__);                        \
      else if (r <= 16) FN<T, 8, 2>(__VA_ARGS__);                       \
      else if (r <= 32) FN<T, 8, 4>(__VA_ARGS__);                       \
      else if (r <= 64) FN<T, 16, 4>(__VA_ARGS__);                      \
      else FN<T, 32, 4>(__VA_ARGS__);                                   \
    } else if constexpr (sizeof(T) == 4) {                              \
      if (r <= 4) FN<T, 4, 1>(__VA_ARGS__);                             \
      else if (r <= 8) FN<T, 4, 2>(__VA_ARGS__);                        \
      else if (r <= 16) FN<T, 4, 4>(__VA_ARGS__);                       \
      else if (r <= 32) { if (variant == 1) FN<T, 4, 8>(__VA_ARGS__); else FN<T, 8, 4>(__VA_ARGS__); } \
      else if (r <= 64) FN<T, 16, 4>(__VA_ARGS__);                      \
      else FN<T, 32, 4>(__VA_ARGS__);                                   \
    } else {                                                            \
      if (r <= 4) FN<T, 2, 2>(__VA_ARGS__);                             \
      else if (r <= 8) FN<T, 2, 4>(__VA_ARGS__);                        \
      else if (r <= 16) FN<T, 2, 8>(__VA_ARGS__);                       \
      else if (r <= 32) FN<T, 4, 8>(__VA_ARGS__);                       \
      else if (r <= 64) FN<T, 8, 8>(__VA_ARGS__);                       \
      else FN<T, 16, 8>(__VA_ARGS__);                                   \
    }                                                                   \
  } while (0)

template <typename T, int LPR, int VEC>
static void p1_cfg(const EdgeAdj& A, long n, int r, const T* R, const double* y, const double* b, double sigma,
                   double* Av, double* wE, double* part, const DevScalars* sc, int nblk, hipStream_t st, double rho,
                   int ncs) {
  if (r == LPR * VEC)
    hipLaunchKernelGGL((k_edges_p1<T, LPR, VEC, true>), dim3(nblk), dim3(kBlock), 0, st, A, n, r, R, y, b, sigma, Av,
                       wE, part, sc, rho, ncs);
  else
    hipLaunchKernelGGL((k_edges_p1<T, LPR, VEC, false>), dim3(nblk), dim3(kBlock), 0, st, A, n, r, R, y, b, sigma, Av,
                       wE, part, sc, rho, ncs);
}
template <typename T, int LPR, int VEC, int S, bool HASS>
static void p2_split(const Cost<typename Acc<T>::type>& C, const EdgeAdj& A, int r, const T* R, const double* wE,
                     double c_tr, double j_coef, const T* G_in, T* G, double* part, const DevScalars* sc, int nblk,
                     hipStream_t st, int ncs) {
  if (r == LPR * VEC)
    hipLaunchKernelGGL((k_edges_p2<T, LPR, VEC, true, S, HASS>), dim3(nblk), dim3(kBlock), 0, st, C, A, r, R, wE, c_tr,
                       j_coef, G_in, G, part, sc, ncs);
  else
    hipLaunchKernelGGL((k_edges_p2<T, LPR, VEC, false, S, HASS>), dim3(nblk), dim3(kBlock), 0, st, C, A, r, R, wE,
                       c_tr, j_coef, G_in, G, part, sc, ncs);
}
// A wave per row when the average row has 8 neighbours for each of its 64 / LPR
// groups.  With one or two lanes per neighbour (FP64, r <= 8) half a neighbour per
// group is enough: the alternative there is one lane walking a row alone, its
// loads 64 rows apart.
template <typename T, int LPR, int VEC>
static void p2_cfg(const Cost<typename Acc<T>::type>& C, const EdgeAdj& A, int r, const T* R, const double* wE,
                   double c_tr, double j_coef, const T* G_in, T* G, double* part, const DevScalars* sc, int nblk,
                   hipStream_t st, int ncs) {
  const float least = LPR <= 2 && sizeof(T) == 8 ? 32.f : 8.f * (kWave / LPR);
  const bool split = A.avg_deg >= least, hass = C.rp || C.ell > 0;
#define ALMBM_P2(S_, HASS_) \
  p2_split<T, LPR, VEC, S_, HASS_>(C, A, r, R, wE, c_tr, j_coef, G_in, G, part, sc, nblk, st, ncs)
  if (split && hass) ALMBM_P2(kWave / LPR, true);
  else if (split) ALMBM_P2(kWave / LPR, false);
  else if (hass) ALMBM_P2(1, true);
  else ALMBM_P2(1, false);
#undef ALMBM_P2
}
template <typename T, int LPR, int VEC>
static void p3_cfg(const Cost<typename Acc<T>::type>& C, const EdgeAdj& A, int r, const T* R, const T* G,
                   const double* y, const double* b, const double* Av, double* part, const DevScalars* sc, int nblk,
                   hipStream_t st, double rho, const EdgeFin& side) {
  const dim3 grid(nblk + (side.part2 ? 1 : 0));
  if (r == LPR * VEC)
    hipLaunchKernelGGL((k_edges_p3<T, LPR, VEC, true>), grid, dim3(kBlock), 0, st, C, A, r, R, G, y, b, Av,
                       part, sc, rho, side);
  else
    hipLaunchKernelGGL((k_edges_p3<T, LPR, VEC, false>), grid, dim3(kBlock), 0, st, C, A, r, R, G, y, b, Av,
                       part, sc, rho, side);
}

// Whether a block of pass 3 adds the totals of passes 1 and 2 (len doubles of partial
// sums; bytes: one gathered row per edge).  It saves a launch and the finalizer's own
// time if pass 3 lasts as long as the block, which has a quarter of a finalizer's
// threads, takes some 0.35 ns a double and starts last: with more than 2048 blocks after
// most of them.  Per step, kernel -> block: completion n = 1000 and 2e4, r = 3, FP64
// (len 2e3, 7e3) 32.6 -> 29.1 and 122 -> 116 us; with a -J term n = 1e5, E = 2e5, r = 32,
// FP32 (3.7e4) 99.6 -> 97.0, n = 5e4, E = 2e5, r = 100, FP32 (8.2e4 and 8e7 bytes) 201 ->
// 184, but n = 1e5, E = 2e5, r = 64, BF16 (7.0e4, 2.6e7) 124 -> 129, n = 7e4, E = 1e5, r =
// 100, BF16 (1.1e5, 2.1e7) 200 -> 210; on chosen grids n = 1e5, E = 1e6, r = 32, FP32 198
// -> 193 with 2048 blocks, 212 -> 219 with 4096.
static bool side_edges12(long len, int nblk, double bytes) {
  return nblk <= 2048 && (len <= 40000 || bytes >= 512.0 * (double)len);
}

template <typename T>
void launch_edges_eval(const Cost<typename Acc<T>::type>& C, const EdgeAdj& A, long n, int r, int variant, const T* R,
                       const double* y, const double* b, double sigma, double c_tr, double j_coef, double rho,
                       double* Av, double* wE, const T* G_in, T* G, double* part, DevScalars* sc, int nblk, int mode,
                       double* f_out, hipStream_t st, EdgeFin* defer) {
  const int ncs = j_coef != 0.0 ? r : 0;
  ALMBM_DISPATCH_EDGES(T, p1_cfg, A, n, r, R, y, b, sigma, Av, wE, part, sc, nblk, st, rho, ncs);
  // pass 2 waits for the finalizer of pass 1 only for the trace row's w_0 and the
  // column sums; it may then reuse its table (part holds NUM_P + kMaxR per block)
  const bool wait = c_tr != 0.0 || ncs > 0;
  double* part2 = wait ? part : part + (long)nblk * E1_N;
  EdgeFin fin{part, nullptr, nblk, ncs, sc, y, b, sigma, c_tr, Av, mode, nullptr};
  if (wait) hipLaunchKernelGGL(k_fin_edges12, dim3(1), dim3(kFin), 0, st, fin);
  ALMBM_DISPATCH_EDGES(T, p2_cfg, C, A, r, R, wE, c_tr, j_coef, G_in, G, part2, sc, nblk, st, ncs);
  fin.part1 = wait ? nullptr : part;
  fin.part2 = part2;
  fin.f_out = f_out;
  if (defer && side_edges12((long)nblk * (E2_N + ncs + (wait ? 0 : E1_N)), nblk, (double)A.E * r * sizeof(T)))
    *defer = fin;
  else
    hipLaunchKernelGGL(k_fin_edges12, dim3(1), dim3(kFin), 0, st, fin);
}
template <typename T>
double* launch_edges_p3(const Cost<typename Acc<T>::type>& C, const EdgeAdj& A, int r, int variant, const T* R,
                        const T* G, const double* y, const double* b, const double* Av, double* part,
                        const DevScalars* sc, int nblk, hipStream_t st, double rho, const EdgeFin& side) {
  // behind the rows of passes 1 and 2 that the side block reads: at most 4 + kMaxR of
  // a block's NUM_P + kMaxR, and pass 3 has 8
  if (side.part2) part += (side.part2 - part) + (long)nblk * (E2_N + side.ncs);
  ALMBM_DISPATCH_EDGES(T, p3_cfg, C, A, r, R, G, y, b, Av, part, sc, nblk, st, rho, side);
  return part;
}
static_assert(E1_N + E2_N + E3_N <= NUM_P + kMaxR && E2_N + kMaxR + E3_N <= NUM_P + kMaxR);
void launch_fin_edges3(const double* part, int nb, int r, DevScalars* sc, const double* y, const double* b,
                       double sigma, double c_tr, double j_coef, int mode, double* coeffs_out, double* t_out,
                       hipStream_t st) {
  hipLaunchKernelGGL(k_fin_edges3, dim3(1), dim3(kFin), 0, st, part, nb, r, sc, y, b, sigma, c_tr, j_coef, mode,
                     coeffs_out, t_out);
}

#define ALMBM_INST_E(T)                                                                                          \
  template void launch_edges_eval<T>(const Cost<Acc<T>::type>&, const EdgeAdj&, long, int, int, const T*,        \
                                     const double*, const double*, double, double, double, double, double*,      \
                                     double*, const T*, T*, double*, DevScalars*, int, int, double*, hipStream_t, \
                                     EdgeFin*);                                                                  \
  template double* launch_edges_p3<T>(const Cost<Acc<T>::type>&, const EdgeAdj&, int, int, const T*, const T*,       \
                                   const double*, const double*, const double*, double*, const DevScalars*, int, \
                                   hipStream_t, double, const EdgeFin&);

ALMBM_INST_E(double)
ALMBM_INST_E(float)
ALMBM_INST_E(bf16)

}  // namespace almbm
