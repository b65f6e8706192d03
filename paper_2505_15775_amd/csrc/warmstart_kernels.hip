// Learned warm start for the dual y0 of ALM-BM (MaxCut-type problems with the
// diagonal constraint family): per-vertex graph features, a small MLP
// (n_in -> h -> h -> 1, ReLU, FP32) forward and backward passes with
// deterministic gradient reductions, and the Adam update.  The MLP's products
// run on the FP32 matrix instructions: at 2.6 kflop per 40 bytes of a vertex
// (h = 32) the vector ALUs, fed one weight at a time, were the bound.
#include "launch.hpp"

namespace almbm {

constexpr int kWsFeat = 8;    // features per vertex

// Features of vertex i (row i of the cost):
//   f0 = log1p(deg_i), f1 = sum_j |S_ij|, f2 = sum_j S_ij, f3 = d_i,
//   f4 = d_i - sum_j |S_ij| (a Gershgorin bound: y_i <= it keeps Z(y) PSD),
//   f5 mean and f6 max of the neighbours' f0, f7 mean of their f1.
// Pass 1 leaves (f0, f1) of every vertex as one 8-byte pair; pass 2 gathers the
// neighbours' pairs (one random access per entry instead of one for each of two
// tables) and writes whole feature rows.  Both walk a row with kWsLpr lanes and
// kWsUnroll entries in flight per lane; the float sums of pass 2 still run over
// a row in its order (each lane adds all of its row group's values in turn).
// Pass 1 streams the cost, pass 2 is bound by the gathers.  n = 1e6, 8e6 entries: 115 + 344 us with a thread per row
// and two gathered tables, 24 + 98 us (82e9 gathers/s) now.
constexpr int kWsLpr = 4;  // quad_lane below works on groups of four
constexpr int kWsUnroll = 4;

__device__ __forceinline__ void ws_row_range(const Cost<double>& C, long i, long& k0, long& k1) {
  k0 = k1 = 0;
  if (C.ell > 0) {
    k0 = i * (long)C.ell;
    k1 = k0 + C.ell;
  } else if (C.rp) {
    k0 = C.rp[i];
    k1 = C.rp[i + 1];
  }
}

__global__ void __launch_bounds__(kBlock)
k_ws_feat1(Cost<double> C, float2* __restrict__ pair) {
  const long i = ((long)blockIdx.x * kBlock + threadIdx.x) / kWsLpr;
  const int lane = threadIdx.x % kWsLpr;
  if (i >= C.n) return;
  long k0, k1;
  ws_row_range(C, i, k0, k1);
  double sa = 0.0;
  int deg = 0;
  for (long k = k0 + lane; k < k1; k += kWsLpr * kWsUnroll) {
#pragma unroll
    for (int u = 0; u < kWsUnroll; ++u) {
      const long kk = k + u * kWsLpr;
      const double v = kk < k1 ? C.cv[kk] : 0.0;
      const int j = kk < k1 ? C.ci[kk] : (int)i;
      if (v != 0.0 && j != i) {
        sa += fabs(v);
        ++deg;
      }
    }
  }
  sa = group_sum<kWsLpr>(sa);
  deg = group_sum<kWsLpr>(deg);
  if (lane == 0) pair[i] = make_float2(log1pf((float)deg), (float)sa);
}

// Value of lane L (0..3) of the lane's group of four.
template <int L>
__device__ __forceinline__ float quad_lane(float x) {
  constexpr int ctrl = L | L << 2 | L << 4 | L << 6;  // quad_perm [L, L, L, L]
  return __uint_as_float(__builtin_amdgcn_mov_dpp(__float_as_uint(x), ctrl, 0xf, 0xf, true));
}
__device__ __forceinline__ void add_in_order(float& s, float x) {
  s += quad_lane<0>(x);
  s += quad_lane<1>(x);
  s += quad_lane<2>(x);
  s += quad_lane<3>(x);
}

__global__ void __launch_bounds__(kBlock)
k_ws_feat2(Cost<double> C, const float2* __restrict__ pair, float* __restrict__ F) {
  const long i = ((long)blockIdx.x * kBlock + threadIdx.x) / kWsLpr;
  const int lane = threadIdx.x % kWsLpr;
  if (i >= C.n) return;
  long k0, k1;
  ws_row_range(C, i, k0, k1);
  double sa = 0.0, s = 0.0;
  float sum = 0.f, mx = 0.f, s1 = 0.f;
  int cnt = 0;
  for (long kb = k0; kb < k1; kb += kWsLpr * kWsUnroll) {  // the same trips for the four lanes
    const long k = kb + lane;
    double v[kWsUnroll];
    int j[kWsUnroll];
    float2 pj[kWsUnroll];
#pragma unroll
    for (int u = 0; u < kWsUnroll; ++u) {
      const long kk = k + u * kWsLpr;
      v[u] = kk < k1 ? C.cv[kk] : 0.0;
      j[u] = kk < k1 ? C.ci[kk] : (int)i;
    }
#pragma unroll
    for (int u = 0; u < kWsUnroll; ++u) pj[u] = pair[j[u]];
#pragma unroll
    for (int u = 0; u < kWsUnroll; ++u) {
      const bool use = v[u] != 0.0 && j[u] != i;
      add_in_order(sum, use ? pj[u].x : 0.f);
      add_in_order(s1, use ? pj[u].y : 0.f);
      if (!use) continue;
      sa += fabs(v[u]);
      s += v[u];
      mx = fmaxf(mx, pj[u].x);
      ++cnt;
    }
  }
  sa = group_sum<kWsLpr>(sa);
  s = group_sum<kWsLpr>(s);
  cnt = group_sum<kWsLpr>(cnt);
#pragma unroll
  for (int o = kWsLpr / 2; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o, kWsLpr));
  if (lane != 0) return;
  const double di = C.dg ? C.dg[i] : 0.0;
  const float inv = cnt ? 1.f / (float)cnt : 0.f;
  const float f[kWsFeat] = {log1pf((float)cnt), (float)sa, (float)s, (float)di, (float)(di - sa),
                            sum * inv,          mx,        s1 * inv};
  __builtin_memcpy(F + i * kWsFeat, f, sizeof(f));
}

// Parameter layout (floats): W1[nin][h], b1[h], W2[h][h], b2[h], W3[h], b3[1].
__device__ __forceinline__ int ws_nparams(int nin, int h) { return nin * h + h + h * h + h + h + 1; }

// Stage the parameters in LDS (<= 8*64 + 64 + 64*64 + 64 + 64 + 1 floats).
__device__ __forceinline__ void ws_load_params(const float* __restrict__ P, float* __restrict__ S, int np) {
  for (int k = threadIdx.x; k < np; k += kBlock) S[k] = P[k];
  __syncthreads();
}

// The MLP on tiles of 32 vertices per wave, transposed: with the weights as the A
// operand of v_mfma_f32_32x32x2f32 and the vertices as its columns, lane l holds
// column l % 32 and accumulator register r the row ws_row(r, l / 32) of a block
// of 32.  The hidden unit computed in row c is ws_unit_of(c), chosen so that
// register r holds unit 2 r in the lower and 2 r + 1 in the upper half of the
// wave: a layer's accumulators are then the next layer's B operands as they
// stand, one register per step, and the units are added in their natural order.
// The instruction adds its two products one after the other, so every
// pre-activation is the same chain of FP32 fused multiply-adds as a loop over
// the inputs.  h = 16 is a block of 32 with zero weights, half of its steps left
// out.
typedef float ws_acc16 __attribute__((ext_vector_type(16)));
typedef float ws_acc4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ constexpr int ws_row(int r, int half) { return (r & 3) + 8 * (r >> 2) + 4 * half; }
__device__ __forceinline__ constexpr int ws_unit(int r, int half) { return 2 * r + half; }
__device__ __forceinline__ constexpr int ws_unit_of(int row) {
  return ws_unit((row & 3) + 4 * (row >> 3), (row >> 2) & 1);
}

template <int H> struct WsShape {
  static constexpr int B = (H + 31) / 32;      // blocks of 32 hidden units
  static constexpr int HP = 32 * B;            // padded width
  static constexpr int KS = H >= 32 ? 16 : 8;  // steps of a product over one block of units
};

// z[b][r] = bias[unit] (zero past H).
template <int H>
__device__ __forceinline__ void ws_bias(const float* __restrict__ bias, int half, ws_acc16 (&z)[WsShape<H>::B]) {
#pragma unroll
  for (int b = 0; b < WsShape<H>::B; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int u = 32 * b + ws_unit(r, half);
      z[b][r] = (H >= 32 || u < H) ? bias[u] : 0.f;
    }
}

// Features half, half + 2, half + 4, half + 6 of vertex v, standardised (zero for
// absent ones).
__device__ __forceinline__ void ws_inputs(const float* __restrict__ X, long v, bool in, int nin, int half,
                                          const float (&m)[4], const float (&d)[4], float (&x)[4]) {
  float raw[kWsFeat];
#pragma unroll
  for (int k = 0; k < kWsFeat; ++k) raw[k] = 0.f;
  if (in) load_some<float, kWsFeat>(X + v * nin, nin, raw);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float f = half ? raw[2 * q + 1] : raw[2 * q];
    x[q] = (in && 2 * q + half < nin) ? (f - m[q]) * d[q] : 0.f;
  }
}
__device__ __forceinline__ void ws_scaling(const float* __restrict__ mu, const float* __restrict__ isd, int nin,
                                           int half, float (&m)[4], float (&d)[4]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int f = 2 * q + half;
    m[q] = f < nin ? mu[f] : 0.f;
    d[q] = f < nin ? isd[f] : 0.f;
  }
}

// Hidden layers of a tile: pre-activations z1, z2 from the inputs x.  S: the
// parameters in LDS.
template <int H>
__device__ __forceinline__ void ws_hidden(const float* __restrict__ S, int nin, int col, int half, const float (&x)[4],
                                          ws_acc16 (&z1)[WsShape<H>::B], ws_acc16 (&z2)[WsShape<H>::B]) {
  using W = WsShape<H>;
  const float* W1 = S;
  const float* b1 = W1 + nin * H;
  const float* W2 = b1 + H;
  const float* b2 = W2 + H * H;
  ws_bias<H>(b1, half, z1);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int f = 2 * q + half;
#pragma unroll
    for (int b = 0; b < W::B; ++b) {
      const int o = 32 * b + ws_unit_of(col);
      const float w = (f < nin && (H >= 32 || o < H)) ? W1[f * H + o] : 0.f;
      z1[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(w, x[q], z1[b], 0, 0, 0);
    }
  }
  ws_bias<H>(b2, half, z2);
#pragma unroll
  for (int ib = 0; ib < W::B; ++ib)
#pragma unroll
    for (int st = 0; st < W::KS; ++st) {
      const float a = fmaxf(z1[ib][st], 0.f);
      const int i = 32 * ib + ws_unit(st, half);
#pragma unroll
      for (int ob = 0; ob < W::B; ++ob) {
        const int o = 32 * ob + ws_unit_of(col);
        const float w = (H >= 32 || o < H) ? W2[i * H + o] : 0.f;
        z2[ob] = __builtin_amdgcn_mfma_f32_32x32x2f32(w, a, z2[ob], 0, 0, 0);
      }
    }
}

// Output of the tile's columns, units in order (both halves of the wave get it).
template <int H>
__device__ __forceinline__ float ws_output(const float* __restrict__ S, int nin,
                                           const ws_acc16 (&z2)[WsShape<H>::B]) {
  const float* W3 = S + nin * H + H + H * H + H;
  float y = W3[H];
#pragma unroll
  for (int b = 0; b < WsShape<H>::B; ++b)
#pragma unroll
    for (int r = 0; r < WsShape<H>::KS; ++r) {
      // swapping a register with itself leaves the lower half's value in both halves, and the upper's
      const unsigned a = __float_as_uint(fmaxf(z2[b][r], 0.f));
      const auto both = __builtin_amdgcn_permlane32_swap(a, a, false, false);
      y = fmaf(__uint_as_float(both[0]), W3[32 * b + 2 * r], y);
      y = fmaf(__uint_as_float(both[1]), W3[32 * b + 2 * r + 1], y);
    }
  return y;
}

// Bound by the matrix cores (n = 1e6, h = 32: 20 instructions of 64 cycles per 32
// vertices, 16 us of them): 313 us on the vector ALUs, 39 us (67 TFLOP/s) now.
template <int H>
__global__ void __launch_bounds__(kBlock)
k_ws_forward(const float* __restrict__ P, int nin, const float* __restrict__ mu, const float* __restrict__ isd,
             long n, const float* __restrict__ X, double* __restrict__ out) {
  using W = WsShape<H>;
  __shared__ float S[kWsFeat * H + H + H * H + H + H + 1];
  ws_load_params(P, S, ws_nparams(nin, H));
  const int lane = threadIdx.x % kWave, half = lane / 32, col = lane % 32;
  float m[4], d[4];
  ws_scaling(mu, isd, nin, half, m, d);
  const long nw = (long)gridDim.x * (kBlock / kWave);
  for (long t = (long)blockIdx.x * (kBlock / kWave) + threadIdx.x / kWave; t * 32 < n; t += nw) {
    const long v = t * 32 + col;
    const bool in = v < n;
    float x[4];
    ws_inputs(X, v, in, nin, half, m, d, x);
    ws_acc16 z1[W::B], z2[W::B];
    ws_hidden<H>(S, nin, col, half, x, z1, z2);
    const float y = ws_output<H>(S, nin, z2);
    if (in && half == 0) out[v] = (double)y;
  }
}

// Column means of an n x 8 feature array (fixed-order two-level reduction over at
// most 64 blocks, what the caller's workspace holds).  A thread reads one half
// of a row at a time.
__global__ void __launch_bounds__(kFin)
k_ws_pool(const float* __restrict__ F, long n, double* __restrict__ part) {
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  const long chunk = (n + gridDim.x - 1) / gridDim.x;
  const long lo = (long)blockIdx.x * chunk;
  const long hi = lo + chunk < n ? lo + chunk : n;
  constexpr int U = 4;
  for (long k = 2 * lo + threadIdx.x; k < 2 * hi; k += (long)kFin * U) {
    float f[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long kk = k + (long)u * kFin;
      f[u][0] = f[u][1] = f[u][2] = f[u][3] = 0.f;
      if (kk < 2 * hi) __builtin_memcpy(f[u], F + kk * 4, sizeof(f[u]));
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int q = 0; q < 4; ++q) acc[q] += (double)f[u][q];
  }
  __shared__ double red[kFin / kWave][kWsFeat];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  const double x = wave_sum_many<4, 2>(acc, lane);  // value lane / 16 over the lanes of one half (lane % 2)
  if (lane % 16 < 2) red[wave][4 * (lane % 2) + lane / 16] = x;
  __syncthreads();
  if (threadIdx.x < kWsFeat) {
    double t = 0.0;
    for (int w = 0; w < kFin / kWave; ++w) t += red[w][threadIdx.x];
    part[(long)blockIdx.x * kWsFeat + threadIdx.x] = t;
  }
}

__global__ void __launch_bounds__(kFin)
k_ws_pool_fin(const double* __restrict__ part, int nb, long n, double* __restrict__ out) {
  __shared__ double tot[kWsFeat];
  fin_rows<kWsFeat>(part, nb, tot);
  if (threadIdx.x < kWsFeat) out[threadIdx.x] = n > 0 ? tot[threadIdx.x] / (double)n : 0.0;
}

// Forward + backward of the mean squared error (1/n) sum_v (f(x_v) - t_v)^2.
// A block owns a contiguous range of vertices and walks it 128 rows at a time,
// each wave a tile of 32.  The deltas of the hidden layers are matrix products
// like the forward pass (the weights transposed as A operand); the weight
// gradients are products over the tile's vertices, whose operands have a lane
// per unit and come back from LDS transposed: dW2 = a1^T d2 and, with x
// extended by a column of ones, dW1 and db1 = [x 1]^T d1 (16 x 16 x 4 tiles).
// The waves' gradients are added in wave order, the blocks' later in block
// order, so the gradient is deterministic.  Bound by the matrix cores and LDS;
// 262 144 rows, h = 32: 260 us on the vector ALUs, 43 us (48 TFLOP/s) now.
template <int H>
__global__ void __launch_bounds__(kBlock)
k_ws_backward(const float* __restrict__ P, int nin, const float* __restrict__ mu, const float* __restrict__ isd, long n,
              const float* __restrict__ X, const float* __restrict__ T, float inv_n, float* __restrict__ gpart,
              double* __restrict__ lpart) {
  using W = WsShape<H>;
  constexpr int NW = kBlock / kWave;
  constexpr int LD = W::HP + 4;  // row stride of the transposed tiles
  constexpr int NPMAX = kWsFeat * H + H + H * H + H + H + 1;
  __shared__ float S[NPMAX];
  __shared__ float sA[NW][32][LD], sD[NW][32][LD];
  __shared__ float sX[NW][32][kWsFeat + 1];
  __shared__ double lred[NW];
  static_assert(NW * 32 * LD >= NPMAX, "the gradient is added up in sA");
  const int np = ws_nparams(nin, H);
  ws_load_params(P, S, np);
  const float* W2 = S + nin * H + H;
  const float* W3 = W2 + H * H + H;
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave, half = lane / 32, col = lane % 32;
  float m[4], d[4];
  ws_scaling(mu, isd, nin, half, m, d);
  ws_acc16 gW2[W::B][W::B];  // [block of i][block of o]
  ws_acc4 gW1[W::HP / 16];   // rows: features, then ones; 16 units each
  float gb2[W::B][16], gW3[W::B][16], gb3 = 0.f;
#pragma unroll
  for (int b = 0; b < W::B; ++b) {
#pragma unroll
    for (int c = 0; c < W::B; ++c)
#pragma unroll
      for (int r = 0; r < 16; ++r) gW2[b][c][r] = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) gb2[b][r] = gW3[b][r] = 0.f;
  }
#pragma unroll
  for (int b = 0; b < W::HP / 16; ++b)
#pragma unroll
    for (int r = 0; r < 4; ++r) gW1[b][r] = 0.f;
  const long chunk = (n + gridDim.x - 1) / gridDim.x;
  const long lo = (long)blockIdx.x * chunk;
  const long hi = lo + chunk < n ? lo + chunk : n;
  double loss = 0.0;
  for (long base = lo; base < hi; base += 32 * NW) {
    const long v = base + 32 * wave + col;
    const bool in = v < hi;
    float x[4];
    ws_inputs(X, v, in, nin, half, m, d, x);
    const float target = in ? T[v] : 0.f;
    ws_acc16 z1[W::B], z2[W::B], d1[W::B];
    ws_hidden<H>(S, nin, col, half, x, z1, z2);
    const float e = in ? ws_output<H>(S, nin, z2) - target : 0.f;
    const float dout = 2.f * e * inv_n;
    if (half == 0) {
      loss += (double)e * (double)e;
      gb3 += dout;
    }
    // d2 in place of z2, dW3 and db2 on the way
#pragma unroll
    for (int b = 0; b < W::B; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int u = 32 * b + ws_unit(r, half);
        const float w3 = (H >= 32 || u < H) ? W3[u] : 0.f;
        const float z = z2[b][r];
        gW3[b][r] += fmaxf(z, 0.f) * dout;
        z2[b][r] = z > 0.f ? dout * w3 : 0.f;
        gb2[b][r] += z2[b][r];
        d1[b][r] = 0.f;
      }
    // d1 = relu'(z1) W2 d2
#pragma unroll
    for (int ob = 0; ob < W::B; ++ob)
#pragma unroll
      for (int st = 0; st < W::KS; ++st) {
        const int o = 32 * ob + ws_unit(st, half);
#pragma unroll
        for (int ib = 0; ib < W::B; ++ib) {
          const int i = 32 * ib + ws_unit_of(col);
          const float w = (H >= 32 || i < H) ? W2[i * H + o] : 0.f;
          d1[ib] = __builtin_amdgcn_mfma_f32_32x32x2f32(w, z2[ob][st], d1[ib], 0, 0, 0);
        }
      }
    // a1 and d2 to LDS, a vertex per row, units at their accumulator rows
#pragma unroll
    for (int b = 0; b < W::B; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int c = 32 * b + ws_row(r, half);
        sA[wave][col][c] = fmaxf(z1[b][r], 0.f);
        sD[wave][col][c] = z2[b][r];
      }
#pragma unroll
    for (int q = 0; q < 4; ++q) sX[wave][col][2 * q + half] = x[q];
    if (half == 0) sX[wave][col][kWsFeat] = 1.f;
    __syncthreads();
#pragma unroll
    for (int st = 0; st < 16; ++st) {
      const int row = 2 * st + half;
      float a[W::B], g[W::B];
#pragma unroll
      for (int b = 0; b < W::B; ++b) {
        a[b] = sA[wave][row][32 * b + col];
        g[b] = sD[wave][row][32 * b + col];
      }
#pragma unroll
      for (int ib = 0; ib < W::B; ++ib)
#pragma unroll
        for (int ob = 0; ob < W::B; ++ob)
          gW2[ib][ob] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[ib], g[ob], gW2[ib][ob], 0, 0, 0);
    }
    __syncthreads();
    // d1 in place of a1
#pragma unroll
    for (int b = 0; b < W::B; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) sA[wave][col][32 * b + ws_row(r, half)] = z1[b][r] > 0.f ? d1[b][r] : 0.f;
    __syncthreads();
#pragma unroll
    for (int st = 0; st < 8; ++st) {
      const int row = 4 * st + lane / 16, f = lane % 16;
      const float a = f <= kWsFeat ? sX[wave][row][f] : 0.f;
#pragma unroll
      for (int b = 0; b < W::HP / 16; ++b)
        gW1[b] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, sA[wave][row][16 * b + f], gW1[b], 0, 0, 0);
    }
    __syncthreads();
  }
  // the waves' gradients, added in wave order into G (LDS)
  float* G = &sA[0][0][0];
  const int ob1 = nin * H, oW2 = ob1 + H, ob2 = oW2 + H * H, oW3 = ob2 + H, ob3 = oW3 + H;
  __syncthreads();
  for (int k = threadIdx.x; k < np; k += kBlock) G[k] = 0.f;
  float sb2[W::B], sW3[W::B];  // unit ws_unit((lane % 32) / 2, half) of each block
#pragma unroll
  for (int b = 0; b < W::B; ++b) {
    sb2[b] = wave_sum_many<16, 1, 16>(gb2[b], lane);
    sW3[b] = wave_sum_many<16, 1, 16>(gW3[b], lane);
  }
  gb3 = wave_sum(gb3);
  for (int w = 0; w < NW; ++w) {
    __syncthreads();
    if (wave != w) continue;
#pragma unroll
    for (int ib = 0; ib < W::B; ++ib)
#pragma unroll
      for (int ob = 0; ob < W::B; ++ob)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int i = 32 * ib + ws_unit(r, half), o = 32 * ob + ws_unit_of(col);
          if (H >= 32 || (i < H && o < H)) G[oW2 + i * H + o] += gW2[ib][ob][r];
        }
#pragma unroll
    for (int b = 0; b < W::HP / 16; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int f = 4 * (lane / 16) + r, c = 16 * b + lane % 16;
        const int o = c / 32 * 32 + ws_unit_of(c % 32);
        if (o < H && f < nin) G[f * H + o] += gW1[b][r];
        if (o < H && f == kWsFeat) G[ob1 + o] += gW1[b][r];
      }
    if (lane % 2 == 0) {
#pragma unroll
      for (int b = 0; b < W::B; ++b) {
        const int u = 32 * b + ws_unit(col / 2, half);
        if (u < H) {
          G[ob2 + u] += sb2[b];
          G[oW3 + u] += sW3[b];
        }
      }
    }
    if (lane == 0) G[ob3] += gb3;
  }
  __syncthreads();
  for (int k = threadIdx.x; k < np; k += kBlock) gpart[(long)blockIdx.x * np + k] = G[k];
  loss = wave_sum(loss);
  if (lane == 0) lred[wave] = loss;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < NW; ++w) t += lred[w];
    lpart[blockIdx.x] = t;
  }
}

// grad[k] = sum over blocks of gpart[b][k]; loss = (1/n) sum of the per-block
// squared errors.  A block takes 32 parameters, thread (row group, parameter)
// the rows of its group (kFin / 32 groups) in FP64, four in flight, and the
// groups are added in order.
// One thread per parameter walking all 512 rows took 146 us, this 8 us.
constexpr int kWsRedK = 32;
__global__ void __launch_bounds__(kFin)
k_ws_reduce(const float* __restrict__ gpart, const double* __restrict__ lpart, int nb, int np, double inv_n,
            float* __restrict__ grad, double* __restrict__ loss_out) {
  constexpr int NG = kFin / kWsRedK, U = 4;
  __shared__ double buf[NG][kWsRedK];
  __shared__ double tot;
  const int kk = threadIdx.x % kWsRedK, g = threadIdx.x / kWsRedK;
  const int k = blockIdx.x * kWsRedK + kk;
  double a = 0.0;
  for (int b = g; b < nb; b += NG * U) {
    float v[U];
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = (k < np && b + u * NG < nb) ? gpart[(long)(b + u * NG) * np + k] : 0.f;
#pragma unroll
    for (int u = 0; u < U; ++u) a += (double)v[u];
  }
  buf[g][kk] = a;
  __syncthreads();
  if (g == 0 && k < np) {
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < NG; ++q) t += buf[q][kk];
    grad[k] = (float)t;
  }
  if (blockIdx.x == 0 && loss_out) {
    fin_rows<1>(lpart, nb, &tot);
    if (threadIdx.x == 0) *loss_out = tot * inv_n;
  }
}

// Adam (Kingma & Ba, 2015), bias-corrected.
__global__ void __launch_bounds__(kBlock)
k_ws_adam(float* __restrict__ P, const float* __restrict__ g, float* __restrict__ m, float* __restrict__ v, int np,
          float lr, float b1, float b2, float eps, float c1, float c2) {
  const int k = blockIdx.x * kBlock + threadIdx.x;
  if (k >= np) return;
  const float gk = g[k];
  const float mk = b1 * m[k] + (1.f - b1) * gk;
  const float vk = b2 * v[k] + (1.f - b2) * gk * gk;
  m[k] = mk;
  v[k] = vk;
  P[k] -= lr * (mk / c1) / (sqrtf(vk / c2) + eps);
}

// ---- launchers -------------------------------------------------------------------

void launch_ws_features(const Cost<double>& C, float* F, float2* pair, hipStream_t st) {
  const int nb = (int)((C.n * kWsLpr + kBlock - 1) / kBlock);
  hipLaunchKernelGGL(k_ws_feat1, dim3(nb), dim3(kBlock), 0, st, C, pair);
  hipLaunchKernelGGL(k_ws_feat2, dim3(nb), dim3(kBlock), 0, st, C, pair, F);
}

int ws_param_count(int nin, int h) { return nin * h + h + h * h + h + h + 1; }

bool launch_ws_forward(const float* P, int nin, int h, const float* mu, const float* isd, long n, const float* X,
                       double* out, hipStream_t st) {
  long nb = (n + 32 * (kBlock / kWave) - 1) / (32 * (kBlock / kWave));
  if (nb > 1024) nb = 1024;
  if (nb < 1) nb = 1;
  if (h == 16) hipLaunchKernelGGL(k_ws_forward<16>, dim3(nb), dim3(kBlock), 0, st, P, nin, mu, isd, n, X, out);
  else if (h == 32) hipLaunchKernelGGL(k_ws_forward<32>, dim3(nb), dim3(kBlock), 0, st, P, nin, mu, isd, n, X, out);
  else if (h == 64) hipLaunchKernelGGL(k_ws_forward<64>, dim3(nb), dim3(kBlock), 0, st, P, nin, mu, isd, n, X, out);
  else return false;
  return true;
}

void launch_ws_pool(const float* F, long n, double* part, int nb, double* out, hipStream_t st) {
  hipLaunchKernelGGL(k_ws_pool, dim3(nb), dim3(kFin), 0, st, F, n, part);
  hipLaunchKernelGGL(k_ws_pool_fin, dim3(1), dim3(kFin), 0, st, part, nb, n, out);
}

bool launch_ws_backward(const float* P, int nin, int h, const float* mu, const float* isd, long n, const float* X,
                        const float* T, float* gpart, double* lpart, int nb, float* grad, double* loss,
                        hipStream_t st) {
  const float inv_n = n > 0 ? 1.f / (float)n : 0.f;
  if (h == 16)
    hipLaunchKernelGGL(k_ws_backward<16>, dim3(nb), dim3(kBlock), 0, st, P, nin, mu, isd, n, X, T, inv_n, gpart,
                       lpart);
  else if (h == 32)
    hipLaunchKernelGGL(k_ws_backward<32>, dim3(nb), dim3(kBlock), 0, st, P, nin, mu, isd, n, X, T, inv_n, gpart,
                       lpart);
  else if (h == 64)
    hipLaunchKernelGGL(k_ws_backward<64>, dim3(nb), dim3(kBlock), 0, st, P, nin, mu, isd, n, X, T, inv_n, gpart,
                       lpart);
  else
    return false;
  const int np = ws_param_count(nin, h);
  hipLaunchKernelGGL(k_ws_reduce, dim3((np + kWsRedK - 1) / kWsRedK), dim3(kFin), 0, st, gpart, lpart, nb, np,
                     n > 0 ? 1.0 / (double)n : 0.0, grad, loss);
  return true;
}

void launch_ws_adam(float* P, const float* g, float* m, float* v, int np, float lr, float b1, float b2, float eps,
                    int step, hipStream_t st) {
  const float c1 = 1.f - powf(b1, (float)step), c2 = 1.f - powf(b2, (float)step);
  hipLaunchKernelGGL(k_ws_adam, dim3((np + kBlock - 1) / kBlock), dim3(kBlock), 0, st, P, g, m, v, np, lr, b1, b2,
                     eps, c1, c2);
}

}  // namespace almbm
