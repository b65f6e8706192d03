// Device-side helpers shared by the ALM-BM kernels (gfx950, wave64).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace almbm {

constexpr int kBlock = 256;          // threads per block for every row kernel
constexpr int kWave = 64;            // CDNA wavefront width
constexpr int kNumXcd = 8;           // MI355X: 8 XCDs, blocks dispatched round robin

// bfloat16 storage: 16 high bits of an IEEE binary32.
struct bf16 {
  uint16_t bits;
};

__device__ __forceinline__ float bf16_to_f32(uint16_t h) {
  return __uint_as_float(static_cast<uint32_t>(h) << 16);
}

// Round a binary32 to the nearest bfloat16, ties to even; NaN stays NaN.
__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u && (u & 0x007fffffu)) return static_cast<uint16_t>((u >> 16) | 0x40u);
  uint32_t lsb = (u >> 16) & 1u;
  u += 0x7fffu + lsb;
  return static_cast<uint16_t>(u >> 16);
}

// Storage type -> arithmetic type.
template <typename T> struct Acc { using type = float; };
template <> struct Acc<double> { using type = double; };

template <typename T> __device__ __forceinline__ typename Acc<T>::type to_acc(T v) { return v; }
template <> __device__ __forceinline__ float to_acc<bf16>(bf16 v) { return bf16_to_f32(v.bits); }

template <typename T> __device__ __forceinline__ T from_acc(typename Acc<T>::type v) { return v; }
template <> __device__ __forceinline__ bf16 from_acc<bf16>(float v) { return bf16{f32_to_bf16(v)}; }

// Value rounded to storage precision and back (what a store then load would give).
template <typename T> __device__ __forceinline__ typename Acc<T>::type round_st(typename Acc<T>::type v) {
  return to_acc<T>(from_acc<T>(v));
}

// ---- row fragments: LPR lanes hold one row of r <= LPR*VEC elements ----------
//
// Lane l of a row group owns columns [l*VEC, l*VEC+VEC).  FULL means
// r == LPR*VEC, so a lane's slice is contiguous and aligned to VEC*sizeof(T)
// bytes and is moved with one vector access.

template <int BYTES> struct VecWord;
template <> struct VecWord<2> { using type = uint16_t; };
template <> struct VecWord<4> { using type = uint32_t; };
template <> struct VecWord<8> { using type = uint2; };
template <> struct VecWord<16> { using type = uint4; };
template <> struct VecWord<32> { struct type { uint4 a, b; }; };
template <> struct VecWord<64> { struct type { uint4 a, b, c, d; }; };

// The first m (any int) of N elements at p, aligned to one element only, with
// the widest accesses that fit: all N at once when m >= N, else the two halves.
// Global accesses need no more than that alignment here; the copies leave the
// choice of instruction to the compiler.
template <typename T, int N>
__device__ __forceinline__ void load_some(const T* __restrict__ p, int m, typename Acc<T>::type* out) {
  if (m >= N) {
    T e[N];
    __builtin_memcpy(e, p, N * sizeof(T));
#pragma unroll
    for (int v = 0; v < N; ++v) out[v] = to_acc<T>(e[v]);
  } else if constexpr (N > 1) {
    load_some<T, N / 2>(p, m, out);
    load_some<T, N / 2>(p + N / 2, m - N / 2, out + N / 2);
  } else {
    out[0] = typename Acc<T>::type(0);
  }
}
template <typename T, int N>
__device__ __forceinline__ void store_some(T* __restrict__ p, int m, const typename Acc<T>::type* in) {
  if (m >= N) {
    T e[N];
#pragma unroll
    for (int v = 0; v < N; ++v) e[v] = from_acc<T>(in[v]);
    __builtin_memcpy(p, e, N * sizeof(T));
  } else if constexpr (N > 1) {
    store_some<T, N / 2>(p, m, in);
    store_some<T, N / 2>(p + N / 2, m - N / 2, in + N / 2);
  }
}

template <typename T, int VEC, bool FULL>
__device__ __forceinline__ void load_frag(const T* __restrict__ row, int lane, int r,
                                          typename Acc<T>::type (&out)[VEC]) {
  if constexpr (FULL) {
    using W = typename VecWord<VEC * sizeof(T)>::type;
    W w = *reinterpret_cast<const W*>(row + lane * VEC);
    const T* e = reinterpret_cast<const T*>(&w);
#pragma unroll
    for (int v = 0; v < VEC; ++v) out[v] = to_acc<T>(e[v]);
  } else {
    load_some<T, VEC>(row + lane * VEC, r - lane * VEC, out);
  }
}

template <typename T, int VEC, bool FULL>
__device__ __forceinline__ void store_frag(T* __restrict__ row, int lane, int r,
                                           const typename Acc<T>::type (&in)[VEC]) {
  if constexpr (FULL) {
    using W = typename VecWord<VEC * sizeof(T)>::type;
    W w;
    T* e = reinterpret_cast<T*>(&w);
#pragma unroll
    for (int v = 0; v < VEC; ++v) e[v] = from_acc<T>(in[v]);
    *reinterpret_cast<W*>(row + lane * VEC) = w;
  } else {
    store_some<T, VEC>(row + lane * VEC, r - lane * VEC, in);
  }
}

// Sum over the LPR lanes of a row group (all lanes of the group get the sum).
template <int LPR, typename V>
__device__ __forceinline__ V group_sum(V x) {
#pragma unroll
  for (int o = LPR / 2; o > 0; o >>= 1) x += __shfl_xor(x, o, LPR);
  return x;
}

template <typename V>
__device__ __forceinline__ V wave_sum(V x) {
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) x += __shfl_xor(x, o, kWave);
  return x;
}

// Deterministic block sum of NS doubles per thread; result written by thread 0
// to out[0..NS).  Fixed order: lanes by butterfly, then waves in index order.
template <int NS>
__device__ __forceinline__ void block_sum_store(double (&acc)[NS], double* __restrict__ out) {
  __shared__ double red[kBlock / kWave][NS];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    double v = wave_sum(acc[s]);
    if (lane == 0) red[wave][s] = v;
  }
  __syncthreads();
  if (threadIdx.x < NS) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kBlock / kWave; ++w) t += red[w][threadIdx.x];
    out[threadIdx.x] = t;
  }
}

// Sums of P (a power of two) values per lane over the lanes of a wave that
// agree in l % LOW, by halving: in each step a lane keeps one half of its values
// and adds the partner's copy of that half, so that P + log2(64 / LOW) - log2 P
// shuffles do the work of P log2(64 / LOW).  Needs P <= 64 / LOW.  Lane l ends
// with the total of value l / (64 / P).
template <int P, int LOW = 1, int BIT = kWave / 2, typename V>
__device__ __forceinline__ V wave_sum_many(const V (&v)[P], int lane) {
  if constexpr (P == 1) {
    V x = v[0];
#pragma unroll
    for (int o = BIT; o >= LOW; o >>= 1) x += __shfl_xor(x, o, kWave);
    return x;
  } else {
    static_assert(BIT >= LOW, "more values than lanes to spread them over");
    V w[P / 2];
    const bool up = (lane & BIT) != 0;
#pragma unroll
    for (int k = 0; k < P / 2; ++k) {
      const V keep = up ? v[k + P / 2] : v[k];
      const V send = up ? v[k] : v[k + P / 2];
      w[k] = keep + __shfl_xor(send, BIT, kWave);
    }
    return wave_sum_many<P / 2, LOW, BIT / 2>(w, lane);
  }
}
constexpr int pow2_at_least(int x) {
  int p = 1;
  while (p < x) p *= 2;
  return p;
}

// Deterministic block sum of NS <= 64 doubles per thread into out[0..NS) (the
// many-slot counterpart of block_sum_store).
template <int NS>
__device__ __forceinline__ void block_sum_many(const double (&acc)[NS], double* __restrict__ out) {
  constexpr int P = pow2_at_least(NS);
  __shared__ double red[kBlock / kWave][P];
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  double v[P];
#pragma unroll
  for (int s = 0; s < P; ++s) v[s] = s < NS ? acc[s] : 0.0;
  const double x = wave_sum_many<P>(v, lane);
  if (lane % (kWave / P) == 0) red[wave][lane / (kWave / P)] = x;
  __syncthreads();
  if (threadIdx.x < NS) {
    double t = 0.0;
#pragma unroll
    for (int w = 0; w < kBlock / kWave; ++w) t += red[w][threadIdx.x];
    out[threadIdx.x] = t;
  }
}

// Totals of a table of per-block partial sums, by one block of kFin threads:
// out[s] (shared, ns <= kFin doubles) = sum over the rows of part[row * ns + s].  The
// table is read as one flat array, thread t taking elements t, t + A, ... with
// A the largest multiple of ns up to kFin, so that loads are coalesced and a
// thread stays on one column; kFinUnroll of them are in flight per thread.  A
// wave then adds each column's A / ns threads.  Fixed order, independent of
// timing, and the same for any THREADS, the threads of the block that runs it (fewer
// take several of the kFin threads' shares).  Bound by the latency of one CU's loads: 4096 x 15 doubles took 18 us
// with 256 threads walking rows (15 strided loads a row, 15 block reductions by
// shuffles) and take 11 us this way.  Every thread of the block must call it.
constexpr int kFin = 1024;
constexpr int kFinUnroll = 16;
template <int THREADS = kFin>
__device__ __forceinline__ void fin_table(const double* __restrict__ part, int rows, int ns, double* __restrict__ out) {
  const int A = kFin / ns * ns;
  __shared__ double buf[kFin];
  const long len = (long)rows * ns;
  for (int t = threadIdx.x; t < A; t += THREADS) {
    double a = 0.0;
    for (long k = t; k < len; k += (long)kFinUnroll * A) {
      double v[kFinUnroll];
#pragma unroll
      for (int u = 0; u < kFinUnroll; ++u) v[u] = k + (long)u * A < len ? part[k + (long)u * A] : 0.0;
#pragma unroll
      for (int o = kFinUnroll / 2; o > 0; o >>= 1)
#pragma unroll
        for (int u = 0; u < o; ++u) v[u] += v[u + o];
      a += v[0];
    }
    buf[t] = a;
  }
  __syncthreads();
  const int lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
  for (int s = wave; s < ns; s += THREADS / kWave) {
    double a = 0.0;
    for (int g = lane; g < A / ns; g += kWave) a += buf[g * ns + s];
    a = wave_sum(a);
    if (lane == 0) out[s] = a;
  }
  __syncthreads();
}
template <int NS, int THREADS = kFin>
__device__ __forceinline__ void fin_rows(const double* __restrict__ part, int rows, double* __restrict__ out) {
  fin_table<THREADS>(part, rows, NS, out);
}

// Rows owned by this block: the row range is split into gridDim.x contiguous
// chunks and blocks are renumbered so that the blocks the hardware sends to one
// XCD (blockIdx % 8 equal) own one contiguous eighth of the rows; neighbour rows
// of banded or mesh-like patterns then stay in that XCD's L2.  With spread the
// blocks keep their order, so that consecutive chunks go to different XCDs:
// where the row lengths are skewed, the long rows often sit together.
struct RowChunk {
  long lo, hi;
};
__device__ __forceinline__ RowChunk row_chunk(long n, bool spread = false, int blocks = 0) {
  const long nb = blocks ? blocks : gridDim.x;  // the first `blocks` of the grid
  long vb = blockIdx.x;
  if (nb % kNumXcd == 0 && !spread) {
    const long per = nb / kNumXcd;
    vb = (blockIdx.x % kNumXcd) * per + blockIdx.x / kNumXcd;
  }
  const long chunk = (n + nb - 1) / nb;
  long lo = vb * chunk;
  long hi = lo + chunk;
  if (lo > n) lo = n;
  if (hi > n) hi = n;
  return {lo, hi};
}

// Counter-based uniform in [-1, 1) from (seed, index): the SplitMix64 output
// function (Steele, Lea, Flood, "Fast splittable pseudorandom number
// generators", OOPSLA 2014) applied to seed * golden + index.
__device__ __forceinline__ double counter_uniform(uint64_t seed, uint64_t idx) {
  uint64_t z = seed * 0x9e3779b97f4a7c15ull + (idx + 1) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  z = z ^ (z >> 31);
  return static_cast<double>(z >> 11) * (2.0 / 9007199254740992.0) - 1.0;
}

}  // namespace almbm
