// Kernels of the graph preprocessing of Graph-SNMPBB (Section 2.2): K nearest neighbours
// by brute force, the union-symmetrised neighbour pattern as CSR, the Gaussian (or
// unweighted) similarity values and the normalised Laplacian I - D^{-1/2} V D^{-1/2} of
// eq. (2.3).  Distances and degrees are formed in FP64, so the integer decisions (which
// points are neighbours) are taken in the precision of the FP64 reference.
#include "common.hpp"
#include "kernels.hpp"

namespace snmf {

// ----------------------------------------------------------------------------- kNN
// The K smallest (distance, index) pairs of every point, distances the FP64 sums of squared
// differences in coordinate order.  A workgroup takes 16 query points; its four wavefronts
// share the candidates (16-point tiles w, w + 4, ... counted from the queries' own tile, so
// that points stored near each other meet first).
//
// Screening: the FP64 matrix cores (16x16x4) form s_ij = |x_j|^2 - 2 <x_i, x_j> of a tile, and
// a pair goes on when s_ij <= T_i - |x_i|^2 + err, T_i being the exact K-th distance found
// for query i so far by any of the four wavefronts.  The roundings of |x_i|^2,
// |x_j|^2 and s_ij come to at most 2 dim 2^-53 |x_i|^2 + 3 dim 2^-53 |x_j|^2, err is
// 4 (dim + 4) 2^-53 of the two, so no pair whose computed distance is below or equal to T_i is left out: the result is
// that of the exhaustive search, bit for bit, whatever the data (norms near the overflow
// are held as -inf, which passes with every partner; 1e-290 covers what underflows).
// First limit: every fourth tile is formed once before, each lane keeping the minimum of
// its s_ij per query: 64 (K > 16: 128) minima over disjoint candidates, whose K-th smallest
// (rounded up) bounds the K-th distance.  Some 4 K pairs per query pass it later; without
// it every tile had pairs to queue while the lists grew.
// Selection: pairs that pass are queued per query in LDS; a queue of more than 48 is
// emptied by the wavefront: one pair per lane, its exact distance, and, if any comes before
// the list's K-th pair, a bitonic sort and a bitonic merge with the query's sorted list
// (ties to the lower index at every step).
// At n = 20000, dim = 16, K = 10 the products take 163 + 41 us at the FP64 matrix rate;
// 473 us in all, 879 us without the first limit (one wavefront per query with every
// distance formed from per-lane rows of X: 1953 us, bound by the uncoalesced loads).
typedef double kd4 __attribute__((ext_vector_type(4)));
constexpr int kKnnQueue = 64;  // queued pairs per query and wavefront: one per lane

__host__ __device__ constexpr size_t knn_lds_wave(int kb) {  // bytes of LDS per wavefront
  return (size_t)16 * kb * 12 + 16 * kKnnQueue * 4;
}

__device__ __forceinline__ bool knn_less(double d, int32_t i, double e, int32_t j) {
  return (d < e) | ((d == e) & (i < j));
}
// LDS that one lane writes and another lane of the same wavefront reads: in order in the
// hardware, and kept so by the compiler.
__device__ __forceinline__ void knn_order() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}
// The value of lane ^ M: cross-lane moves inside a row of 16, LDS permutes across rows.
template <int M>
__device__ __forceinline__ int knn_xor(int v) {
  if constexpr (M == 1)
    return __builtin_amdgcn_update_dpp(v, v, 0xB1, 0xf, 0xf, true);  // quad_perm 1 0 3 2
  else if constexpr (M == 2)
    return __builtin_amdgcn_update_dpp(v, v, 0x4E, 0xf, 0xf, true);  // quad_perm 2 3 0 1
  else if constexpr (M == 4) {
    const int u = __builtin_amdgcn_update_dpp(v, v, 0x1B, 0xf, 0xf, true);  // lane ^ 3
    return __builtin_amdgcn_update_dpp(u, u, 0x141, 0xf, 0xf, true);        // lane ^ 7
  } else if constexpr (M == 8)
    return __builtin_amdgcn_update_dpp(v, v, 0x128, 0xf, 0xf, true);  // row_ror 8
  else
    return __shfl_xor(v, M);
}
// One compare-exchange with the lane M away; the lower (up) or higher pair stays.
template <int M>
__device__ __forceinline__ void knn_swap(double& d, int32_t& i, bool up) {
  const long long b = __double_as_longlong(d);
  const int lo = knn_xor<M>((int)b), hi = knn_xor<M>((int)(b >> 32));
  const double e = __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
  const int32_t j = knn_xor<M>(i);
  if (knn_less(e, j, d, i) == up) {
    d = e;
    i = j;
  }
}
// The steps M, M / 2, ... 1 of a merge into runs of K, alternately increasing and decreasing
// (K = 64: one increasing run).
template <int K, int M>
__device__ __forceinline__ void knn_steps(double& d, int32_t& i) {
  knn_swap<M>(d, i, ((threadIdx.x & M) == 0) == ((threadIdx.x & 63 & K) == 0));
  if constexpr (M > 1) knn_steps<K, M / 2>(d, i);
}
// Lanes hold a bitonic sequence of 64 pairs; on return it is increasing.
__device__ __forceinline__ void knn_merge64(double& d, int32_t& i) {
  knn_steps<64, 32>(d, i);
}
// N = 16: the first 16 lanes are sorted, the others hold nothing (infinity).  Lanes 0-15 of
// the step K = 16 lie in an increasing run.
template <int N>
__device__ __forceinline__ void knn_sort(double& d, int32_t& i) {
  knn_steps<2, 1>(d, i);
  knn_steps<4, 2>(d, i);
  knn_steps<8, 4>(d, i);
  knn_steps<16, 8>(d, i);
  if constexpr (N == 64) {
    knn_steps<32, 16>(d, i);
    knn_steps<64, 32>(d, i);
  }
}

// KS MFMA k-steps cover the coordinates.  FULL (dim = 4 KS, a multiple of 16): coordinate
// 16 b + 4 g + s in step 4 b + s of lane group g, four consecutive ones per load; else 4 s + g.
template <bool FULL>
__device__ __forceinline__ constexpr int knn_coord(int step, int g) {
  return FULL ? 16 * (step >> 2) + 4 * g + (step & 3) : 4 * step + g;
}

template <typename T, int KS, bool FULL>
__global__ __launch_bounds__(kThreads, KS <= 4 ? 5 : KS == 8 && !FULL ? 4 : 1) void k_knn(const T* __restrict__ X, int64_t n, int dim,
                                                  int K, int kb, const double* __restrict__ nrm,
                                                  int32_t* __restrict__ nbr) {
  extern __shared__ __attribute__((aligned(16))) unsigned char knn_lds[];
  __shared__ unsigned long long sT[16];  // bits of the exact K-th distances (nonnegative)
  __shared__ double sN[16];                         // the queries' norms, rounded down
  __shared__ int sC[4][16];                         // queue lengths, 65 and more: a list too
  const int lane = threadIdx.x & 63, c16 = lane & 15, g = lane >> 4;
  const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  unsigned char* const base = knn_lds + (size_t)wv * knn_lds_wave(kb);
  double* const ld = (double*)base;                 // 16 lists of kb distances, increasing
  int32_t* const li = (int32_t*)(ld + 16 * kb);     // and their points
  int32_t* const qu = li + 16 * kb;                 // 16 queues
  const int64_t q0 = (int64_t)blockIdx.x * 16;
  const double inf = __builtin_inf();
  const double c1 = 4.0 * (dim + 4) * 0x1p-53, up = 1.0 + 0x1p-46;
  // queries: MFMA operand A[m = lane % 16][k], times -2
  double qa[KS];
  {
    const int64_t i = q0 + c16 < n ? q0 + c16 : n - 1;
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const int c = knn_coord<FULL>(s, g);
      qa[s] = c < dim ? -2.0 * (double)X[i * dim + c] : 0.0;
    }
  }
  double thr[4] = {inf, inf, inf, inf};
  auto limits = [&]() {
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const double t = __longlong_as_double(
          (long long)*(volatile unsigned long long*)&sT[g + 4 * v]);
      thr[v] = t * up - sN[g + 4 * v] + 1e-290;
    }
  };
  auto distance = [&](int64_t i, int64_t j) __attribute__((always_inline)) {
    const T* __restrict__ xi = X + i * dim;
    const T* __restrict__ xj = X + j * dim;
    double d = 0.0;
    if constexpr (FULL) {
      for (int k = 0; k < dim; k += 16) {
        T a[16], b[16];
        __builtin_memcpy(a, xi + k, sizeof(a));
        __builtin_memcpy(b, xj + k, sizeof(b));
#pragma unroll
        for (int q = 0; q < 16; ++q) {
          const double t = (double)a[q] - (double)b[q];
          d = __builtin_fma(t, t, d);
        }
      }
      return d;
    }
#pragma unroll 4
    for (int k = 0; k < dim; ++k) {
      const double t = (double)xi[k] - (double)xj[k];
      d = __builtin_fma(t, t, d);
    }
    return d;
  };
  // empties the queue of query m, c pairs, into its list
  auto flush = [&](int m, int c) __attribute__((always_inline)) {
    knn_order();
    const int64_t i = q0 + m;
    const double kd = ld[m * kb + K - 1];
    const int32_t ki = li[m * kb + K - 1];
    double d = inf;
    int32_t j = 0x7fffffff;
    if (lane < c) {
      j = qu[m * kKnnQueue + lane];
      d = distance(i, j);
      if (!knn_less(d, j, kd, ki)) {  // (an infinite distance comes before an empty place)
        d = inf;
        j = 0x7fffffff;
      }
    }
    if (!__any(j != 0x7fffffff)) return;
    if (c <= 16)
      knn_sort<16>(d, j);
    else
      knn_sort<64>(d, j);
    // the lowest 64 of two increasing sequences: elementwise minimum of one and the other
    // reversed, a bitonic sequence
    const int rv = 63 - lane;
    const double e = rv < kb ? ld[m * kb + rv] : inf;
    const int32_t f = rv < kb ? li[m * kb + rv] : 0x7fffffff;
    if (knn_less(e, f, d, j)) {
      d = e;
      j = f;
    }
    knn_merge64(d, j);
    knn_order();
    if (lane < kb) {
      ld[m * kb + lane] = d;
      li[m * kb + lane] = j;
    }
    if (lane == K - 1) atomicMin(&sT[m], (unsigned long long)__double_as_longlong(d));
  };
  const int64_t nt = (n + 15) / 16, own = blockIdx.x;
  // candidates: operand B[k][lane % 16] and |x_j|^2 of a tile, the next tile's in flight
  T xb[KS], xn[KS];
  double nc, nn;
  const int cl = nt * 16 == n ? c16 : c16 < (int)(n - (nt - 1) * 16) ? c16 : 0;  // last tile
  const int o_all = FULL ? c16 * dim + 4 * g : c16 * dim;
  const int o_last = FULL ? cl * dim + 4 * g : cl * dim;
  // tile is alike over the wavefront
  auto load = [&](T (&x)[KS], double& nrmj, int64_t tile) __attribute__((always_inline)) {
    const T* __restrict__ xj = X + tile * 16 * dim;
    const int o = tile == nt - 1 ? o_last : o_all;
    if constexpr (FULL) {
#pragma unroll
      for (int b = 0; b < KS / 4; ++b) {
        T t[4];
        __builtin_memcpy(t, xj + o + 16 * b, 4 * sizeof(T));
#pragma unroll
        for (int s = 0; s < 4; ++s) x[4 * b + s] = t[s];
      }
    } else {
#pragma unroll
      for (int s = 0; s < KS; ++s) {  // past dim: a valid coordinate against a zero of A
        const int c = knn_coord<FULL>(s, g);
        x[s] = xj[o + (c < dim ? c : 0)];
      }
    }
    nrmj = nrm[tile * 16 + (tile == nt - 1 ? cl : c16)];
  };
  auto tile_of = [&](int64_t s) {
    const int64_t t = own + wv + 4 * s;
    return t < nt ? t : t - nt;
  };
  const int64_t ns = (nt - wv + 3) / 4;  // tiles of this wavefront (own + wv + 4 s < 2 nt)
  // the first limit: tiles s = 1, 5, 9, ... (not the queries' own), whole ones only
  {
    double mn[2][4];
#pragma unroll
    for (int v = 0; v < 4; ++v) mn[0][v] = mn[1][v] = inf;
    if (ns > 1) load(xb, nc, tile_of(1));
    int set = 0;
    for (int64_t s = 1; s < ns; s += 4) {
      load(xn, nn, tile_of(s + 4 < ns ? s + 4 : s));
      const double n0 = nc < 0.0 || (tile_of(s) + 1) * 16 > n ? inf : nc * (1.0 + c1);
      kd4 acc = {n0, n0, n0, n0};
#pragma unroll
      for (int k = 0; k < KS; ++k)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[k], (double)xb[k], acc, 0, 0, 0);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        mn[0][v] = __builtin_fmin(mn[0][v], set ? inf : acc[v]);
        mn[1][v] = __builtin_fmin(mn[1][v], set ? acc[v] : inf);
      }
      set ^= 1;
#pragma unroll
      for (int k = 0; k < KS; ++k) xb[k] = xn[k];
      nc = nn;
    }
    // per query 16 (two sets: 32) minima of every wavefront, in the space of the lists
    const bool two = kb > 16;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      double* const at = ld + (g + 4 * v) * kb + c16;
      at[0] = two ? mn[0][v] : __builtin_fmin(mn[0][v], mn[1][v]);
      if (two) at[16] = mn[1][v];
    }
    __syncthreads();
    for (int m = wv; m < 16; m += 4) {
      const double* const src = (const double*)(knn_lds + (size_t)g * knn_lds_wave(kb)) + m * kb;
      double d = src[c16];
      int32_t at = lane;
      knn_sort<64>(d, at);
      if (two) {
        double e = src[16 + c16];
        int32_t f = lane;
        knn_sort<64>(e, f);
        e = __shfl(e, 63 - lane);
        d = __builtin_fmin(d, e);
        knn_merge64(d, at);
      }
      if (lane == K - 1) {
        const double nm = nrm[q0 + m < n ? q0 + m : n - 1];
        const double t = nm < 0.0 ? inf : (d + nm * (1.0 + c1)) * up + 1e-290;
        sT[m] = (unsigned long long)__double_as_longlong(t > 0.0 ? t : 0.0);
        sN[m] = nm * (1.0 - c1);
      }
    }
    __syncthreads();
  }
  for (int e = lane; e < 16 * kb; e += kWave) {
    ld[e] = inf;
    li[e] = 0x7fffffff;
  }
  knn_order();
  int cnt[4] = {0, 0, 0, 0};  // queue lengths of queries g + 4 v, alike over a lane group
  unsigned listed = 0;          // queries with a list
  auto queued = [&](int m) {
    const int mine = m < 4 ? cnt[0] : m < 8 ? cnt[1] : m < 12 ? cnt[2] : cnt[3];
    return __builtin_amdgcn_readlane(mine, 16 * (m & 3));
  };
  auto visit = [&](const T (&x)[KS], double nrmj, int64_t tile) __attribute__((always_inline)) {
    const double n0 = nrmj * (1.0 - c1);
    kd4 acc = {n0, n0, n0, n0};
#pragma unroll
    for (int k = 0; k < KS; ++k)
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(qa[k], (double)x[k], acc, 0, 0, 0);
    // not greater: NaN passes
    unsigned long long pass[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) pass[v] = __ballot(!(acc[v] > thr[v]));
    if ((pass[0] | pass[1] | pass[2] | pass[3]) == 0) return;
    const int64_t j = tile * 16 + c16;
    bool full = false;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      if (pass[v] == 0) continue;
      const int m = g + 4 * v;
      const bool ok = !(acc[v] > thr[v]) && j < n && j != q0 + m && q0 + m < n;
      const unsigned bits = (unsigned)(__ballot(ok) >> (16 * g)) & 0xffffu;
      if (ok) qu[m * kKnnQueue + cnt[v] + __popc(bits & ((1u << c16) - 1u))] = (int32_t)j;
      cnt[v] += __popc(bits);
      full |= cnt[v] > kKnnQueue - 16;
    }
    if (__any(full)) {
      for (int m = 0; m < 16; ++m) {
        const int c = queued(m);
        if (c <= kKnnQueue - 16) continue;
        flush(m, c);
        listed |= 1u << m;
#pragma unroll
        for (int v = 0; v < 4; ++v)
          if (m == g + 4 * v) cnt[v] = 0;
      }
      knn_order();
      limits();
    }
  };
  limits();
  if (ns > 0) load(xb, nc, tile_of(0));
  for (int64_t s = 0; s < ns; ++s) {
    load(xn, nn, tile_of(s + 1 < ns ? s + 1 : s));
    visit(xb, nc, tile_of(s));
    if ((s & 15) == 15) limits();  // what the other wavefronts have found since
#pragma unroll
    for (int k = 0; k < KS; ++k) xb[k] = xn[k];
    nc = nn;
  }
  for (int m = 0; m < 16; ++m) {
    const int c = queued(m);
    if (lane == 0) sC[wv][m] = (listed >> m & 1) ? kKnnQueue + 1 + c : c;
  }
  __syncthreads();
  // Queries whose queues together fit one wavefront and have no list yet: one sort.
  unsigned rest = 0;
  for (int m = 0; m < 16; ++m)
    if (sC[0][m] + sC[1][m] + sC[2][m] + sC[3][m] > kKnnQueue) rest |= 1u << m;
  rest = __builtin_amdgcn_readfirstlane(rest);
  for (int m = wv; m < 16; m += 4) {
    if (q0 + m >= n || (rest >> m & 1)) continue;
    int at = lane, w = 0;
    while (w < 4 && at >= sC[w][m]) at -= sC[w++][m];
    double d = inf;
    int32_t j = 0x7fffffff;
    if (w < 4) {
      j = ((const int32_t*)(knn_lds + (size_t)w * knn_lds_wave(kb) + (size_t)16 * kb *
                            12))[m * kKnnQueue + at];
      d = distance(q0 + m, j);
    }
    knn_sort<64>(d, j);
    if (lane < K) nbr[(q0 + m) * K + lane] = j;
  }
  if (rest == 0) return;
  for (unsigned left = rest; left; left &= left - 1) {
    const int m = __ffs((int)left) - 1, c = queued(m);
    if (c > 0) flush(m, c);
  }
  __syncthreads();
  // the four wavefronts' lists of query m
  for (int m = wv; m < 16; m += 4) {
    if (q0 + m >= n || !(rest >> m & 1)) continue;
    double d = inf;
    int32_t j = 0x7fffffff;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const double* const wd = (const double*)(knn_lds + (size_t)w * knn_lds_wave(kb));
      const int32_t* const wi = (const int32_t*)(wd + 16 * kb);
      const int at = w == 0 ? lane : 63 - lane;
      const double e = at < kb ? wd[m * kb + at] : inf;
      const int32_t f = at < kb ? wi[m * kb + at] : 0x7fffffff;
      if (w == 0) {
        d = e;
        j = f;
      } else {
        if (knn_less(e, f, d, j)) {
          d = e;
          j = f;
        }
        knn_merge64(d, j);
      }
    }
    if (lane < K) nbr[(q0 + m) * K + lane] = j;
  }
}

// One wavefront per query point i; its coordinates are staged in LDS.  Lane l scans the
// candidates j = l, l + 64, ... (increasing j) and keeps the KB smallest (distance, j)
// pairs in a sorted register list (a candidate that ties with a kept one goes after it,
// so within a lane ties keep the lower index).  The wave then takes the K smallest over
// all lanes by K rounds of a (distance, index) minimum across lanes, the winning lane
// dropping its head.  The point itself is skipped.  Serves few points (knn_wave_max) and
// points that the screen of k_knn cannot separate (knn_inseparable).
template <typename T, int KB>
__global__ __launch_bounds__(kThreads) void k_knn_wave(const T* __restrict__ X, int64_t n, int dim,
                                                       int K, int32_t* __restrict__ nbr) {
  __shared__ double sq[kThreads / kWave][kKnnMaxDim];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t i = (int64_t)blockIdx.x * (kThreads / kWave) + wv;
  const bool valid = i < n;  // the waves past n stay for the barrier, then leave
  if (valid)
    for (int c = lane; c < dim; c += kWave) sq[wv][c] = (double)X[i * dim + c];
  __syncthreads();
  if (!valid) return;
  double dist[KB];
  int32_t idx[KB];
#pragma unroll
  for (int q = 0; q < KB; ++q) {
    dist[q] = __builtin_inf();
    idx[q] = 0x7fffffff;
  }
  for (int64_t j = lane; j < n; j += kWave) {
    if (j == i) continue;
    const T* __restrict__ xj = X + j * dim;
    double d = 0.0;
    for (int c = 0; c < dim; ++c) {
      const double t = sq[wv][c] - (double)xj[c];
      d = __builtin_fma(t, t, d);
    }
    // a distance beyond the largest double counts as that: an infinite one would not come
    // before an empty place
    d = __builtin_fmin(d, 1.7976931348623157e308);
    if (d < dist[KB - 1]) {
#pragma unroll
      for (int q = KB - 1; q > 0; --q) {
        const bool sh = d < dist[q - 1];
        const bool here = !sh && d < dist[q];
        const double nd = sh ? dist[q - 1] : (here ? d : dist[q]);
        const int32_t ni = sh ? idx[q - 1] : (here ? (int32_t)j : idx[q]);
        dist[q] = nd;
        idx[q] = ni;
      }
      if (d < dist[0]) {
        dist[0] = d;
        idx[0] = (int32_t)j;
      }
    }
  }
  for (int t = 0; t < K; ++t) {
    double bd = dist[0];
    int32_t bi = idx[0];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const double od = __shfl_xor(bd, o);
      const int32_t oi = __shfl_xor(bi, o);
      if (od < bd || (od == bd && oi < bi)) {
        bd = od;
        bi = oi;
      }
    }
    if (lane == 0) nbr[i * K + t] = bi;
    if (idx[0] == bi) {  // the lane that held the winner drops its head
#pragma unroll
      for (int q = 0; q < KB - 1; ++q) {
        dist[q] = dist[q + 1];
        idx[q] = idx[q + 1];
      }
      dist[KB - 1] = __builtin_inf();
      idx[KB - 1] = 0x7fffffff;
    }
  }
}

// |x_i|^2 in FP64; -inf where a product could overflow.  near[q] += points within 1.25 err of
// probe q, kKnnProbes points spread over the array: where that is most of them the screen
// separates nothing (knn_inseparable).
template <typename T>
__global__ __launch_bounds__(kThreads) void k_knn_norms(const T* __restrict__ X, int64_t n,
                                                        int dim, double* __restrict__ nrm,
                                                        unsigned* __restrict__ near) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const bool in = i < n;
  const T* __restrict__ xi = X + (in ? i : n - 1) * dim;
  double d = 0.0, pn[kKnnProbes], pd[kKnnProbes];
#pragma unroll
  for (int q = 0; q < kKnnProbes; ++q) pn[q] = pd[q] = 0.0;
  for (int c = 0; c < dim; ++c) {
    const double t = (double)xi[c];
    d = __builtin_fma(t, t, d);
#pragma unroll
    for (int q = 0; q < kKnnProbes; ++q) {
      const double p = (double)X[n / kKnnProbes * q * dim + c];
      pn[q] = __builtin_fma(p, p, pn[q]);
      pd[q] = __builtin_fma(t - p, t - p, pd[q]);
    }
  }
  if (in) nrm[i] = d < 1e290 ? d : -__builtin_inf();
  const double c1 = 1.25 * 4.0 * (dim + 4) * 0x1p-53;
#pragma unroll
  for (int q = 0; q < kKnnProbes; ++q) {
    const unsigned long long b = __ballot(in && (d >= 1e290 || pd[q] <= c1 * (d + pn[q])));
    if (b && (threadIdx.x & 63) == 0) atomicAdd(&near[q], (unsigned)__popcll(b));
  }
}

// ----------------------------------------------------------------------------- pattern
// True if i is among the K neighbours of j.
__device__ __forceinline__ bool lists(const int32_t* __restrict__ nbr, int K, int64_t j,
                                      int64_t i) {
  for (int t = 0; t < K; ++t)
    if (nbr[j * K + t] == (int32_t)i) return true;
  return false;
}

// cnt[j] += 1 for every edge i -> j whose reverse j -> i is not listed (the union adds i to
// row j).
__global__ __launch_bounds__(kThreads) void k_knn_incount(const int32_t* __restrict__ nbr,
                                                          int64_t n, int K,
                                                          unsigned* __restrict__ cnt) {
  const int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (e >= n * K) return;
  const int64_t i = e / K;
  const int64_t j = nbr[e];
  if (!lists(nbr, K, j, i)) atomicAdd(&cnt[j], 1u);
}

// rowptr[0] = 0, rowptr[i + 1] = rowptr[i] + K + cnt[i] + diag, in one workgroup: pieces of
// 8 rows per thread staged through LDS, a block scan of the threads' sums per piece
// (n = 20000: 19 us; 42 us with one contiguous chunk of all rows per thread).
constexpr int kScanThreads = 1024, kScanPer = 8;
__global__ __launch_bounds__(kScanThreads) void k_knn_rowptr(const unsigned* __restrict__ cnt,
                                                             int64_t n, int K, int diag,
                                                             int64_t* __restrict__ rowptr) {
  __shared__ unsigned sc[kScanThreads * (kScanPer + 1)];
  __shared__ int64_t wsum[kScanThreads / kWave];
  const int t = threadIdx.x, lane = t & 63, wv = t >> 6;
  int64_t run = 0;
  for (int64_t i0 = 0; i0 < n; i0 += kScanThreads * kScanPer) {
#pragma unroll
    for (int u = 0; u < kScanPer; ++u) {
      const int e = u * kScanThreads + t;
      sc[e + e / kScanPer] = i0 + e < n ? cnt[i0 + e] + (unsigned)(K + diag) : 0u;
    }
    __syncthreads();
    unsigned v[kScanPer];
    int64_t mine = 0;
#pragma unroll
    for (int u = 0; u < kScanPer; ++u) {
      v[u] = sc[t * (kScanPer + 1) + u];
      mine += v[u];
    }
    int64_t inc = mine;  // inclusive scan over the wave
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int64_t up = __shfl_up(inc, o);
      if (lane >= o) inc += up;
    }
    if (lane == 63) wsum[wv] = inc;
    __syncthreads();
    int64_t before = run, all = 0;
#pragma unroll
    for (int w = 0; w < kScanThreads / kWave; ++w) {
      if (w < wv) before += wsum[w];
      all += wsum[w];
    }
    int64_t at = before + inc - mine;
#pragma unroll
    for (int u = 0; u < kScanPer; ++u) {
      const int64_t i = i0 + (int64_t)t * kScanPer + u;
      if (i < n) rowptr[i] = at;
      at += v[u];
    }
    run += all;
    __syncthreads();
  }
  if (t == 0) rowptr[n] = run;
}

// Row i: its own K neighbours (and i itself when diag) first; cursor[i] = where the
// union's additions to row i begin.
__global__ __launch_bounds__(kThreads) void k_knn_own(const int32_t* __restrict__ nbr, int64_t n,
                                                      int K, int diag,
                                                      const int64_t* __restrict__ rowptr,
                                                      int32_t* __restrict__ col,
                                                      unsigned long long* __restrict__ cursor) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  int64_t p = rowptr[i];
  for (int t = 0; t < K; ++t) col[p++] = nbr[i * K + t];
  if (diag) col[p++] = (int32_t)i;
  cursor[i] = (unsigned long long)p;
}

// The union's additions: i is appended to row j for every edge i -> j without its reverse.
__global__ __launch_bounds__(kThreads) void k_knn_add(const int32_t* __restrict__ nbr, int64_t n,
                                                      int K, int32_t* __restrict__ col,
                                                      unsigned long long* __restrict__ cursor) {
  const int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (e >= n * K) return;
  const int64_t i = e / K;
  const int64_t j = nbr[e];
  if (lists(nbr, K, j, i)) return;
  const unsigned long long p = atomicAdd(&cursor[j], 1ull);
  col[p] = (int32_t)i;
}

// Sort every row's columns (all different; the order the additions arrived in is not
// deterministic, the sorted row is): one wavefront per row puts every column at its rank.
// Rows of up to 64 are held in registers, longer ones are ranked into tmp and copied back
// (n = 20000, rows of 17 on average: 12 us; 379 us with one thread's insertion sort per
// row).
__global__ __launch_bounds__(kThreads) void k_sort_rows(const int64_t* __restrict__ rowptr,
                                                        int64_t n, int32_t* __restrict__ col,
                                                        int32_t* __restrict__ tmp) {
  const int64_t i = (int64_t)blockIdx.x * (kThreads / kWave) + threadIdx.x / kWave;
  if (i >= n) return;
  const int lane = threadIdx.x & 63;
  const int64_t b = rowptr[i], c = rowptr[i + 1] - b;
  if (c <= kWave) {
    const int32_t v = lane < c ? col[b + lane] : 0x7fffffff;
    int rank = 0;
    for (int k = 0; k < (int)c; ++k) rank += __builtin_amdgcn_readlane(v, k) < v ? 1 : 0;
    if (lane < c) col[b + rank] = v;
    return;
  }
  for (int64_t z0 = 0; z0 < c; z0 += kWave) {
    const int32_t v = z0 + lane < c ? col[b + z0 + lane] : 0x7fffffff;
    int64_t rank = 0;
    for (int64_t k0 = 0; k0 < c; k0 += kWave) {
      const int32_t u = k0 + lane < c ? col[b + k0 + lane] : 0x7fffffff;
#pragma unroll 16
      for (int k = 0; k < kWave; ++k) rank += __builtin_amdgcn_readlane(u, k) < v ? 1 : 0;
    }
    if (z0 + lane < c) tmp[b + rank] = v;
  }
  __threadfence_block();  // the wavefront's stores before its loads of other lanes' entries
  for (int64_t z = lane; z < c; z += kWave) col[b + z] = *(volatile int32_t*)(tmp + b + z);
}

// ----------------------------------------------------------------------------- values
// v_ij = exp(-||x_i - x_j||^2 / (2 sigma^2)) (sigma > 0) or 1, 0 on the diagonal; the
// degree d_i = sum_j v_ij (FP64).  Sixteen lanes per row.
constexpr int kRowLanes = 16;
template <typename T>
__global__ __launch_bounds__(kThreads) void k_knn_values(const T* __restrict__ X, int64_t n,
                                                         int dim, double sigma,
                                                         const int64_t* __restrict__ rowptr,
                                                         const int32_t* __restrict__ col,
                                                         double* __restrict__ v,
                                                         double* __restrict__ deg) {
  const int64_t i = ((int64_t)blockIdx.x * kThreads + threadIdx.x) / kRowLanes;
  const int q = threadIdx.x % kRowLanes;
  if (i >= n) return;
  const double inv = sigma > 0.0 ? 1.0 / (2.0 * sigma * sigma) : 0.0;
  double d = 0.0;
  for (int64_t z = rowptr[i] + q; z < rowptr[i + 1]; z += kRowLanes) {
    const int64_t j = col[z];
    double w = 0.0;
    if (j != i) {
      w = 1.0;
      if (sigma > 0.0) {
        double s2 = 0.0;
        for (int c = 0; c < dim; ++c) {
          const double t = (double)X[i * dim + c] - (double)X[j * dim + c];
          s2 = __builtin_fma(t, t, s2);
        }
        w = exp(-s2 * inv);
      }
    }
    v[z] = w;
    d += w;
  }
#pragma unroll
  for (int o = kRowLanes / 2; o > 0; o >>= 1) d += __shfl_xor(d, o);
  if (q == 0) deg[i] = d;
}

// Output values: the similarity itself, or L_ij = [i == j] - s_i v_ij s_j with
// s = d^{-1/2} (0 where d = 0).  Sixteen lanes per row (n = 20000: 6.5 us; 48 us with one
// thread per row).
template <typename T>
__global__ __launch_bounds__(kThreads) void k_knn_out(int64_t n, int laplacian,
                                                      const int64_t* __restrict__ rowptr,
                                                      const int32_t* __restrict__ col,
                                                      const double* __restrict__ v,
                                                      const double* __restrict__ deg,
                                                      T* __restrict__ val) {
  const int64_t i = ((int64_t)blockIdx.x * kThreads + threadIdx.x) / kRowLanes;
  if (i >= n) return;
  const double si = deg[i] > 0.0 ? 1.0 / sqrt(deg[i]) : 0.0;
  for (int64_t z = rowptr[i] + threadIdx.x % kRowLanes; z < rowptr[i + 1]; z += kRowLanes) {
    if (!laplacian) {
      val[z] = (T)v[z];
      continue;
    }
    const int64_t j = col[z];
    const double sj = deg[j] > 0.0 ? 1.0 / sqrt(deg[j]) : 0.0;
    val[z] = (T)((j == i ? 1.0 : 0.0) - si * v[z] * sj);
  }
}

// flag[0] += number of non-finite coordinates (the search needs finite distances).
template <typename T>
__global__ __launch_bounds__(kThreads) void k_count_nonfinite(const T* __restrict__ X,
                                                              int64_t count,
                                                              unsigned* __restrict__ flag) {
  unsigned bad = 0;
  for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < count;
       e += (int64_t)gridDim.x * kThreads) {
    const double a = (double)X[e];
    if (!(a - a == 0.0)) ++bad;
  }
  if (bad) atomicAdd(flag, bad);
}

// ----------------------------------------------------------------------------- launchers
template <typename T>
void launch_count_nonfinite(const T* X, int64_t count, unsigned* flag, hipStream_t s) {
  int64_t nb = (count + kThreads - 1) / kThreads;
  if (nb > 4096) nb = 4096;
  if (nb < 1) nb = 1;
  hipLaunchKernelGGL(k_count_nonfinite<T>, dim3((unsigned)nb), dim3(kThreads), 0, s, X, count,
                     flag);
}
template void launch_count_nonfinite<float>(const float*, int64_t, unsigned*, hipStream_t);
template void launch_count_nonfinite<double>(const double*, int64_t, unsigned*, hipStream_t);

template <typename T, int KS, bool FULL>
static void knn_go(const T* X, int64_t n, int dim, int K, const double* nrm, int32_t* nbr,
                   hipStream_t s) {
  const int kb = K <= 16 ? 16 : K <= 32 ? 32 : 64;
  const size_t lds = 4 * knn_lds_wave(kb);
  if (lds > 60 * 1024)
    (void)hipFuncSetAttribute((const void*)k_knn<T, KS, FULL>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL((k_knn<T, KS, FULL>), dim3((unsigned)((n + 15) / 16)), dim3(kThreads), lds, s,
                     X, n, dim, K, kb, nrm, nbr);
}
// Points up to which one wavefront per query is the faster search: the whole chip works on
// some 20 us where k_knn has too few workgroups (a call screened / with a wavefront per query,
// n = 1000, 2100, 2500, 3000, 4000: FP32 dim = 10, K = 10 1.31 1.00 0.93 0.91 0.73, K = 16 1.48
// 1.16 1.08 1.05 0.85, K = 20 1.56 1.08 1.04 0.99 0.76).  Lists of more than 32 cost the wavefront
// most of its registers (K = 40: 1.20 0.59 0.60 0.58 0.43), long rows its uncoalesced loads,
// where the screen loads whole blocks of 16 coordinates (FP64, dim = 32, K = 16: 1.33 0.59 0.53
// 0.48 0.32; FP64, dim = 24, K = 20: 1.61 1.09 1.02 0.96 0.68).
static int64_t knn_wave_max(int dim, int K, size_t esz) {
  if (K > 32 || dim > 24 || (dim == 16 && esz == 8)) return 2000;
  return K <= 10 ? 2400 : K <= 16 ? 3000 : 2600;
}

bool knn_screened(int64_t n, int dim, int K, size_t esz) { return n > knn_wave_max(dim, K, esz); }

// More than half of the points lie within the rounding of the screen of one of the probes:
// nearly every pair would pass it and be formed twice (n = 20000, dim = 16, K = 10, all points
// equal: 2166 us screened, 1432 with a wavefront per query; FP32 points of unit spread around
// 1e7: 3211 and 2462).
bool knn_inseparable(const unsigned* near, int64_t n) {
  unsigned most = 0;
  for (int q = 0; q < kKnnProbes; ++q) most = near[q] > most ? near[q] : most;
  return 2 * (int64_t)most > n;
}

template <typename T>
void launch_knn_norms(const T* X, int64_t n, int dim, double* nrm, unsigned* near, hipStream_t s) {
  hipLaunchKernelGGL(k_knn_norms<T>, dim3((unsigned)((n + kThreads - 1) / kThreads)),
                     dim3(kThreads), 0, s, X, n, dim, nrm, near);
}

template <typename T>
void launch_knn(const T* X, int64_t n, int dim, int K, const double* nrm, int32_t* nbr,
                hipStream_t s) {
  if (!nrm) {
    const dim3 grid((unsigned)((n + kThreads / kWave - 1) / (kThreads / kWave))), block(kThreads);
    if (K <= 16)
      hipLaunchKernelGGL((k_knn_wave<T, 16>), grid, block, 0, s, X, n, dim, K, nbr);
    else if (K <= 32)
      hipLaunchKernelGGL((k_knn_wave<T, 32>), grid, block, 0, s, X, n, dim, K, nbr);
    else
      hipLaunchKernelGGL((k_knn_wave<T, 64>), grid, block, 0, s, X, n, dim, K, nbr);
    return;
  }
  if (dim == 16) knn_go<T, 4, true>(X, n, dim, K, nrm, nbr, s);
  else if (dim == 32) knn_go<T, 8, true>(X, n, dim, K, nrm, nbr, s);
  else if (dim == 48) knn_go<T, 12, true>(X, n, dim, K, nrm, nbr, s);
  else if (dim == 64) knn_go<T, 16, true>(X, n, dim, K, nrm, nbr, s);
  else if (dim <= 4) knn_go<T, 1, false>(X, n, dim, K, nrm, nbr, s);
  else if (dim <= 8) knn_go<T, 2, false>(X, n, dim, K, nrm, nbr, s);
  else if (dim <= 16) knn_go<T, 4, false>(X, n, dim, K, nrm, nbr, s);
  else if (dim <= 32) knn_go<T, 8, false>(X, n, dim, K, nrm, nbr, s);
  else knn_go<T, 16, false>(X, n, dim, K, nrm, nbr, s);
}

static unsigned blocks_of(int64_t m) { return (unsigned)((m + kThreads - 1) / kThreads); }

void launch_knn_pattern_count(const int32_t* nbr, int64_t n, int K, int diag, unsigned* cnt,
                              int64_t* rowptr, hipStream_t s) {
  hipLaunchKernelGGL(k_knn_incount, dim3(blocks_of(n * K)), dim3(kThreads), 0, s, nbr, n, K, cnt);
  hipLaunchKernelGGL(k_knn_rowptr, dim3(1), dim3(kScanThreads), 0, s, (const unsigned*)cnt, n, K,
                     diag, rowptr);
}

void launch_knn_pattern_fill(const int32_t* nbr, int64_t n, int K, int diag,
                             const int64_t* rowptr, int32_t* col, unsigned long long* cursor,
                             int32_t* tmp, hipStream_t s) {
  hipLaunchKernelGGL(k_knn_own, dim3(blocks_of(n)), dim3(kThreads), 0, s, nbr, n, K, diag, rowptr,
                     col, cursor);
  hipLaunchKernelGGL(k_knn_add, dim3(blocks_of(n * K)), dim3(kThreads), 0, s, nbr, n, K, col,
                     cursor);
  hipLaunchKernelGGL(k_sort_rows, dim3(blocks_of(n * kWave)), dim3(kThreads), 0, s, rowptr, n, col,
                     tmp);
}

template <typename T>
void launch_knn_values(const T* X, int64_t n, int dim, double sigma, int laplacian,
                       const int64_t* rowptr, const int32_t* col, double* v, double* deg, T* val,
                       hipStream_t s) {
  hipLaunchKernelGGL(k_knn_values<T>, dim3(blocks_of(n * kRowLanes)), dim3(kThreads), 0, s, X, n, dim, sigma,
                     rowptr, col, v, deg);
  hipLaunchKernelGGL(k_knn_out<T>, dim3(blocks_of(n * kRowLanes)), dim3(kThreads), 0, s, n, laplacian, rowptr,
                     col, (const double*)v, (const double*)deg, val);
}

template void launch_knn_norms<float>(const float*, int64_t, int, double*, unsigned*, hipStream_t);
template void launch_knn_norms<double>(const double*, int64_t, int, double*, unsigned*, hipStream_t);
template void launch_knn<float>(const float*, int64_t, int, int, const double*, int32_t*,
                                hipStream_t);
template void launch_knn<double>(const double*, int64_t, int, int, const double*, int32_t*,
                                 hipStream_t);
template void launch_knn_values<float>(const float*, int64_t, int, double, int, const int64_t*,
                                       const int32_t*, double*, double*, float*, hipStream_t);
template void launch_knn_values<double>(const double*, int64_t, int, double, int, const int64_t*,
                                        const int32_t*, double*, double*, double*, hipStream_t);

}  // namespace snmf
