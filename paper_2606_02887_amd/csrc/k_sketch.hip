// Kernels of the randomized range finder of LAI-SNMPBB (Section 2.3) and of the SVD start
// (Section 4.2): wide products A X (X with up to 128 columns), tall-skinny Gram products
// X^T Y in FP64 with a fixed summation order, a one-workgroup Cholesky factorisation with
// the inverse of its triangular factor, tall-skinny products X M, a one-workgroup Jacobi
// eigensolver and the selection of the dominant eigenpairs.
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"
#include "rho.hpp"

namespace snmf {

// ----------------------------------------------------------------------------- A X
// CSR: one wavefront per row; lane c owns the VEC consecutive columns c VEC .. of each block
// of 64 VEC columns (VEC = 2 for even w: one vector load per nonzero and block).  The row's
// (column, value) pairs are loaded 64 at a time, the next row's first 64 and the extent of
// the row after it while this row gathers, and broadcast by lane reads.  The rows of X of
// up to 32 nonzeros are requested before the first is used (long rows), of 8 or 16 in the
// rest of a row; every column's terms are added in storage order.  Bound by the gathers'
// latency: the longest rows of a power-law graph are one chain each (n = 200000, 2e6
// nonzeros, w = 74: 1208 us with one nonzero in flight per wavefront, 265 us so, on average
// 1800 wavefronts resident).
template <typename T, int VEC>
__global__ __launch_bounds__(kThreads) void k_spmm_wide(const int64_t* __restrict__ rowptr,
                                                        const int32_t* __restrict__ col,
                                                        const T* __restrict__ val,
                                                        const T* __restrict__ X, int64_t n, int w,
                                                        T* __restrict__ Y) {
  constexpr int NBLK = kSketchMaxW / (64 * VEC);
  typedef T vec __attribute__((ext_vector_type(2)));
  const int lane = threadIdx.x & 63;
  const int64_t wave = __builtin_amdgcn_readfirstlane(
      (int)(((int64_t)blockIdx.x * kThreads + threadIdx.x) / kWave));
  const int64_t nwaves = (int64_t)gridDim.x * (kThreads / kWave);
  // columns of a lane; a lane past the last reads the first columns and stores nothing
  bool own[NBLK];
  int at[NBLK];
#pragma unroll
  for (int q = 0; q < NBLK; ++q) {
    const int c = (q * 64 + lane) * VEC;
    own[q] = c < w;
    at[q] = own[q] ? c : 0;
  }
  T acc[NBLK][VEC];
  auto load = [&](const T* __restrict__ xr, T (&x)[NBLK][VEC]) {
#pragma unroll
    for (int q = 0; q < NBLK; ++q) {
      if (VEC == 2) {
        const vec t = *(const vec*)(xr + at[q]);
        x[q][0] = t[0];
        x[q][VEC - 1] = t[1];
      } else {
        x[q][0] = xr[at[q]];
      }
    }
  };
  auto add = [&](T v, const T (&x)[NBLK][VEC]) {
#pragma unroll
    for (int q = 0; q < NBLK; ++q)
#pragma unroll
      for (int u = 0; u < VEC; ++u) acc[q][u] += v * x[q][u];
  };
  auto value = [&](T mv, int k) -> T {
    if constexpr (sizeof(T) == 8) return readlane_d(mv, k);
    else return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(mv), k));
  };
  // nonzeros k .. k + U - 1 of the 64 held by the lanes, those at or past cnt left out
  // (their loads repeat the last one's)
  auto batch = [&](auto uc, int k, int cnt, int mc, T mv) {
    constexpr int U = decltype(uc)::value;
    T x[U][NBLK][VEC];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int kk = k + u < cnt ? k + u : cnt - 1;
      load(X + (int64_t)__builtin_amdgcn_readlane(mc, kk) * w, x[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (k + u < cnt) add(value(mv, k + u), x[u]);
  };
  if (wave >= n) return;
  const int64_t last = n - 1;
  int64_t b = rowptr[wave], e = rowptr[wave + 1];
  int64_t r1 = wave + nwaves < n ? wave + nwaves : last;
  int64_t b1 = rowptr[r1], e1 = rowptr[r1 + 1];
  int mc = lane < e - b ? col[b + lane] : 0;
  T mv = lane < e - b ? val[b + lane] : T(0);
  for (int64_t row = wave; row < n; row += nwaves) {
    const int64_t r2 = row + 2 * nwaves < n ? row + 2 * nwaves : last;
    const int64_t b2 = rowptr[r2], e2 = rowptr[r2 + 1];
    const int mc1 = lane < e1 - b1 ? col[b1 + lane] : 0;
    const T mv1 = lane < e1 - b1 ? val[b1 + lane] : T(0);
#pragma unroll
    for (int q = 0; q < NBLK; ++q)
#pragma unroll
      for (int v = 0; v < VEC; ++v) acc[q][v] = T(0);
    for (int64_t zb = b; zb < e; zb += kWave) {
      if (zb > b) {
        mc = lane < e - zb ? col[zb + lane] : 0;
        mv = lane < e - zb ? val[zb + lane] : T(0);
      }
      const int cnt = e - zb < kWave ? (int)(e - zb) : kWave;
      int k = 0;
      for (; k + 32 <= cnt; k += 32) batch(std::integral_constant<int, 32>{}, k, cnt, mc, mv);
      for (; cnt - k > 8; k += 16) batch(std::integral_constant<int, 16>{}, k, cnt, mc, mv);
      if (k < cnt) batch(std::integral_constant<int, 8>{}, k, cnt, mc, mv);
    }
    T* __restrict__ yr = Y + row * w;
#pragma unroll
    for (int q = 0; q < NBLK; ++q)
      if (own[q]) {
#pragma unroll
        for (int v = 0; v < VEC; ++v) yr[at[q] + v] = acc[q][v];
      }
    b = b1;
    e = e1;
    b1 = b2;
    e1 = e2;
    mc = mc1;
    mv = mv1;
  }
}

// Dense A (n x n, leading dimension ld): 64-row output tiles, K in chunks of 32 staged in
// LDS; thread t owns row t % 64 of the tile and columns t / 64 + 4 q (accumulated in T,
// K in increasing order).
template <typename T>
__global__ __launch_bounds__(kThreads) void k_dense_wide(const T* __restrict__ A, int64_t ld,
                                                         const T* __restrict__ X, int64_t n, int w,
                                                         T* __restrict__ Y) {
  __shared__ T sA[64][33];
  __shared__ T sX[32][kSketchMaxW];
  const int t = threadIdx.x, rr = t & 63, cg = t >> 6;
  const int64_t row0 = (int64_t)blockIdx.x * 64;
  T acc[kSketchMaxW / 4];
#pragma unroll
  for (int q = 0; q < kSketchMaxW / 4; ++q) acc[q] = T(0);
  for (int64_t k0 = 0; k0 < n; k0 += 32) {
    __syncthreads();
    for (int e = t; e < 64 * 32; e += kThreads) {
      const int i = e >> 5, kk = e & 31;
      const int64_t gi = row0 + i, gk = k0 + kk;
      sA[i][kk] = (gi < n && gk < n) ? A[gi * ld + gk] : T(0);
    }
    for (int e = t; e < 32 * w; e += kThreads) {
      const int kk = e / w, c = e - kk * w;
      const int64_t gk = k0 + kk;
      sX[kk][c] = gk < n ? X[gk * w + c] : T(0);
    }
    __syncthreads();
    for (int kk = 0; kk < 32; ++kk) {
      const T a = sA[rr][kk];
#pragma unroll
      for (int q = 0; q < kSketchMaxW / 4; ++q) {
        const int c = cg + 4 * q;
        if (c < w) acc[q] += a * sX[kk][c];
      }
    }
  }
  const int64_t gi = row0 + rr;
  if (gi < n) {
#pragma unroll
    for (int q = 0; q < kSketchMaxW / 4; ++q) {
      const int c = cg + 4 * q;
      if (c < w) Y[gi * w + c] = acc[q];
    }
  }
}

// ----------------------------------------------------------------------------- X^T Y
typedef double sd4 __attribute__((ext_vector_type(4)));

// Partial C_b = X_b^T Y_b over the rows of slab b = blockIdx.x in FP64 on the FP64 matrix
// cores (16x16x4, rows as K; the instruction is one FMA chain over its four rows, so an
// entry is the chain over the slab's rows in order).  The rows are staged in LDS as FP64,
// CH at a time in two buffers with the next two chunks' loads in registers, one barrier per
// chunk; of the NB^2 tiles of 16 x 16 entries, NB = ceil(w / 16) (Y = X: the NB (NB + 1) / 2
// of the upper block triangle, written to both halves, so the Gram is exactly symmetric)
// wave v takes tiles v, v + 8, ... (tile 0 once more where there are none left, never
// stored).  Lane l supplies X[l / 16][16 qa + l % 16] and Y[l / 16][16 qb + l % 16] of a
// k-step and holds D[l / 16 + 4 v][l % 16].
// Bound by the FP64 matrix rate: n = 200000, w = 74 needs 15 tiles of 64 cycles per four
// rows, 20 us over 1024 SIMDs; measured 47 us (299 us on the vector units from LDS).
template <int NB, bool SYM>
struct TsGram {
  static constexpr int CH = SYM ? (NB > 6 ? 32 : 64) : (NB > 6 ? 16 : 32);  // rows of a chunk
  static constexpr int NM = SYM ? 1 : 2;
  static constexpr int NT = SYM ? NB * (NB + 1) / 2 : NB * NB;
  static constexpr int TPW = (NT + 7) / 8;                   // tiles of a wave
  static constexpr int PITCH = NB % 2 ? 16 * NB : 16 * NB + 16;  // 32 mod 64 words
  static constexpr size_t LDS = (size_t)2 * NM * CH * PITCH * 8;
};

template <typename T, int NB, bool SYM>
__global__ __launch_bounds__(512) void k_tsgram(const T* __restrict__ X, const T* __restrict__ Y,
                                                int64_t n, int w, int64_t rows_per,
                                                double* __restrict__ part) {
  typedef TsGram<NB, SYM> C;
  constexpr int CH = C::CH, NM = C::NM, NT = C::NT, TPW = C::TPW, PITCH = C::PITCH;
  constexpr int one = CH * PITCH, NL = CH / 4;
  extern __shared__ __attribute__((aligned(16))) double ts_lds[];  // [buffer][X, Y][CH x PITCH]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t r0 = (int64_t)blockIdx.x * rows_per;
  const int64_t r1 = r0 + rows_per < n ? r0 + rows_per : n;
  int ia[TPW], ib[TPW], qa[TPW], qb[TPW];  // tiles of this wave
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    int t = wave + 8 * i;
    if (t >= NT) t = 0;
    if (SYM) {
      int a = 0;
      while (t >= NB - a) {
        t -= NB - a;
        ++a;
      }
      qa[i] = a;
      qb[i] = a + t;
    } else {
      qa[i] = t / NB;
      qb[i] = t - qa[i] * NB;
    }
    ia[i] = (lane >> 4) * PITCH + (lane & 15) + 16 * qa[i];
    ib[i] = (lane >> 4) * PITCH + (lane & 15) + 16 * qb[i] + (NM - 1) * one;
  }
  sd4 acc[TPW];
#pragma unroll
  for (int i = 0; i < TPW; ++i) acc[i] = sd4{0.0, 0.0, 0.0, 0.0};
  for (int e = tid; e < 2 * NM * one; e += 512) ts_lds[e] = 0.0;  // columns past w stay zero
  // thread t loads column t % 128 of rows t / 128 + 4 i of a chunk
  const int c = tid & 127, rr = tid >> 7;
  const bool cok = c < w;
  const unsigned off = (unsigned)(rr * w + (cok ? c : 0));
  T xa[NM][NL], xb[NM][NL];
  auto load = [&](T (&xv)[NM][NL], int64_t k0) {
    if (k0 + CH <= r1) {
      const T* const px = X + k0 * w;
      const T* const py = Y + k0 * w;
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        xv[0][i] = px[off + (unsigned)(4 * i * w)];
        if (!SYM) xv[NM - 1][i] = py[off + (unsigned)(4 * i * w)];
      }
    } else {  // the slab's last chunk, or past it: rows clamped to a valid one
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int64_t row = k0 + rr + 4 * i;
        const int64_t a = (row < r1 ? row : r1 - 1) * w + (cok ? c : 0);
        xv[0][i] = X[a];
        if (!SYM) xv[NM - 1][i] = Y[a];
      }
    }
  };
  load(xa, r0);
  load(xb, r0 + CH);
  __syncthreads();
  auto chunk = [&](T (&xv)[NM][NL], int64_t k0, double* s0) {
    if (cok) {
      double* const d = s0 + rr * PITCH + c;
      const int left = (int)(r1 - k0 < CH ? r1 - k0 : CH) - rr;  // rows past the slab add zeros
#pragma unroll
      for (int i = 0; i < NL; ++i)
#pragma unroll
        for (int q = 0; q < NM; ++q)
          d[q * one + 4 * i * PITCH] = 4 * i < left ? (double)xv[q][i] : 0.0;
    }
    __syncthreads();
    load(xv, k0 + 2 * CH);
#pragma unroll(TPW > 2 ? 4 : 8)
    for (int s = 0; s < CH / 4; ++s)
#pragma unroll
      for (int i = 0; i < TPW; ++i)
        acc[i] = __builtin_amdgcn_mfma_f64_16x16x4f64(s0[ia[i] + 4 * s * PITCH],
                                                      s0[ib[i] + 4 * s * PITCH], acc[i], 0, 0, 0);
  };
  for (int64_t k0 = r0; k0 < r1; k0 += 2 * CH) {
    chunk(xa, k0, ts_lds);
    chunk(xb, k0 + CH, ts_lds + NM * one);
  }
  double* __restrict__ out = part + (size_t)blockIdx.x * w * w;
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    if (wave + 8 * i >= NT) continue;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int a = 16 * qa[i] + (lane >> 4) + 4 * v, b = 16 * qb[i] + (lane & 15);
      if (a >= w || b >= w) continue;
      if (!SYM) {
        out[a * w + b] = acc[i][v];
      } else if (qa[i] < qb[i] || a <= b) {
        out[a * w + b] = acc[i][v];
        out[b * w + a] = acc[i][v];
      }
    }
  }
}

// C = sum over slabs of the partials, in slab order (at most 256 slabs): a workgroup takes
// 16 entries, thread t loads those of slab t, and one lane per entry adds its slabs from
// LDS (65 us for 256 slabs at w = 74 with one load in flight per entry, 7.7 us so).
__global__ __launch_bounds__(kThreads) void k_tsgram_reduce(const double* __restrict__ part,
                                                            int nb, int ww,
                                                            double* __restrict__ C) {
  __shared__ double sp[kThreads][17];
  const int t = threadIdx.x, e0 = blockIdx.x * 16;
  if (t < nb) {
    double v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = part[(size_t)t * ww + (e0 + u < ww ? e0 + u : ww - 1)];
#pragma unroll
    for (int u = 0; u < 16; ++u) sp[t][u] = v[u];
  }
  __syncthreads();
  if (t >= 16 || e0 + t >= ww) return;
  double s = 0.0;
#pragma unroll 16
  for (int b = 0; b < nb; ++b) s += sp[b][t];
  C[e0 + t] = s;
}

// ----------------------------------------------------------------------------- Cholesky
// One workgroup: G + s I = R^T R with s = shift_rel tr(G) (R upper triangular, the rows
// eliminated in order), then Rinv = R^{-1} by back substitution, one column per lane, a
// w x w global array (w <= 128).  flag[0] is set when a pivot is not positive (the sketch
// has lost rank beyond what the shift covers).
//
// Factorisation: the Schur complement stays in registers (thread (x, y) of 32 x 32 holds
// the entries (y + 32 a, x + 32 b)).  By symmetry the multipliers R_ji of step j are row j
// itself, so one row is all that a step broadcasts: the 32 lanes that own row j + 1 take its
// pivot from a lane, divide by its root and put the row in LDS, one barrier per step (the
// entries left of the diagonal collect values that nothing reads).  Back
// substitution: X_ic = -(sum_{k > i} R_ik X_kc) / R_ii is one FMA chain over k in increasing
// order, R_ik an LDS broadcast and X_kc a row of LDS (X in Rinv itself where both do not
// fit, w > 96), eight terms at a time with the next eight requested across rows; R and X are
// padded with zeros, so no term is conditional.  Both phases are chains of w steps:
// 93 us at w = 74 (492 us with R in global memory, three barriers per step).
template <int NE, bool XL>
__global__ __launch_bounds__(1024) void k_chol_inv(const double* __restrict__ G, int w,
                                                   double shift_rel, double* __restrict__ Rinv,
                                                   int32_t* __restrict__ flag) {
  constexpr int PR = 32 * NE + 8, PX = 32 * NE;            // row pitches
  extern __shared__ __attribute__((aligned(16))) double chol_lds[];
  double* const sR = chol_lds;                             // R: w rows, zeros from column w
  double* const sX = chol_lds + w * PR;                    // X: w + 8 rows, zeros below
  __shared__ double srow[2][kSketchMaxW];
  __shared__ double sdiag[kSketchMaxW];
  const int tid = threadIdx.x, x = tid & 31, y = tid >> 5;
  if (tid < w) sdiag[tid] = G[tid * w + tid];
  double m[NE][NE];
#pragma unroll
  for (int a = 0; a < NE; ++a)
#pragma unroll
    for (int b = 0; b < NE; ++b) {
      const int i = y + 32 * a, c = x + 32 * b;
      m[a][b] = i < w && c < w ? G[i * w + c] : 0.0;
    }
  for (int e = tid; e < w * PR; e += 1024) sR[e] = 0.0;
  if (XL)
    for (int e = tid; e < (w + 8) * PX; e += 1024) sX[e] = 0.0;
  for (int e = tid; e < w * w; e += 1024) Rinv[e] = 0.0;
  __syncthreads();
  double tr = 0.0;
  for (int i = 0; i < w; ++i) tr += sdiag[i];
  const double sh = shift_rel * tr;
#pragma unroll
  for (int a = 0; a < NE; ++a)
    if (x == y) m[a][a] += sh;
  bool bad = false;
  // row i (the NE values r of each of its 32 lanes) scaled by its pivot's root and stored
  auto finish_row = [&](int i, const double (&r)[NE]) {
    double d = 0.0;
#pragma unroll
    for (int b = 0; b < NE; ++b)
      if (b == i / 32) d = readlane_d(r[b], ((i & 1) << 5) | (i & 31));
    const bool ok = d > 0.0;
    bad = bad || !ok;
    const double p = ok ? sqrt(d) : 1.0;
#pragma unroll
    for (int b = 0; b < NE; ++b) {
      const int c = x + 32 * b;
      const double v = c == i ? p : r[b] / p;
      if (c >= i && c < w) {
        srow[i & 1][c] = v;
        sR[i * PR + c] = v;
      }
    }
  };
  if (y == 0) finish_row(0, m[0]);
  __syncthreads();
  for (int j = 0; j + 1 < w; ++j) {
    const double* const row = srow[j & 1];
    const int jn = j + 1;
    double rc[NE];
#pragma unroll
    for (int b = 0; b < NE; ++b) rc[b] = row[x + 32 * b];
    // row j + 1 first: the next step waits for it
    if (y == (jn & 31)) {
      const double l = row[jn];
#pragma unroll
      for (int a = 0; a < NE; ++a)
        if (a == jn / 32) {
#pragma unroll
          for (int b = 0; b < NE; ++b) m[a][b] = __builtin_fma(-l, rc[b], m[a][b]);
          finish_row(jn, m[a]);
        }
    }
#pragma unroll
    for (int a = 0; a < NE; ++a) {
      const int i = y + 32 * a;
      if (i > jn && i < w) {
        const double l = row[i];
#pragma unroll
        for (int b = 0; b < NE; ++b) m[a][b] = __builtin_fma(-l, rc[b], m[a][b]);
      }
    }
    __syncthreads();
  }
  if (bad && x == 0) flag[0] = 1;
  const int wv = tid / kWave;
  if (wv * kWave >= w) return;
  const int c = tid < w ? tid : w - 1;  // a lane past the last column repeats it, not stored
  const int last = __builtin_amdgcn_readfirstlane((wv + 1) * kWave < w ? (wv + 1) * kWave : w) - 1;
  const double xcc = 1.0 / sR[c * PR + c];
  if (XL) {
    if (tid < w) sX[c * PX + c] = xcc;
    double rv[2][8], xv[2][8];
    auto fetch = [&](double (&r)[8], double (&v)[8], int i, int k) {
      const double* const ri = sR + i * PR + k;
      const double* const xk = sX + k * PX + c;
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        r[u] = ri[u];
        v[u] = xk[u * PX];
      }
    };
    double xn = c == last ? xcc : 0.0;  // X_{i+1,c}, formed just before row i needs it
    int i = last - 1, k = last;
    double acc = 0.0, rii = 1.0, rin = 1.0;
    if (i >= 0) {
      fetch(rv[0], xv[0], i, k);
      rii = sR[i * PR + i];
    }
    auto step = [&](double (&r)[8], double (&v)[8], double (&rn)[8], double (&vn)[8]) {
      const bool end = k + 8 > last;  // the row's last eight
      const int i2 = end ? i - 1 : i, k2 = end ? i : k + 8, il = i2 < 0 ? 0 : i2;
      fetch(rn, vn, il, k2);
      rin = sR[il * PR + il];
      if (k == i + 1) v[0] = xn;
#pragma unroll
      for (int u = 0; u < 8; ++u) acc = __builtin_fma(r[u], v[u], acc);
      if (end) {
        const double xi = -acc / rii;
        xn = i < c ? xi : (c == i ? xcc : 0.0);
        if (i < c && tid < w) sX[i * PX + c] = xi;
        acc = 0.0;
        rii = rin;
      }
      i = i2;
      k = k2;
    };
    while (i >= 0) {
      step(rv[0], xv[0], rv[1], xv[1]);
      if (i < 0) break;
      step(rv[1], xv[1], rv[0], xv[0]);
    }
    if (tid < w)
      for (int q = 0; q <= c; ++q) Rinv[q * w + c] = sX[q * PX + c];
  } else {
    if (tid < w) Rinv[c * w + c] = xcc;
    for (int i = last - 1; i >= 0; --i) {
      double acc = 0.0;
      for (int k = i + 1; k <= last; ++k)
        acc = __builtin_fma(sR[i * PR + k], k <= c ? Rinv[k * w + c] : 0.0, acc);
      if (i < c && tid < w) Rinv[i * w + c] = -acc / sR[i * PR + i];
    }
  }
}

// ----------------------------------------------------------------------------- X M
// Q (n x c) = Y (n x w) M (w x c, FP64), optionally |.|, on the FP64 matrix cores (16x16x4):
// M is staged once per workgroup in LDS (rows past w and columns past c are zeros), a
// wavefront takes tiles of 16 rows, NB = ceil(w / 16) blocks of columns (c <= w).  Lane l (row
// l % 16, group g = l / 16) supplies the values k = 4 s + g of its row in k-step s; a whole
// tile is requested at once, one tile ahead.  The instruction is one FMA chain over its
// four k, so an entry is the chain over k in increasing order.  Bound by the FP64 matrix
// rate (31 us at n = 200000, w = c = 74; 24 us for the bytes at copy rate): 58 us
// (222 us on the vector units, one row per four threads).
template <typename T, int NB>
__global__ __launch_bounds__(512) void k_tsmm(const T* __restrict__ Y, int64_t n, int w,
                                              const double* __restrict__ M, int c, int absval,
                                              T* __restrict__ Q) {
  constexpr int NS = 4 * NB;                        // k-steps, ceil(w / 16) blocks of four
  constexpr int pitch = NB % 2 ? 16 * NB : 16 * NB + 16;  // 32 mod 64 words
  extern __shared__ __attribute__((aligned(16))) double tsmm_m[];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  {
    constexpr int NE = 4 * NS * pitch, NL = (NE + 511) / 512;
    double t[NL];  // every load requested before the first is used
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int e = tid + 512 * i, k = e / pitch, j = e - k * pitch;
      t[i] = M[k < w && j < c ? k * c + j : 0];
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int e = tid + 512 * i, k = e / pitch, j = e - k * pitch;
      if (e < NE) tsmm_m[e] = k < w && j < c ? t[i] : 0.0;
    }
  }
  __syncthreads();
  const int r16 = lane & 15, g = lane >> 4;
  const int64_t ntile = (n + 15) / 16, step = (int64_t)gridDim.x * 8;
  T y[NS], yn[NS];
  auto load = [&](T (&t)[NS], int64_t tile) {
    const int64_t row = tile * 16 + r16;
    const T* __restrict__ yr = Y + (row < n ? row : n - 1) * w;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int k = 4 * s + g;
      t[s] = yr[s < NS - 4 || k < w ? k : 0];
    }
  };
  int64_t tile = (int64_t)blockIdx.x * 8 + wave;
  if (tile >= ntile) return;
  load(y, tile);
  for (; tile < ntile; tile += step) {
    load(yn, tile + step < ntile ? tile + step : tile);
    asm volatile("" ::: "memory");  // M is read again from LDS: kept in registers it spills
    sd4 acc[NB];
#pragma unroll
    for (int q = 0; q < NB; ++q) acc[q] = sd4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const double a = s < NS - 4 || 4 * s + g < w ? (double)y[s] : 0.0;
      const double* __restrict__ mr = tsmm_m + (4 * s + g) * pitch + r16;
#pragma unroll
      for (int q = 0; q < NB; ++q)
        acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, mr[16 * q], acc[q], 0, 0, 0);
    }
#pragma unroll
    for (int q = 0; q < NB; ++q)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t i = tile * 16 + g + 4 * v;
        const int j = 16 * q + r16;
        if (i < n && j < c) Q[i * c + j] = (T)(absval ? fabs(acc[q][v]) : acc[q][v]);
      }
#pragma unroll
    for (int s = 0; s < NS; ++s) y[s] = yn[s];
  }
}

// ----------------------------------------------------------------------------- Jacobi
// Eigen-decomposition S = V diag(ev) V^T of S = (Tin + Tin^T) / 2 (w x w, FP64) by cyclic
// Jacobi rotations.  A sweep runs w' - 1 rounds (w' = w rounded up to even) of w'/2
// disjoint pairs in the round-robin order: player 0 stays, players 1 .. w'-1 rotate, and
// pairs holding the padding player w are skipped.  For pair (p, q) the rotation
// c = 1/sqrt(1 + t^2), s = t c, t = sgn(th) / (|th| + sqrt(th^2 + 1)),
// th = (a_qq - a_pp) / (2 a_pq) zeroes a_pq; all rotations of a round update the rows
// first, then the columns and V (the pairs are disjoint, so this is their product).
// Sweeps stop when the off-diagonal part is below 1e-15 of the matrix (Frobenius) or
// after 50 sweeps.
//
// k_jacobi runs the rotations on the matrix alone, one workgroup, the matrix in LDS (w <=
// 128): a round is the w'/2 rotations and then the 2 x 2 blocks (t, u), t <= u, of the pairs
// t and u, each by one thread, mirrored to (u, t); it records every round's (c, s) and
// their number.  k_jacobi_vec then applies them to V, whose rows are independent: one
// wavefront per row, no barrier.  Bound by the chain of rounds (some ten sweeps of w' - 1):
// 515 + 102 us at w = 74 for both (7.9 ms with the matrix and V in global memory).
__device__ __forceinline__ void jacobi_pair(int t, int round, int m, int& p, int& q) {
  const int a = t == 0 ? 0 : ((t - 1 + round) % (m - 1)) + 1;
  const int b = ((m - 2 - t + round) % (m - 1)) + 1;
  p = a < b ? a : b;
  q = a < b ? b : a;
}

constexpr int kJacobiThreads = 1024;
__global__ __launch_bounds__(kJacobiThreads) void k_jacobi(const double* __restrict__ Tin, int w,
                                                           double2* __restrict__ rot,
                                                           int* __restrict__ nrounds,
                                                           double* __restrict__ ev) {
  extern __shared__ __attribute__((aligned(16))) double jac_a[];  // m x (m + 1)
  __shared__ double s_c[kSketchMaxW / 2], s_s[kSketchMaxW / 2];
  __shared__ int s_p[kSketchMaxW / 2], s_q[kSketchMaxW / 2];
  __shared__ double sred[2 * (kJacobiThreads / kWave)];
  const int tid = threadIdx.x;
  const int m = w < 2 ? 2 : (w + 1) & ~1, np = m / 2, ld = m + 1;
  double* A = jac_a;
  for (int e = tid; e < m * m; e += kJacobiThreads) {
    const int i = e / m, j = e - i * m;
    A[i * ld + j] = i < w && j < w ? 0.5 * (Tin[i * w + j] + Tin[j * w + i]) : 0.0;
  }
  // the blocks (t, u), t <= u, of this thread: numbers tid, tid + 1024, ... row by row
  constexpr int MB = (kSketchMaxW / 2 * (kSketchMaxW / 2 + 1) / 2 + kJacobiThreads - 1) / kJacobiThreads;
  int bt[MB], bu[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    int e = tid + i * kJacobiThreads, t = 0;
    if (e >= np * (np + 1) / 2) {
      bt[i] = -1;
      bu[i] = 0;
      continue;
    }
    while (e >= np - t) {
      e -= np - t;
      ++t;
    }
    bt[i] = t;
    bu[i] = t + e;
  }
  // the players of pair tid, round 0; a sweep is a full turn
  int pa = tid == 0 ? 0 : tid, pb = m - 1 - tid;
  int done = 0;
  __syncthreads();
  for (int sweep = 0; sweep < 50; ++sweep) {
    double off = 0.0, tot = 0.0;
    for (int e = tid; e < w * w; e += kJacobiThreads) {
      const int i = e / w, j = e - i * w;
      const double a = A[i * ld + j];
      tot = __builtin_fma(a, a, tot);
      if (i != j) off = __builtin_fma(a, a, off);
    }
    off = wave_sum(off);
    tot = wave_sum(tot);
    if ((tid & 63) == 0) {
      sred[2 * (tid >> 6)] = off;
      sred[2 * (tid >> 6) + 1] = tot;
    }
    __syncthreads();
    double o2 = 0.0, t2 = 0.0;
    for (int q = 0; q < kJacobiThreads / kWave; ++q) {
      o2 += sred[2 * q];
      t2 += sred[2 * q + 1];
    }
    if (!(o2 > 1e-30 * t2)) break;  // the same sums in every thread
    for (int round = 0; round < m - 1; ++round) {
      if (tid < np) {
        const int p = pa < pb ? pa : pb, q = pa < pb ? pb : pa;
        if (tid > 0) pa = pa == m - 1 ? 1 : pa + 1;  // the players move on
        pb = pb == m - 1 ? 1 : pb + 1;
        double c = 1.0, s = 0.0;
        if (q < w) {
          const double apq = A[p * ld + q];
          if (apq != 0.0) {
            const double th = (A[q * ld + q] - A[p * ld + p]) / (2.0 * apq);
            const double at = fabs(th), h = __builtin_fma(th, th, 1.0);
            // roots by the refined hardware estimate: the chain of divisions and roots is
            // half of a round; beyond 1e150 th^2 overflows and t = 1 / (2 th)
            const double t = at < 1e150 ? (th >= 0.0 ? 1.0 : -1.0) / __builtin_fma(h, rsqrt_nr(h), at)
                                        : 0.5 / th;
            c = rsqrt_nr(__builtin_fma(t, t, 1.0));
            s = t * c;
          }
        }
        s_c[tid] = c;
        s_s[tid] = s;
        s_p[tid] = p;
        s_q[tid] = q;
        rot[(size_t)done * np + tid] = make_double2(c, s);
      }
      ++done;
      __syncthreads();
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        if (bt[i] < 0) continue;
        const int t = bt[i], u = bu[i];
        const int p = s_p[t], q = s_q[t], g = s_p[u], h = s_q[u];
        const double ct = s_c[t], st = s_s[t], cu = s_c[u], su = s_s[u];
        const double a00 = A[p * ld + g], a01 = A[p * ld + h];
        const double a10 = A[q * ld + g], a11 = A[q * ld + h];
        const double b00 = ct * a00 - st * a10, b01 = ct * a01 - st * a11;
        const double b10 = st * a00 + ct * a10, b11 = st * a01 + ct * a11;
        const double d00 = cu * b00 - su * b01, d01 = su * b00 + cu * b01;
        const double d10 = cu * b10 - su * b11, d11 = su * b10 + cu * b11;
        A[p * ld + g] = d00;
        A[p * ld + h] = d01;
        A[q * ld + g] = d10;
        A[q * ld + h] = d11;
        if (t != u) {
          A[g * ld + p] = d00;
          A[h * ld + p] = d01;
          A[g * ld + q] = d10;
          A[h * ld + q] = d11;
        }
      }
      __syncthreads();
    }
  }
  for (int i = tid; i < w; i += kJacobiThreads) ev[i] = A[i * ld + i];
  if (tid == 0) nrounds[0] = done;
}

__global__ __launch_bounds__(kWave) void k_jacobi_vec(const double2* __restrict__ rot,
                                                      const int* __restrict__ nrounds, int w,
                                                      double* __restrict__ V) {
  __shared__ double v[kSketchMaxW];
  constexpr int U = 8;  // rounds of rotations requested at once
  const int lane = threadIdx.x, i = blockIdx.x;
  const int m = w < 2 ? 2 : (w + 1) & ~1, np = m / 2;
  for (int j = lane; j < m; j += kWave) v[j] = j == i ? 1.0 : 0.0;
  __builtin_amdgcn_wave_barrier();
  const int nr = nrounds[0], mine = lane < np ? lane : 0;
  int round = 0;
  for (int k0 = 0; k0 < nr; k0 += U) {
    double2 cs[U];
#pragma unroll
    for (int u = 0; u < U; ++u) cs[u] = rot[(size_t)(k0 + u < nr ? k0 + u : nr - 1) * np + mine];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (k0 + u >= nr) continue;
      int p, q;
      jacobi_pair(mine, round, m, p, q);
      const double a = v[p], b = v[q];
      __builtin_amdgcn_wave_barrier();
      if (lane < np && q < w) {
        v[p] = cs[u].x * a - cs[u].y * b;
        v[q] = cs[u].y * a + cs[u].x * b;
      }
      __builtin_amdgcn_wave_barrier();
      round = round + 1 == m - 1 ? 0 : round + 1;
    }
  }
  for (int j = lane; j < w; j += kWave) V[i * w + j] = v[j];
}

// ----------------------------------------------------------------------------- selection
// The k eigenpairs of largest |ev| (ties: lower index first): lam[j] = ev[o_j] and
// M[a][j] = V[a][o_j], times sqrt(|ev[o_j]|) when sqrt_scale is set.  One workgroup.
__global__ __launch_bounds__(kThreads) void k_sketch_select(const double* __restrict__ ev,
                                                            const double* __restrict__ V, int w,
                                                            int k, int sqrt_scale,
                                                            double* __restrict__ lam,
                                                            double* __restrict__ M) {
  __shared__ int order[kSketchMaxW];
  // every slot holds a valid index even if a non-finite eigenvalue breaks the ranking
  for (int i = threadIdx.x; i < kSketchMaxW; i += kThreads) order[i] = i < w ? i : 0;
  __syncthreads();
  for (int i = threadIdx.x; i < w; i += kThreads) {
    const double ai = fabs(ev[i]);
    int rank = 0;
    for (int j = 0; j < w; ++j) {
      const double aj = fabs(ev[j]);
      rank += (aj > ai) || (aj == ai && j < i);
    }
    if (rank < k) order[rank] = i;
  }
  __syncthreads();
  if (lam)
    for (int j = threadIdx.x; j < k; j += kThreads) lam[j] = ev[order[j]];
  for (int e = threadIdx.x; e < w * k; e += kThreads) {
    const int a = e / k, j = e - a * k;
    double v = V[a * w + order[j]];
    if (sqrt_scale) v *= sqrt(fabs(ev[order[j]]));
    M[e] = v;
  }
}

// ----------------------------------------------------------------------------- launchers
template <typename T>
void launch_sketch_spmm(const int64_t* rowptr, const int32_t* col, const T* val, const T* X,
                        int64_t n, int w, T* Y, hipStream_t s) {
  int64_t nb = (n + 3) / 4;
  if (nb > 8192) nb = 8192;
  if (nb < 1) nb = 1;
  // rows of X start on even elements of an aligned X: two columns per load
  if (w % 2 == 0 && (uintptr_t)X % (2 * sizeof(T)) == 0)
    hipLaunchKernelGGL((k_spmm_wide<T, 2>), dim3((unsigned)nb), dim3(kThreads), 0, s, rowptr, col,
                       val, X, n, w, Y);
  else
    hipLaunchKernelGGL((k_spmm_wide<T, 1>), dim3((unsigned)nb), dim3(kThreads), 0, s, rowptr, col,
                       val, X, n, w, Y);
}
template <typename T>
void launch_sketch_dense(const T* A, int64_t ld, const T* X, int64_t n, int w, T* Y,
                         hipStream_t s) {
  hipLaunchKernelGGL(k_dense_wide<T>, dim3((unsigned)((n + 63) / 64)), dim3(kThreads), 0, s, A, ld,
                     X, n, w, Y);
}
int sketch_slabs(int64_t n, int64_t* rows_per) {
  int64_t rp = (n + 255) / 256;
  if (rp < 256) rp = 256;
  *rows_per = rp;
  return (int)((n + rp - 1) / rp);
}
template <typename T, bool SYM>
static void tsgram_slabs(const T* X, const T* Y, int64_t n, int w, int nslab, int64_t rp,
                         double* part, hipStream_t s) {
  auto go = [&](auto nbc) {
    constexpr int NB = decltype(nbc)::value;
    constexpr size_t lds = TsGram<NB, SYM>::LDS;
    if (lds > 64 * 1024)
      (void)hipFuncSetAttribute((const void*)k_tsgram<T, NB, SYM>,
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL((k_tsgram<T, NB, SYM>), dim3((unsigned)nslab), dim3(512), lds, s, X, Y, n,
                       w, rp, part);
  };
  switch ((w + 15) / 16) {
    case 1: go(std::integral_constant<int, 1>{}); break;
    case 2: go(std::integral_constant<int, 2>{}); break;
    case 3: go(std::integral_constant<int, 3>{}); break;
    case 4: go(std::integral_constant<int, 4>{}); break;
    case 5: go(std::integral_constant<int, 5>{}); break;
    case 6: go(std::integral_constant<int, 6>{}); break;
    case 7: go(std::integral_constant<int, 7>{}); break;
    default: go(std::integral_constant<int, 8>{});
  }
}
template <typename T>
void launch_tsgram(const T* X, const T* Y, int64_t n, int w, double* part, double* C,
                   hipStream_t s) {
  int64_t rp = 0;
  const int nb = sketch_slabs(n, &rp);
  if (X == Y)
    tsgram_slabs<T, true>(X, Y, n, w, nb, rp, part, s);
  else
    tsgram_slabs<T, false>(X, Y, n, w, nb, rp, part, s);
  hipLaunchKernelGGL(k_tsgram_reduce, dim3((unsigned)((w * w + 15) / 16)), dim3(kThreads), 0, s,
                     (const double*)part, nb, w * w, C);
}
template <int NE>
static void chol_blocks(const double* G, int w, double shift_rel, double* Rinv, int32_t* flag,
                        hipStream_t s) {
  const size_t lr = (size_t)w * (32 * NE + 8) * 8, lx = (size_t)(w + 8) * 32 * NE * 8;
  const bool xl = lr + lx <= 156 * 1024;  // 160 KB of LDS less the static rows
  const size_t lds = lr + (xl ? lx : 0);
  const void* const k = xl ? (const void*)k_chol_inv<NE, true> : (const void*)k_chol_inv<NE, false>;
  if (lds > 60 * 1024)
    (void)hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (xl)
    hipLaunchKernelGGL((k_chol_inv<NE, true>), dim3(1), dim3(1024), lds, s, G, w, shift_rel, Rinv,
                       flag);
  else
    hipLaunchKernelGGL((k_chol_inv<NE, false>), dim3(1), dim3(1024), lds, s, G, w, shift_rel, Rinv,
                       flag);
}
void launch_chol_inv(const double* G, int w, double shift_rel, double* Rinv, int32_t* flag,
                     hipStream_t s) {
  switch ((w + 31) / 32) {
    case 1: chol_blocks<1>(G, w, shift_rel, Rinv, flag, s); break;
    case 2: chol_blocks<2>(G, w, shift_rel, Rinv, flag, s); break;
    case 3: chol_blocks<3>(G, w, shift_rel, Rinv, flag, s); break;
    default: chol_blocks<4>(G, w, shift_rel, Rinv, flag, s);
  }
}
template <typename T, int NB>
static void tsmm_blocks(const T* Y, int64_t n, int w, const double* M, int c, int absval, T* Q,
                        hipStream_t s) {
  const size_t lds = (size_t)16 * NB * (NB % 2 ? 16 * NB : 16 * NB + 16) * 8;
  if (lds > 64 * 1024)
    (void)hipFuncSetAttribute((const void*)k_tsmm<T, NB>,
                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  // two workgroups per CU share the tiles (M is staged once per workgroup)
  int64_t nb = (n + 127) / 128;
  if (nb > 512) nb = 512;
  hipLaunchKernelGGL((k_tsmm<T, NB>), dim3((unsigned)nb), dim3(512), lds, s, Y, n, w, M, c, absval,
                     Q);
}
template <typename T>
void launch_tsmm(const T* Y, int64_t n, int w, const double* M, int c, int absval, T* Q,
                 hipStream_t s) {
  switch ((w + 15) / 16) {  // c <= w
    case 1: tsmm_blocks<T, 1>(Y, n, w, M, c, absval, Q, s); break;
    case 2: tsmm_blocks<T, 2>(Y, n, w, M, c, absval, Q, s); break;
    case 3: tsmm_blocks<T, 3>(Y, n, w, M, c, absval, Q, s); break;
    case 4: tsmm_blocks<T, 4>(Y, n, w, M, c, absval, Q, s); break;
    case 5: tsmm_blocks<T, 5>(Y, n, w, M, c, absval, Q, s); break;
    case 6: tsmm_blocks<T, 6>(Y, n, w, M, c, absval, Q, s); break;
    case 7: tsmm_blocks<T, 7>(Y, n, w, M, c, absval, Q, s); break;
    default: tsmm_blocks<T, 8>(Y, n, w, M, c, absval, Q, s);
  }
}
size_t jacobi_rot_bytes(int w) {
  const int m = w < 2 ? 2 : (w + 1) & ~1;
  return (size_t)50 * (m - 1) * (m / 2) * sizeof(double2) + 256;
}
void launch_jacobi(const double* Tin, int w, void* rot, double* V, double* ev, hipStream_t s) {
  const int m = w < 2 ? 2 : (w + 1) & ~1;
  const size_t lds = (size_t)m * (m + 1) * 8;
  if (lds > 60 * 1024)
    (void)hipFuncSetAttribute((const void*)k_jacobi, hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)lds);
  int* nr = (int*)rot;
  double2* cs = (double2*)((char*)rot + 256);
  hipLaunchKernelGGL(k_jacobi, dim3(1), dim3(kJacobiThreads), lds, s, Tin, w, cs, nr, ev);
  hipLaunchKernelGGL(k_jacobi_vec, dim3(w), dim3(kWave), 0, s, (const double2*)cs,
                     (const int*)nr, w, V);
}
void launch_sketch_select(const double* ev, const double* V, int w, int k, int sqrt_scale,
                          double* lam, double* M, hipStream_t s) {
  hipLaunchKernelGGL(k_sketch_select, dim3(1), dim3(kThreads), 0, s, ev, V, w, k, sqrt_scale, lam,
                     M);
}

#define SNMF_SKETCH_INST(T)                                                                       \
  template void launch_sketch_spmm<T>(const int64_t*, const int32_t*, const T*, const T*, int64_t, \
                                      int, T*, hipStream_t);                                      \
  template void launch_sketch_dense<T>(const T*, int64_t, const T*, int64_t, int, T*,             \
                                       hipStream_t);                                              \
  template void launch_tsgram<T>(const T*, const T*, int64_t, int, double*, double*, hipStream_t); \
  template void launch_tsmm<T>(const T*, int64_t, int, const double*, int, int, T*, hipStream_t);
SNMF_SKETCH_INST(float)
SNMF_SKETCH_INST(double)

}  // namespace snmf
