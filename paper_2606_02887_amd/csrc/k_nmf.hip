// Kernels of NMPBB for rectangular NMF (eq. (1.1)): the products V P and V^T P of a dense
// m x n matrix with an n x r or m x r partner, and the transpose of a CSR matrix (column
// counts, their scan, the scatter and a per-row sort that makes the result deterministic).
#include "common.hpp"
#include "kernels.hpp"
#include "rho.hpp"

namespace snmf {

// B (rows x r) = V P (trans = 0: V is rows x K, row-major, leading dimension ld) or V^T P
// (trans = 1: V is K x rows).  64 output rows per workgroup, K in chunks of 32 staged in
// LDS; thread t owns row t % 64 and columns t / 64 + 4 q; accumulation in T, K in order.
// Skipped when the solve is done.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_rect_apass(const T* __restrict__ V, int64_t ld,
                                                         int64_t rows, int64_t K, int trans,
                                                         const T* __restrict__ P, int r,
                                                         T* __restrict__ B,
                                                         const State* __restrict__ st) {
  if (st->done) return;
  __shared__ T sA[64][33];
  __shared__ T sP[32][kMaxRank];
  const int t = threadIdx.x, rr = t & 63, cg = t >> 6;
  const int64_t row0 = (int64_t)blockIdx.x * 64;
  T acc[kMaxRank / 4];
#pragma unroll
  for (int q = 0; q < kMaxRank / 4; ++q) acc[q] = T(0);
  for (int64_t k0 = 0; k0 < K; k0 += 32) {
    __syncthreads();
    for (int e = t; e < 64 * 32; e += kThreads) {
      int i, kk;
      if (trans) {  // consecutive threads read consecutive entries of one row of V
        kk = e >> 6;
        i = e & 63;
      } else {
        i = e >> 5;
        kk = e & 31;
      }
      const int64_t gi = row0 + i, gk = k0 + kk;
      T a = T(0);
      if (gi < rows && gk < K) a = trans ? V[gk * ld + gi] : V[gi * ld + gk];
      sA[i][kk] = a;
    }
    for (int e = t; e < 32 * r; e += kThreads) {
      const int kk = e / r, c = e - kk * r;
      const int64_t gk = k0 + kk;
      sP[kk][c] = gk < K ? P[gk * r + c] : T(0);
    }
    __syncthreads();
    for (int kk = 0; kk < 32; ++kk) {
      const T a = sA[rr][kk];
#pragma unroll
      for (int q = 0; q < kMaxRank / 4; ++q) {
        const int c = cg + 4 * q;
        if (c < r) acc[q] += a * sP[kk][c];
      }
    }
  }
  const int64_t gi = row0 + rr;
  if (gi < rows) {
#pragma unroll
    for (int q = 0; q < kMaxRank / 4; ++q) {
      const int c = cg + 4 * q;
      if (c < r) B[gi * r + c] = acc[q];
    }
  }
}

// CSR of m rows with columns in [0, ncols): flags[0] += bad row pointers, flags[1] +=
// columns out of range, flags[2] += columns not strictly increasing within a row.
__global__ __launch_bounds__(kThreads) void k_csr_check_rect(const int64_t* __restrict__ rowptr,
                                                             const int32_t* __restrict__ col,
                                                             int64_t m, int64_t ncols,
                                                             int64_t nnz,
                                                             unsigned* __restrict__ flags) {
  unsigned bp = 0, bc = 0, us = 0;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < m;
       i += (int64_t)gridDim.x * kThreads) {
    const int64_t b = rowptr[i], e = rowptr[i + 1];
    if (b < 0 || e < b || e > nnz) {
      ++bp;
      continue;
    }
    int32_t prev = -1;
    for (int64_t z = b; z < e; ++z) {
      const int32_t c = col[z];
      if (c < 0 || c >= ncols) ++bc;
      if (c <= prev) ++us;
      prev = c;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0 && (rowptr[0] != 0 || rowptr[m] != nnz))
    atomicAdd(&flags[0], 1u);
  if (bp) atomicAdd(&flags[0], bp);
  if (bc) atomicAdd(&flags[1], bc);
  if (us) atomicAdd(&flags[2], us);
}

// cnt[c] = entries of column c.
__global__ __launch_bounds__(kThreads) void k_csr_colcount(const int32_t* __restrict__ col,
                                                           int64_t nnz,
                                                           unsigned* __restrict__ cnt) {
  const int64_t z = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (z < nnz) atomicAdd(&cnt[col[z]], 1u);
}

// out[0] = 0, out[i + 1] = out[i] + cnt[i] (one workgroup: chunk sums scanned in thread
// order), and cursor[i] = out[i].
__global__ __launch_bounds__(kThreads) void k_scan_counts(const unsigned* __restrict__ cnt,
                                                          int64_t n, int64_t* __restrict__ out,
                                                          unsigned long long* __restrict__ cursor) {
  __shared__ int64_t tot[kThreads];
  const int64_t chunk = (n + kThreads - 1) / kThreads;
  const int64_t b = (int64_t)threadIdx.x * chunk;
  const int64_t e = b + chunk < n ? b + chunk : n;
  int64_t s = 0;
  for (int64_t i = b; i < e; ++i) s += cnt[i];
  tot[threadIdx.x] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    int64_t run = 0;
    for (int q = 0; q < kThreads; ++q) {
      const int64_t v = tot[q];
      tot[q] = run;
      run += v;
    }
    out[n] = run;
  }
  __syncthreads();
  int64_t run = tot[threadIdx.x];
  for (int64_t i = b; i < e; ++i) {
    out[i] = run;
    cursor[i] = (unsigned long long)run;
    run += cnt[i];
  }
}

// Entry (i, c, v) of V goes to row c of V^T at the next free place of that row.
template <typename T>
__global__ __launch_bounds__(kThreads) void k_csr_scatter_t(const int64_t* __restrict__ rowptr,
                                                            const int32_t* __restrict__ col,
                                                            const T* __restrict__ val, int64_t m,
                                                            unsigned long long* __restrict__ cursor,
                                                            int32_t* __restrict__ colT,
                                                            T* __restrict__ valT) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= m) return;
  for (int64_t z = rowptr[i]; z < rowptr[i + 1]; ++z) {
    const unsigned long long p = atomicAdd(&cursor[col[z]], 1ull);
    colT[p] = (int32_t)i;
    valT[p] = val[z];
  }
}

// Sort every row of V^T by column, values alongside (one thread per row; the rows' column
// indices are distinct, so the result is unique).
template <typename T>
__global__ __launch_bounds__(kThreads) void k_csr_sort_pairs(const int64_t* __restrict__ rowptr,
                                                             int64_t n, int32_t* __restrict__ col,
                                                             T* __restrict__ val) {
  const int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (i >= n) return;
  const int64_t b = rowptr[i], e = rowptr[i + 1];
  for (int64_t a = b + 1; a < e; ++a) {
    const int32_t c = col[a];
    const T v = val[a];
    int64_t q = a - 1;
    while (q >= b && col[q] > c) {
      col[q + 1] = col[q];
      val[q + 1] = val[q];
      --q;
    }
    col[q + 1] = c;
    val[q + 1] = v;
  }
}

// ----------------------------------------------------------------------------- FP32 MFMA
typedef float f32x16n __attribute__((ext_vector_type(16)));

// Split-K panels of V^T P (the H-step) and V P (the W-step): panel y of the N x r product
// holds the sums over k in chunk y (kchunk rows of P, a multiple of 16), every sum in
// increasing k on v_mfma_f32_32x32x2f32.  The general path is that of the symmetric A-pass
// (k_apass_dense.hip), with a transposed copy of V for the W-step; for r in (32, 64] and
// aligned V these wide kernels serve both from V itself.  A wave computes 128 output rows and
// all ranks (rank m = 2 c + b in M-block b: P is loaded two ranks at a time), so a k-pair
// feeds 8 MFMAs from one 16-byte load of V (the general kernel: 4 from two 4-byte loads);
// 16 k (ROWS: 8) per batch, the next batch in flight during this one's 64 (32) MFMAs, one
// load among every few MFMAs.  Two wavefronts' registers fit a SIMD, so that the workgroup of rho finds a place
// beside a tile workgroup (with 288 registers the last tile waited for it: 106 us).
// ROWS = false (V^T P): lane (c, h) = (lane % 32, lane / 32) loads V[k + h][j0 + 4c .. +3],
// column block q = rows j0 + 4c + q of the product.
// ROWS = true (V P): lane c reads 8 consecutive k of row j0 + 32 q + c of V, both halves of
// the wave the same 32 bytes; half h takes the k of its parity.
// With rj.G set the grid has one more row of workgroups, the first, whose first workgroup
// computes rho = ||G||_2 (rho.hpp).  Skipped when the solve is done.
// V 8192 x 4096, r = 64: V^T P 47, V P 59 us (FP32 matrix rate 28, V from memory 27, the
// panels' stores 7 and more), up to 88 beside a rho of all r steps (52 alone); the general
// kernel took 74 and 97 us, the transposed copy 58 us and 134 MB per call.
typedef float f32x4n __attribute__((ext_vector_type(4)));

template <bool ROWS>
__global__ __launch_bounds__(256, 2) void k_rect_f32w(const float* __restrict__ V, int64_t ld,
                                                      const float* __restrict__ P, int64_t K,
                                                      int64_t N, int r, int64_t kchunk,
                                                      float* __restrict__ Bpart, int64_t pstride,
                                                      const State* __restrict__ st, RhoJob rj) {
  if (st->done) return;
  int64_t y = blockIdx.y;
  if (rj.G) {
    if (y == 0) {
      if (blockIdx.x == 0) rho_body(rj.G, rj.r, rj.st);
      return;
    }
    --y;
  }
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 31, h = lane >> 5;
  const int64_t j0 = ((int64_t)blockIdx.x * 4 + wave) * 128;
  if (j0 >= N) return;
  const int64_t kb = y * kchunk;
  const int64_t ke = kb + kchunk < K ? kb + kchunk : K;
  f32x16n acc[2][4];
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[mb][nb][v] = 0.0f;
  // rows and ranks out of range read a clamped, valid address; they are never stored
  const float* prow = P + (2 * c + 1 < r ? 2 * c : 0);
  const float* vrow[ROWS ? 4 : 1];
  if constexpr (ROWS) {
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
      const int64_t j = j0 + 32 * nb + c;
      vrow[nb] = V + (j < N ? j : N - 1) * ld;
    }
  } else {
    vrow[0] = V + (j0 + 4 * c + 3 < N ? j0 + 4 * c : N - 4);  // N % 4 == 0 here
  }
  constexpr int U = ROWS ? 4 : 8;  // k-pairs per batch
  struct Batch {
    f32x4n x[ROWS ? 2 * U : U];
    float2 p[U];
  } qa, qb;
  auto load = [&](Batch& q, int64_t k0) __attribute__((always_inline)) {
    if constexpr (ROWS) {
#pragma unroll
      for (int t = 0; t < U / 2; ++t)
#pragma unroll
        for (int nb = 0; nb < 4; ++nb) q.x[4 * t + nb] = *(const f32x4n*)(vrow[nb] + k0 + 4 * t);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t kk = k0 + 2 * u + h;
      if constexpr (!ROWS) q.x[u] = __builtin_nontemporal_load((const f32x4n*)(vrow[0] + kk * ld));
      q.p[u] = *(const float2*)(prow + kk * r);
    }
  };
  auto mma = [&](const Batch& q) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float pv[2] = {q.p[u].x, q.p[u].y};
#pragma unroll
      for (int nb = 0; nb < 4; ++nb) {
        float a;
        if constexpr (ROWS) {
          const f32x4n x = q.x[4 * (u >> 1) + nb];
          a = h ? x[2 * (u & 1) + 1] : x[2 * (u & 1)];
        } else {
          a = q.x[u][nb];
        }
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
          acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(pv[mb], a, acc[mb][nb], 0, 0, 0);
      }
    }
  };
  const int64_t nbat = ke > kb ? (ke - kb) / (2 * U) : 0;
  const int64_t klast = kb + (nbat > 0 ? nbat - 1 : 0) * 2 * U;
  int64_t k = kb, b = 0;
  if (nbat > 0) load(qa, k);
  for (; b + 2 <= nbat; b += 2) {
    // a prefetch past the last batch reads the last one again: no load is conditional
    load(qb, k + 2 * U);
    mma(qa);
    load(qa, k + 4 * U < klast ? k + 4 * U : klast);
    mma(qb);
    k += 4 * U;
#pragma unroll
    for (int i = 0; i < 2 * U; ++i) {
      if constexpr (ROWS) {
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);  // a load, MFMAs
        __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
      } else {
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
      }
    }
  }
  if (b < nbat) {
    mma(qa);
    k += 2 * U;
  }
  for (; k < ke; k += 2) {  // the end of K
    const int64_t kk = k + h;
    const bool kin = kk < ke;
    const int64_t kc = kin ? kk : ke - 1;
    float2 p = *(const float2*)(prow + kc * r);
    f32x4n x;
    if constexpr (ROWS) {
#pragma unroll
      for (int nb = 0; nb < 4; ++nb) x[nb] = vrow[nb][kc];
    } else {
      x = *(const f32x4n*)(vrow[0] + kc * ld);
    }
    const float pv[2] = {kin ? p.x : 0.0f, kin ? p.y : 0.0f};
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
      const float a = kin ? x[nb] : 0.0f;
#pragma unroll
      for (int mb = 0; mb < 2; ++mb)
        acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x2f32(pv[mb], a, acc[mb][nb], 0, 0, 0);
    }
  }
  // D[row][column]: lane (c, h) holds column c and row 8 (v / 4) + 4 h + v % 4 of a block in
  // register v; rows v, v + 1 of both M-blocks are four consecutive ranks
  float* out = Bpart + y * pstride;
#pragma unroll
  for (int nb = 0; nb < 4; ++nb) {
    const int64_t j = ROWS ? j0 + 32 * nb + c : j0 + 4 * c + nb;
    if (j >= N) continue;
#pragma unroll
    for (int v = 0; v < 16; v += 2) {
      const int m = 2 * (8 * (v >> 2) + 4 * h + (v & 3));
      const float o[4] = {acc[0][nb][v], acc[1][nb][v], acc[0][nb][v + 1], acc[1][nb][v + 1]};
      if (m + 3 < r) __builtin_memcpy(out + j * r + m, o, 16);
      else if (m + 1 < r) __builtin_memcpy(out + j * r + m, o, 8);
    }
  }
}

// AT (cols x rows) = A^T for A rows x cols (leading dimension lda): 64 x 64 tiles through
// LDS, reads and writes along rows.
template <typename T>
__global__ __launch_bounds__(256) void k_transpose(const T* __restrict__ A, int64_t rows,
                                                   int64_t cols, int64_t lda, T* __restrict__ AT) {
  __shared__ T t[64][65];
  const int64_t r0 = (int64_t)blockIdx.y * 64, c0 = (int64_t)blockIdx.x * 64;
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  for (int i = ty; i < 64; i += 4) {
    const int64_t rr = r0 + i, cc = c0 + tx;
    t[i][tx] = (rr < rows && cc < cols) ? A[rr * lda + cc] : T(0);
  }
  __syncthreads();
  for (int i = ty; i < 64; i += 4) {
    const int64_t cc = c0 + i, rr = r0 + tx;
    if (cc < cols && rr < rows) AT[cc * rows + rr] = t[tx][i];
  }
}

static unsigned nblk(int64_t m) {
  int64_t b = (m + kThreads - 1) / kThreads;
  return (unsigned)(b < 1 ? 1 : b);
}

template <typename T>
void launch_rect_apass(const T* V, int64_t ld, int64_t rows, int64_t K, int trans, const T* P,
                       int r, T* B, const State* st, hipStream_t s) {
  hipLaunchKernelGGL(k_rect_apass<T>, dim3((unsigned)((rows + 63) / 64)), dim3(kThreads), 0, s, V,
                     ld, rows, K, trans, P, r, B, st);
}

void launch_csr_check_rect(const int64_t* rowptr, const int32_t* col, int64_t m, int64_t ncols,
                           int64_t nnz, unsigned* flags, hipStream_t s) {
  unsigned b = nblk(m);
  if (b > 4096) b = 4096;
  hipLaunchKernelGGL(k_csr_check_rect, dim3(b), dim3(kThreads), 0, s, rowptr, col, m, ncols, nnz,
                     flags);
}

template <typename T>
void launch_csr_transpose(const int64_t* rowptr, const int32_t* col, const T* val, int64_t m,
                          int64_t ncols, int64_t nnz, unsigned* cnt, unsigned long long* cursor,
                          int64_t* rowptrT, int32_t* colT, T* valT, hipStream_t s) {
  (void)hipMemsetAsync(cnt, 0, (size_t)ncols * sizeof(unsigned), s);
  if (nnz > 0)
    hipLaunchKernelGGL(k_csr_colcount, dim3(nblk(nnz)), dim3(kThreads), 0, s, col, nnz, cnt);
  hipLaunchKernelGGL(k_scan_counts, dim3(1), dim3(kThreads), 0, s, (const unsigned*)cnt, ncols,
                     rowptrT, cursor);
  hipLaunchKernelGGL(k_csr_scatter_t<T>, dim3(nblk(m)), dim3(kThreads), 0, s, rowptr, col, val, m,
                     cursor, colT, valT);
  hipLaunchKernelGGL(k_csr_sort_pairs<T>, dim3(nblk(ncols)), dim3(kThreads), 0, s,
                     (const int64_t*)rowptrT, ncols, colT, valT);
}

RectSplit rect_split(int64_t K, int64_t N) {
  RectSplit sp;
  sp.gx = (int)((N + 255) / 256);
  int64_t want = (512 + sp.gx - 1) / sp.gx;          // about two workgroups per CU
  int64_t most = (K + 63) / 64;                      // chunks of at least 64 rows
  if (want > most) want = most;
  if (want < 1) want = 1;
  sp.kchunk = ((K + want - 1) / want + 15) / 16 * 16;  // whole batches of eight k-pairs
  sp.ksplit = (int)((K + sp.kchunk - 1) / sp.kchunk);
  return sp;
}

bool rect_f32_wide(const void* V, int64_t ld, int64_t rows, int64_t cols, int r) {
  return r > 32 && r % 2 == 0 && cols % 4 == 0 && ld % 4 == 0 && ((uintptr_t)V & 15) == 0;
}

void launch_rect_f32(const float* V, int64_t ld, const float* VT, int trans, const float* P,
                     int64_t K, int64_t N, int r, const RectSplit& sp, float* Bpart,
                     const State* st, hipStream_t s, const RhoJob& rj) {
  if (rect_f32_wide(V, ld, trans ? K : N, trans ? N : K, r)) {
    const dim3 grid((unsigned)((N + 511) / 512), (unsigned)(sp.ksplit + (rj.G ? 1 : 0)));
    if (trans)
      hipLaunchKernelGGL(k_rect_f32w<false>, grid, dim3(256), 0, s, V, ld, P, K, N, r, sp.kchunk,
                         Bpart, N * r, st, rj);
    else
      hipLaunchKernelGGL(k_rect_f32w<true>, grid, dim3(256), 0, s, V, ld, P, K, N, r, sp.kchunk,
                         Bpart, N * r, st, rj);
    return;
  }
  launch_apass_f32_panels(trans ? V : VT, trans ? ld : N, P, K, N, r, sp.kchunk,
                          dim3((unsigned)sp.gx, (unsigned)sp.ksplit), Bpart, N * r, st, s, rj);
}

template <typename T>
void launch_transpose(const T* A, int64_t rows, int64_t cols, int64_t lda, T* AT, hipStream_t s) {
  hipLaunchKernelGGL(k_transpose<T>, dim3((unsigned)((cols + 63) / 64), (unsigned)((rows + 63) / 64)),
                     dim3(256), 0, s, A, rows, cols, lda, AT);
}
template void launch_transpose<float>(const float*, int64_t, int64_t, int64_t, float*, hipStream_t);
template void launch_transpose<double>(const double*, int64_t, int64_t, int64_t, double*,
                                       hipStream_t);

template void launch_rect_apass<float>(const float*, int64_t, int64_t, int64_t, int, const float*,
                                       int, float*, const State*, hipStream_t);
template void launch_rect_apass<double>(const double*, int64_t, int64_t, int64_t, int,
                                        const double*, int, double*, const State*, hipStream_t);
template void launch_csr_transpose<float>(const int64_t*, const int32_t*, const float*, int64_t,
                                          int64_t, int64_t, unsigned*, unsigned long long*,
                                          int64_t*, int32_t*, float*, hipStream_t);
template void launch_csr_transpose<double>(const int64_t*, const int32_t*, const double*, int64_t,
                                           int64_t, int64_t, unsigned*, unsigned long long*,
                                           int64_t*, int32_t*, double*, hipStream_t);

}  // namespace snmf
