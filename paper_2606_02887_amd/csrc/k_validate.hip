// Input checks of the C ABI run on the device: ||x||^2 with negative / non-finite counts
// over a strided 2-D region, and CSR structure and symmetry checks.
#include "common.hpp"
#include "kernels.hpp"

namespace snmf {

// {sum of squares, negatives, non-finite} over rows x cols with leading dimension ld, in
// pieces of kStatSeg elements of a row (a contiguous array is one row), eight loads in flight
// per thread and no division per element; k_stats_sum adds the workgroups' sums.  Bound by
// the copy rate: 8192 x 4096 floats 30 us (179 us with one load in flight, a 64-bit division
// per element and the sums finished by the last workgroup to arrive; 128 us with that
// finish alone, whose device-scope fence every workgroup pays for).
constexpr int kStatSeg = kThreads * 8;
template <typename T>
__global__ __launch_bounds__(kThreads) void k_stats2d(const T* __restrict__ x, int64_t rows,
                                                      int64_t cols, int64_t ld, int64_t nseg,
                                                      double* __restrict__ part) {
  __shared__ double sred[kThreads / kWave * 3];
  double v[3] = {0.0, 0.0, 0.0};
  for (int64_t it = blockIdx.x; it < rows * nseg; it += gridDim.x) {
    const int64_t row = it / nseg, c0 = (it - row * nseg) * kStatSeg;
    const int left = (int)(cols - c0 < kStatSeg ? cols - c0 : kStatSeg);
    const T* __restrict__ p = x + row * ld + c0;
    T a[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const int e = u * kThreads + (int)threadIdx.x;
      a[u] = p[e < left ? e : 0];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const double d = (double)a[u];
      const bool in = u * kThreads + (int)threadIdx.x < left, fin = d - d == 0.0;
      const double ok = in && fin ? d : 0.0;
      v[0] = __builtin_fma(ok, ok, v[0]);
      v[1] += in && d < 0.0 && fin ? 1.0 : 0.0;
      v[2] += in && !fin ? 1.0 : 0.0;
    }
  }
  block_sum<3>(v, sred);
  if (threadIdx.x == 0)
    for (int j = 0; j < 3; ++j) part[(size_t)blockIdx.x * kNumPart + j] = v[j];
}
__global__ __launch_bounds__(kThreads) void k_stats_sum(const double* __restrict__ part, int nb,
                                                        double* __restrict__ out) {
  __shared__ double sred[kThreads / kWave * 3];
  double t[3];
  reduce_partials<3>(part, nb, t, sred);
  if (threadIdx.x == 0)
    for (int j = 0; j < 3; ++j) out[j] = t[j];
}

// CSR structure: flags[0] += bad rowptr, flags[1] += column out of range,
// flags[2] += unsorted or repeated column within a row.  One wavefront per row (a thread
// per row made a power-law graph's longest row one chain: 276 us at n = 200000, 2e6
// nonzeros, 37 us so).
__global__ __launch_bounds__(kThreads) void k_csr_structure(const int64_t* __restrict__ rowptr,
                                                            const int32_t* __restrict__ col,
                                                            int64_t n, int64_t nnz,
                                                            unsigned* __restrict__ flags) {
  const int lane = threadIdx.x & (kWave - 1);
  unsigned bad_ptr = 0, bad_col = 0, unsorted = 0;
  const int64_t step = (int64_t)gridDim.x * (kThreads / kWave);
  for (int64_t i = (int64_t)blockIdx.x * (kThreads / kWave) + threadIdx.x / kWave; i < n;
       i += step) {
    const int64_t b = rowptr[i], e = rowptr[i + 1];
    if (b < 0 || e < b || e > nnz) {
      if (lane == 0) ++bad_ptr;
      continue;
    }
    for (int64_t z = b + lane; z < e; z += kWave) {
      const int32_t cc = col[z], prev = z > b ? col[z - 1] : -1;
      if (cc < 0 || cc >= n) ++bad_col;
      if (cc <= prev) ++unsorted;
    }
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (rowptr[0] != 0 || rowptr[n] != nnz) atomicAdd(&flags[0], 1u);
  }
  if (bad_ptr) atomicAdd(&flags[0], bad_ptr);
  if (bad_col) atomicAdd(&flags[1], bad_col);
  if (unsorted) atomicAdd(&flags[2], unsorted);
}

// Symmetry of a CSR matrix with sorted rows: for every stored (i, j, v) row j must hold
// column i with the same value.  flags[3] += mismatches.  One thread per nonzero, its row
// found by bisection of rowptr (a structure that k_csr_structure has passed): a thread per
// row left the longest rows of a power-law graph to one thread each (5180 us at
// n = 200000, 2e6 nonzeros, 118 us so).
template <typename T>
__global__ __launch_bounds__(kThreads) void k_csr_symmetry(const int64_t* __restrict__ rowptr,
                                                           const int32_t* __restrict__ col,
                                                           const T* __restrict__ val, int64_t n,
                                                           int64_t nnz,
                                                           unsigned* __restrict__ flags) {
  unsigned bad = 0;
  for (int64_t z = (int64_t)blockIdx.x * kThreads + threadIdx.x; z < nnz;
       z += (int64_t)gridDim.x * kThreads) {
    int64_t a = 0, b = n;  // the last row i with rowptr[i] <= z lies in [a, b)
    while (b - a > 1) {
      const int64_t mid = (a + b) >> 1;
      if (rowptr[mid] <= z) a = mid;
      else b = mid;
    }
    const int64_t i = a, j = col[z];
    int64_t lo = rowptr[j], hi = rowptr[j + 1] - 1;
    bool found = false;
    while (lo <= hi) {
      const int64_t mid = (lo + hi) >> 1;
      const int32_t cm = col[mid];
      if (cm == i) {
        found = val[mid] == val[z];
        break;
      }
      if (cm < i) lo = mid + 1;
      else hi = mid - 1;
    }
    if (!found) ++bad;
  }
  if (bad) atomicAdd(&flags[3], bad);
}

// Symmetry of a dense n x n matrix (leading dimension ld): workgroup (bx, by), by <= bx,
// stages the 32 x 32 tile at (block row by, block column bx) in LDS and compares it with
// the mirrored tile read row by row.  flags[3] += entries with
// |a_ij - a_ji| > tol max(|a_ij|, |a_ji|) (NaN entries count as mismatches).
template <typename T>
__global__ __launch_bounds__(kThreads) void k_dense_symmetry(const T* __restrict__ A, int64_t n,
                                                             int64_t ld, double tol,
                                                             unsigned* __restrict__ flags) {
  if (blockIdx.y > blockIdx.x) return;
  __shared__ T tile[32][33];
  const int64_t i0 = (int64_t)blockIdx.y * 32, j0 = (int64_t)blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;   // 32 x 8 threads
  for (int q = ty; q < 32; q += 8) {
    const int64_t i = i0 + q, j = j0 + tx;
    tile[q][tx] = (i < n && j < n) ? A[i * ld + j] : T(0);
  }
  __syncthreads();
  unsigned bad = 0;
  for (int q = ty; q < 32; q += 8) {
    const int64_t j = j0 + q, i = i0 + tx;                    // entry (j, i) of the mirror
    if (i < n && j < n) {
      const double a = (double)A[j * ld + i];
      const double b = (double)tile[tx][q];                    // entry (i, j)
      const double m = fmax(fabs(a), fabs(b));
      if (!(fabs(a - b) <= tol * m)) ++bad;
    }
  }
  if (bad) atomicAdd(&flags[3], bad);
}

template <typename T>
void launch_dense_symmetry(const T* A, int64_t n, int64_t ld, double tol, unsigned* flags,
                           hipStream_t s) {
  const int64_t nt = (n + 31) / 32;
  hipLaunchKernelGGL(k_dense_symmetry<T>, dim3((unsigned)nt, (unsigned)nt), dim3(kThreads), 0, s,
                     A, n, ld, tol, flags);
}
template void launch_dense_symmetry<float>(const float*, int64_t, int64_t, double, unsigned*,
                                           hipStream_t);
template void launch_dense_symmetry<double>(const double*, int64_t, int64_t, double, unsigned*,
                                            hipStream_t);

template <typename T>
void launch_stats2d(const T* x, int64_t rows, int64_t cols, int64_t ld, double* part, double* out,
                    hipStream_t s) {
  if (ld == cols) {
    cols *= rows;
    rows = 1;
  }
  const int64_t nseg = (cols + kStatSeg - 1) / kStatSeg;
  int64_t nb = rows * nseg;
  if (nb < 1) nb = 1;
  if (nb > kMaxGrid) nb = kMaxGrid;
  hipLaunchKernelGGL(k_stats2d<T>, dim3((unsigned)nb), dim3(kThreads), 0, s, x, rows, cols, ld,
                     nseg, part);
  hipLaunchKernelGGL(k_stats_sum, dim3(1), dim3(kThreads), 0, s, (const double*)part, (int)nb, out);
}

void launch_csr_structure(const int64_t* rowptr, const int32_t* col, int64_t n, int64_t nnz,
                          unsigned* flags, hipStream_t s) {
  int64_t nb = (n + kThreads / kWave - 1) / (kThreads / kWave);
  if (nb > 8192) nb = 8192;
  if (nb < 1) nb = 1;
  hipLaunchKernelGGL(k_csr_structure, dim3((unsigned)nb), dim3(kThreads), 0, s, rowptr, col, n,
                     nnz, flags);
}

template <typename T>
void launch_csr_symmetry(const int64_t* rowptr, const int32_t* col, const T* val, int64_t n,
                         int64_t nnz, unsigned* flags, hipStream_t s) {
  int64_t nb = (nnz + kThreads - 1) / kThreads;
  if (nb > 8192) nb = 8192;
  if (nb < 1) nb = 1;
  hipLaunchKernelGGL(k_csr_symmetry<T>, dim3((unsigned)nb), dim3(kThreads), 0, s, rowptr, col,
                     val, n, nnz, flags);
}

template void launch_stats2d<float>(const float*, int64_t, int64_t, int64_t, double*, double*,
                                    hipStream_t);
template void launch_stats2d<double>(const double*, int64_t, int64_t, int64_t, double*, double*,
                                     hipStream_t);
template void launch_csr_symmetry<float>(const int64_t*, const int32_t*, const float*, int64_t,
                                         int64_t, unsigned*, hipStream_t);
template void launch_csr_symmetry<double>(const int64_t*, const int32_t*, const double*, int64_t,
                                          int64_t, unsigned*, hipStream_t);

// Solve start, after the copy and check of the start: clear the device state, store ||A||^2
// and the start time; one wavefront (one thread storing the whole struct took 41 us).
static_assert(sizeof(State) % 8 == 0, "State is cleared in 8-byte words");
__device__ __forceinline__ void reset_state(State* st, double normA2) {
  uint64_t* const w = (uint64_t*)st;
  for (int e = threadIdx.x; e < (int)(sizeof(State) / 8); e += kWave) w[e] = 0;
  __syncthreads();
  if (threadIdx.x == 0) {
    st->normA2 = normA2;
    st->t0 = wall_clock64();
  }
}
__global__ __launch_bounds__(kWave) void k_reset_state(State* st, double normA2,
                                                       const uint64_t* bad, uint32_t seq) {
  const int done = bad && copy_bad(*bad, seq);
  reset_state(st, normA2);
  if (threadIdx.x == 0) st->done = done;
}
void launch_reset_state(State* st, double normA2, hipStream_t s, const uint64_t* bad,
                        uint32_t seq) {
  hipLaunchKernelGGL(k_reset_state, dim3(1), dim3(kWave), 0, s, st, normA2, bad, seq);
}

// Batched solve start: one State per instance.
__global__ __launch_bounds__(kWave) void k_breset(State* states, const BInst* inst) {
  reset_state(states + blockIdx.x, inst[blockIdx.x].normA2);
}
void launch_breset(State* states, const BInst* inst, int ninst, hipStream_t s) {
  hipLaunchKernelGGL(k_breset, dim3(ninst), dim3(kWave), 0, s, states, inst);
}

// Batched solve end: every instance's results in one compact array.
__global__ __launch_bounds__(kThreads) void k_bout(const State* __restrict__ states, int ninst,
                                                   BOut* __restrict__ out) {
  const int i = blockIdx.x * kThreads + threadIdx.x;
  if (i >= ninst) return;
  const State& h = states[i];
  BOut o;
  o.status = h.status;
  o.outer = h.outer;
  o.converged_at = h.converged_at;
  o.pad = 0;
  o.inner_total = h.inner_total;
  o.ls_evals = h.ls_evals;
  o.ls_exhausted = h.ls_exhausted;
  o.res = h.res_last;
  o.resww = h.resww_last;
  o.sym = h.sym_last;
  o.pg = h.pg_last;
  o.f = h.f_last;
  o.normA2 = h.normA2;
  o.t_last = h.t_hstep - h.t0;
  o.t_conv = h.t_conv;
  out[i] = o;
}
void launch_bout(const State* states, int ninst, BOut* out, hipStream_t s) {
  hipLaunchKernelGGL(k_bout, dim3((ninst + kThreads - 1) / kThreads), dim3(kThreads), 0, s, states,
                     ninst, out);
}

// The starts of a solve copied in (to both factors) and checked, or its results copied out,
// in one launch: sixteen elements per thread, all loaded before the first is stored.  The
// checks and copies they replace were a launch each, and a host wait per array.
constexpr int kCopyPer = 16;
template <typename T>
__global__ __launch_bounds__(kThreads) void k_copy(CopyTab t, int check, uint64_t* bad,
                                                  uint32_t seq) {
  if (bad && !check && copy_bad(*bad, seq)) return;
  int q = 0;
  while (q + 1 < t.n && (int)blockIdx.x >= t.blk0[q + 1]) ++q;
  const CopySeg& g = t.s[q];
  const int64_t at = (int64_t)((int)blockIdx.x - t.blk0[q]) * (kThreads * kCopyPer);
  const int left = (int)(g.count - at < kThreads * kCopyPer ? g.count - at : kThreads * kCopyPer);
  const T* __restrict__ src = (const T*)g.src + at;
  T* __restrict__ d0 = (T*)g.d0 + at;
  T v[kCopyPer];
#pragma unroll
  for (int u = 0; u < kCopyPer; ++u) {
    const int e = u * kThreads + (int)threadIdx.x;
    v[u] = src[e < left ? e : 0];
  }
  bool neg = false, nonfin = false;
#pragma unroll
  for (int u = 0; u < kCopyPer; ++u) {
    const int e = u * kThreads + (int)threadIdx.x;
    if (e < left) d0[e] = v[u];
    const bool fin = v[u] - v[u] == T(0);
    nonfin = nonfin || !fin;
    neg = neg || (fin && v[u] < T(0));
  }
  if (g.d1) {
    T* __restrict__ d1 = (T*)g.d1 + at;
#pragma unroll
    for (int u = 0; u < kCopyPer; ++u) {
      const int e = u * kThreads + (int)threadIdx.x;
      if (e < left) d1[e] = v[u];
    }
  }
  if (bad && check && (neg || nonfin))
    atomicMax((unsigned long long*)bad,
              (unsigned long long)seq << 32 | (uint32_t)~(2u * (uint32_t)(t.base + q) + (nonfin ? 0u : 1u)));
}
template <typename T>
void launch_copy(CopyTab& t, bool check, uint64_t* bad, uint32_t seq, hipStream_t s) {
  int64_t nb = 0;
  for (int q = 0; q < t.n; ++q) {
    t.blk0[q] = (int32_t)nb;
    nb += (t.s[q].count + kThreads * kCopyPer - 1) / (kThreads * kCopyPer);
  }
  t.blk0[t.n] = (int32_t)nb;
  if (nb < 1) return;
  hipLaunchKernelGGL(k_copy<T>, dim3((unsigned)nb), dim3(kThreads), 0, s, t, check ? 1 : 0, bad,
                     seq);
}
template void launch_copy<float>(CopyTab&, bool, uint64_t*, uint32_t, hipStream_t);
template void launch_copy<double>(CopyTab&, bool, uint64_t*, uint32_t, hipStream_t);

// flag = 1 when every instance of a batched solve is done.
__global__ __launch_bounds__(256) void k_all_done(const State* states, int ninst, int32_t* flag) {
  __shared__ int s_any;
  if (threadIdx.x == 0) s_any = 0;
  __syncthreads();
  int open = 0;
  for (int i = threadIdx.x; i < ninst; i += blockDim.x) open |= states[i].done == 0;
  if (open) s_any = 1;
  __syncthreads();
  if (threadIdx.x == 0) flag[0] = s_any ? 0 : 1;
}
void launch_all_done(const State* states, int ninst, int32_t* flag, hipStream_t s) {
  hipLaunchKernelGGL(k_all_done, dim3(1), dim3(256), 0, s, states, ninst, flag);
}

// Flat BF16 split of count floats.
__device__ __forceinline__ uint16_t bf16_rne_v(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7f800000u) == 0x7f800000u) return (uint16_t)((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__global__ __launch_bounds__(kThreads) void k_split_flat(const float* __restrict__ x, int64_t count,
                                                         uint16_t* __restrict__ hi,
                                                         uint16_t* __restrict__ lo) {
  for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < count;
       e += (int64_t)gridDim.x * kThreads) {
    const float a = x[e];
    const uint16_t h = bf16_rne_v(a);
    hi[e] = h;
    lo[e] = bf16_rne_v(a - __uint_as_float((uint32_t)h << 16));
  }
}
void launch_split_flat(const float* x, int64_t count, uint16_t* hi, uint16_t* lo, hipStream_t s) {
  int64_t nb = (count + kThreads - 1) / kThreads;
  if (nb > 65536) nb = 65536;
  if (nb < 1) nb = 1;
  hipLaunchKernelGGL(k_split_flat, dim3((unsigned)nb), dim3(kThreads), 0, s, x, count, hi, lo);
}

}  // namespace snmf
