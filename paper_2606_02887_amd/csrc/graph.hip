// Host side and C ABI of the graph preprocessing of Graph-SNMPBB (Section 2.2; include/
// snmf.h snmf_knn / snmf_knn_graph): neighbours, the union pattern, the similarity values
// and the normalised Laplacian, every step in the kernels of k_graph.hip.
#include <hip/hip_runtime.h>

#include <string>

#include "../../include/snmf.h"
#include "common.hpp"
#include "host.hpp"
#include "kernels.hpp"

using namespace snmf;

namespace {

snmf_status check_points(const void* X, int64_t n, int dim, int K, int prec) {
  if (!X) return fail(SNMF_E_ARG, "X is required");
  if (prec != SNMF_F32 && prec != SNMF_F64) return fail(SNMF_E_ARG, "prec must be F32 or F64");
  if (n < 2 || n >= ((int64_t)1 << 31)) return fail(SNMF_E_SHAPE, "n must lie in [2, 2^31)");
  if (dim < 1 || dim > kKnnMaxDim) return fail(SNMF_E_SHAPE, "dim must lie in [1, 64]");
  if (K < 1 || K > kKnnMaxK) return fail(SNMF_E_SHAPE, "K must lie in [1, 64]");
  if (K > n - 1) return fail(SNMF_E_SHAPE, "K must not exceed n - 1");
  return SNMF_OK;
}

// E_NONFINITE unless every coordinate is finite, then the neighbours.  nrm: n doubles, flag:
// kFlagWords device words of scratch.  The norms that the screened search needs are formed
// before the host wait of the check, which brings their near counts along.
constexpr int kFlagWords = 8, kNearWord = 4;
template <typename T>
snmf_status check_points_finite(const T* X, int64_t n, int dim, unsigned* flag, double* nrm,
                                bool* inseparable, hipStream_t s) {
  const size_t bytes = (nrm ? kFlagWords : 1) * sizeof(unsigned);
  HIP_TRY(hipMemsetAsync(flag, 0, bytes, s));
  launch_count_nonfinite<T>(X, n * dim, flag, s);
  if (nrm) launch_knn_norms<T>(X, n, dim, nrm, flag + kNearWord, s);
  HIP_TRY(hipGetLastError());
  unsigned f[kFlagWords] = {};
  HIP_TRY(hipMemcpyAsync(f, flag, bytes, hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  if (f[0]) return fail(SNMF_E_NONFINITE, "X has NaN/Inf entries");
  *inseparable = knn_inseparable(f + kNearWord, n);
  return SNMF_OK;
}

snmf_status knn_any(const void* X, int64_t n, int dim, int K, int prec, double* nrm,
                    unsigned* flag, int32_t* nbr, hipStream_t s) {
  if (!knn_screened(n, dim, K, elt_size(prec))) nrm = nullptr;
  bool inseparable = false;
  SNMF_TRY(prec == SNMF_F64
               ? check_points_finite<double>((const double*)X, n, dim, flag, nrm, &inseparable, s)
               : check_points_finite<float>((const float*)X, n, dim, flag, nrm, &inseparable, s));
  if (inseparable) nrm = nullptr;
  if (prec == SNMF_F64)
    launch_knn<double>((const double*)X, n, dim, K, nrm, nbr, s);
  else
    launch_knn<float>((const float*)X, n, dim, K, nrm, nbr, s);
  HIP_TRY(hipGetLastError());
  return SNMF_OK;
}

}  // namespace

extern "C" {

snmf_status snmf_knn(const void* X, int64_t n, int32_t dim, int32_t K, int32_t prec,
                     int32_t* nbr_out, void* stream) {
  SNMF_TRY(check_points(X, n, dim, K, prec));
  if (!nbr_out) return fail(SNMF_E_ARG, "nbr_out is required");
  hipStream_t s = (hipStream_t)stream;
  DevBuf pool;  // the flags of the check, the squared norms
  HIP_TRY(hipMalloc(&pool.p, 256 + (size_t)n * 8));
  SNMF_TRY(knn_any(X, n, dim, K, prec, (double*)((char*)pool.p + 256), (unsigned*)pool.p, nbr_out,
                   s));
  HIP_TRY(hipStreamSynchronize(s));
  return SNMF_OK;
}

snmf_status snmf_knn_graph(const void* X, int64_t n, int32_t dim, int32_t K, double sigma,
                           int32_t laplacian, int32_t prec, int64_t* rowptr_out,
                           int32_t* col_out, void* val_out, int64_t capacity, int64_t* nnz_out,
                           void* stream) {
  SNMF_TRY(check_points(X, n, dim, K, prec));
  if (!rowptr_out || !col_out || !val_out || !nnz_out)
    return fail(SNMF_E_ARG, "rowptr_out, col_out, val_out and nnz_out are required");
  if (!(sigma >= 0.0) || !(sigma < 1e300)) return fail(SNMF_E_ARG, "sigma must be >= 0 and finite");
  const int diag = laplacian ? 1 : 0;
  const int64_t bound = n * (2 * (int64_t)K + diag);
  if (capacity < bound)
    return fail(SNMF_E_SHAPE, "capacity must be at least n (2 K + [laplacian]) = " +
                                  std::to_string(bound));
  hipStream_t s = (hipStream_t)stream;
  // scratch: neighbours, counts, cursors, degrees, FP64 similarity values
  const size_t b_nbr = ((size_t)n * K * 4 + 255) / 256 * 256;
  const size_t b_cnt = ((size_t)n * 4 + 255) / 256 * 256;
  const size_t b_cur = ((size_t)n * 8 + 255) / 256 * 256;
  const size_t b_deg = ((size_t)n * 8 + 255) / 256 * 256;
  const size_t b_v = ((size_t)bound * 8 + 255) / 256 * 256;
  DevBuf pool;
  HIP_TRY(hipMalloc(&pool.p, b_nbr + b_cnt + b_cur + b_deg + b_v + 256));
  char* base = (char*)pool.p;
  int32_t* nbr = (int32_t*)base;
  unsigned* cnt = (unsigned*)(base + b_nbr);
  unsigned long long* cursor = (unsigned long long*)(base + b_nbr + b_cnt);
  double* deg = (double*)(base + b_nbr + b_cnt + b_cur);
  double* v = (double*)(base + b_nbr + b_cnt + b_cur + b_deg);
  SNMF_TRY(knn_any(X, n, dim, K, prec, deg,  // deg is free until the values
                   (unsigned*)(base + b_nbr + b_cnt + b_cur + b_deg + b_v), nbr, s));
  HIP_TRY(hipMemsetAsync(cnt, 0, (size_t)n * 4, s));
  launch_knn_pattern_count(nbr, n, K, diag, cnt, rowptr_out, s);
  launch_knn_pattern_fill(nbr, n, K, diag, rowptr_out, col_out, cursor, (int32_t*)v, s);
  if (prec == SNMF_F64)
    launch_knn_values<double>((const double*)X, n, dim, sigma, laplacian, rowptr_out, col_out, v,
                              deg, (double*)val_out, s);
  else
    launch_knn_values<float>((const float*)X, n, dim, sigma, laplacian, rowptr_out, col_out, v,
                             deg, (float*)val_out, s);
  HIP_TRY(hipGetLastError());
  int64_t nnz = 0;
  HIP_TRY(hipMemcpyAsync(&nnz, rowptr_out + n, 8, hipMemcpyDeviceToHost, s));
  HIP_TRY(hipStreamSynchronize(s));
  *nnz_out = nnz;
  return SNMF_OK;
}

}  // extern "C"
