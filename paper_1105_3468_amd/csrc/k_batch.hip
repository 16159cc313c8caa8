// Kernels of the multi-right-hand-side solve: one launch processes up to
// BATCH_MAX columns, so the matrix, the aggregates and the factors are read
// once for all of them.  A batch of vectors is column-major: column c starts
// at base + c * ld (ld a multiple of 64 elements, so every column is aligned
// like a single vector).
//
//   k_spmm           y_c = A x_c, or y_c = b_c - A x_c (the FGMRES residual),
//                    or y_c = z_c - A^T P e_c (the adjoint cycle's residual)
//   k_restrict_cols  r_c = P^T z_c (members in ascending order)
//   k_prolong_cols   q_c = t_c + P e_c
//   k_cols_from_rows / k_rows_from_cols: between the caller's (N, nrhs)
//                    row-major arrays and the column-major batch
#include <algorithm>
#include <type_traits>

#include "gmg_internal.h"
#include "kcommon.h"

namespace gmg {

constexpr int BROWS = 256;    // rows per workgroup of the sparse products
constexpr int BCAP = 3072;    // (column, value) pairs of a tile staged in LDS

constexpr int SPMM_LOADS = 16;  // loads of x a lane has in flight

// One workgroup owns BROWS consecutive rows.  When the tile's entries fit in
// LDS they are first staged there with coalesced loads; then each lane runs
// its own row, reading the entry once and the nb columns' values of x at that
// entry (consecutive lanes hold consecutive rows, so for fixed column and
// entry position the gathers are nearly contiguous).  Column group blockIdx.y
// of CB columns.
// MODE 0: y = A x; 1: y = b - A x; 2: y = b - A (P e), x indexed through agg
// and rsx apart from row to row.
template <class T, class TB, int MODE, int CB>
__global__ __launch_bounds__(BROWS) void k_spmm(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                                const T* __restrict__ v, const int* __restrict__ agg,
                                                const T* __restrict__ x, size_t ldx, size_t rsx,
                                                const TB* __restrict__ b, size_t ldb, T* __restrict__ y, size_t ldy,
                                                int nb) {
  constexpr int U = SPMM_LOADS / CB;  // entries of a row in flight
  __shared__ int sc[BCAP];
  __shared__ T sv[BCAP];
  const int r0 = blockIdx.x * BROWS;
  const int r1 = min(r0 + BROWS, n);
  const int e0 = rp[r0], e1 = rp[r1];
  const int row = r0 + threadIdx.x;
  const int c0 = blockIdx.y * CB;
  nb = min(CB, nb - c0);
  x += c0 * ldx;
  y += c0 * ldy;
  if (MODE != 0) b += c0 * ldb;
  const bool staged = e1 - e0 <= BCAP;
  if (staged) {
    for (int e = e0 + threadIdx.x; e < e1; e += BROWS) {
      sc[e - e0] = ci[e];
      sv[e - e0] = v[e];
    }
    __syncthreads();
  }
  if (row >= r1) return;
  TB bv[CB];
  T acc[CB];
#pragma unroll
  for (int c = 0; c < CB; ++c) {
    acc[c] = (T)0;
    if (MODE != 0) bv[c] = c < nb ? b[c * ldb + row] : (TB)0;
  }
  const int p0 = rp[row], p1 = rp[row + 1];
  for (int p = p0; p < p1; p += U) {
    int j[U];
    T a[U], xv[U][CB];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int q = min(p + u, p1 - 1);
      j[u] = staged ? sc[q - e0] : ci[q];
      a[u] = staged ? sv[q - e0] : v[q];
    }
    if (MODE == 2) {
#pragma unroll
      for (int u = 0; u < U; ++u) j[u] = agg[j[u]];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int c = 0; c < CB; ++c) xv[u][c] = c < nb ? x[c * ldx + (MODE == 2 ? j[u] * rsx : j[u])] : (T)0;
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (p + u < p1) {
#pragma unroll
        for (int c = 0; c < CB; ++c) acc[c] += a[u] * xv[u][c];
      }
  }
#pragma unroll
  for (int c = 0; c < CB; ++c)
    if (c < nb) y[c * ldy + row] = MODE == 0 ? acc[c] : (T)bv[c] - acc[c];
}

template <class T, class TB, int MODE>
static void spmm_launch(int n, const int* rp, const int* ci, const T* v, const int* agg, const T* x, size_t ldx,
                        size_t rsx, const TB* b, size_t ldb, T* y, size_t ldy, int nb, hipStream_t s) {
  if (n <= 0) return;
  if (nb < 1 || nb > BATCH_MAX) fail(GMG_ERR_INVALID_ARG, "spmm: bad column count");
  const int blocks = (n + BROWS - 1) / BROWS;
  auto go = [&](auto cb) {
    constexpr int CB = decltype(cb)::value;
    hipLaunchKernelGGL((k_spmm<T, TB, MODE, CB>), dim3(blocks, (nb + CB - 1) / CB), dim3(BROWS), 0, s, n, rp, ci, v,
                       agg, x, ldx, rsx, b, ldb, y, ldy, nb);
  };
  // All columns in one workgroup read the matrix once; with few workgroups a
  // product is a row's chain of loads, one trip to L2 per entry, and columns
  // go to more workgroups with several entries in flight instead (us, product
  // / fine residual of 16 columns, with 16, 4 and 2 columns a workgroup:
  // 32^2 7.5 / 8.1, 5.6 / 5.2, 4.7 / 5.3; 160^2 9.5 / 13.3, 7.8 / 10.1, 8.1 /
  // 10.3; 512^2, 4 and 8: 37, 29 against 28).
  if (blocks <= 64) go(std::integral_constant<int, 2>());
  else if (blocks < 256) go(std::integral_constant<int, 4>());
  else go(std::integral_constant<int, BATCH_MAX>());
  HIPCK(hipGetLastError());
}

template <class T>
void launch_spmm(int n, const int* rp, const int* ci, const T* v, const T* x, size_t ldx, T* y, size_t ldy, int nb,
                 hipStream_t s) {
  spmm_launch<T, T, 0>(n, rp, ci, v, nullptr, x, ldx, 1, (const T*)nullptr, 0, y, ldy, nb, s);
}
template void launch_spmm<double>(int, const int*, const int*, const double*, const double*, size_t, double*, size_t,
                                  int, hipStream_t);
template void launch_spmm<float>(int, const int*, const int*, const float*, const float*, size_t, float*, size_t,
                                 int, hipStream_t);

void launch_residual_cols(int n, const int* rp, const int* ci, const double* v, const double* x, size_t ldx,
                          const double* b, size_t ldb, double* r, size_t ldr, int nb, hipStream_t s) {
  spmm_launch<double, double, 1>(n, rp, ci, v, nullptr, x, ldx, 1, b, ldb, r, ldr, nb, s);
}

void launch_resid_adj_cols(int n, const int* rp, const int* ci, const double* v, const int* agg, const double* ec,
                           CoarseCols lc, const double* z, size_t ldz, double* out, size_t ldo, int nb,
                           hipStream_t s) {
  spmm_launch<double, double, 2>(n, rp, ci, v, agg, ec, lc.col, lc.row, z, ldz, out, ldo, nb, s);
}

// r_c = z_c - A t_c over the column batch (t in the cycle's precision T, z
// in FP64): the fine residual of the smoothed iterate
template <class T>
void launch_resid_fine_cols(int n, const int* rp, const int* ci, const T* v, const T* t, size_t ldt, const double* z,
                            size_t ldz, T* r, size_t ldr, int nb, hipStream_t s) {
  spmm_launch<T, double, 1>(n, rp, ci, v, nullptr, t, ldt, 1, z, ldz, r, ldr, nb, s);
}
template void launch_resid_fine_cols<double>(int, const int*, const int*, const double*, const double*, size_t,
                                             const double*, size_t, double*, size_t, int, hipStream_t);
template void launch_resid_fine_cols<float>(int, const int*, const int*, const float*, const float*, size_t,
                                            const double*, size_t, float*, size_t, int, hipStream_t);

// rc_c[I] = sum over members (ascending) of z_c[k]; reset_c[I] <- sentinel
// (column blockIdx.y, coarse columns ldc apart)
template <class T>
__global__ void k_restrict_cols(int nc, const int* __restrict__ aptr, const int* __restrict__ amem,
                                const T* __restrict__ z, size_t ldz, T* __restrict__ rc, T* __restrict__ reset,
                                size_t ldc) {
  const int I = blockIdx.x * blockDim.x + threadIdx.x;
  if (I >= nc) return;
  z += blockIdx.y * ldz;
  T s = (T)0;
  for (int m = aptr[I]; m < aptr[I + 1]; ++m) s += z[amem[m]];
  rc[blockIdx.y * ldc + I] = s;
  if (reset) reset[blockIdx.y * ldc + I] = sentinel_of<T>(0);
}

// The same into rows of CW columns (zeros past the batch's nb).  A workgroup
// takes 64 aggregates: its waves gather CW / 4 columns each, lanes along the
// aggregates (near members of a column share lines), and the rows leave
// through LDS coalesced.
template <class T, int CW>
__global__ __launch_bounds__(256) void k_restrict_rows(int nc, const int* __restrict__ aptr,
                                                       const int* __restrict__ amem, const T* __restrict__ z,
                                                       size_t ldz, T* __restrict__ rc, T* __restrict__ reset, int nb) {
  __shared__ T sh[64][CW + 1];
  constexpr int NC = CW / 4;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int I0 = blockIdx.x * 64, I = I0 + lane;
  const int m0 = I < nc ? aptr[I] : 0, m1 = I < nc ? aptr[I + 1] : 0;
  T acc[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) acc[c] = (T)0;
  for (int m = m0; m < m1; m += 8) {
    int k[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) k[u] = m + u < m1 ? amem[m + u] : -1;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
      const int col = wave + 4 * c;
      if (col >= nb) break;
      T v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = k[u] >= 0 ? z[col * ldz + k[u]] : (T)0;
#pragma unroll
      for (int u = 0; u < 8; ++u)
        if (k[u] >= 0) acc[c] += v[u];
    }
  }
#pragma unroll
  for (int c = 0; c < NC; ++c) sh[lane][wave + 4 * c] = acc[c];
  __syncthreads();
  const int rows = min(64, nc - I0);
  for (int o = threadIdx.x; o < rows * CW; o += 256) {
    rc[(size_t)I0 * CW + o] = sh[o / CW][o & (CW - 1)];
    reset[(size_t)I0 * CW + o] = sentinel_of<T>(0);
  }
}

#define GMG_COLS_WIDTH(cw, CALL)                                       \
  do {                                                                 \
    if ((cw) == 4) CALL(4);                                            \
    else if ((cw) == 8) CALL(8);                                       \
    else if ((cw) == 16) CALL(16);                                     \
    else fail(GMG_ERR_INVALID_ARG, "coarse columns: bad row width");   \
  } while (0)

template <class T>
void launch_restrict_cols(int nc, const int* aptr, const int* amem, const T* z, size_t ldz, T* rc, T* reset,
                          CoarseCols lc, int nb, hipStream_t s) {
  if (nc <= 0) return;
  if (lc.col == 1) {
#define GMG_RESTRICT(CW_)                                                                                             \
  hipLaunchKernelGGL((k_restrict_rows<T, CW_>), dim3((nc + 63) / 64), dim3(256), 0, s, nc, aptr, amem, z, ldz, rc,    \
                     reset, nb)
    GMG_COLS_WIDTH(lc.width, GMG_RESTRICT);
#undef GMG_RESTRICT
  } else {
    hipLaunchKernelGGL(k_restrict_cols<T>, dim3((nc + 255) / 256, nb), dim3(256), 0, s, nc, aptr, amem, z, ldz, rc,
                       reset, lc.col);
  }
  HIPCK(hipGetLastError());
}
template void launch_restrict_cols<double>(int, const int*, const int*, const double*, size_t, double*, double*,
                                           CoarseCols, int, hipStream_t);
template void launch_restrict_cols<float>(int, const int*, const int*, const float*, size_t, float*, float*,
                                          CoarseCols, int, hipStream_t);

// q_c[k] = t_c[k] + ec_c[agg[k]] (in T, widened); t_c[k] <- sentinel if
// reset_t (t was polled)
template <class T>
__global__ void k_prolong_cols(int n, const int* __restrict__ agg, T* __restrict__ t, size_t ldt,
                               const T* __restrict__ ec, size_t ldc, double* __restrict__ q, size_t ldq,
                               int reset_t) {
  t += blockIdx.y * ldt;
  ec += blockIdx.y * ldc;
  q += blockIdx.y * ldq;
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x) {
    const T val = t[k] + ec[agg[k]];
    q[k] = (double)val;
    if (reset_t) t[k] = sentinel_of<T>(0);
  }
}
// The same from rows of CW coarse columns: a lane reads its aggregate's row
// once, in 16-byte pieces, and the columns of t and q follow lane by lane.
template <class T, int CW>
__global__ __launch_bounds__(256) void k_prolong_rows(int n, const int* __restrict__ agg, T* __restrict__ t,
                                                      size_t ldt, const T* __restrict__ ec, double* __restrict__ q,
                                                      size_t ldq, int nb, int reset_t) {
  constexpr int V = 16 / sizeof(T);
  typedef T vec __attribute__((ext_vector_type(V)));
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < n; k += gridDim.x * blockDim.x) {
    const vec* row = reinterpret_cast<const vec*>(ec + (size_t)agg[k] * CW);
    vec e[CW / V];
    T tv[CW];
#pragma unroll
    for (int u = 0; u < CW / V; ++u) e[u] = row[u];
#pragma unroll
    for (int c = 0; c < CW; ++c) tv[c] = c < nb ? t[c * ldt + k] : (T)0;
#pragma unroll
    for (int c = 0; c < CW; ++c)
      if (c < nb) {
        const T val = tv[c] + e[c / V][c % V];
        q[c * ldq + k] = (double)val;
        if (reset_t) t[c * ldt + k] = sentinel_of<T>(0);
      }
  }
}
template <class T>
void launch_prolong_cols(int n, const int* agg, T* t, size_t ldt, const T* ec, CoarseCols lc, double* q, size_t ldq,
                         int nb, bool reset_t, hipStream_t s) {
  if (n <= 0) return;
  if (lc.col == 1) {
    const unsigned g = (unsigned)std::min<int64_t>(4096, ((int64_t)n + 255) / 256);
#define GMG_PROLONG(CW_) \
  hipLaunchKernelGGL((k_prolong_rows<T, CW_>), dim3(g), dim3(256), 0, s, n, agg, t, ldt, ec, q, ldq, nb, reset_t ? 1 : 0)
    GMG_COLS_WIDTH(lc.width, GMG_PROLONG);
#undef GMG_PROLONG
  } else {
    const unsigned g = (unsigned)std::min<int64_t>(1024, ((int64_t)n + 255) / 256);
    hipLaunchKernelGGL(k_prolong_cols<T>, dim3(g, nb), dim3(256), 0, s, n, agg, t, ldt, ec, lc.col, q, ldq, reset_t ? 1 : 0);
  }
  HIPCK(hipGetLastError());
}
template void launch_prolong_cols<double>(int, const int*, double*, size_t, const double*, CoarseCols, double*, size_t,
                                          int, bool, hipStream_t);
template void launch_prolong_cols<float>(int, const int*, float*, size_t, const float*, CoarseCols, double*, size_t,
                                         int, bool, hipStream_t);

// out_c[i] = X[i * nrhs + c0 + c] for c < nb (column blockIdx.y), and back
__global__ void k_cols_from_rows(const double* __restrict__ X, int nrhs, int c0, double* __restrict__ out, size_t ld,
                                 int64_t n) {
  const int c = blockIdx.y;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    out[c * ld + i] = X[i * nrhs + c0 + c];
}
__global__ void k_rows_from_cols(double* __restrict__ X, int nrhs, int c0, const double* __restrict__ in, size_t ld,
                                 int64_t n) {
  const int c = blockIdx.y;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    X[i * nrhs + c0 + c] = in[c * ld + i];
}
void launch_cols_from_rows(const double* X, int nrhs, int c0, double* out, size_t ld, int64_t n, int nb,
                           hipStream_t s) {
  if (n <= 0) return;
  const unsigned g = (unsigned)std::min<int64_t>(1024, (n + 255) / 256);
  hipLaunchKernelGGL(k_cols_from_rows, dim3(g, nb), dim3(256), 0, s, X, nrhs, c0, out, ld, n);
  HIPCK(hipGetLastError());
}
void launch_rows_from_cols(double* X, int nrhs, int c0, const double* in, size_t ld, int64_t n, int nb,
                           hipStream_t s) {
  if (n <= 0) return;
  const unsigned g = (unsigned)std::min<int64_t>(1024, (n + 255) / 256);
  hipLaunchKernelGGL(k_rows_from_cols, dim3(g, nb), dim3(256), 0, s, X, nrhs, c0, in, ld, n);
  HIPCK(hipGetLastError());
}

}  // namespace gmg
