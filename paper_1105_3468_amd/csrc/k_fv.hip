// Finite-volume assembly of the convection-diffusion matrix A(kappa) and the
// gradients of a loss through the solve (dL/dkappa, dL/dA on the pattern).
//
// Discretisation of Eq. (pde): cell-centred finite volumes on [0,1]^dim,
// h = 1/n, row i + n j (+ n^2 k), rows scaled by the cell volume; harmonic
// face transmissibility T = 2 kc km / ((kc + km) h^2); Dirichlet faces y = 0, 1
// add 2 kc / h^2; Neumann faces add nothing; first-order upwind convection on
// face-averaged velocities.  The arithmetic order matches the generator that
// builds the same matrices on the host, so both give identical bits.
#include "gmg_internal.h"
#include "kcommon.h"

#pragma clang fp contract(off)

namespace gmg {

struct FvGeom {
  int n, dim;
  const double* fvel[3];
};

// face velocity of direction d at face index f (0..n) for the cell line (a, b)
// of the other coordinates; memory order of the face arrays is x fastest.
__device__ __forceinline__ double face_vel(const FvGeom& g, int d, const int* ijk, int f) {
  const int n = g.n;
  if (g.dim == 2) {
    if (d == 0) return g.fvel[0][(size_t)ijk[1] * (n + 1) + f];
    return g.fvel[1][(size_t)f * n + ijk[0]];
  }
  if (d == 0) return g.fvel[0][((size_t)ijk[2] * n + ijk[1]) * (n + 1) + f];
  if (d == 1) return g.fvel[1][((size_t)ijk[2] * (n + 1) + f) * n + ijk[0]];
  return g.fvel[2][((size_t)f * n + ijk[1]) * n + ijk[0]];
}

// First entry of row c (c = N: all entries): 2 dim + 1 per cell before it,
// less one for every cell before it that lies on the low or high side of a
// direction.  With stride s = n^d, runs of s cells share coordinate d, and s n
// cells pass through all of its values.
__device__ __forceinline__ int fv_row_start(int n, int dim, int c) {
  int start = (2 * dim + 1) * c;
  for (int d = 0, s = 1; d < dim; ++d, s *= n) {
    const int q = c / (s * n), r = c - q * (s * n);
    start -= 2 * q * s + min(r, s) + max(0, r - (n - 1) * s);
  }
  return start;
}

// One thread per row.  The row pointers have a closed form, so pattern and
// values take one launch without counting and scanning.  A workgroup's
// entries are consecutive in memory: the rows put theirs together in LDS and
// the workgroup writes them out coalesced (a lane storing its own row touches
// a line of its own per entry).  128^3 cells: count + scan + fill took 356 us
// (fill 118 us); this takes 85 us.  An assembly and a gradient, with what both
// calls cost beside their kernels, went from 440 to 172 us.
constexpr int FV_ROWS = 256;
__global__ __launch_bounds__(FV_ROWS) void k_fv_fill(FvGeom g, const double* __restrict__ kap, int* __restrict__ rp,
                                                     int* __restrict__ ci, double* __restrict__ v, int N) {
  __shared__ double sv[FV_ROWS * 7];
  __shared__ int sc[FV_ROWS * 7];
  const int n = g.n, dim = g.dim;
  const int c0 = blockIdx.x * FV_ROWS, c = c0 + threadIdx.x;
  const int first = fv_row_start(n, dim, c0);
  if (c < N) {
    const double h = 1.0 / n, h2 = h * h;
    int ijk[3] = {c % n, (c / n) % n, dim == 3 ? c / (n * n) : 0};
    const int stride[3] = {1, n, n * n};
    const double kc = kap[c];
    double diag = 0.0, lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0};
    bool has_lo[3] = {false, false, false}, has_hi[3] = {false, false, false};
    for (int d = 0; d < dim; ++d) {
      const double Flo = face_vel(g, d, ijk, ijk[d]);
      const double Fhi = face_vel(g, d, ijk, ijk[d] + 1);
      const double out_hi = Fhi, out_lo = -Flo;
      double dint = 0.0;
      if (ijk[d] < n - 1) {
        const double km = kap[c + stride[d]];
        const double T = 2.0 * kc * km / ((kc + km) * h2);
        dint += T;
        has_hi[d] = true;
        hi[d] = (0.0 - T) + fmin(out_hi, 0.0) / h;
      }
      if (ijk[d] > 0) {
        const double km = kap[c - stride[d]];
        const double T = 2.0 * km * kc / ((km + kc) * h2);
        dint += T;
        has_lo[d] = true;
        lo[d] = (0.0 - T) + fmin(out_lo, 0.0) / h;
      }
      const double conv = fmax(out_hi, 0.0) / h + fmax(out_lo, 0.0) / h;
      diag += dint;
      diag += conv;
      if (d == 1) {
        if (ijk[1] == 0) diag += 2.0 * kc / h2;
        if (ijk[1] == n - 1) diag += 2.0 * kc / h2;
      }
    }
    const int start = fv_row_start(n, dim, c);
    rp[c] = start;
    if (c == N - 1) rp[N] = fv_row_start(n, dim, N);
    int o = start - first;
    for (int d = dim - 1; d >= 0; --d)
      if (has_lo[d]) { sc[o] = c - stride[d]; sv[o] = lo[d]; ++o; }
    sc[o] = c;
    sv[o] = diag;
    ++o;
    for (int d = 0; d < dim; ++d)
      if (has_hi[d]) { sc[o] = c + stride[d]; sv[o] = hi[d]; ++o; }
  }
  __syncthreads();
  const int count = fv_row_start(n, dim, min(c0 + FV_ROWS, N)) - first;
  for (int e = threadIdx.x; e < count; e += FV_ROWS) {
    ci[first + e] = sc[e];
    v[first + e] = sv[e];
  }
}

static void launch_fv_fill(int n, int dim, const double* kappa, const double* vel_x, const double* vel_y,
                           const double* vel_z, int* rp, int* ci, double* v, int N, hipStream_t s) {
  FvGeom g{n, dim, {vel_x, vel_y, dim == 3 ? vel_z : nullptr}};
  hipLaunchKernelGGL(k_fv_fill, dim3((N + FV_ROWS - 1) / FV_ROWS), dim3(FV_ROWS), 0, s, g, kappa, rp, ci, v, N);
  HIPCK(hipGetLastError());
}

// dL/dkappa_c = - sum_r [ sum over interior faces f of c of dT_f/dkappa_c
//   (lam_c - lam_m)(x_c - x_m) + sum over Dirichlet faces of (2/h^2) lam_c x_c ]
// G = 2^LG lanes per cell share its right-hand sides (lane t takes t, t + G,
// ...), so that lanes read consecutive values of the row-major arrays; one
// lane per cell reads a line of its own per value instead.
template <int LG>
__global__ __launch_bounds__(256) void k_fv_grad(int n, int dim, const double* __restrict__ kap,
                                                 const double* __restrict__ lam, const double* __restrict__ x,
                                                 int nrhs, double* __restrict__ grad, int N) {
  constexpr int G = 1 << LG;
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int sub = (int)(t & (G - 1));
  const bool in = (t >> LG) < N;  // idle lanes take part in the shuffles
  const int c = in ? (int)(t >> LG) : N - 1;
  const double h = 1.0 / n, h2 = h * h;
  int ijk[3] = {c % n, (c / n) % n, dim == 3 ? c / (n * n) : 0};
  const int stride[3] = {1, n, n * n};
  const double kc = kap[c];
  double gsum = 0.0;
  for (int d = 0; d < dim; ++d) {
    for (int side = 0; side < 2; ++side) {
      const bool inside = side ? ijk[d] < n - 1 : ijk[d] > 0;
      if (inside) {
        const int m = side ? c + stride[d] : c - stride[d];
        const double km = kap[m];
        const double s = kc + km;
        const double dT = 2.0 * km * km / (s * s * h2);
        double acc = 0.0;
        for (int r = sub; r < nrhs; r += G)
          acc += (lam[(size_t)c * nrhs + r] - lam[(size_t)m * nrhs + r]) *
                 (x[(size_t)c * nrhs + r] - x[(size_t)m * nrhs + r]);
        gsum += dT * acc;
      } else if (d == 1) {
        double acc = 0.0;
        for (int r = sub; r < nrhs; r += G) acc += lam[(size_t)c * nrhs + r] * x[(size_t)c * nrhs + r];
        gsum += (2.0 / h2) * acc;
      }
    }
  }
#pragma unroll
  for (int off = G >> 1; off > 0; off >>= 1) gsum += __shfl_xor(gsum, off, 64);
  if (in && sub == 0) grad[c] = -gsum;
}

// G = 2^LG lanes per row share the right-hand sides, as above.
template <int LG>
__global__ __launch_bounds__(256) void k_pattern_grad(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                                      const double* __restrict__ lam, const double* __restrict__ x,
                                                      int nrhs, double* __restrict__ g) {
  constexpr int G = 1 << LG;
  const int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  const int64_t i = t >> LG;
  const int sub = (int)(t & (G - 1));
  if (i >= n) return;  // whole groups leave together
  for (int p = rp[i]; p < rp[i + 1]; ++p) {
    const int j = ci[p];
    double s = 0.0;
    for (int r = sub; r < nrhs; r += G) s += lam[(size_t)i * nrhs + r] * x[(size_t)j * nrhs + r];
#pragma unroll
    for (int off = G >> 1; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
    if (sub == 0) g[p] = -s;
  }
}

// lanes per cell or row for nrhs right-hand sides: the largest power of two
// that keeps them all busy, at most 16 (a 128-byte line of values), and fewer
// where a launch cannot have that many threads
#define GMG_FV_LANES(nrhs, KERNEL, items, ...)                                                                  \
  do {                                                                                                          \
    int lg_ = (nrhs) >= 16 ? 4 : (nrhs) >= 8 ? 3 : (nrhs) >= 4 ? 2 : (nrhs) >= 2 ? 1 : 0;                       \
    while (lg_ > 0 && ((int64_t)(items) << lg_) > kMaxThreads - 255) --lg_;                                     \
    const dim3 grid_((unsigned)((((int64_t)(items) << lg_) + 255) / 256));                                      \
    if (lg_ == 0) hipLaunchKernelGGL(KERNEL<0>, grid_, dim3(256), 0, s, __VA_ARGS__);                           \
    else if (lg_ == 1) hipLaunchKernelGGL(KERNEL<1>, grid_, dim3(256), 0, s, __VA_ARGS__);                      \
    else if (lg_ == 2) hipLaunchKernelGGL(KERNEL<2>, grid_, dim3(256), 0, s, __VA_ARGS__);                      \
    else if (lg_ == 3) hipLaunchKernelGGL(KERNEL<3>, grid_, dim3(256), 0, s, __VA_ARGS__);                      \
    else hipLaunchKernelGGL(KERNEL<4>, grid_, dim3(256), 0, s, __VA_ARGS__);                                    \
  } while (0)

}  // namespace gmg

using namespace gmg;

template <class F>
static gmg_status fv_guard(F&& f) {
  try {
    set_error_message("");
    return f();
  } catch (const Error& e) {
    set_error_message(e.msg);
    return e.code;
  }
}

extern "C" int64_t gmg_fv_nnz(int n, int dim) {
  if (n < 1 || (dim != 2 && dim != 3)) return -1;
  const int64_t N = dim == 2 ? (int64_t)n * n : (int64_t)n * n * n;
  return (int64_t)(2 * dim + 1) * N - (int64_t)2 * dim * (N / n);
}

extern "C" gmg_status gmg_fv_assemble(int n, int dim, const double* kappa, const double* vel_x,
                                      const double* vel_y, const double* vel_z, int32_t* rowptr, int32_t* col,
                                      double* val, void* stream) {
  return fv_guard([&]() -> gmg_status {
    if (n < 1 || (dim != 2 && dim != 3) || !kappa || !vel_x || !vel_y || (dim == 3 && !vel_z) || !rowptr ||
        !col || !val)
      return GMG_ERR_INVALID_ARG;
    const int64_t N64 = dim == 2 ? (int64_t)n * n : (int64_t)n * n * n;
    if (N64 >= (1LL << 31) / 8) return GMG_ERR_INVALID_ARG;
    const int N = (int)N64;
    hipStream_t s = (hipStream_t)stream;
    launch_fv_fill(n, dim, kappa, vel_x, vel_y, vel_z, rowptr, col, val, N, s);
    HIPCK(hipStreamSynchronize(s));
    return GMG_OK;
  });
}

extern "C" gmg_status gmg_fv_assemble_noalloc(int n, int dim, const double* kappa, const double* vel_x,
                                              const double* vel_y, const double* vel_z, int32_t* rowptr,
                                              int32_t* col, double* val, void* stream) {
  return fv_guard([&]() -> gmg_status {
    // every argument is checked before any device call
    if (n < 1 || (dim != 2 && dim != 3) || !kappa || !vel_x || !vel_y || (dim == 3 && !vel_z) || !rowptr ||
        !col || !val)
      return GMG_ERR_INVALID_ARG;
    const int64_t N64 = dim == 2 ? (int64_t)n * n : (int64_t)n * n * n;
    if (N64 > GMG_FV_NOALLOC_MAX_CELLS) {
      set_error_message("gmg_fv_assemble_noalloc: " + std::to_string(N64) + " cells exceed the limit of " +
                        std::to_string((long long)GMG_FV_NOALLOC_MAX_CELLS));
      return GMG_ERR_INVALID_ARG;
    }
    launch_fv_fill(n, dim, kappa, vel_x, vel_y, vel_z, rowptr, col, val, (int)N64, (hipStream_t)stream);
    return GMG_OK;
  });
}

extern "C" gmg_status gmg_fv_kappa_grad(int n, int dim, const double* kappa, const double* lambda,
                                        const double* x, int nrhs, double* grad, void* stream) {
  return fv_guard([&]() -> gmg_status {
    if (n < 1 || (dim != 2 && dim != 3) || !kappa || !lambda || !x || !grad || nrhs < 1)
      return GMG_ERR_INVALID_ARG;
    const int N = dim == 2 ? n * n : n * n * n;
    hipStream_t s = (hipStream_t)stream;
    GMG_FV_LANES(nrhs, k_fv_grad, N, n, dim, kappa, lambda, x, nrhs, grad, N);
    HIPCK(hipGetLastError());
    HIPCK(hipStreamSynchronize(s));
    return GMG_OK;
  });
}

extern "C" gmg_status gmg_pattern_grad(int64_t n, const int32_t* rowptr, const int32_t* col, const double* lambda,
                                       const double* x, int nrhs, double* gval, void* stream) {
  return fv_guard([&]() -> gmg_status {
    if (n < 1 || !rowptr || !col || !lambda || !x || !gval || nrhs < 1) return GMG_ERR_INVALID_ARG;
    hipStream_t s = (hipStream_t)stream;
    GMG_FV_LANES(nrhs, k_pattern_grad, n, (int)n, rowptr, col, lambda, x, nrhs, gval);
    HIPCK(hipGetLastError());
    HIPCK(hipStreamSynchronize(s));
    return GMG_OK;
  });
}
