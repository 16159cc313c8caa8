// Krylov-subspace vector kernels of FGMRES: block multi-dot products, the
// projections (two reads of the basis per step), norms, scaling and the
// solution update.  Reductions are deterministic (no floating-point
// atomics): every block writes its partial sums and they are added in block
// order, so repeated runs are bitwise identical.  Up to KDEF blocks a column
// the kernel that needs the sums adds the partials in each of its blocks;
// beyond, the last block to finish adds them.  There the partials are
// published like the sweeps' results: relaxed agent-scope stores into a buffer
// reset to a NaN sentinel, polled by the last block, which resets them again.
// No fence is needed; an agent-scope fence writes the whole L2 back and cost
// ~40 us per launch here.
#include <algorithm>

#include "gmg_internal.h"
#include "kcommon.h"

namespace gmg {

constexpr int KB = 256;          // threads per block
constexpr int KGRID = 512;       // blocks of the reduction kernels
constexpr int KMAX = 32;         // vectors per fused register-resident pass
constexpr int KPART = KMAX + 1;  // partial sums per block: a product per vector and a norm
// Up to KDEF blocks a column, the next kernel adds the partials: counting the
// blocks, and the last one's reads, took more than the rest of a small
// reduction (an FGMRES step of a short solve, with the exchanges of wave_sums:
// 64^2 78 -> 70 us, 32^2 in 16 columns 99 -> 90 us).  With the line at 64
// blocks the reads at the start of every block cost more: 512^2 in 16 columns
// (64 blocks each) 685 -> 701 us a step, 160^2 (50 blocks) 128 -> 130.
constexpr int KDEF = 32;
constexpr int KLDS = 2048;       // vectors per LDS-staged pass (longest basis)
// many-vector passes (a basis longer than KMAX)
constexpr int MKB = 512;          // threads per block
constexpr int MROWS = 64;         // rows per chunk (two per thread)
constexpr int MG = MKB / (MROWS / 2);  // vector groups per block
constexpr int MGRID = 256;        // blocks (one per CU)
constexpr int MMAX = 384;         // longest basis they take (24 vectors per thread group)
constexpr int MPIPE2 = 12;        // the same when two products are taken
constexpr int MPARTS = 32;        // thread groups adding the block partials of one vector
constexpr int MPIPE = 16;         // up to this many vectors per thread, the next chunk is loaded early
constexpr int MSTR = MMAX + 8;    // stride of a block's row of partials (one extra slot for a norm)

// Keeps the machine scheduler from sinking the loads issued above it into the
// arithmetic below: without it the compiler reuses one register pair for all
// K basis loads of an element and waits for each in turn.
#define ALL_LOADS_ISSUED() __builtin_amdgcn_sched_barrier(0)

// Sums of the M values a[0 .. M) over the wave's lanes, each added in the order
// of a tree over lane distances 32, 16, .., 1.  At every distance a lane keeps
// half of its values and gives the other half to its partner, so M values
// cost about M + 6 exchanges instead of 6 M (a tree per value spent more on
// LDS permutes than a small reduction on its loads).  Afterwards a lane with
// cnt > 0 holds the sum of value `base` in a[0].
__device__ __forceinline__ double lane_swap(double lo, double hi, int off, bool up) {
  if (off == 32 || off == 16) {
    // lanes without bit `off` take lo + their partner's lo, the others hi
    const uint64_t x = __builtin_bit_cast(uint64_t, lo), y = __builtin_bit_cast(uint64_t, hi);
    uint32_t xl = (uint32_t)x, xh = (uint32_t)(x >> 32), yl = (uint32_t)y, yh = (uint32_t)(y >> 32);
    if (off == 32) {
      const auto l = __builtin_amdgcn_permlane32_swap(xl, yl, false, false);
      const auto h = __builtin_amdgcn_permlane32_swap(xh, yh, false, false);
      xl = l[0], yl = l[1], xh = h[0], yh = h[1];
    } else {
      const auto l = __builtin_amdgcn_permlane16_swap(xl, yl, false, false);
      const auto h = __builtin_amdgcn_permlane16_swap(xh, yh, false, false);
      xl = l[0], yl = l[1], xh = h[0], yh = h[1];
    }
    return __builtin_bit_cast(double, (uint64_t)xh << 32 | xl) + __builtin_bit_cast(double, (uint64_t)yh << 32 | yl);
  }
  return (up ? hi : lo) + __shfl_xor(up ? lo : hi, off, 64);
}
template <int M, int OFF, int K>
__device__ __forceinline__ void wave_sums(double (&a)[K], int lane, int& base, int& cnt) {
  if constexpr (OFF > 0) {
    constexpr int H = (M + 1) / 2;
    const bool up = (lane & OFF) != 0;
#pragma unroll
    for (int i = 0; i < H; ++i) a[i] = lane_swap(a[i], i + H < M ? a[i + H < M ? i + H : i] : 0.0, OFF, up);
    base += up ? H : 0;
    cnt = up ? cnt - H : (cnt < H ? cnt : H);
    wave_sums<H, OFF / 2, K>(a, lane, base, cnt);
  }
}

// sum of the partials p[b * KPART], b < nblk, in block order
__device__ __forceinline__ double sum_parts(const double* __restrict__ p, int nblk) {
  double s = 0.0;
  for (int b0 = 0; b0 < nblk; b0 += 8) {
    double v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = b0 + u < nblk ? p[(size_t)(b0 + u) * KPART] : 0.0;
#pragma unroll
    for (int u = 0; u < 8; ++u) s += v[u];
  }
  return s;
}

// dpart: the blocks' sums are left there, plain stores, for the next kernel
// to add (a reduction of few blocks: counting the blocks and the last one's
// reading cost more than every block of the next kernel adding them).
template <int K>
__device__ __forceinline__ void block_reduce_store(double (&acc)[K], int kcount, double* partial,
                                                   unsigned* counter, double* result, double* dpart = nullptr) {
  __shared__ double sh[KB / 64][K];
  __shared__ bool last;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int base = 0, cnt = K;
  wave_sums<K, 32, K>(acc, lane, base, cnt);
  if (cnt > 0) sh[wave][base] = acc[0];
  __syncthreads();
  if (threadIdx.x < kcount) {
    double s = 0.0;
#pragma unroll
    for (int w = 0; w < KB / 64; ++w) s += sh[w][threadIdx.x];
    if (dpart) {
      dpart[(size_t)blockIdx.x * KPART + threadIdx.x] = s;
    } else {
      if (is_sentinel(s)) s = __builtin_nan("");
      st_agent(&partial[(size_t)blockIdx.x * KPART + threadIdx.x], s);
    }
  }
  if (dpart) return;
  __syncthreads();
  if (threadIdx.x == 0) {
    unsigned t = atomicAdd(counter, 1u);
    last = (t == gridDim.x - 1);
  }
  __syncthreads();
  if (last) {
    // all threads take part: thread t adds blocks part, part + NP, ... of
    // vector k (t = part * K + k), then thread k adds the NP parts in order
    constexpr int NP = KB / K;
    __shared__ double sh2[NP][K];
    const int k = threadIdx.x % K, part = threadIdx.x / K;
    if (part < NP) {
      double s = 0.0;
      if (k < kcount) {
        // 16 partials in flight at a time, added in block order; a partial
        // not yet visible is polled (its block stored it before counting)
        double* pp = partial + k;
        for (unsigned b0 = part; b0 < gridDim.x; b0 += 16 * NP) {
          double v[16];
#pragma unroll
          for (int u = 0; u < 16; ++u) {
            const unsigned b = b0 + u * NP;
            v[u] = b < gridDim.x ? ld_agent(pp + (size_t)b * KPART) : 0.0;
          }
#pragma unroll
          for (int u = 0; u < 16; ++u) {
            const unsigned b = b0 + u * NP;
            if (b < gridDim.x) {
              unsigned spins = 0;
#pragma clang loop unroll(disable)
              while (is_sentinel(v[u])) {
                if (++spins > (1u << 22)) { v[u] = __builtin_nan(""); break; }  // bounded
                __builtin_amdgcn_s_sleep(1);
                v[u] = ld_agent(pp + (size_t)b * KPART);
              }
              s += v[u];
              st_agent(pp + (size_t)b * KPART, sentinel_of<double>(0));
            }
          }
        }
      }
      sh2[part][k] = s;
    }
    __syncthreads();
    if (threadIdx.x < kcount) {
      double s = 0.0;
      for (int q = 0; q < NP; ++q) s += sh2[q][threadIdx.x];
      result[threadIdx.x] = s;
    }
    if (threadIdx.x == 0) *counter = 0u;
  }
}

// result[k] = sum_i V[k][i] w[i], k < K.  The vector count is a compile-time
// constant so the K loads of an element are unconditional and all in flight.
// Batched forms (several independent FGMRES recurrences per launch): column
// c = blockIdx.y works on V + c * vcol, w + c * wcol and writes result +
// c * rcol, with its own block partials and counter.
#define KRYLOV_COLUMN()                                   \
  do {                                                    \
    const size_t col_ = blockIdx.y;                       \
    V += col_ * vcol;                                     \
    w += col_ * wcol;                                     \
    result += col_ * rcol;                                \
    partial += col_ * (size_t)KGRID * KPART;               \
    counter += col_;                                      \
  } while (0)

// Two rows per lane and 16-byte loads; vectors start on 64-row boundaries, and
// their padding is loaded but never counted.
__device__ __forceinline__ double2 ld2(const double* p) { return *reinterpret_cast<const double2*>(p); }

// a value that all lanes share, in scalar registers (32 coefficients in vector
// registers do not fit beside 32 rows of the basis)
__device__ __forceinline__ double uniform(double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)b), hi = __builtin_amdgcn_readfirstlane((uint32_t)(b >> 32));
  return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo);
}

// The projection of up to KMAX vectors is classical Gram-Schmidt twice, the
// second pass of a vector taken together with the first pass of the next one:
// - k_multidot: the newest vector V[K - 1], projected once and normalised, is
//   projected again, v <- (v - sum_k fix[k] V[k]) fix[K - 1], and written back;
//   in the same read h = V^T w with it.
// - k_update: w <- w - V h, and s = V^T w and ||w||^2 in the same read.
// - k_normalize: y = w / ||w||, and the next k_multidot's coefficients
//   fix = s / ||w|| and scale 1 / sqrt(1 - |fix|^2).
// The Hessenberg column is h + s over ||w|| sqrt(1 - |fix|^2), as after a second
// pass.  The preconditioner sees the vector projected once, which a flexible
// method allows: z_j is any vector, and only V has to be orthonormal.  Two
// reads of the basis and one vector written a step; a second pass of its own
// reads it a third time (27 vectors of 16 columns of 262k rows: 201 + 194 +
// 181 us).  Correcting the coefficients with the basis' Gram matrix instead,
// c = (2I - G) h, also takes two reads, but leaves the rounding of w - V c in
// the basis: max |V^T V - I| of 2e-14 where two passes give 7e-16, and 1e-10
// where a step cancels by 1e5.
template <int K>
__global__ __launch_bounds__(KB) void k_multidot(const double* __restrict__ V, size_t ld,
                                                 const double* __restrict__ fix, double* __restrict__ last,
                                                 const double* __restrict__ w, int64_t n, double* partial,
                                                 unsigned* counter, double* result, double* dpart, size_t vcol,
                                                 size_t wcol, size_t rcol, size_t fcol) {
  KRYLOV_COLUMN();
  last += blockIdx.y * vcol;
  if (dpart) dpart += blockIdx.y * (size_t)KDEF * KPART;
  fix += blockIdx.y * fcol;
  double f[K];
#pragma unroll
  for (int k = 0; k < K; ++k) f[k] = K > 1 ? uniform(fix[k]) : 0.0;
  double acc[K];
#pragma unroll
  for (int k = 0; k < K; ++k) acc[k] = 0.0;
  for (int64_t i = 2 * (blockIdx.x * (int64_t)KB + threadIdx.x); i < n; i += 2 * (int64_t)gridDim.x * KB) {
    const double2 wi = ld2(w + i);
    double2 v[K];
#pragma unroll
    for (int k = 0; k < K - 1; ++k) v[k] = ld2(V + k * ld + i);
    double2 u = ld2(last + i);
    ALL_LOADS_ISSUED();
    if constexpr (K > 1) {
#pragma unroll
      for (int k = 0; k < K - 1; ++k) {
        u.x -= f[k] * v[k].x;
        u.y -= f[k] * v[k].y;
      }
      u.x *= f[K - 1];
      u.y *= f[K - 1];
    }
    v[K - 1] = u;
    if (i + 1 < n) {
      if constexpr (K > 1) *reinterpret_cast<double2*>(last + i) = u;
#pragma unroll
      for (int k = 0; k < K; ++k) acc[k] += v[k].x * wi.x + v[k].y * wi.y;
    } else {
      if constexpr (K > 1) last[i] = u.x;
#pragma unroll
      for (int k = 0; k < K; ++k) acc[k] += v[k].x * wi.x;
    }
  }
  block_reduce_store<K>(acc, K, partial, counter, result, dpart);
}

// hpart: h is the sum of the gridDim.x partials k_multidot left there, which
// every block adds; block 0 stores it.
template <int K>
__global__ __launch_bounds__(KB) void k_update(const double* __restrict__ V, size_t ld, double* h,
                                               double* __restrict__ w, int64_t n, double* partial, unsigned* counter,
                                               double* result, const double* __restrict__ hpart, double* dpart,
                                               size_t vcol, size_t wcol, size_t rcol, size_t hcol) {
  KRYLOV_COLUMN();
  h += blockIdx.y * hcol;
  if (dpart) dpart += blockIdx.y * (size_t)KDEF * KPART;
  __shared__ double hs[K];
  if (threadIdx.x < K) {
    if (hpart) {
      const double t = sum_parts(hpart + blockIdx.y * (size_t)KDEF * KPART + threadIdx.x, gridDim.x);
      hs[threadIdx.x] = t;
      if (blockIdx.x == 0) h[threadIdx.x] = t;
    } else {
      hs[threadIdx.x] = h[threadIdx.x];
    }
  }
  __syncthreads();
  double acc[K + 1], hk[K];
#pragma unroll
  for (int k = 0; k < K; ++k) { acc[k] = 0.0; hk[k] = uniform(hs[k]); }
  acc[K] = 0.0;
  for (int64_t i = 2 * (blockIdx.x * (int64_t)KB + threadIdx.x); i < n; i += 2 * (int64_t)gridDim.x * KB) {
    double2 v[K];
    double2 s = ld2(w + i);
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = ld2(V + k * ld + i);
    ALL_LOADS_ISSUED();
#pragma unroll
    for (int k = 0; k < K; ++k) {
      s.x -= hk[k] * v[k].x;
      s.y -= hk[k] * v[k].y;
    }
    if (i + 1 < n) {
      *reinterpret_cast<double2*>(w + i) = s;
#pragma unroll
      for (int k = 0; k < K; ++k) acc[k] += v[k].x * s.x + v[k].y * s.y;
      acc[K] += s.x * s.x + s.y * s.y;
    } else {
      w[i] = s.x;
#pragma unroll
      for (int k = 0; k < K; ++k) acc[k] += v[k].x * s.x;
      acc[K] += s.x * s.x;
    }
  }
  block_reduce_store<K + 1>(acc, K + 1, partial, counter, result, dpart);
}

void red_init(RedWork& rw, hipStream_t s) {
  rw.blocks = KGRID;
  rw.partial.alloc((size_t)KGRID * KPART * KCOLS);
  rw.counter.alloc(KCOLS);
  rw.dpart.alloc((size_t)2 * KDEF * KPART * KCOLS);
  rw.result.alloc(2 * KLDS + 8);
  rw.mpart.alloc((size_t)2 * MGRID * MSTR);
  launch_fill_u32(rw.counter.p, 0u, KCOLS, s);
  launch_fill_f64_bits(rw.partial.p, SENT64, (size_t)KGRID * KPART * KCOLS, s);
}

// Back to the state red_init leaves (every partial the sentinel, counters
// zero), after a reduction may have given up on a partial (its bounded wait
// ran out): a partial that lands later must not be read by the next one.
void red_reset(RedWork& rw, hipStream_t s) {
  launch_fill_u32(rw.counter.p, 0u, KCOLS, s);
  launch_fill_f64_bits(rw.partial.p, SENT64, (size_t)KGRID * KPART * KCOLS, s);
}

// Blocks of a reduction over n rows in nb columns: two rows a lane, at most
// KGRID blocks a column and, for a batch, four blocks a CU in all (every block
// ends with a reduction per vector: 16 columns of 262k rows in 512 blocks each
// spent most of their time there).
static unsigned red_grid(int64_t n, int nb = 1) {
  int64_t g = (n + 2 * KB - 1) / (2 * KB);
  const int64_t cap = nb > 1 ? std::max(32, 1024 / nb) : KGRID;
  if (g > cap) g = cap;
  if (g < 1) g = 1;
  return (unsigned)g;
}

// The partials of k_multidot (which 0) and k_update (which 1) where the
// next kernel adds them: up to KDEF blocks a column.
static double* deferred(RedWork& rw, int64_t n, int nb, int which) {
  return red_grid(n, nb) <= KDEF ? rw.dpart.p + (size_t)which * KDEF * KPART * KCOLS : nullptr;
}

// launch KERNEL<kc> for 1 <= kc <= 32
#define GMG_K4(KERNEL, B, ...)                                           \
  case B + 1: hipLaunchKernelGGL(KERNEL<B + 1>, __VA_ARGS__); break;    \
  case B + 2: hipLaunchKernelGGL(KERNEL<B + 2>, __VA_ARGS__); break;    \
  case B + 3: hipLaunchKernelGGL(KERNEL<B + 3>, __VA_ARGS__); break;    \
  case B + 4: hipLaunchKernelGGL(KERNEL<B + 4>, __VA_ARGS__); break;
#define GMG_DISPATCH_K(kc, KERNEL, ...)                                                                   \
  do {                                                                                                    \
    switch (kc) {                                                                                         \
      GMG_K4(KERNEL, 0, __VA_ARGS__) GMG_K4(KERNEL, 4, __VA_ARGS__) GMG_K4(KERNEL, 8, __VA_ARGS__)         \
      GMG_K4(KERNEL, 12, __VA_ARGS__) GMG_K4(KERNEL, 16, __VA_ARGS__) GMG_K4(KERNEL, 20, __VA_ARGS__)      \
      GMG_K4(KERNEL, 24, __VA_ARGS__) GMG_K4(KERNEL, 28, __VA_ARGS__)                                     \
      default: fail(GMG_ERR_INVALID_ARG, "vector count out of range");                                    \
    }                                                                                                     \
  } while (0)

static void check_cols(const BatchCols& bc) {
  if (bc.nb < 1 || bc.nb > KCOLS) fail(GMG_ERR_INVALID_ARG, "Krylov kernels: bad column count");
}
void launch_multidot(double* V, size_t ld, int k, const double* fix, const double* w, int64_t n, RedWork& rw,
                     double* result, hipStream_t s, const BatchCols& bc) {
  if (k < 1 || k > KMAX) fail(GMG_ERR_INVALID_ARG, "multidot: bad vector count");
  check_cols(bc);
  GMG_DISPATCH_K(k, k_multidot, dim3(red_grid(n, bc.nb), bc.nb), dim3(KB), 0, s, V, ld, fix, V + (size_t)(k - 1) * ld,
                 w, n, rw.partial.p, rw.counter.p, result, deferred(rw, n, bc.nb, 0), bc.vcol, bc.wcol, bc.rcol,
                 bc.fcol);
  HIPCK(hipGetLastError());
}
void launch_update(const double* V, size_t ld, int k, double* h, double* w, int64_t n, RedWork& rw, double* result,
                   hipStream_t s, const BatchCols& bc) {
  if (k < 1 || k > KMAX) fail(GMG_ERR_INVALID_ARG, "update: bad vector count");
  check_cols(bc);
  GMG_DISPATCH_K(k, k_update, dim3(red_grid(n, bc.nb), bc.nb), dim3(KB), 0, s, V, ld, h, w, n, rw.partial.p,
                 rw.counter.p, result, deferred(rw, n, bc.nb, 0), deferred(rw, n, bc.nb, 1), bc.vcol, bc.wcol, bc.rcol,
                 bc.hcol);
  HIPCK(hipGetLastError());
}

// v <- (v - sum_{k < row} fix[k] V[k]) fix[row], the newest vector V[row] = v
// projected again, where no k_multidot does it (KMAX vectors before it)
__global__ __launch_bounds__(KB) void k_again(double* V, size_t ld, int row, const double* __restrict__ fix,
                                              int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)KB + threadIdx.x; i < n; i += (int64_t)gridDim.x * KB) {
    double u = V[(size_t)row * ld + i];
#pragma unroll 16
    for (int k = 0; k < row; ++k) u -= fix[k] * V[(size_t)k * ld + i];
    V[(size_t)row * ld + i] = u * fix[row];
  }
}
void launch_again(double* V, size_t ld, int row, const double* fix, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  const unsigned g = (unsigned)std::min<int64_t>(8192, (n + KB - 1) / KB);
  hipLaunchKernelGGL(k_again, dim3(g), dim3(KB), 0, s, V, ld, row, fix, n);
  HIPCK(hipGetLastError());
}

__global__ __launch_bounds__(KB) void k_norm2(const double* __restrict__ x, int64_t n, double* partial,
                                              unsigned* counter, double* result, size_t xcol, size_t rcol) {
  x += blockIdx.y * xcol;
  result += blockIdx.y * rcol;
  partial += blockIdx.y * (size_t)KGRID * KPART;
  counter += blockIdx.y;
  double acc[1] = {0.0};
  for (int64_t i = blockIdx.x * (int64_t)KB + threadIdx.x; i < n; i += (int64_t)gridDim.x * KB) {
    const double v = x[i];
    acc[0] += v * v;
  }
  block_reduce_store<1>(acc, 1, partial, counter, result);
}
void launch_norm2(const double* x, int64_t n, RedWork& rw, double* result, hipStream_t s, int nb, size_t xcol,
                  size_t rcol) {
  if (nb < 1 || nb > KCOLS) fail(GMG_ERR_INVALID_ARG, "norm2: bad column count");
  hipLaunchKernelGGL(k_norm2, dim3(red_grid(n, nb), nb), dim3(KB), 0, s, x, n, rw.partial.p, rw.counter.p, result, xcol,
                     rcol);
  HIPCK(hipGetLastError());
}

// y_c = x_c / sqrt(nrm2[c * rcol]) for the columns c < nb (zero when the
// norm is zero); x_c = x + c * xcol, y_c = y + c * ycol
__global__ void k_normalize_cols(const double* __restrict__ x, size_t xcol, const double* __restrict__ nrm2,
                                 size_t rcol, double* __restrict__ y, size_t ycol, int64_t n) {
  const double nv = nrm2[blockIdx.y * rcol];
  const double hn = sqrt(nv);
  const double a = hn != 0.0 ? 1.0 / hn : 0.0;
  x += blockIdx.y * xcol;
  y += blockIdx.y * ycol;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    y[i] = a * x[i];
}
void launch_normalize_cols(const double* x, size_t xcol, const double* nrm2, size_t rcol, double* y, size_t ycol,
                           int64_t n, int nb, hipStream_t s) {
  if (n <= 0) return;
  int64_t g = (n + 255) / 256;
  if (g > 2048) g = 2048;
  hipLaunchKernelGGL(k_normalize_cols, dim3((unsigned)g, nb), dim3(256), 0, s, x, xcol, nrm2, rcol, y, ycol, n);
  HIPCK(hipGetLastError());
}

__global__ void k_scale(const double* __restrict__ x, double a, double* __restrict__ y, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    y[i] = a * x[i];
}
void launch_scale(const double* x, double a, double* y, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  int64_t g = (n + 255) / 256;
  if (g > 8192) g = 8192;
  hipLaunchKernelGGL(k_scale, dim3((unsigned)g), dim3(256), 0, s, x, a, y, n);
  HIPCK(hipGetLastError());
}

// y = x / ||x|| (zero when the norm is zero) and the coefficients of its second
// projection, from dots[0..row) = V^T x and dots[row] = ||x||^2: fix[i] = dots[i] /
// ||x||, fix[row] = 1 / sqrt(1 - |fix|^2) (zero when x lies in the basis).  The
// step's column goes to the host from here as well (a copy of its own cost 3 us
// a step): host[0..row) = h, host[row..2 row) = dots and host[2 row] =
// ||x||^2 (1 - |fix|^2).  parts: dots is the sum of the nparts partials k_update
// left there.  gram (may be null): y's row of the basis' Gram matrix, whose
// vectors up to here are orthonormal.  Column blockIdx.y of a batch.
__global__ void k_normalize(const double* __restrict__ x, double* __restrict__ y, int64_t n, int row,
                            const double* __restrict__ dots, double* __restrict__ fix, double* __restrict__ gram,
                            size_t ldg, const double* __restrict__ h, double* __restrict__ host,
                            const double* __restrict__ parts, int nparts, size_t xcol, size_t ycol, size_t dcol,
                            size_t fcol, size_t hcol) {
  x += blockIdx.y * xcol;
  y += blockIdx.y * ycol;
  dots += blockIdx.y * dcol;
  if (parts) parts += blockIdx.y * (size_t)KDEF * KPART;
  const double nv = parts ? sum_parts(parts + row, nparts) : dots[row];
  const double hn = sqrt(nv);
  const double a = hn != 0.0 ? 1.0 / hn : 0.0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    y[i] = a * x[i];
  if (blockIdx.x == 0) {
    __shared__ double sq[KMAX];
    fix += blockIdx.y * fcol;
    h += blockIdx.y * hcol;
    host += blockIdx.y * hcol;
    const int i = threadIdx.x;
    if (i < row) {
      const double d = parts ? sum_parts(parts + i, nparts) : dots[i];
      const double f = d * a;
      fix[i] = f;
      sq[i] = f * f;
      host[i] = h[i];
      host[row + i] = d;
      if (gram) {
        gram[(size_t)row * ldg + i] = 0.0;
        gram[(size_t)i * ldg + row] = 0.0;
      }
    }
    __syncthreads();
    if (i == 0) {
      double rest = 1.0;
      for (int k = 0; k < row; ++k) rest -= sq[k];
      if (rest < 0.0) rest = 0.0;
      fix[row] = rest > 0.0 ? 1.0 / sqrt(rest) : 0.0;
      host[2 * row] = nv * rest;
      if (gram) gram[(size_t)row * ldg + row] = 1.0;
    }
  }
}
void launch_normalize(const double* x, double* y, int64_t n, int row, const double* dots, double* fix, double* gram,
                      size_t ldg, const double* h, double* host, RedWork& rw, hipStream_t s, const BatchCols& bc) {
  if (n <= 0) return;
  if (row < 1 || row > KMAX) fail(GMG_ERR_INVALID_ARG, "normalize: bad vector count");
  check_cols(bc);
  const double* parts = deferred(rw, n, bc.nb, 1);
  const int64_t g = std::min<int64_t>((n + 255) / 256, 8192 / bc.nb);
  hipLaunchKernelGGL(k_normalize, dim3((unsigned)g, bc.nb), dim3(256), 0, s, x, y, n, row, dots, fix, gram, ldg, h,
                     host, parts, parts ? (int)red_grid(n, bc.nb) : 0, bc.wcol, bc.vcol, bc.rcol, bc.fcol, bc.hcol);
  HIPCK(hipGetLastError());
}

// The same for a basis of more than KMAX vectors: y's Gram row, G[row][i] =
// G[i][row] = dots[i] / ||x|| (i < row, when have_dots: else the next projection
// takes it), takes the place of a second projection, and the column is
// host[0 .. 2 row) = col[0 .. 2 row), host[2 row] = ||x||^2.
__global__ void k_normalize_gram(const double* __restrict__ x, double* __restrict__ y, int64_t n, int row,
                                 const double* __restrict__ dots, int have_dots, double* __restrict__ gram,
                                 size_t ldg, const double* __restrict__ col, double* __restrict__ host) {
  const double nv = dots[row];
  const double hn = sqrt(nv);
  const double a = hn != 0.0 ? 1.0 / hn : 0.0;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    y[i] = a * x[i];
  if (blockIdx.x == 0) {
    for (int i = threadIdx.x; i < row && have_dots; i += blockDim.x) {
      const double gv = dots[i] * a;
      gram[(size_t)row * ldg + i] = gv;
      gram[(size_t)i * ldg + row] = gv;
    }
    for (int i = threadIdx.x; i < 2 * row; i += blockDim.x) host[i] = col[i];
    if (threadIdx.x == 0) {
      gram[(size_t)row * ldg + row] = 1.0;
      host[2 * row] = nv;
    }
  }
}
void launch_normalize_gram(const double* x, double* y, int64_t n, int row, const double* dots, bool have_dots,
                           double* gram, size_t ldg, const double* col, double* host, hipStream_t s) {
  if (n <= 0) return;
  const int64_t g = std::min<int64_t>((n + 255) / 256, 8192);
  hipLaunchKernelGGL(k_normalize_gram, dim3((unsigned)g), dim3(256), 0, s, x, y, n, row, dots, have_dots ? 1 : 0,
                     gram, ldg, col, host);
  HIPCK(hipGetLastError());
}

template <int K>
__global__ void k_xupdate(double* __restrict__ x, const double* __restrict__ Z, size_t ld, int kc,
                          const double* __restrict__ c, int64_t n, size_t xcol, size_t zcol, size_t ccol) {
  x += blockIdx.y * xcol;
  Z += blockIdx.y * zcol;
  c += blockIdx.y * ccol;
  double ck[K];
#pragma unroll
  for (int k = 0; k < K; ++k) ck[k] = c[k];
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
    double v[K];
    double s = x[i];
#pragma unroll
    for (int k = 0; k < K; ++k) v[k] = Z[k * ld + i];
    ALL_LOADS_ISSUED();
#pragma unroll
    for (int k = 0; k < K; ++k) s += ck[k] * v[k];
    x[i] = s;
  }
}

// Any number of vectors: w <- w - sum_k h[k] V[k] with the coefficients staged
// in LDS, and result[0] = ||w_new||^2.  Used when the basis has more vectors
// than one fused pass holds in registers.
__global__ __launch_bounds__(KB) void k_update_many(const double* __restrict__ V, size_t ld, int kc,
                                                    const double* __restrict__ h, double* __restrict__ w,
                                                    int64_t n, double* partial, unsigned* counter,
                                                    double* result) {
  __shared__ double hs[KLDS];
  for (int k = threadIdx.x; k < kc; k += KB) hs[k] = h[k];
  __syncthreads();
  double acc[1] = {0.0};
  for (int64_t i = blockIdx.x * (int64_t)KB + threadIdx.x; i < n; i += (int64_t)gridDim.x * KB) {
    double s = w[i];
    int k = 0;
    for (; k + 16 <= kc; k += 16) {
      double v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = V[(size_t)(k + u) * ld + i];
      ALL_LOADS_ISSUED();
#pragma unroll
      for (int u = 0; u < 16; ++u) s -= hs[k + u] * v[u];
    }
    for (; k < kc; ++k) s -= hs[k] * V[(size_t)k * ld + i];
    w[i] = s;
    acc[0] += s * s;
  }
  block_reduce_store<1>(acc, 1, partial, counter, result);
}

void launch_update_many(const double* V, size_t ld, int k, const double* h, double* w, int64_t n, RedWork& rw,
                        double* result, hipStream_t s) {
  if (k < 1 || k > KLDS) fail(GMG_ERR_INVALID_ARG, "update_many: bad vector count");
  hipLaunchKernelGGL(k_update_many, dim3(red_grid(n)), dim3(KB), 0, s, V, ld, k, h, w, n, rw.partial.p,
                     rw.counter.p, result);
  HIPCK(hipGetLastError());
}

// ----------------------------------------------------- many-vector passes
// For a basis longer than one register-resident pass: rows are taken in
// chunks of MROWS; thread (r, g) of a block holds rows 2r and 2r + 1 of the
// chunk (one 16-byte load) for the basis vectors g, g + MG, g + 2 MG, ...
// (PER of them, loads all in flight) and keeps their running dot products in
// registers across chunks.  A chunk reads 512 contiguous bytes of each
// vector: shorter segments of many vectors 8 MB apart cost HBM efficiency.
// The block's per-vector sums (over r, in order) go to mpart[block][k]; a
// second kernel adds the blocks in order.  Rows at or past n (the padding up
// to ld, which is a multiple of 64) are loaded but count as zero.
constexpr int MRT = MROWS / 2;    // threads along a chunk's rows

template <int PER>
__device__ __forceinline__ void many_block_sums(const double (&acc)[PER], int kc, double* mpart) {
  // acc[u] of thread (r, g) belongs to vector g + MG u; sum over r in order
  __shared__ double red[MRT][MG + 1];
  const int r = threadIdx.x % MRT, g = threadIdx.x / MRT;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    if (MG * u >= kc) break;  // the same for every thread of the block
    red[r][g] = acc[u];
    __syncthreads();
    if (threadIdx.x < MG) {
      double t = 0.0;
      for (int q = 0; q < MRT; ++q) t += red[q][threadIdx.x];
      const int k = threadIdx.x + MG * u;
      if (k < kc) mpart[(size_t)blockIdx.x * MSTR + k] = t;
    }
    __syncthreads();
  }
}

// the two rows of thread r in chunk c of V's vector k (zero past n)
__device__ __forceinline__ double2 many_load(const double* __restrict__ V, size_t ld, int k, int64_t i, int64_t n,
                                             bool ok) {
  double2 x = ok ? *reinterpret_cast<const double2*>(V + (size_t)k * ld + i) : make_double2(0.0, 0.0);
  if (i >= n) x.x = 0.0;
  if (i + 1 >= n) x.y = 0.0;
  return x;
}

// h[k] = V[k] . w for k < kc (block partials); the next chunk's loads are
// issued before the current chunk's products.  DUAL: also V[k] . w2, in the
// same read of V (partials mpart2).
template <int PER, bool DUAL>
__global__ __launch_bounds__(MKB) void k_multidot_many(const double* __restrict__ V, size_t ld, int kc,
                                                       const double* __restrict__ w, const double* __restrict__ w2,
                                                       int64_t n, double* __restrict__ mpart,
                                                       double* __restrict__ mpart2) {
  const int r = threadIdx.x % MRT, g = threadIdx.x / MRT;
  double acc[PER], acc2[DUAL ? PER : 1];
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    acc[u] = 0.0;
    if constexpr (DUAL) acc2[u] = 0.0;
  }
  const int64_t nch = (n + MROWS - 1) / MROWS;
  double2 v[PER], wi, wi2;
  auto load = [&](double2 (&x)[PER], double2& xw, double2& xw2, int64_t c) {
    const int64_t i = c * MROWS + 2 * r;
    const bool ok = c < nch;
    xw = many_load(w, 0, 0, i, n, ok);
    if constexpr (DUAL) xw2 = many_load(w2, 0, 0, i, n, ok);
#pragma unroll
    for (int u = 0; u < PER; ++u) x[u] = many_load(V, ld, g + MG * u, i, n, ok && g + MG * u < kc);
  };
  auto add = [&](int u) {
    acc[u] += v[u].x * wi.x + v[u].y * wi.y;
    if constexpr (DUAL) acc2[u] += v[u].x * wi2.x + v[u].y * wi2.y;
  };
  if constexpr (PER <= (DUAL ? MPIPE2 : MPIPE)) {
    load(v, wi, wi2, blockIdx.x);
    for (int64_t ch = blockIdx.x; ch < nch; ch += gridDim.x) {
      double2 vn[PER], wn, wn2;
      load(vn, wn, wn2, ch + gridDim.x);
      ALL_LOADS_ISSUED();
#pragma unroll
      for (int u = 0; u < PER; ++u) {
        add(u);
        v[u] = vn[u];
      }
      wi = wn;
      if constexpr (DUAL) wi2 = wn2;
    }
  } else {
    for (int64_t ch = blockIdx.x; ch < nch; ch += gridDim.x) {
      load(v, wi, wi2, ch);
      ALL_LOADS_ISSUED();
#pragma unroll
      for (int u = 0; u < PER; ++u) add(u);
    }
  }
  many_block_sums<PER>(acc, kc, mpart);
  if constexpr (DUAL) many_block_sums<PER>(acc2, kc, mpart2);
}

// A barrier that orders LDS accesses only: global loads issued before it stay
// in flight (__syncthreads would also wait for them).
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// w <- w - sum_k h[k] V[k]; block partials of V[k] . w_new and of ||w_new||^2
// (slot kc).  A chunk's new w needs every vector
// group's partial sum (two barriers per chunk), so the next chunk's basis
// values (and w) are loaded before them.  The grid walks the rows from the
// last chunk down to the first: the preceding multidot pass walked them
// upwards, so the basis rows it read last are still in the 256 MB memory-side
// cache when this pass starts (block b takes chunks nch-1-b, nch-1-b-grid, ...).
template <int PER>
__global__ __launch_bounds__(MKB) void k_update_dot_many(const double* __restrict__ V, size_t ld, int kc,
                                                         const double* __restrict__ h, double* __restrict__ w,
                                                         int64_t n, double* __restrict__ mpart) {
  __shared__ double pr[MROWS][MG + 1];
  __shared__ double wn[MROWS];
  __shared__ double hs[MMAX];
  const int r = threadIdx.x % MRT, g = threadIdx.x / MRT;
  for (int k = threadIdx.x; k < MG * PER; k += MKB) hs[k] = k < kc ? h[k] : 0.0;
  __syncthreads();
  double acc[PER];
#pragma unroll
  for (int u = 0; u < PER; ++u) acc[u] = 0.0;
  const int64_t nch = (n + MROWS - 1) / MROWS;
  double2 v[PER];
  // step c of the walk is chunk nch - 1 - c
  auto load = [&](double2 (&x)[PER], int64_t c) {
    const int64_t i = (nch - 1 - c) * MROWS + 2 * r;
    const bool ok = c < nch;
#pragma unroll
    for (int u = 0; u < PER; ++u) x[u] = many_load(V, ld, g + MG * u, i, n, ok && g + MG * u < kc);
  };
  // threads 0..MROWS-1 also hold w of their row of the chunk (loaded one
  // chunk ahead, like the basis values)
  auto load_w = [&](int64_t c) {
    const int64_t ii = (nch - 1 - c) * MROWS + threadIdx.x;
    return (threadIdx.x < MROWS && c < nch && ii < n) ? w[ii] : 0.0;
  };
  double wc = load_w(blockIdx.x);
  double nacc = 0.0;  // threads 0..MROWS-1 (wave 0): squares of their rows of w_new
  if constexpr (PER <= MPIPE) load(v, blockIdx.x);
  for (int64_t c = blockIdx.x; c < nch; c += gridDim.x) {
    const int64_t ch = nch - 1 - c;
    double2 vn[PER];
    const double wnext = load_w(c + gridDim.x);
    if constexpr (PER <= MPIPE) load(vn, c + gridDim.x);
    else load(v, c);
    double p0 = 0.0, p1 = 0.0;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const double hk = hs[g + MG * u];
      p0 += hk * v[u].x;
      p1 += hk * v[u].y;
    }
    pr[2 * r][g] = p0;
    pr[2 * r + 1][g] = p1;
    lds_barrier();
    if (threadIdx.x < MROWS) {
      const int64_t ii = ch * MROWS + threadIdx.x;
      double t = 0.0;
      if (ii < n) {
        t = wc;
        for (int q = 0; q < MG; ++q) t -= pr[threadIdx.x][q];
        w[ii] = t;
      }
      wn[threadIdx.x] = t;
      nacc += t * t;
    }
    wc = wnext;
    lds_barrier();
    const double w0 = wn[2 * r], w1 = wn[2 * r + 1];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      acc[u] += v[u].x * w0 + v[u].y * w1;
      if constexpr (PER <= MPIPE) v[u] = vn[u];
    }
  }
  __syncthreads();
  many_block_sums<PER>(acc, kc, mpart);
  static_assert(MROWS == 64, "the norm is reduced within wave 0");
  if (threadIdx.x < MROWS) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) nacc += __shfl_down(nacc, off, 64);
    if (threadIdx.x == 0) mpart[(size_t)blockIdx.x * MSTR + kc] = nacc;
  }
}

// result[k] = sum over blocks b (in order) of mpart[b][k]; 8 vectors per
// block, MPARTS thread groups each adding every MPARTS-th block, then the
// groups in order
__global__ __launch_bounds__(KB) void k_colsum(const double* __restrict__ mpart, int nb, int kc,
                                               double* __restrict__ result) {
  constexpr int NC = KB / MPARTS;
  __shared__ double sh[MPARTS][NC];
  const int c = threadIdx.x % NC, part = threadIdx.x / NC;
  const int k = blockIdx.x * NC + c;
  double s = 0.0;
  if (k < kc) {
    constexpr int IN = MGRID / MPARTS;
    double v[IN];
#pragma unroll
    for (int u = 0; u < IN; ++u) {
      const int b = part + u * MPARTS;
      v[u] = b < nb ? mpart[(size_t)b * MSTR + k] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < IN; ++u) s += v[u];
  }
  sh[part][c] = s;
  __syncthreads();
  if (threadIdx.x < NC && k < kc) {
    double t = 0.0;
    for (int q = 0; q < MPARTS; ++q) t += sh[q][threadIdx.x];
    result[k] = t;
  }
}

static unsigned many_grid(int64_t n) {
  int64_t g = (n + MROWS - 1) / MROWS;
  if (g > MGRID) g = MGRID;
  if (g < 1) g = 1;
  return (unsigned)g;
}

#define GMG_MANY(KERNEL, kc, ...)                                                  \
  do {                                                                             \
    const int per_ = (kc + MG - 1) / MG;                                           \
    if (per_ <= 8) hipLaunchKernelGGL(KERNEL(8), __VA_ARGS__);                     \
    else if (per_ <= 16) hipLaunchKernelGGL(KERNEL(16), __VA_ARGS__);              \
    else hipLaunchKernelGGL(KERNEL(24), __VA_ARGS__);                              \
  } while (0)
#define GMG_DOT(PER_) (k_multidot_many<PER_, false>)
#define GMG_DOT2(PER_) (k_multidot_many<PER_, true>)
#define GMG_UPDATE(PER_) (k_update_dot_many<PER_>)

static_assert(MMAX <= 24 * MG, "the widest many-vector instance holds 24 vectors per group");
int many_max() { return MMAX; }

static void colsum(const double* mpart, unsigned nb, int k, double* result, hipStream_t s) {
  hipLaunchKernelGGL(k_colsum, dim3((k + KB / MPARTS - 1) / (KB / MPARTS)), dim3(KB), 0, s, mpart, (int)nb, k, result);
}

void launch_multidot_many(const double* V, size_t ld, int k, const double* w, int64_t n, RedWork& rw, double* result,
                          hipStream_t s, const double* w2, double* result2) {
  if (k < 1 || k > MMAX) fail(GMG_ERR_INVALID_ARG, "multidot_many: bad vector count");
  const unsigned nb = many_grid(n);
  double* m2 = rw.mpart.p + (size_t)MGRID * MSTR;
  if (w2) {
    GMG_MANY(GMG_DOT2, k, dim3(nb), dim3(MKB), 0, s, V, ld, k, w, w2, n, rw.mpart.p, m2);
    colsum(m2, nb, k, result2, s);
  } else {
    GMG_MANY(GMG_DOT, k, dim3(nb), dim3(MKB), 0, s, V, ld, k, w, w2, n, rw.mpart.p, m2);
  }
  colsum(rw.mpart.p, nb, k, result, s);
  HIPCK(hipGetLastError());
}

void launch_update_dot_many(const double* V, size_t ld, int k, const double* h, double* w, int64_t n, RedWork& rw,
                            double* result, hipStream_t s) {
  if (k < 1 || k > MMAX) fail(GMG_ERR_INVALID_ARG, "update_dot_many: bad vector count");
  const unsigned nb = many_grid(n);
  GMG_MANY(GMG_UPDATE, k, dim3(nb), dim3(MKB), 0, s, V, ld, k, h, w, n, rw.mpart.p);
  colsum(rw.mpart.p, nb, k + 1, result, s);
  HIPCK(hipGetLastError());
}

// Gram-corrected coefficients of one projection: with G = V^T V (unit
// diagonal taken as exact), c = h + d, d_i = -sum_{l != i} G[i][l] h[l],
// i.e. c = (2I - G) h, the first-order form of G^{-1} h and, in exact
// arithmetic, what a second classical Gram-Schmidt pass, V^T (w - V h) = h - G
// h, adds.  It makes up for what the basis has lost, but the rounding of w - V c
// itself, about eps ||w||, stays in the new vector, where a second pass removes
// it: products with the basis are left at eps ||w|| / ||w - V c||, and enter G.
// One wave per coefficient, lanes over l, added in a fixed order.
// `fresh`: the products of the last vector with the basis, when its Gram row
// was not taken as it was formed; used in the row's place and stored there.
__global__ __launch_bounds__(64) void k_gram_coef(int kc, const double* __restrict__ h, double* gram, size_t ldg,
                                                  const double* __restrict__ fresh, double* __restrict__ d,
                                                  double* __restrict__ c) {
  const int i = blockIdx.x, lane = threadIdx.x;
  const double* gi = gram + (size_t)i * ldg;
  double s = 0.0;
  for (int l = lane; l < kc; l += 64) {
    const double g = !fresh ? gi[l] : i == kc - 1 ? fresh[l] : l == kc - 1 ? fresh[i] : gi[l];
    if (l != i) s += g * h[l];
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) s += __shfl_down(s, off, 64);
  if (lane == 0) {
    d[i] = -s;
    c[i] = h[i] + (-s);
    if (fresh && i < kc - 1) {
      gram[(size_t)(kc - 1) * ldg + i] = fresh[i];
      gram[(size_t)i * ldg + kc - 1] = fresh[i];
    }
  }
}
void launch_gram_coef(int kc, const double* h, double* gram, size_t ldg, const double* fresh, double* d, double* c,
                      hipStream_t s) {
  if (kc < 1) return;
  hipLaunchKernelGGL(k_gram_coef, dim3(kc), dim3(64), 0, s, kc, h, gram, ldg, fresh, d, c);
  HIPCK(hipGetLastError());
}
#undef GMG_MANY
#undef GMG_DOT
#undef GMG_DOT2
#undef GMG_UPDATE


__global__ __launch_bounds__(KB) void k_xupdate_many(double* __restrict__ x, const double* __restrict__ Z, size_t ld,
                                                     int kc, const double* __restrict__ c, int64_t n) {
  __shared__ double cs[KLDS];
  for (int k = threadIdx.x; k < kc; k += KB) cs[k] = c[k];
  __syncthreads();
  for (int64_t i = blockIdx.x * (int64_t)KB + threadIdx.x; i < n; i += (int64_t)gridDim.x * KB) {
    double s = x[i];
    int k = 0;
    for (; k + 16 <= kc; k += 16) {
      double v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = Z[(size_t)(k + u) * ld + i];
      ALL_LOADS_ISSUED();
#pragma unroll
      for (int u = 0; u < 16; ++u) s += cs[k + u] * v[u];
    }
    for (; k < kc; ++k) s += cs[k] * Z[(size_t)k * ld + i];
    x[i] = s;
  }
}

__global__ void k_get_col(const double* __restrict__ X, int nrhs, int col, double* __restrict__ x, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    x[i] = X[i * nrhs + col];
}
__global__ void k_set_col(double* __restrict__ X, int nrhs, int col, const double* __restrict__ x, int64_t n) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    X[i * nrhs + col] = x[i];
}
void launch_get_col(const double* X, int nrhs, int col, double* x, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  int64_t g = (n + 255) / 256;
  if (g > 8192) g = 8192;
  hipLaunchKernelGGL(k_get_col, dim3((unsigned)g), dim3(256), 0, s, X, nrhs, col, x, n);
  HIPCK(hipGetLastError());
}
void launch_set_col(double* X, int nrhs, int col, const double* x, int64_t n, hipStream_t s) {
  if (n <= 0) return;
  int64_t g = (n + 255) / 256;
  if (g > 8192) g = 8192;
  hipLaunchKernelGGL(k_set_col, dim3((unsigned)g), dim3(256), 0, s, X, nrhs, col, x, n);
  HIPCK(hipGetLastError());
}

void launch_xupdate(double* x, const double* Z, size_t ld, int k, const double* c, int64_t n, hipStream_t s, int nb,
                    size_t xcol, size_t zcol, size_t ccol) {
  if (n <= 0 || k <= 0) return;
  if (nb < 1 || nb > KCOLS || (nb > 1 && k > KMAX)) fail(GMG_ERR_INVALID_ARG, "xupdate: bad column count");
  int64_t g = (n + 255) / 256;
  if (g > 4096) g = 4096;
  if (nb > 1 && g > 1024) g = 1024;
  if (k <= KMAX) {
    GMG_DISPATCH_K(k, k_xupdate, dim3((unsigned)g, nb), dim3(256), 0, s, x, Z, ld, k, c, n, xcol, zcol, ccol);
  } else {
    if (k > KLDS) fail(GMG_ERR_INVALID_ARG, "xupdate: bad vector count");
    hipLaunchKernelGGL(k_xupdate_many, dim3((unsigned)g), dim3(KB), 0, s, x, Z, ld, k, c, n);
  }
  HIPCK(hipGetLastError());
}

}  // namespace gmg
