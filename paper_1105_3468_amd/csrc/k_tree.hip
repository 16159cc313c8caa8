// Triangular solves over the nested-dissection tree (coarse ILUT factors).
//
// With the coarse unknowns numbered by nested dissection, an elimination only
// creates entries between a row and the rows of its own tree node or of the
// node's descendants (strictly lower part) or ancestors (strictly upper
// part).  So a lower solve can run bottom-up over the tree and an upper solve
// top-down: a node's rows are x = T^{-1} (rhs - E x_outside), where T is the
// node's diagonal block and the rows outside it that E refers to are final by
// then.  The diagonal blocks of separators are nearly dense after fill, and a
// substitution through one costs a dependent step per row; instead T^{-1} is
// formed once at setup (dense, zeros in the other triangle; column-major up to
// 64 rows, packed by the slices that read it beyond) and the solve applies it as
// a matrix-vector product, whose rows are independent and are split over several
// workgroups.
//
// One launch runs a whole solve as a list of tasks in tree order (lower:
// heights ascending; upper: descending).  For a node with terms outside it,
// helper tasks first compute rhs - (those terms) for slices of its rows,
// polling the published results of other nodes (value-as-flag, as in the
// sweeps), and publish them to a staging vector that doubles as its own
// ready flag; the node's slice tasks poll them, multiply, and publish their
// rows.  Every task waits only on earlier tasks.  Workgroups start in order on
// each XCD, so a solve that has the device, or shares it with kernels that do
// not wait, makes progress; beside another kernel that polls, each could fill
// the XCD that the other's next workgroup waits for.  Every wait is bounded: it
// then ends with an error.
#include <algorithm>

#include "gmg_internal.h"
#include "kcommon.h"

namespace gmg {

constexpr int TREE_THREADS = 256;
constexpr int TREE_BATCH = 8;   // helper loads in flight per lane
constexpr int TREE_MBATCH = 16; // inverse-block loads in flight per lane

template <class T>
__device__ __forceinline__ T tree_poll(const T* p, int* abort_flag, uint64_t limit) {
  T v = ld_agent(p);
  if (!is_sentinel(v)) return v;
  const uint64_t t0 = wall_clock64();
  unsigned it = 0;
#pragma clang loop unroll(disable)
  while (is_sentinel(v)) {
    __builtin_amdgcn_s_sleep(1);
    v = ld_agent(p);
    if (is_sentinel(v) && (++it & 63u) == 0) {
      if (ld_agent(abort_flag)) return (T)__builtin_nan("");
      if (wall_clock64() - t0 > limit) {
        st_agent(abort_flag, 1);
        return (T)__builtin_nan("");
      }
    }
  }
  return v;
}

// task[8t ..]: helper: 0, lo, s, r0, r1, node, 1, log2 G
//               slice:  1, lo, s, a, b, node, has_ext | log2 R << 1, slices
//               pair:   2, lo, s, node, lo', s', node', 0 (lower solves): two
//                       nodes of at most 64 rows without outside entries, one
//                       slice each, one per half of the workgroup (s' = 0:
//                       none), so that a tree's many leaves fit the workgroups
//                       resident at once
template <class T, class TR, bool LOWER>
__global__ __launch_bounds__(TREE_THREADS, 6) void k_tree(const int* __restrict__ task,
                                                          const int64_t* __restrict__ boff,
                                                          const int* __restrict__ erp, const int* __restrict__ ecol,
                                                          const T* __restrict__ eval, const T* __restrict__ inv,
                                                          int* ncount, const TR* rhs, T* out, T* ext, TR* reset_rhs,
                                                          int* abort_flag, uint64_t limit) {
  extern __shared__ __align__(16) unsigned char tree_smem[];
  T* y = reinterpret_cast<T*>(tree_smem);
  const int* tk = task + 8 * (size_t)blockIdx.x;
  const int kind = tk[0];

  if (kind == 0) {
    // ------------------------------------------------------------ helper
    // rows [r0, r1) of the node: ext[r] = rhs[r] - sum over entries outside
    // the node, G lanes per row, TREE_BATCH loads in flight per lane, pending
    // values polled as a group
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int r0 = tk[3], r1 = tk[4], lg = tk[7];
    const int G = 1 << lg, per_wave = 64 >> lg;
    const int slot = lane >> lg, sub = lane & (G - 1);
    for (int rb = r0 + wave * per_wave; rb < r1; rb += (TREE_THREADS / 64) * per_wave) {
      const int r = rb + slot;
      const bool active = r < r1;
      T acc = (T)0;
      TR rh = (TR)0;
      if (active && sub == 0) rh = rhs[r];
      if (active) {
        const int q1 = erp[r + 1];
        for (int q = erp[r] + sub; q < q1; q += G * TREE_BATCH) {
          int c[TREE_BATCH];
          T v[TREE_BATCH], a[TREE_BATCH];
          unsigned need = 0;
#pragma unroll
          for (int u = 0; u < TREE_BATCH; ++u) {
            const int qq = q + u * G < q1 ? q + u * G : q1 - 1;
            c[u] = ecol[qq];
            a[u] = eval[qq];
            if (q + u * G < q1) need |= 1u << u;
          }
#pragma unroll
          for (int u = 0; u < TREE_BATCH; ++u) v[u] = ld_agent(out + c[u]);
#pragma unroll
          for (int u = 0; u < TREE_BATCH; ++u)
            if ((need >> u & 1u) && is_sentinel(v[u])) v[u] = tree_poll(out + c[u], abort_flag, limit);
#pragma unroll
          for (int u = 0; u < TREE_BATCH; ++u)
            if (need >> u & 1u) acc += a[u] * v[u];
        }
      }
      for (int off = G >> 1; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
      if (active && sub == 0) {
        T e = (T)rh - acc;
        if (is_sentinel(e)) e = (T)__builtin_nan("");
        st_agent(ext + r, e);
        if (reset_rhs) reset_rhs[r] = sentinel_of<TR>(0);
      }
    }
    return;
  }

  // ------------------------------------------------------- node slice
  // rows [a, b) of the node: x = Tinv[a:b, cols] y[cols], cols = [0, b)
  // (lower) or [a, s) (upper); R rows per slice, G = 256 / R column groups,
  // each thread one row and one group's columns, then a fixed-order sum of the
  // groups' partial sums
  // a pair task: threads [0, 128) take the first node, [128, 256) the second
  // (lower solves only: an upper solve's nodes without outside entries are
  // the few at the top of the tree)
  const bool pair = LOWER && kind == 2;
  const int half = pair ? (int)(threadIdx.x >> 7) : 0;
  const int tid = pair ? (int)(threadIdx.x & 127) : (int)threadIdx.x;
  const int nthr = pair ? TREE_THREADS / 2 : TREE_THREADS;
  const int lo = tk[1 + (pair ? 3 * half : 0)], s = tk[2 + (pair ? 3 * half : 0)];
  const int a = pair ? 0 : tk[3], b = pair ? s : tk[4], node = pair ? tk[3 + 3 * half] : tk[5];
  const int has_ext = pair ? 0 : tk[6] & 1, lgR = pair ? 6 : tk[6] >> 1, nsl = pair ? 1 : tk[7];
  const int j0 = LOWER ? 0 : a, j1 = LOWER ? b : s;
  __shared__ T part_all[TREE_THREADS];
  __shared__ int last_slice[2];
  T* part = part_all + half * (TREE_THREADS / 2);
  y += half * 64;  // a pair's second node: y holds at least 128 values then
  const int R = 1 << lgR, G = nthr >> lgR;
  const int rl = tid & (R - 1), cg = tid >> lgR;
  const int i = a + rl < b ? a + rl : a;
  const int ncol = j1 - j0, cw = (ncol + G - 1) / G;
  const int jg = j0 + cg * cw, jge = jg + cw < j1 ? jg + cw : j1;
  // the inverse of a triangular block is triangular: row i has no terms
  // past its diagonal (lower: columns <= i, upper: columns >= i), so each
  // thread reads only its row's side of the diagonal
  const int jb = LOWER ? jg : (jg > i ? jg : i);
  const int je = LOWER ? (jge < i + 1 ? jge : i + 1) : jge;
  // columns of the slice's rows: `cs` apart (tree_packed)
  const bool packed = s > kTreeLeaf;
  const int cs = packed ? R : s;
  const T* col = inv + boff[node] + (packed ? (int64_t)a * s + (i - a) : (int64_t)i);
  // the first batch of the block's entries does not depend on the
  // right-hand side: in flight while the inputs are awaited
  T m[TREE_MBATCH];
#pragma unroll
  for (int u = 0; u < TREE_MBATCH; ++u) m[u] = jb + u < je ? col[(int64_t)(jb + u) * cs] : (T)0;
  // the slice's right-hand side: all loads issued first, pending ones polled
  // (s <= kTreeMaxRows, checked on the host)
  constexpr int YK = kTreeMaxRows / TREE_THREADS;
  {
    T v[YK];
#pragma unroll
    for (int k = 0; k < YK; ++k) {
      const int r = j0 + tid + k * nthr;
      if (r < j1) v[k] = has_ext ? ld_agent(ext + lo + r) : (T)rhs[lo + r];
    }
#pragma unroll
    for (int k = 0; k < YK; ++k) {
      const int r = j0 + tid + k * nthr;
      if (r < j1) {
        if (has_ext && is_sentinel(v[k])) v[k] = tree_poll(ext + lo + r, abort_flag, limit);
        y[r - j0] = v[k];
      }
    }
  }
  __syncthreads();
  T acc = (T)0;
#pragma unroll
  for (int u = 0; u < TREE_MBATCH; ++u)
    if (jb + u < je) acc += m[u] * y[jb + u - j0];
  for (int j = jb + TREE_MBATCH; j < je; j += TREE_MBATCH) {
#pragma unroll
    for (int u = 0; u < TREE_MBATCH; ++u) m[u] = j + u < je ? col[(int64_t)(j + u) * cs] : (T)0;
#pragma unroll
    for (int u = 0; u < TREE_MBATCH; ++u)
      if (j + u < je) acc += m[u] * y[j + u - j0];
  }
  part[tid] = acc;
  __syncthreads();
  if (tid < R && a + tid < b) {
    T x = (T)0;
    for (int g = 0; g < G; ++g) x += part[g * R + tid];
    if (!isfinite(x)) {
      // a zero entry's term is no term, whatever the value beside it
      const int k1 = LOWER ? a + tid + 1 : j1;
      x = (T)0;
      for (int k = LOWER ? j0 : a + tid; k < k1; ++k)
        if (const T e = inv[boff[node] + (packed ? (int64_t)a * s + tid : (int64_t)(a + tid)) + (int64_t)k * cs];
            e != (T)0)
          x += e * y[k - j0];
    }
    if (is_sentinel(x)) x = (T)__builtin_nan("");
    st_agent(out + lo + a + tid, x);
  }
  // the last slice of the node to get here resets what the slices read (the
  // counter is left at zero for the next solve).  Every slice has its inputs
  // in LDS by now; the count comes after the results are published so that
  // its round trip is not on the dependency chain, and a node of one slice
  // needs none.
  if (tid == 0) {
    bool last = true;
    if (nsl > 1) {
      const int t = atomicAdd(ncount + node, 1);
      last = t == nsl - 1;
      if (last) st_agent(ncount + node, 0);
    }
    last_slice[half] = last;
  }
  __syncthreads();
  if (last_slice[half]) {
    for (int r = tid; r < s; r += nthr) {
      if (has_ext) st_agent(ext + lo + r, sentinel_of<T>(0));
      else if (reset_rhs) reset_rhs[lo + r] = sentinel_of<TR>(0);
    }
  }
}

static uint64_t tree_limit_ticks() {
  static uint64_t ticks = 0;
  if (!ticks) {
    int dev = 0, khz = 0;
    (void)hipGetDevice(&dev);
    if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess || khz <= 0) {
      (void)hipGetLastError();
      khz = 100000;
    }
    ticks = (uint64_t)khz * 1000ull * 4ull;  // 4 seconds
  }
  return ticks;
}

template <class T>
void launch_tree(const TreeSolve& ts, const void* rhs, bool rhs_is_f64, T* out, T* reset_rhs, T* ext, int* abort_flag,
                 hipStream_t s) {
  if (ts.ntasks == 0) return;
  constexpr bool F32 = sizeof(T) == 4;
  const T* ev = F32 ? (const T*)ts.eval32.p : (const T*)ts.eval.p;
  const T* iv = F32 ? (const T*)ts.inv32.p : (const T*)ts.inv.p;
  const size_t lds = (size_t)std::max(ts.max_rows, 128) * sizeof(T);  // a pair task's two nodes: 2 x 64
  const uint64_t lim = tree_limit_ticks();
#define GMG_TREE(TR_, LO_, RHS_, RESET_)                                                                           \
  do {                                                                                                             \
    static bool attr = false;                                                                                      \
    if (!attr) {                                                                                                   \
      HIPCK(hipFuncSetAttribute(reinterpret_cast<const void*>(&k_tree<T, TR_, LO_>),                               \
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)(kTreeMaxRows * sizeof(double)))); \
      attr = true;                                                                                                 \
    }                                                                                                              \
    hipLaunchKernelGGL((k_tree<T, TR_, LO_>), dim3(ts.ntasks), dim3(TREE_THREADS), lds, s, ts.task.p, ts.boff.p,   \
                       ts.erp.p, ts.ecol.p, ev, iv, ts.ncount.p, (const TR_*)RHS_, out, ext, RESET_, abort_flag,   \
                       lim);                                                                                       \
  } while (0)
#define GMG_TREE_RHS(TR_, RHS_, RESET_)                \
  do {                                                 \
    if (ts.lower) GMG_TREE(TR_, true, RHS_, RESET_);   \
    else GMG_TREE(TR_, false, RHS_, RESET_);           \
  } while (0)
  if (rhs_is_f64 && F32) GMG_TREE_RHS(double, rhs, (double*)nullptr);
  else GMG_TREE_RHS(T, rhs, reset_rhs);
#undef GMG_TREE_RHS
#undef GMG_TREE
  HIPCK(hipGetLastError());
}
template void launch_tree<double>(const TreeSolve&, const void*, bool, double*, double*, double*, int*, hipStream_t);
template void launch_tree<float>(const TreeSolve&, const void*, bool, float*, float*, float*, int*, hipStream_t);

// ------------------------------------------------- several right-hand sides
// The same solve for CW = 4, 8 or 16 columns in one launch, vectors row-major
// (value (r, c) at r * CW + c, columns past the batch's zero).  A node's rows
// are then X = Tinv (B - E X_outside) with CW-column matrices: the product
// with the inverse runs on the matrix cores, every entry of the factor is
// read once for all columns, and a row's values, polled or not, are one
// contiguous piece.  With a workgroup per task and column instead the 16
// columns of a 512^2 grid took 205 + 165 us for the lower and the upper solve,
// most of it workgroups queueing.
//
// ctask[8t ..]: helper: 0, r0, r1, wide, log2 G;  slice: 1, lo, s, a, b, node, has_ext | log2 R << 1, slices
//
// v_mfma_*_16x16x4: lane l holds A[l % 16][l / 16] and B[l / 16][l % 16]; D's
// row of register r is 4 r + l / 16 in FP64, 4 (l / 16) + r in FP32.
typedef double f64x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
template <class T>
struct Mma;
template <>
struct Mma<double> {
  using acc = f64x4;
  static __device__ __forceinline__ acc mul(double a, double b, acc c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int r, int q) { return 4 * r + q; }
};
template <>
struct Mma<float> {
  using acc = f32x4;
  static __device__ __forceinline__ acc mul(float a, float b, acc c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int row(int r, int q) { return 4 * q + r; }
};

constexpr int TREE_HB = 8;   // helper loads in flight per lane
constexpr int TREE_KB = 8;   // products of four columns of the inverse whose operands are in flight together

// Operands of up to NK consecutive products of the four-column steps k, k + 4,
// ...: the values of the right-hand side at rows kk < ke (polled when POLL)
template <class T, int CW, int NK>
__device__ __forceinline__ void cols_operand(const T* y, int k, int ke, int q, int l16, bool poll, int* abort_flag,
                                             uint64_t limit, T (&b)[NK]) {
#pragma unroll
  for (int u = 0; u < NK; ++u) {
    const int kk = k + 4 * u + q;
    const bool in = kk < ke && l16 < CW;
    b[u] = in ? (poll ? ld_agent(y + (size_t)kk * CW + l16) : y[(size_t)kk * CW + l16]) : (T)0;
  }
  if (poll) {
#pragma unroll
    for (int u = 0; u < NK; ++u)
      if (is_sentinel(b[u])) b[u] = tree_poll(y + (size_t)(k + 4 * u + q) * CW + l16, abort_flag, limit);
  }
}

template <class T, bool LOWER, int CW>
__global__ __launch_bounds__(TREE_THREADS, 7) void k_tree_cols(const int* __restrict__ ctask,
                                                            const int64_t* __restrict__ boff,
                                                            const int* __restrict__ erp, const int* __restrict__ ecol,
                                                            const T* __restrict__ eval, const T* __restrict__ inv,
                                                            int* ncount, const T* rhs, T* out, T* ext, T* reset_rhs,
                                                            int* abort_flag, uint64_t limit) {
  constexpr int NT = 4;  // row tiles of a slice at most (a leaf of 64 rows)
  __shared__ T part[TREE_THREADS / 64][NT * 16][CW + 1];
  __shared__ int last_slice;
  const int* tk = ctask + 8 * (size_t)blockIdx.x;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (tk[0] == 0) {
    // helper: ext[r] = rhs[r] - sum over entries outside the node.  CW lanes hold
    // an entry's columns; a wave's 64 / CW such groups are shared by its rows,
    // G to a row, TREE_HB entries in flight each.  `wide`: all four waves share
    // the one row (a long row taken by one wave waits for round after round)
    constexpr int E = 64 / CW, W = TREE_THREADS / 64;
    // past a row's end: load its last entry again (16 columns: branches around
    // the loads cost more, 117 against 97 us on the 512^2 grid) or nothing (4
    // and 8 columns: more such loads in a wave, 64 against 78 us)
    constexpr bool kAll = CW == 16;
    const bool wide = tk[3] != 0;
    const int G = wide ? E : min(1 << tk[4], E), rows = E / G;  // powers of two
    const int c = lane & (CW - 1), slot = lane / CW / G, sub = lane / CW & (G - 1);
    for (int rb = wide ? tk[1] : tk[1] + wave * rows; rb < tk[2]; rb += W * rows) {
      const int r = rb + slot;
      const bool active = r < tk[2];
      const size_t at = (size_t)r * CW + c;
      const T rh = active && sub == 0 ? rhs[at] : (T)0;
      const int q1 = active ? erp[r + 1] : 0, step = (wide ? W : 1) * G * TREE_HB;
      T acc = (T)0;
      for (int q = (active ? erp[r] : 0) + sub + (wide ? wave * E * TREE_HB : 0); q < q1; q += step) {
        int cc[TREE_HB];
        T v[TREE_HB], a[TREE_HB];
#pragma unroll
        for (int u = 0; u < TREE_HB; ++u) {
          const bool in = kAll || q + u * G < q1;
          const int qq = min(q + u * G, q1 - 1);
          cc[u] = in ? ecol[qq] : 0;
          a[u] = in ? eval[qq] : (T)0;
        }
#pragma unroll
        for (int u = 0; u < TREE_HB; ++u)
          v[u] = kAll || q + u * G < q1 ? ld_agent(out + (size_t)cc[u] * CW + c) : (T)0;
#pragma unroll
        for (int u = 0; u < TREE_HB; ++u)
          if (is_sentinel(v[u])) v[u] = tree_poll(out + (size_t)cc[u] * CW + c, abort_flag, limit);
#pragma unroll
        for (int u = 0; u < TREE_HB; ++u)
          if (q + u * G < q1) acc += a[u] * v[u];
      }
      for (int off = CW; off < CW * G; off <<= 1) acc += __shfl_xor(acc, off, 64);
      if (wide) {
        if (sub == 0) part[wave][0][c] = acc;
        __syncthreads();
        acc = (T)0;
#pragma unroll
        for (int w = 0; w < W; ++w) acc += part[w][0][c];
      }
      if (active && sub == 0 && (!wide || wave == 0)) {
        T e = rh - acc;
        if (is_sentinel(e)) e = (T)__builtin_nan("");
        st_agent(ext + at, e);
        if (reset_rhs) reset_rhs[at] = sentinel_of<T>(0);
      }
    }
    return;
  }
  // slice: rows [a, b) of the node, in tiles of 16; the four waves share the
  // columns [k0, k1) of the inverse (its other triangle holds zeros) and their
  // sums are added in order
  const int lo = tk[1], s = tk[2], a = tk[3], b = tk[4], node = tk[5], has_ext = tk[6] & 1, nsl = tk[7];
  const int k0 = LOWER ? 0 : a, k1 = LOWER ? b : s;
  const int per = (k1 - k0 + 15) / 16 * 4;
  const int kb = k0 + wave * per, ke = min(kb + per, k1);
  const int l16 = lane & 15, q = lane >> 4;
  const T* M = inv + boff[node];
  const T* y = (has_ext ? ext : rhs) + (size_t)lo * CW;
  using Acc = typename Mma<T>::acc;
  const int tiles = (b - a + 15) / 16;
  auto store = [&](int t, const Acc& acc) {
    if (l16 < CW) {
#pragma unroll
      for (int r = 0; r < 4; ++r) part[wave][16 * t + Mma<T>::row(r, q)][l16] = acc[r];
    }
  };
  if (tiles > 1) {  // a leaf: at most 64 columns, 16 of them per wave
    T m[NT][4];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const int i = a + 16 * t + l16, kk = kb + 4 * u + q;
        m[t][u] = i < b && kk < ke ? M[(int64_t)kk * s + i] : (T)0;  // not packed
      }
    T v[4];
    cols_operand<T, CW>(y, kb, ke, q, l16, has_ext != 0, abort_flag, limit, v);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      Acc acc = {};
#pragma unroll
      for (int u = 0; u < 4; ++u) acc = Mma<T>::mul(m[t][u], v[u], acc);
      store(t, acc);
    }
  } else {
    const int i = a + l16, lgR = tk[6] >> 1, R = 1 << lgR;
    const bool packed = s > kTreeLeaf;
    const int cs = packed ? R : s;
    const T* col = M + (packed ? (int64_t)(i >> lgR) * R * s + (i & (R - 1)) : (int64_t)i);
    Acc acc = {};
    for (int k = kb; k < ke; k += 4 * TREE_KB) {
      T m[TREE_KB], v[TREE_KB];
      // the inverse's entries are in flight while the inputs are awaited
#pragma unroll
      for (int u = 0; u < TREE_KB; ++u) {
        const int kk = k + 4 * u + q;
        m[u] = i < b && kk < ke ? col[(int64_t)kk * cs] : (T)0;
      }
      cols_operand<T, CW>(y, k, ke, q, l16, has_ext != 0, abort_flag, limit, v);
#pragma unroll
      for (int u = 0; u < TREE_KB; ++u) acc = Mma<T>::mul(m[u], v[u], acc);
    }
    store(0, acc);
  }
  __syncthreads();
  for (int o = threadIdx.x; o < (b - a) * CW; o += TREE_THREADS) {
    const int rr = o / CW, c = o & (CW - 1);
    T x = (T)0;
#pragma unroll
    for (int w = 0; w < TREE_THREADS / 64; ++w) x += part[w][rr][c];
    if (!isfinite(x)) {  // without the terms of zero entries, as in k_tree
      const int i = a + rr, lgR = tk[6] >> 1, R = 1 << lgR, cs = s > kTreeLeaf ? R : s;
      const T* col = M + (s > kTreeLeaf ? (int64_t)(i >> lgR) * R * s + (i & (R - 1)) : (int64_t)i);
      x = (T)0;
      for (int k = k0; k < k1; ++k)
        if (const T e = col[(int64_t)k * cs]; e != (T)0) x += e * ld_agent(y + (size_t)k * CW + c);
    }
    if (is_sentinel(x)) x = (T)__builtin_nan("");
    st_agent(out + (size_t)(lo + a) * CW + o, x);
  }
  // the last slice of the node resets what the slices read (as in k_tree)
  if (threadIdx.x == 0) {
    bool last = true;
    if (nsl > 1) {
      const int t = atomicAdd(ncount + node, 1);
      last = t == nsl - 1;
      if (last) st_agent(ncount + node, 0);
    }
    last_slice = last;
  }
  __syncthreads();
  if (last_slice) {
    for (int o = threadIdx.x; o < s * CW; o += TREE_THREADS) {
      if (has_ext) st_agent(ext + (size_t)lo * CW + o, sentinel_of<T>(0));
      else if (reset_rhs) reset_rhs[(size_t)lo * CW + o] = sentinel_of<T>(0);
    }
  }
}

int tree_cols(int nb) { return nb <= 4 ? 4 : nb <= 8 ? 8 : 16; }

template <class T>
void launch_tree_cols(const TreeSolve& ts, const T* rhs, T* out, T* reset_rhs, T* ext, int* abort_flag, hipStream_t s,
                      int cw) {
  const int list = cw < 16 ? 0 : 1;
  if (ts.nctasks[list] == 0) return;
  constexpr bool F32 = sizeof(T) == 4;
  const T* ev = F32 ? (const T*)ts.eval32.p : (const T*)ts.eval.p;
  const T* iv = F32 ? (const T*)ts.inv32.p : (const T*)ts.inv.p;
  const uint64_t lim = tree_limit_ticks();
#define GMG_TREE_COLS(LO_, CW_)                                                                                      \
  hipLaunchKernelGGL((k_tree_cols<T, LO_, CW_>), dim3(ts.nctasks[list]), dim3(TREE_THREADS), 0, s, ts.ctask[list].p, ts.boff.p,  \
                     ts.erp.p, ts.ecol.p, ev, iv, ts.ncount.p, rhs, out, ext, reset_rhs, abort_flag, lim)
  if (cw == 4) {
    if (ts.lower) GMG_TREE_COLS(true, 4);
    else GMG_TREE_COLS(false, 4);
  } else if (cw == 8) {
    if (ts.lower) GMG_TREE_COLS(true, 8);
    else GMG_TREE_COLS(false, 8);
  } else if (cw == 16) {
    if (ts.lower) GMG_TREE_COLS(true, 16);
    else GMG_TREE_COLS(false, 16);
  } else {
    fail(GMG_ERR_INVALID_ARG, "tree solve: bad column count");
  }
#undef GMG_TREE_COLS
  HIPCK(hipGetLastError());
}
template void launch_tree_cols<double>(const TreeSolve&, const double*, double*, double*, double*, int*, hipStream_t,
                                       int);
template void launch_tree_cols<float>(const TreeSolve&, const float*, float*, float*, float*, int*, hipStream_t, int);

// ---------------------------------------------------------------- setup
// Inverse of a node's diagonal block T (unit diagonal, or diagonal 1/dinv), by
// blocks of 64 rows: the 64 x 64 diagonal blocks first (k_tree_inv_diag),
// then the blocks off the diagonal (k_tree_inv_off), column by column:
//   lower: X_IJ = -D_I sum_{J <= K < I} T_IK X_KJ, I ascending,
//   upper: X_IJ = -D_I sum_{I < K <= J} T_IK X_KJ, I descending,
// D_I the inverse of T_II.  The sums are matrix products and run on the
// matrix cores in FP64 (the same fused multiply-adds as a substitution, in
// another order).  A substitution of one row per step, whatever the node's
// size, took 57 ms for the 2048-row blocks of a 128^3 grid's coarse factor.
constexpr int INV_B = 64;    // rows of a block
constexpr int INV_W = 16;    // columns per workgroup of k_tree_inv_off

// One wave per diagonal block; lane c solves for column c of the inverse, its
// unknowns in registers, T in LDS (every lane reads the same entry).
// itask[8t ..]: first row (of the factor), s, first row in the node, rows, node
template <bool LOWER, bool DIAG>
__global__ __launch_bounds__(INV_B) void k_tree_inv_diag(const int* __restrict__ itask,
                                                         const int64_t* __restrict__ boff,
                                                         const double* __restrict__ blk,
                                                         const double* __restrict__ dinv, double* __restrict__ inv) {
  __shared__ __align__(16) double Tl[INV_B * (INV_B + 1)];
  __shared__ double dl[INV_B];
  const int* t = itask + 8 * (size_t)blockIdx.x;
  const int lo = t[0], s = t[1], b0 = t[2], bs = t[3], node = t[4];
  const int lane = threadIdx.x;
  const double* Tb = blk + boff[node] + (int64_t)b0 * s + b0;
  double* M = inv + boff[node] + (int64_t)b0 * s + b0;
  // the block padded with the identity
  for (int k0 = 0; k0 < INV_B; k0 += 16) {
    double v[16];
#pragma unroll
    for (int u = 0; u < 16; ++u) v[u] = (k0 + u < bs && lane < bs) ? Tb[(int64_t)(k0 + u) * s + lane] : 0.0;
#pragma unroll
    for (int u = 0; u < 16; ++u) Tl[(k0 + u) * INV_B + lane] = v[u];
  }
  if (DIAG) dl[lane] = lane < bs ? dinv[lo + lane] : 1.0;
  __syncthreads();
  double x[INV_B];
#pragma unroll
  for (int i = 0; i < INV_B; ++i) x[i] = i == lane ? 1.0 : 0.0;
#pragma unroll
  for (int step = 0; step < INV_B; ++step) {
    const int k = LOWER ? step : INV_B - 1 - step;
    if (k < bs) {  // the same for every lane
      const double xk = DIAG ? dl[k] * x[k] : x[k];
      x[k] = xk;
      if (LOWER) {
#pragma unroll
        for (int i = k + 1; i < INV_B; ++i) x[i] -= Tl[k * INV_B + i] * xk;
      } else {
#pragma unroll
        for (int i = 0; i < k; ++i) x[i] -= Tl[k * INV_B + i] * xk;
      }
    }
  }
  bool fin = true;
#pragma unroll
  for (int i = 0; i < INV_B; ++i) fin = fin && isfinite(x[i]);
  const bool redo = __any(!fin);
  __syncthreads();
  double* X = Tl + lane * (INV_B + 1);  // column `lane` of the inverse
  if (redo) {
    // an entry overflowed: again, without the terms of zero entries
    for (int i = 0; i < INV_B; ++i) X[i] = i == lane ? 1.0 : 0.0;
    for (int step = 0; step < bs; ++step) {
      const int k = LOWER ? step : bs - 1 - step;
      double xk = X[k];
      if (DIAG && xk != 0.0) X[k] = xk = xk * dl[k];
      if (xk == 0.0) continue;
      for (int i = LOWER ? k + 1 : 0; i < (LOWER ? bs : k); ++i)
        if (const double e = Tb[(int64_t)k * s + i]; e != 0.0) X[i] -= e * xk;
    }
  } else {
#pragma unroll
    for (int i = 0; i < INV_B; ++i) X[i] = x[i];
  }
  __syncthreads();
  if (lane < bs)
    for (int c = 0; c < bs; ++c) M[(int64_t)c * s + lane] = Tl[c * (INV_B + 1) + lane];
}

// INV_W columns of a node's inverse, below (above) their diagonal block.  Four
// waves take 16 rows each of the 64-row block at hand; a wave's operands come
// from T (16 consecutive rows of four columns) and from the columns computed
// so far, which the workgroup wrote itself.
// v_mfma_f64_16x16x4: lane l holds A[l % 16][l / 16], B[l / 16][l % 16] and, in
// register r, D[4 r + l / 16][l % 16].
// itask[8t ..]: s, first column in the node, node
template <bool LOWER>
__global__ __launch_bounds__(256) void k_tree_inv_off(const int* __restrict__ itask, const int64_t* __restrict__ boff,
                                                      const double* __restrict__ blk, double* inv) {
  __shared__ double Ss[INV_B][INV_W + 1];
  const int* t = itask + 8 * (size_t)blockIdx.x;
  const int s = t[0], c0 = t[1], node = t[2];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l16 = lane & 15, kq = lane >> 4;
  const double* T = blk + boff[node];
  double* M = inv + boff[node];
  const int J = c0 / INV_B, nb = (s + INV_B - 1) / INV_B;
  const int c = c0 + l16;
  const bool col = c < s;
  const double* X = M + (int64_t)(col ? c : c0) * s;
  constexpr int KU = 8;  // matrix products whose operands are in flight together
  for (int I = LOWER ? J + 1 : J - 1; LOWER ? I < nb : I >= 0; I += LOWER ? 1 : -1) {
    const int row = I * INV_B + 16 * wave + l16;
    const bool rok = row < s;
    const int k0 = LOWER ? J * INV_B : (I + 1) * INV_B, k1 = LOWER ? I * INV_B : min((J + 1) * INV_B, s);
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    for (int k = k0; k < k1; k += 4 * KU) {
      double a[KU], b[KU];
#pragma unroll
      for (int u = 0; u < KU; ++u) {
        const int kk = k + 4 * u + kq;
        a[u] = rok && kk < k1 ? T[(int64_t)kk * s + row] : 0.0;
        b[u] = col && kk < k1 ? X[kk] : 0.0;
      }
#pragma unroll
      for (int u = 0; u < KU; ++u) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b[u], acc, 0, 0, 0);
    }
    // entries that overflowed: again without the terms of zero entries
    auto again = [&](int i, int q0, int q1, const double* A, auto&& value) {
      double t = 0.0;
      for (int q = q0; q < q1; ++q)
        if (const double e = A[(int64_t)q * s + i]; e != 0.0)
          if (const double v = value(q); v != 0.0) t += e * v;
      return t;
    };
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = I * INV_B + 16 * wave + 4 * r + kq;
      double v = acc[r];
      if (!isfinite(v) && i < s && col) v = again(i, k0, k1, T, [&](int q) { return X[q]; });
      Ss[16 * wave + 4 * r + kq][l16] = v;
    }
    __syncthreads();
    f64x4 x = {0.0, 0.0, 0.0, 0.0};
    double a[INV_B / 4];
#pragma unroll
    for (int u = 0; u < INV_B / 4; ++u) {
      const int kk = I * INV_B + 4 * u + kq;
      a[u] = rok && kk < s ? M[(int64_t)kk * s + row] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < INV_B / 4; ++u)
      x = __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], Ss[4 * u + kq][l16], x, 0, 0, 0);
    if (col) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = I * INV_B + 16 * wave + 4 * r + kq;
        double v = x[r];
        if (!isfinite(v) && i < s)
          v = again(i, I * INV_B, min((I + 1) * INV_B, s), M, [&](int q) { return Ss[q - I * INV_B][l16]; });
        if (i < s) M[(int64_t)c * s + i] = -v;
      }
    }
    __syncthreads();  // the next block reads these rows; Ss is free again
  }
}

// The inverses from the column-major work layout (node k's at woff[k]) to the
// solves' layout in FP64 and FP32.  Nodes above kTreeLeaf rows are packed by
// slices: the R rows of a slice of one column are adjacent, and the columns
// follow, so a slice's workgroup streams one contiguous piece.  (In column-
// major order a slice of 8 rows read 64 bytes of every line, the other half
// going to another slice's workgroup; 16 rows straddled lines.)
// growth (may be null): the largest entry of the inverses with the block's
// columns, and its rows, scaled to a unit diagonal (as float bits)
// ptask[8t ..]: s, first column, columns, node, log2 R
constexpr int PACK_COLS = 16;
__global__ __launch_bounds__(256) void k_tree_pack(const int* __restrict__ ptask, const int64_t* __restrict__ woff,
                                                   const int64_t* __restrict__ boff, const double* __restrict__ work,
                                                   double* __restrict__ inv, float* __restrict__ inv32,
                                                   unsigned* growth) {
  const int* t = ptask + 8 * (size_t)blockIdx.x;
  const int s = t[0], j0 = t[1], nj = t[2], node = t[3], lgR = t[4], R = 1 << lgR;
  const double* W = work + woff[node];
  double* O = inv + boff[node];
  float* O32 = inv32 + boff[node];
  if (growth) {
    unsigned by_col = 0, by_row = 0;  // bits of non-negative floats order like the floats, NaN above them all
    for (int e = threadIdx.x; e < nj * s; e += 256) {
      const int j = j0 + e / s, i = e % s;
      const double v = W[(int64_t)j * s + i];
      if (v == 0.0) continue;
      by_col = max(by_col, __float_as_uint((float)fabs(v / W[(int64_t)j * s + j])));
      by_row = max(by_row, __float_as_uint((float)fabs(v / W[(int64_t)i * s + i])));
    }
    for (int off = 32; off > 0; off >>= 1) {
      by_col = max(by_col, (unsigned)__shfl_xor((int)by_col, off, 64));
      by_row = max(by_row, (unsigned)__shfl_xor((int)by_row, off, 64));
    }
    if ((threadIdx.x & 63) == 0) {
      atomicMax(growth, by_col);
      atomicMax(growth + 1, by_row);
    }
  }
  if (s <= kTreeLeaf) {
    for (int e = threadIdx.x; e < nj * s; e += 256) {
      const double v = W[(int64_t)j0 * s + e];
      O[(int64_t)j0 * s + e] = v;
      O32[(int64_t)j0 * s + e] = (float)v;
    }
    return;
  }
  const int slices = (s + R - 1) >> lgR;
  for (int e = threadIdx.x; e < slices * R * nj; e += 256) {
    const int rr = e & (R - 1), j = (e >> lgR) % nj, q = (e >> lgR) / nj, i = (q << lgR) + rr;
    const double v = i < s ? W[(int64_t)(j0 + j) * s + i] : 0.0;
    const int64_t o = ((int64_t)q * s + j0 + j) * R + rr;
    O[o] = v;
    O32[o] = (float)v;
  }
}

void launch_tree_pack(const int* ptask, int npack, const int64_t* woff, const int64_t* boff, const double* work,
                      double* inv, float* inv32, unsigned* growth, hipStream_t s) {
  if (npack == 0) return;
  hipLaunchKernelGGL(k_tree_pack, dim3(npack), dim3(256), 0, s, ptask, woff, boff, work, inv, inv32, growth);
  HIPCK(hipGetLastError());
}
static_assert(kTreePackCols == PACK_COLS, "packing tasks");

void launch_tree_invert(bool lower, const int64_t* woff, const int* dtask, int ndiag, const int* otask, int noff,
                        const double* blk, const double* dinv, double* inv, hipStream_t s) {
  if (ndiag == 0) return;
#define GMG_INV(LO_, DG_) \
  hipLaunchKernelGGL((k_tree_inv_diag<LO_, DG_>), dim3(ndiag), dim3(INV_B), 0, s, dtask, woff, blk, dinv, inv)
  if (lower) {
    if (dinv) GMG_INV(true, true);
    else GMG_INV(true, false);
    if (noff) hipLaunchKernelGGL(k_tree_inv_off<true>, dim3(noff), dim3(256), 0, s, otask, woff, blk, inv);
  } else {
    if (dinv) GMG_INV(false, true);
    else GMG_INV(false, false);
    if (noff) hipLaunchKernelGGL(k_tree_inv_off<false>, dim3(noff), dim3(256), 0, s, otask, woff, blk, inv);
  }
#undef GMG_INV
  HIPCK(hipGetLastError());
}
static_assert(kTreeInvBlock == INV_B && kTreeInvCols == INV_W, "inversion tasks");

// Setup: scatter a factor's rows (entries q in [rp[r] + skip, rp[r+1])) into
// the dense column-major diagonal blocks (entries inside the row's node) and
// the outside-entry lists (erp from the host's count of the same test).  Eight
// lanes per row read its entries side by side; an outside entry's place is its
// rank among the row's outside entries.  (A thread per row, every load a line
// of its own: 0.8 ms for the 1.9M entries of a 512^2 grid's coarse factor.)
constexpr int FILL_G = 8;
__global__ __launch_bounds__(256) void k_tree_fill(int n, const int* __restrict__ rp, const int* __restrict__ ci,
                                                   const double* __restrict__ v, int skip,
                                                   const int* __restrict__ node_of, const int* __restrict__ nlo,
                                                   const int* __restrict__ nsz, const int64_t* __restrict__ boff,
                                                   const int* __restrict__ erp, double* __restrict__ blk,
                                                   int* __restrict__ ecol, double* __restrict__ eval) {
  const int64_t t = (blockIdx.y * (int64_t)gridDim.x + blockIdx.x) * blockDim.x + threadIdx.x;
  const bool in = t / FILL_G < n;  // whole groups; idle ones take part in the ballots
  const int r = in ? (int)(t / FILL_G) : n - 1, sub = (int)(t % FILL_G);
  const int a = node_of[r], lo = nlo[a], sz = nsz[a];
  double* B = blk + boff[a];
  int e = erp[r];
  const int q0 = rp[r] + skip, q1 = in ? rp[r + 1] : q0;
  const int shift = (threadIdx.x & 63) / FILL_G * FILL_G;
  for (int qb = q0; __any(qb < q1); qb += FILL_G) {
    const int q = qb + sub;
    const bool on = q < q1;
    const int c = on ? ci[q] : 0;
    const double x = on ? v[q] : 0.0;
    const bool inside = on && node_of[c] == a;
    if (inside) B[(int64_t)(c - lo) * sz + (r - lo)] = x;
    const unsigned out = (unsigned)(__ballot(on && !inside) >> shift) & ((1u << FILL_G) - 1u);
    if (on && !inside) {
      const int o = e + __popc(out & ((1u << sub) - 1u));
      ecol[o] = c;
      eval[o] = x;
    }
    e += __popc(out);
  }
}

void launch_tree_fill(int n, const int* rp, const int* ci, const double* v, int skip, const int* node_of,
                      const int* nlo, const int* nsz, const int64_t* boff, const int* erp, double* blk, int* ecol,
                      double* eval, hipStream_t s) {
  if (n <= 0) return;
  const int64_t blocks = ((int64_t)n * FILL_G + 255) / 256, most = 1 << 23;
  const dim3 grid((unsigned)std::min(blocks, most), (unsigned)((blocks + most - 1) / most));
  hipLaunchKernelGGL(k_tree_fill, grid, dim3(256), 0, s, n, rp, ci, v, skip, node_of, nlo, nsz, boff,
                     erp, blk, ecol, eval);
  HIPCK(hipGetLastError());
}

}  // namespace gmg
