// Memory-bound kernels: preconditioner sweeps (batched GEMV and pull
// GEMV over slot lists), BSR SpMV (Algorithms 1/2, line "SpMV") with the
// Newton-basis shift fused in, and the tall-skinny pieces of the s-step
// orthogonalisation (Gram matrices, block updates, triangular scaling).
#include <climits>

#include "internal.h"
#include "kernels_vec.h"
#include "lanes.h"

namespace spand {

template <typename T>
__device__ inline T wsum(T v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// ------------------------------------------------------------------ GEMV
// out[oslot[r]] = sum_c op(A)(r, c) in[islot[c]]   (level 0 of the sweeps)
// Bound by HBM: the leaf inverses are most of the bytes of an apply, and the
// two sweeps need only parts of them.  Only a leaf's unknowns next to a
// separator (0:nb) couple to anything: the forward sweep needs just their
// rows of t = A_ss^-1 x_s, and with the couplings' correction c on them the
// backward sweep's A_ss^-1 (x_s + c) is t + A_ss^-1 c on those rows, a product
// with nb columns.  So n^2 + nb^2 elements are read instead of 2 n^2 (measured
// at Factor::sweeps).
// 5.6 TB/s on matrices of ~220 columns (8128 of them in 292 us), 6.05 TB/s on
// leaves of ~580 (forward and backward, 4096 of them: 811 + 825 us, FP32).  With
// four rows' sums shuffled through LDS and their slots loaded after them, no
// load of the matrix in flight meanwhile: 374, 841 + 903 us.
// One workgroup per band of output rows (GemvChunk).  The input is staged
// in LDS.  Bands of one item may run concurrently, so in == out is not
// allowed (the sweeps alternate between two vectors).
// Products accumulate in float64 for either factor precision: a float32
// factor stays one fixed linear operator (rounding the vector to float32 in
// every sweep would make M^-1 differ between applications, which
// right-preconditioned GMRES does not tolerate: the update M^-1 Q y would no
// longer match the basis and the true residual would stall above the
// estimate).
template <typename T>
struct Vec16;
template <>
struct Vec16<float> {
  using V = float4;
  static constexpr int N = 4;
  __device__ static inline void get(const V &v, float *o) { o[0] = v.x; o[1] = v.y; o[2] = v.z; o[3] = v.w; }
};
template <>
struct Vec16<double> {
  using V = double2;
  static constexpr int N = 2;
  __device__ static inline void get(const V &v, double *o) { o[0] = v.x; o[1] = v.y; }
};

template <typename T>
__global__ __launch_bounds__(256) void k_gemv(const GemvDesc *__restrict__ items,
                                              const GemvChunk *__restrict__ chunks,
                                              const double *__restrict__ in,
                                              const double *__restrict__ corr,
                                              const double *__restrict__ add,
                                              double *__restrict__ out) {
  using VW = Vec16<T>;
  constexpr int VN = VW::N;
  const GemvChunk ch = chunks[blockIdx.x];
  GemvDesc d = items[ch.item];
  __shared__ double xs[GEMV_MAXC];
  __shared__ double part[256];
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  if (ch.kind == GEMV_EDGE) d.cols = d.nb;
  auto stage = [&]() {
    for (int c = tid; c < d.cols; c += 256) {
      const int s = gmem<const int32_t>(d.islot)[c];
      double v = ch.kind == GEMV_EDGE ? corr[s] : in[s];
      if (ch.kind == GEMV_INNER && c < d.nb) v += corr[s];
      xs[c] = v;
    }
    __syncthreads();
  };
  const T *A = gmem<const T>(d.A);
  const int32_t *os = gmem<const int32_t>(d.oslot) + ch.row0;
  if (!d.trans) {
    // each wave works on four rows at once; the next four 16-byte loads (of
    // these rows or the next four) are issued before the products of the last
    // ones, and a group's output slots one group ahead, so that the sums over
    // the lanes and the stores run under them.  Rows past the band re-read the
    // band's last row and are discarded.
    constexpr int ST = 64 * VN;
    const int cv = d.cols / VN * VN;     // vectorised part (lda is a multiple of 4)
    const int cl = max(cv - VN, 0);
    typename VW::V cur[4], nxt[4];
    auto load = [&](int rr, int c0, typename VW::V (&v)[4]) {
      const int c = min(c0 + lane * VN, cl);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        v[q] = *reinterpret_cast<const typename VW::V *>(A + (int64_t)(ch.row0 + min(rr + q, ch.nrows - 1)) * d.lda + c);
    };
    auto slot = [&](int rr) { return os[min(rr + (lane >> 4), ch.nrows - 1)]; };   // lanes 16 q ..: row rr + q
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    int rr = wid * 4, c0 = 0;
    load(rr, 0, cur);
    int oc = slot(rr), on = slot(rr + 16);
    stage();
    double ac = ch.kind == GEMV_EDGE ? add[oc] : 0.0;
    while (rr < ch.nrows) {
      const bool last = c0 + ST >= cv;
      const int rn = last ? rr + 16 : rr, cn = last ? 0 : c0 + ST;
      if (rn < ch.nrows) load(rn, cn, nxt);
      double an = 0.0;
      int o2 = 0;
      if (last && rn < ch.nrows) {
        if (ch.kind == GEMV_EDGE) an = add[on];
        o2 = slot(rn + 16);
      }
      __builtin_amdgcn_sched_barrier(0);
      const int c = c0 + lane * VN;
      if (c < cv) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          T e[VN];
          VW::get(cur[q], e);
#pragma unroll
          for (int u = 0; u < VN; ++u) acc[q] += double(e[u]) * xs[c + u];
        }
      }
      if (last) {
        for (int ct = cv + lane; ct < d.cols; ct += 64)
#pragma unroll
          for (int q = 0; q < 4; ++q)
            acc[q] += double(A[(int64_t)(ch.row0 + min(rr + q, ch.nrows - 1)) * d.lda + ct]) * xs[ct];
        const double sum = wave_sum4(acc);
        if ((lane & 15) == 0 && rr + (lane >> 4) < ch.nrows) out[oc] = ch.kind == GEMV_EDGE ? ac + sum : sum;
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = 0.0;
        oc = on;
        ac = an;
        on = o2;
      }
#pragma unroll
      for (int q = 0; q < 4; ++q) cur[q] = nxt[q];
      rr = rn;
      c0 = cn;
    }
  } else {
    // bands of GEMV_TROWS rows: lane = row, each wave takes every fourth
    // column (eight loads in flight per lane), the four sums meet in LDS
    stage();
    double a = 0.0;
    const int r = ch.row0 + min(lane, ch.nrows - 1);
    const T *col = A + r;
    int c = wid;
    for (; c + 28 < d.cols; c += 32) {
      T v[8];
#pragma unroll
      for (int u = 0; u < 8; ++u) v[u] = col[(int64_t)(c + 4 * u) * d.lda];
#pragma unroll
      for (int u = 0; u < 8; ++u) a += double(v[u]) * xs[c + 4 * u];
    }
    for (; c < d.cols; c += 4) a += double(col[(int64_t)c * d.lda]) * xs[c];
    part[tid] = a;
    __syncthreads();
    if (tid < ch.nrows) {
      const double v = (part[tid] + part[tid + 64]) + (part[tid + 128] + part[tid + 192]);
      const int o = os[tid];
      out[o] = ch.kind == GEMV_EDGE ? add[o] + v : v;
    }
  }
}

int launch_gemv(FType t, const GemvDesc *d_items, const GemvChunk *d_chunks, int nchunks,
                const double *in, const double *corr, const double *add, double *out,
                hipStream_t st) {
  if (nchunks <= 0) return SPAND_OK;
  if (t == FType::F64)
    hipLaunchKernelGGL(k_gemv<double>, dim3(nchunks), dim3(256), 0, st, d_items, d_chunks, in,
                       corr, add, out);
  else
    hipLaunchKernelGGL(k_gemv<float>, dim3(nchunks), dim3(256), 0, st, d_items, d_chunks, in,
                       corr, add, out);
  SP_HIP(hipGetLastError());
  return SPAND_OK;
}

// ------------------------------------------------------------------ levels above the leaves
// The sweeps over a level l >= 1 (LevelTask): its clusters are small dense
// matrices (interfaces of ~100 unknowns, interiors of ~60), so a launch is
// bound by latency - of the launch itself and of each step's loads - and the
// steps of a level are fused: one workgroup carries a cluster through the
// couplings to its neighbours (y) and its own matrix (M y), and with P set
// recomputes the neighbours' matrix-vector products it needs without a launch
// of their own.
// Two to six launches a level; one per step and three copies back to x (nine a
// level) against them: 616 and 197 us for the transposed apply at 37x29 p = 1
// FP64 (36 and 14 launches), 1063 and 860 us at 128x128 p = 2 FP32 (3.0 GB, 81
// and 25), 4.46 and 3.87 ms at 256x256 p = 3 FP32.  Loads left to the
// compiler's own schedule (one after another, each waited for): 926, not 860 us.
// The sum of a row never depends on how a level is cut into launches: plain
// rows take LEVEL_LANES lanes in 16-byte vectors and a shuffle tree,
// transposed rows LEVEL_LANES slices of every LEVEL_LANES-th column, and the
// couplings of a cluster accumulate in item order.
constexpr int LEVEL_LANES = 8;

template <typename T>
using GPtr = const T __attribute__((address_space(1))) *;
template <typename T>
__device__ inline GPtr<T> gptr(const void *p) {
  return (GPtr<T>)p;
}
typedef float level_f32x4 __attribute__((ext_vector_type(4)));
typedef double level_f64x2 __attribute__((ext_vector_type(2)));
template <typename T>
struct LevelVec;
template <>
struct LevelVec<float> {
  using V = level_f32x4;
  static constexpr int N = 4;
};
template <>
struct LevelVec<double> {
  using V = level_f64x2;
  static constexpr int N = 2;
};

// sum over the columns of one row of a row-major matrix that lane q of
// LEVEL_LANES takes.  Rows start at any multiple of sizeof(T): up to VN - 1
// elements before the first 16-byte boundary and after the last whole vector
// are scalar.  Four vectors in flight: past the end a load repeats the last
// vector and its products are dropped, and the empty statement keeps the
// loads of a step together (one memory round trip instead of four).
template <typename T>
__device__ inline double level_dot(GPtr<T> row, int n, const double *x, int q) {
  using V = typename LevelVec<T>::V;
  constexpr int VN = LevelVec<T>::N, ST = LEVEL_LANES * VN;
  const int mis = int((reinterpret_cast<uintptr_t>((const T *)row) / sizeof(T)) % VN);
  const int h = min(mis ? VN - mis : 0, n);
  const int cv = h + (n - h) / VN * VN;
  // element q of the head and tail together (at most 2 VN - 2 < LEVEL_LANES)
  const int ns = h + n - cv, cs = q < ns ? (q < h ? q : cv + (q - h)) : 0;
  T es = row[cs];
  if (cv == h) return q < ns ? double(es) * x[cs] : 0.0;
  double a = 0.0;
  for (int c = h + q * VN; c < cv; c += 4 * ST) {
    V v[4];
    int cc[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      cc[u] = min(c + u * ST, cv - VN);
      v[u] = *(GPtr<V>)(row + cc[u]);
    }
    asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(es));
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      double s = a;
#pragma unroll
      for (int w = 0; w < VN; ++w) s += double(v[u][w]) * x[cc[u] + w];
      a = c + u * ST < cv ? s : a;
    }
  }
  const double xe = x[cs];
  return q < ns ? a + double(es) * xe : a;
}

// sum over every LEVEL_LANES-th column from q of one row of the transpose
// (element (c, r) at col[c * ld]); eight loads in flight
template <typename T>
__device__ inline double level_dot_t(GPtr<T> col, int ld, int n, const double *x, int q) {
  double a = 0.0;
  for (int c = q; c < n; c += 8 * LEVEL_LANES) {
    T v[8];
    int cc[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      cc[u] = min(c + u * LEVEL_LANES, n - 1);
      v[u] = col[(int64_t)cc[u] * ld];
    }
    asm volatile("" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]), "+v"(v[6]), "+v"(v[7]));
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const double s = a + double(v[u]) * x[cc[u]];
      a = c + u * LEVEL_LANES < n ? s : a;
    }
  }
  return a;
}

template <typename T, int TRANS>
__global__ __launch_bounds__(1024) void k_level(const LevelTask *__restrict__ tasks,
                                                const LevelItem *__restrict__ items, int tot,
                                                int mmax, int pre, const double *in,
                                                const double *base0, const double *base1,
                                                double *out) {
  extern __shared__ double sm[];
  __shared__ LevelItem its[LEVEL_MAXIT];
  double *xs = sm, *t = xs + tot, *y = pre ? t + tot : t, *part = y + mmax;
  const LevelTask d = tasks[blockIdx.x];
  const int tid = threadIdx.x, nt = blockDim.x, nr = nt / LEVEL_LANES;
  // plain: consecutive lanes share a row; transposed: consecutive lanes take
  // consecutive rows (coalesced), one slice of the columns after the other
  const int rl = TRANS ? tid % nr : tid / LEVEL_LANES, q = TRANS ? tid / nr : tid % LEVEL_LANES;
  const double *bs = d.base ? base1 : base0;
  const int y0 = d.M ? 0 : d.row0, y1 = d.M ? d.m : d.row0 + d.nrows;   // rows of y needed here
  // the first row's base is on its way while the items are staged
  const GPtr<int32_t> slots = gptr<int32_t>(d.slots);
  const double yb = y0 + tid < y1 ? bs[slots[y0 + tid]] : 0.0;
  // one row's sum over its lanes, in lane 0 (plain) or slice 0 (transposed;
  // all threads of the workgroup call it together)
  auto total = [&](double a) {
    if (TRANS) {
      part[tid] = a;
      __syncthreads();
      if (q == 0) {
        a = 0.0;
#pragma unroll
        for (int u = 0; u < LEVEL_LANES; ++u) a += part[u * nr + rl];
      }
      __syncthreads();
    } else {
#pragma unroll
      for (int o = LEVEL_LANES / 2; o > 0; o >>= 1) a += __shfl_xor(a, o, 64);
    }
    return a;
  };
  auto item_of = [&](int ni, int R) {
    int j = 0;
    while (j + 1 < ni && its[j + 1].off <= R) ++j;
    return j;
  };
  for (int ib = d.item_begin; ib < d.item_end;) {
    const int ni = items[ib].nb;
    if (ib > d.item_begin) __syncthreads();   // the batch before is done with its inputs
    if (tid < ni) its[tid] = items[ib + tid];
    __syncthreads();
    const int nin = its[ni - 1].off + its[ni - 1].k;
    for (int R = tid; R < nin; R += nt) {
      const LevelItem &p = its[item_of(ni, R)];
      xs[R] = in[gptr<int32_t>(p.islot)[R - p.off]];
    }
    if (ib == d.item_begin) {
      if (y0 + tid < y1) y[y0 + tid] = yb;
      for (int r = y0 + nt + tid; r < y1; r += nt) y[r] = bs[slots[r]];
    }
    __syncthreads();
    const double *v = xs;
    if (pre) {
      for (int r0 = 0; r0 < nin; r0 += nr) {
        const int R = r0 + rl;
        double a = 0.0;
        if (R < nin) {
          const LevelItem &p = its[item_of(ni, R)];
          const GPtr<T> P = gptr<T>(p.P);
          a = TRANS ? level_dot_t<T>(P + (R - p.off), p.ldp, p.k, xs + p.off, q)
                    : level_dot<T>(P + (int64_t)(R - p.off) * p.ldp, p.k, xs + p.off, q);
        }
        a = total(a);
        if (q == 0 && R < nin) t[R] = a;
      }
      __syncthreads();
      v = t;
    }
    for (int r0 = y0; r0 < y1; r0 += nr) {
      const int r = r0 + rl;
      double a = 0.0;
      if (r < y1)
        for (int j = 0; j < ni; ++j) {
          const LevelItem &p = its[j];
          const GPtr<T> B = gptr<T>(p.B);
          a += TRANS ? level_dot_t<T>(B + r, p.ldb, p.k, v + p.off, q)
                     : level_dot<T>(B + (int64_t)r * p.ldb, p.k, v + p.off, q);
        }
      a = total(a);
      if (q == 0 && r < y1) y[r] -= a;
    }
    ib += ni;
  }
  if (d.item_begin == d.item_end) {
    if (y0 + tid < y1) y[y0 + tid] = yb;
    for (int r = y0 + nt + tid; r < y1; r += nt) y[r] = bs[slots[r]];
  }
  __syncthreads();
  const int rend = d.row0 + d.nrows;
  if (!d.M) {
    for (int r = d.row0 + tid; r < rend; r += nt) out[slots[r]] = y[r];
    return;
  }
  const GPtr<T> M = gptr<T>(d.M);
  for (int r0 = d.row0; r0 < rend; r0 += nr) {
    const int r = r0 + rl;
    double a = 0.0;
    if (r < rend)
      a = TRANS ? level_dot_t<T>(M + r, d.ldm, d.m, y, q) : level_dot<T>(M + (int64_t)r * d.ldm, d.m, y, q);
    a = total(a);
    if (q == 0 && r < rend) out[slots[r]] = a;
  }
}

size_t level_lds_bytes(int tot, int m, int pre, int trans, int nt) {
  return (size_t(tot) * (pre ? 2 : 1) + size_t(m) + (trans ? size_t(nt) : 0)) * 8;
}

int launch_level(FType t, int trans, const LevelTask *d_tasks, int ntasks, const LevelItem *d_items,
                 int tot, int m, int pre, int nt, const double *in, const double *base0,
                 const double *base1, double *out, hipStream_t st) {
  if (ntasks <= 0) return SPAND_OK;
  const size_t lds = level_lds_bytes(tot, m, pre, trans, nt);
  const dim3 g(ntasks), b(nt);
#define LEVEL_LAUNCH(T, TR)                                                                       \
  hipLaunchKernelGGL((k_level<T, TR>), g, b, lds, st, d_tasks, d_items, tot, m, pre, in, base0,   \
                     base1, out)
  if (t == FType::F64) {
    if (trans) LEVEL_LAUNCH(double, 1);
    else LEVEL_LAUNCH(double, 0);
  } else {
    if (trans) LEVEL_LAUNCH(float, 1);
    else LEVEL_LAUNCH(float, 0);
  }
#undef LEVEL_LAUNCH
  SP_HIP(hipGetLastError());
  return SPAND_OK;
}

// ------------------------------------------------------------------ pull
// out[oslot[r]] = base[oslot[r]] + alpha * sum_items op(B_i) in[islot_i]
// (level 0; a group without items copies base to out)
// One workgroup per chunk of at most 64 output rows of a group; the items of
// the group are accumulated in order, in registers (a row is always owned by
// the same lanes).  Per item the input segment is staged in LDS.
//  * op(B) = B: 4 lanes per row with 16-byte loads from each row's first
//    16-byte boundary on (scalar head and tail); the partial sums combine
//    by shuffles.
//  * op(B) = B^T (B stored cols x rows): one lane per output row, four
//    slices of the columns, combined through LDS at the end.
template <typename T, int TRANS>
__global__ __launch_bounds__(256) void k_pull(const PullGroup *__restrict__ groups,
                                              const PullItem *__restrict__ items,
                                              const PullChunk *__restrict__ chunks,
                                              const double *in, const double *base,
                                              double *out, double alpha) {
  using VW = Vec16<T>;
  constexpr int VN = VW::N;
  const PullChunk ch = chunks[blockIdx.x];
  const PullGroup g = groups[ch.group];
  __shared__ double xs[GEMV_MAXC];
  __shared__ double part[256];
  const int tid = threadIdx.x;
  double acc[4] = {0.0, 0.0, 0.0, 0.0};
  for (int it = g.item_begin; it < g.item_end; ++it) {
    const PullItem p = items[it];
    __syncthreads();
    for (int c = tid; c < p.cols; c += 256) xs[c] = in[gmem<const int32_t>(p.islot)[c]];
    __syncthreads();
    const T *B = gmem<const T>(p.B);
    if (!TRANS) {
      // 4 lanes per row, 16-byte loads from the row's first 16-byte
      // boundary on (a row of any leading dimension: the few elements
      // before the boundary and after the last full vector are scalar)
      const int rr = tid >> 2, q = tid & 3;
      double a = 0.0;
      if (rr < ch.nrows) {
        const T *row = B + (int64_t)(ch.row0 + rr) * p.ldb;
        const int mis = int((reinterpret_cast<uintptr_t>(row) / sizeof(T)) % VN);
        const int h = min(mis ? VN - mis : 0, p.cols);
        if (q < h) a += double(row[q]) * xs[q];
        const int cv = h + (p.cols - h) / VN * VN;
#pragma unroll 4
        for (int c = h + q * VN; c < cv; c += 4 * VN) {
          const typename VW::V v = *reinterpret_cast<const typename VW::V *>(row + c);
          T e[VN];
          VW::get(v, e);
#pragma unroll
          for (int u = 0; u < VN; ++u) a += double(e[u]) * xs[c + u];
        }
        for (int c = cv + q; c < p.cols; c += 4) a += double(row[c]) * xs[c];
      }
      a += __shfl_xor(a, 1, 64);
      a += __shfl_xor(a, 2, 64);
      acc[0] += a;
    } else {
      const int rr = tid & 63, cs = tid >> 6;
      if (rr < ch.nrows) {
        const T *col = B + ch.row0 + rr;
        double a0 = 0.0, a1 = 0.0;
        int c = cs;
        for (; c + 4 < p.cols; c += 8) {
          a0 += double(col[(int64_t)c * p.ldb]) * xs[c];
          a1 += double(col[(int64_t)(c + 4) * p.ldb]) * xs[c + 4];
        }
        if (c < p.cols) a0 += double(col[(int64_t)c * p.ldb]) * xs[c];
        acc[0] += a0 + a1;
      }
    }
  }
  auto put = [&](int r, double v) {
    const int o = gmem<const int32_t>(g.oslot)[ch.row0 + r];
    out[o] = (base ? base[o] : 0.0) + alpha * v;
  };
  if (!TRANS) {
    const int rr = tid >> 2;
    if ((tid & 3) == 0 && rr < ch.nrows) put(rr, acc[0]);
  } else {
    part[tid] = acc[0];
    __syncthreads();
    if (tid < ch.nrows) put(tid, (part[tid] + part[tid + 64]) + (part[tid + 128] + part[tid + 192]));
  }
}

int launch_pull2(FType t, const PullGroup *d_groups, const PullItem *d_items,
                 const PullChunk *d_chunks, int nchunks, int trans, const double *in,
                 const double *base, double *out, double alpha, hipStream_t st) {
  if (nchunks <= 0) return SPAND_OK;
  const dim3 g(nchunks), b(256);
  if (t == FType::F64) {
    if (trans) hipLaunchKernelGGL((k_pull<double, 1>), g, b, 0, st, d_groups, d_items, d_chunks, in, base, out, alpha);
    else hipLaunchKernelGGL((k_pull<double, 0>), g, b, 0, st, d_groups, d_items, d_chunks, in, base, out, alpha);
  } else {
    if (trans) hipLaunchKernelGGL((k_pull<float, 1>), g, b, 0, st, d_groups, d_items, d_chunks, in, base, out, alpha);
    else hipLaunchKernelGGL((k_pull<float, 0>), g, b, 0, st, d_groups, d_items, d_chunks, in, base, out, alpha);
  }
  SP_HIP(hipGetLastError());
  return SPAND_OK;
}

// ------------------------------------------------------------------ SpMV
// y = alpha*A x + beta*y + gz*z + gw*w  (row-major b x b BSR blocks).
// G lanes per scalar row, 16-byte loads: one instruction of a lane group
// reads 16*G contiguous bytes of the row segment.  G is picked per block
// size by the autotuner (4, 8 or 16).
typedef double spmv_f64x2 __attribute__((ext_vector_type(2)));
template <int G>
__global__ __launch_bounds__(256) void k_spmv(int n_brows, int bs, const int32_t *__restrict__ rowptr,
                                              const int32_t *__restrict__ colind,
                                              const double *__restrict__ val,
                                              const double *__restrict__ x, double alpha,
                                              double beta, double *__restrict__ y,
                                              const double *__restrict__ z, double gz,
                                              const double *__restrict__ w, double gw) {
  constexpr int RPB = 256 / G;
  const int64_t N = (int64_t)n_brows * bs;
  const int64_t R = (int64_t)blockIdx.x * RPB + (threadIdx.x / G);
  const int sub = threadIdx.x % G;
  double acc = 0.0;
  if (R < N) {
    const int I = int(R / bs), r = int(R % bs);
    const int64_t b2 = (int64_t)bs * bs;
    for (int t = rowptr[I]; t < rowptr[I + 1]; ++t) {
      const double *rowv = val + (int64_t)t * b2 + (int64_t)r * bs;
      const double *xv = x + (int64_t)colind[t] * bs;
      for (int c = sub * 2; c < bs; c += 2 * G) {
        // the matrix is streamed once per product: non-temporal, so that
        // the vector's blocks stay in the caches
        const spmv_f64x2 a = __builtin_nontemporal_load(reinterpret_cast<const spmv_f64x2 *>(rowv + c));
        acc += a[0] * xv[c] + a[1] * xv[c + 1];
      }
    }
  }
#pragma unroll
  for (int o = G / 2; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if (R < N && sub == 0) {
    double v = alpha * acc;
    if (beta != 0.0) v += beta * y[R];
    if (z) v += gz * z[R];
    if (w) v += gw * w[R];
    y[R] = v;
  }
}

// The same product with one wave per element, for the block sizes
// 4 (p + 1)^2 of p = 1 and 2: L = BS / 2 lanes
// cover a block row and S = 64 / L slices of lanes take every S-th row, so an
// instruction reads up to 1 KB of the element's contiguous blocks and a block's
// part of x is read once, not once per row.  A lane keeps the partial sums of
// its K = BS / S rows; LDS adds the L lanes of a row at the end.  U blocks
// of a row are in flight per wave (a cell's five of BS = 16).
// Bound by the one read of the values: 1.9 GB of BS = 36 in 295 us (6.5 TB/s;
// k_spmv 455 us), 2.7 GB of BS = 16 in 424 us (590 us).
template <int BS>
struct SpmvWave {
  static constexpr int L = BS / 2, S = 64 / L, K = BS / S, P = L + 1 - (L & 1);
  static constexpr int U = K < 10 ? 10 / K : 1;
  static_assert(K * S == BS, "slices cover the rows evenly");
};
template <int BS>
__global__ __launch_bounds__(256) void k_spmv_wave(int n_brows, const int32_t *__restrict__ rowptr,
                                                   const int32_t *__restrict__ colind,
                                                   const double *__restrict__ val,
                                                   const double *__restrict__ x, double alpha,
                                                   double beta, double *__restrict__ y,
                                                   const double *__restrict__ z, double gz,
                                                   const double *__restrict__ w, double gw) {
  using W = SpmvWave<BS>;
  constexpr int L = W::L, S = W::S, K = W::K, P = W::P, U = W::U;
  __shared__ double part[4][BS * P];
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int I = blockIdx.x * 4 + wv;
  if (I >= n_brows) return;                // whole waves; each uses its own part of LDS
  const int lane = threadIdx.x & 63;
  const int sl = min(lane / L, S - 1), i = lane % L;      // lanes past S L repeat the last slice's loads
  spmv_f64x2 a[K] = {};
  const int t1 = rowptr[I + 1];
  const int t0 = rowptr[I];
  int J[U];                                // one round ahead of the loads that need it
  auto cols = [&](int t) {
#pragma unroll
    for (int u = 0; u < U; ++u) J[u] = colind[min(t + u, t1 - 1)];
  };
  if (t0 < t1) cols(t0);
  for (int t = t0; t < t1; t += U) {
    spmv_f64x2 xv[U], e[U][K];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const double *blk = val + (int64_t)min(t + u, t1 - 1) * (BS * BS) + sl * BS + 2 * i;
#pragma unroll
      for (int k = 0; k < K; ++k)
        e[u][k] = __builtin_nontemporal_load(reinterpret_cast<const spmv_f64x2 *>(blk + k * S * BS));
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const double *xp = x + (int64_t)J[u] * BS + 2 * i;
      xv[u] = spmv_f64x2{xp[0], xp[1]};
    }
    cols(t + U);
    // every load is issued before the first product (left to itself the
    // compiler moves each to its use, one wait per load)
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int k = 0; k < K; ++k) asm volatile("" : "+v"(e[u][k]));
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (t + u < t1)
#pragma unroll
        for (int k = 0; k < K; ++k) a[k] += e[u][k] * xv[u];
  }
  if (lane < L * S)
#pragma unroll
    for (int k = 0; k < K; ++k) part[wv][(sl + k * S) * P + i] = a[k][0] + a[k][1];
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
  if (lane < BS) {
    const double *pr = part[wv] + lane * P;
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int q = 0; q < L; q += 2) s0 += pr[q], s1 += q + 1 < L ? pr[q + 1] : 0.0;
    const int64_t R = (int64_t)I * BS + lane;
    double v = alpha * (s0 + s1);
    if (beta != 0.0) v += beta * y[R];
    if (z) v += gz * z[R];
    if (w) v += gw * w[R];
    y[R] = v;
  }
}

static int g_spmv_lanes[65] = {0};   // per block size; 0 = not tuned (default 8)

void set_spmv_lanes(int bs, int G) {
  if (bs >= 0 && bs <= 64) g_spmv_lanes[bs] = G;
}
int get_spmv_lanes(int bs) {
  const int g = (bs >= 0 && bs <= 64) ? g_spmv_lanes[bs] : 0;
  return g ? g : 8;
}

int launch_spmv_g(const spand_bsr_t &A, int G, double alpha, const double *x, double beta,
                  double *y, const double *z, double gz, const double *w, double gw,
                  hipStream_t st) {
  const int64_t N = (int64_t)A.n_brows * A.bs;
  if (N == 0) return SPAND_OK;
  const unsigned nb = (unsigned)cdiv(N, 256 / G);
  if (G == 4)
    hipLaunchKernelGGL(k_spmv<4>, dim3(nb), dim3(256), 0, st, A.n_brows, A.bs, A.d_rowptr,
                       A.d_colind, A.d_val, x, alpha, beta, y, z, gz, w, gw);
  else if (G == 16)
    hipLaunchKernelGGL(k_spmv<16>, dim3(nb), dim3(256), 0, st, A.n_brows, A.bs, A.d_rowptr,
                       A.d_colind, A.d_val, x, alpha, beta, y, z, gz, w, gw);
  else
    hipLaunchKernelGGL(k_spmv<8>, dim3(nb), dim3(256), 0, st, A.n_brows, A.bs, A.d_rowptr,
                       A.d_colind, A.d_val, x, alpha, beta, y, z, gz, w, gw);
  SP_HIP(hipGetLastError());
  return SPAND_OK;
}

// y = alpha*A^T x + beta*y + gz*z + gw*w for a structurally symmetric block
// pattern, without a transposed copy: row R = I*bs + r of A^T x sums
// A_JI(c, r) x_J(c) over the blocks (J, I) mirroring row I's blocks (I, J).
// The mirror block is found by binary search in row J; a missing mirror
// contributes nothing (spmv_t_check reports it before the products).
//
// Position of block (J, I), J = colind[t], or -1
__device__ inline int mirror_of(const int32_t *__restrict__ rowptr, const int32_t *__restrict__ colind, int t,
                                int I) {
  const int J = colind[t];
  int lo = rowptr[J], hi = rowptr[J + 1] - 1, pos = -1;
  while (lo <= hi) {
    const int mid = (lo + hi) >> 1;
    const int cm = colind[mid];
    if (cm == I) { pos = mid; break; }
    if (cm < I) lo = mid + 1; else hi = mid - 1;
  }
  return pos;
}

// One lane per output row: for each c the lanes of element I read row c of
// A_JI, bs contiguous doubles.  Small blocks, and values that are not 16-byte
// aligned.
__global__ __launch_bounds__(256) void k_spmv_t(int n_brows, int bs,
                                                const int32_t *__restrict__ rowptr,
                                                const int32_t *__restrict__ colind,
                                                const double *__restrict__ val,
                                                const double *__restrict__ x, double alpha,
                                                double beta, double *__restrict__ y,
                                                const double *__restrict__ z, double gz,
                                                const double *__restrict__ w, double gw) {
  const int64_t N = (int64_t)n_brows * bs;
  const int64_t R = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (R >= N) return;
  const int I = int(R / bs), r = int(R - (int64_t)I * bs);
  const int64_t b2 = (int64_t)bs * bs;
  double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
  for (int t = rowptr[I]; t < rowptr[I + 1]; ++t) {
    const int pos = mirror_of(rowptr, colind, t, I);
    if (pos < 0) continue;
    const double *blk = val + (int64_t)pos * b2 + r;
    const double *xv = x + (int64_t)colind[t] * bs;
    int c = 0;
    for (; c + 4 <= bs; c += 4) {
      a0 += __builtin_nontemporal_load(blk + (int64_t)c * bs) * xv[c];
      a1 += __builtin_nontemporal_load(blk + (int64_t)(c + 1) * bs) * xv[c + 1];
      a2 += __builtin_nontemporal_load(blk + (int64_t)(c + 2) * bs) * xv[c + 2];
      a3 += __builtin_nontemporal_load(blk + (int64_t)(c + 3) * bs) * xv[c + 3];
    }
    for (; c < bs; ++c) a0 += __builtin_nontemporal_load(blk + (int64_t)c * bs) * xv[c];
  }
  double v = alpha * ((a0 + a1) + (a2 + a3));
  if (beta != 0.0) v += beta * y[R];
  if (z) v += gz * z[R];
  if (w) v += gw * w[R];
  y[R] = v;
}

// One wave per element I: L = bs / 2 lanes with 16-byte loads cover a row of a
// block and S = 64 / L slices of lanes take every S-th row, so an instruction
// reads up to 1 KB of contiguous memory; the slices' sums are added at the end.
// The lanes search the mirrors of up to 64 blocks at once; a search a block
// stalls every lane before each block's loads.  Bound by the one read of the
// values: 10.8 GB (bs = 64) in 1.62 ms, 6.7 TB/s; one lane per row 1.74 ms
// with 8-byte loads, 1.70 ms with 16-byte loads.
__global__ __launch_bounds__(256) void k_spmv_t_wave(int n_brows, int bs,
                                                     const int32_t *__restrict__ rowptr,
                                                     const int32_t *__restrict__ colind,
                                                     const double *__restrict__ val,
                                                     const double *__restrict__ x, double alpha,
                                                     double beta, double *__restrict__ y,
                                                     const double *__restrict__ z, double gz,
                                                     const double *__restrict__ w, double gw) {
  const int I = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (I >= n_brows) return;
  const int lane = threadIdx.x & 63;
  const int L = bs >> 1, S = 64 / L;
  const int sl = lane / L, i = lane - sl * L;
  const int64_t b2 = (int64_t)bs * bs;
  const int nst = sl < S ? (bs - sl + S - 1) / S : 0;     // rows of a block this lane reads
  const int nfull = bs / S;                               // ... and every lane of a slice
  spmv_f64x2 a[2] = {};
  const int t1 = rowptr[I + 1];
  for (int t0 = rowptr[I]; t0 < t1; t0 += 64) {
    const int nt = min(64, t1 - t0);
    int Jl = 0, pl = -1;
    if (lane < nt) {
      Jl = colind[t0 + lane];
      pl = mirror_of(rowptr, colind, t0 + lane, I);
    }
    for (int t = 0; t < nt; ++t) {
      const int pos = __builtin_amdgcn_readlane(pl, t);
      if (pos < 0) continue;
      const double *xv = x + (int64_t)__builtin_amdgcn_readlane(Jl, t) * bs + sl;
      const double *blk = val + (int64_t)pos * b2 + (int64_t)sl * bs + 2 * i;
      if (sl < S) {
        auto part = [&](int k, auto un) {
          constexpr int U = decltype(un)::value;
          spmv_f64x2 e[U];
          double xc[U];
#pragma unroll
          for (int q = 0; q < U; ++q) {
            e[q] = __builtin_nontemporal_load(reinterpret_cast<const spmv_f64x2 *>(blk + (k + q) * S * bs));
            xc[q] = xv[(k + q) * S];
          }
#pragma unroll
          for (int q = 0; q < U; ++q) a[q & 1] += e[q] * xc[q];
        };
        int k = 0;
        for (; k + 8 <= nfull; k += 8) part(k, std::integral_constant<int, 8>{});
        if (k + 4 <= nfull) part(k, std::integral_constant<int, 4>{}), k += 4;
        for (; k < nst; ++k) part(k, std::integral_constant<int, 1>{});
      }
    }
  }
  spmv_f64x2 s = a[0] + a[1];
  for (int n = S; n > 1;) {
    const int h = (n + 1) >> 1;
    const double p0 = __shfl(s[0], (lane + h * L) & 63, 64), p1 = __shfl(s[1], (lane + h * L) & 63, 64);
    if (sl + h < n) s[0] += p0, s[1] += p1;
    n = h;
  }
  if (sl == 0) {
    const int64_t R = (int64_t)I * bs + 2 * i;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      double v = alpha * s[q];
      if (beta != 0.0) v += beta * y[R + q];
      if (z) v += gz * z[R + q];
      if (w) v += gw * w[R + q];
      y[R + q] = v;
    }
  }
}

// *flag = 1 if some stored block (I, J) has no mirror (J, I)
__global__ __launch_bounds__(256) void k_spmv_t_check(int n_brows, const int32_t *__restrict__ rowptr,
                                                      const int32_t *__restrict__ colind,
                                                      int *__restrict__ flag) {
  const int I = blockIdx.x * 256 + threadIdx.x;
  if (I >= n_brows) return;
  for (int t = rowptr[I]; t < rowptr[I + 1]; ++t) {
    if (mirror_of(rowptr, colind, t, I) < 0) {
      atomicOr(flag, 1);
      return;
    }
  }
}

int launch_spmv_t_check(const spand_bsr_t &A, int *d_flag, hipStream_t st) {
  if (A.n_brows <= 0) return SPAND_OK;
  hipLaunchKernelGGL(k_spmv_t_check, dim3((unsigned)cdiv(A.n_brows, 256)), dim3(256), 0, st,
                     A.n_brows, A.d_rowptr, A.d_colind, d_flag);
  SP_HIP(hipGetLastError());
  return SPAND_OK;
}

// One wave per element where a block size has it and the values are aligned.
// Kernel time in us, lane groups (8 or 16 lanes, as tuned) / one wave:
//   elements     4         16         36        64       256      1024     16384    65536
//   bs = 16   2.8/2.2   3.5/2.9    3.7/3.2   3.8/3.4   4.9/3.4   7.2/3.7   35/26   140/105
//   bs = 36   5.2/4.8  5.1-7.1/5.8 5.1/6.3   6.8/6.4   8.2/6.8  18.8/9.2  209/129  834/522
// Below 64 elements of 36 neither is always ahead (25 to 49: 4.8-5.2 against
// 5.6-6.3); the call around it takes 15 us.  At bs = 64 a group of 8 lanes reads
// a row's 512 bytes evenly and is faster (10.7 GB: 1.53 ms against 1.65 ms for
// 32 rows' sums per lane).
bool spmv_by_wave(const spand_bsr_t &A) {
  return (A.bs == 16 || A.bs == 36) && (reinterpret_cast<uintptr_t>(A.d_val) & 15) == 0;
}

int launch_spmv(const spand_bsr_t &A, int transpose, double alpha, const double *x, double beta,
                double *y, const double *z, double gz, const double *w, double gw,
                hipStream_t st) {
  if (!transpose && spmv_by_wave(A)) {
    if (A.n_brows <= 0) return SPAND_OK;
    auto *k = A.bs == 16 ? k_spmv_wave<16> : k_spmv_wave<36>;
    hipLaunchKernelGGL(k, dim3((unsigned)cdiv(A.n_brows, 4)), dim3(256), 0, st, A.n_brows, A.d_rowptr, A.d_colind,
                       A.d_val, x, alpha, beta, y, z, gz, w, gw);
    SP_HIP(hipGetLastError());
    return SPAND_OK;
  }
  if (!transpose) return launch_spmv_g(A, get_spmv_lanes(A.bs), alpha, x, beta, y, z, gz, w, gw, st);
  const int64_t N = (int64_t)A.n_brows * A.bs;
  if (N == 0) return SPAND_OK;
  // From bs = 10 on an element fills 50 or more of a wave's 64 lanes (8: 32,
  // 4: 8, 2: 2).
  if (A.bs >= 10 && A.bs <= 64 && A.bs % 2 == 0 && (reinterpret_cast<uintptr_t>(A.d_val) & 15) == 0)
    hipLaunchKernelGGL(k_spmv_t_wave, dim3((unsigned)cdiv(A.n_brows, 4)), dim3(256), 0, st, A.n_brows, A.bs,
                       A.d_rowptr, A.d_colind, A.d_val, x, alpha, beta, y, z, gz, w, gw);
  else
    hipLaunchKernelGGL(k_spmv_t, dim3((unsigned)cdiv(N, 256)), dim3(256), 0, st, A.n_brows, A.bs,
                       A.d_rowptr, A.d_colind, A.d_val, x, alpha, beta, y, z, gz, w, gw);
  SP_HIP(hipGetLastError());
  return SPAND_OK;
}

// d_out[t] = alpha * u_I v_J^T for every stored block: bound by the one write
// of out, W = 2 adjacent columns per 16-byte store where bs is even and out is
// 16-byte aligned.  A thread's row and column advance by constants.  1.34 GB
// written in 0.37 ms; with a division and an 8-byte store per element 0.52 ms.
template <int W>
__global__ __launch_bounds__(256) void k_pattern_outer(int n_brows, int bs,
                                                       const int32_t *__restrict__ rowptr,
                                                       const int32_t *__restrict__ colind,
                                                       const double *__restrict__ u,
                                                       const double *__restrict__ v, double alpha,
                                                       double *__restrict__ out) {
  const int I = blockIdx.x;
  if (I >= n_brows) return;
  typedef double vec __attribute__((ext_vector_type(W)));
  const int b2 = bs * bs, dr = W * 256 / bs, dc = W * 256 % bs;
  const int r0 = W * threadIdx.x / bs, c0 = W * threadIdx.x % bs;
  for (int t = rowptr[I]; t < rowptr[I + 1]; ++t) {
    const int J = colind[t];
    int r = r0, c = c0;
    for (int idx = W * threadIdx.x; idx < b2; idx += W * 256) {
      const double au = alpha * u[(int64_t)I * bs + r];
      vec o;
#pragma unroll
      for (int q = 0; q < W; ++q) o[q] = au * v[(int64_t)J * bs + c + q];
      *reinterpret_cast<vec *>(out + (int64_t)t * b2 + idx) = o;
      r += dr, c += dc;
      if (c >= bs) c -= bs, ++r;
    }
  }
}

int launch_pattern_outer(const spand_bsr_t &P, const double *u, const double *v, double alpha,
                         double *out, hipStream_t st) {
  if (P.n_brows <= 0) return SPAND_OK;
  if (P.bs % 2 == 0 && (reinterpret_cast<uintptr_t>(out) & 15) == 0)
    hipLaunchKernelGGL(k_pattern_outer<2>, dim3(P.n_brows), dim3(256), 0, st, P.n_brows, P.bs,
                       P.d_rowptr, P.d_colind, u, v, alpha, out);
  else
    hipLaunchKernelGGL(k_pattern_outer<1>, dim3(P.n_brows), dim3(256), 0, st, P.n_brows, P.bs,
                       P.d_rowptr, P.d_colind, u, v, alpha, out);
  SP_HIP(hipGetLastError());
  return SPAND_OK;
}

// ------------------------------------------------------------------ vectors
__global__ void k_fill(double *x, int64_t n, double v) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    x[i] = v;
}
__global__ void k_iota(int32_t *x, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    x[i] = int32_t(i);
}
// y = a*x + b*y  with a, b optionally read from device scalars:
// a = ca * (pa ? *pa : 1) [* (inva ? 1/ *inva : 1)]
__global__ void k_axpby(int64_t n, const double *__restrict__ x, double *__restrict__ y,
                        double ca, const double *pa, int inva, double cb) {
  double a = ca;
  if (pa) a *= inva ? 1.0 / *pa : *pa;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    double v = a * x[i];
    if (cb != 0.0) v += cb * y[i];
    y[i] = v;
  }
}

int vec_fill(double *x, int64_t n, double v, hipStream_t st) {
  if (n <= 0) return SPAND_OK;
  hipLaunchKernelGGL(k_fill, dim3((unsigned)std::min<int64_t>(4096, cdiv(n, 256))), dim3(256), 0,
                     st, x, n, v);
  SP_HIP(hipGetLastError());
  return SPAND_OK;
}
int vec_iota(int32_t *x, int64_t n, hipStream_t st) {
  if (n <= 0) return SPAND_OK;
  hipLaunchKernelGGL(k_iota, dim3((unsigned)std::min<int64_t>(4096, cdiv(n, 256))), dim3(256), 0,
                     st, x, n);
  SP_HIP(hipGetLastError());
  return SPAND_OK;
}
int vec_axpby(int64_t n, const double *x, double *y, double ca, const double *pa, int inva,
              double cb, hipStream_t st) {
  if (n <= 0) return SPAND_OK;
  hipLaunchKernelGGL(k_axpby, dim3((unsigned)std::min<int64_t>(4096, cdiv(n, 256))), dim3(256), 0,
                     st, n, x, y, ca, pa, inva, cb);
  SP_HIP(hipGetLastError());
  return SPAND_OK;
}

// ------------------------------------------------------------------ tall-skinny
// Partial Gram: part[chunk][i][j] = sum_{r in chunk} X[i*ldx + r] * W[j*ldw + r]
// (X: N x a, W: N x s, both column-major).  Chunks of TS_CHUNK rows.
__global__ __launch_bounds__(256) void k_gram_part(int64_t N, const double *__restrict__ X,
                                                   int64_t ldx, int a,
                                                   const double *__restrict__ W, int64_t ldw,
                                                   int s, double *__restrict__ part) {
  __shared__ double ws[TS_CHUNK][TS_MAXS + 1];
  const int64_t r0 = (int64_t)blockIdx.x * TS_CHUNK;
  const int rows = int(std::min<int64_t>(TS_CHUNK, N - r0));
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  for (int idx = tid; idx < TS_CHUNK * s; idx += 256) {
    const int j = idx / TS_CHUNK, r = idx % TS_CHUNK;
    ws[r][j] = r < rows ? W[(int64_t)j * ldw + r0 + r] : 0.0;
  }
  __syncthreads();
  double *outp = part + (int64_t)blockIdx.x * a * s;
  for (int i = wid; i < a; i += 4) {
    double acc[TS_MAXS];
#pragma unroll
    for (int j = 0; j < TS_MAXS; ++j) acc[j] = 0.0;
    const double *xc = X + (int64_t)i * ldx + r0;
    for (int r = lane; r < rows; r += 64) {
      const double xv = xc[r];
#pragma unroll
      for (int j = 0; j < TS_MAXS; ++j)
        if (j < s) acc[j] += xv * ws[r][j];
    }
#pragma unroll
    for (int j = 0; j < TS_MAXS; ++j) {
      if (j < s) {
        const double v = wsum(acc[j]);
        if (lane == 0) outp[(int64_t)i * s + j] = v;
      }
    }
  }
}

// out[i*ldo + j] = sum over chunks; one workgroup per output, fixed
// partition and tree order (deterministic)
__global__ __launch_bounds__(256) void k_gram_reduce(const double *__restrict__ part, int nchunk,
                                                     int a, int s, double *__restrict__ out,
                                                     int ldo) {
  __shared__ double red[256];
  const int idx = blockIdx.x;
  double v = 0.0;
  for (int c = threadIdx.x; c < nchunk; c += 256) v += part[(int64_t)c * a * s + idx];
  red[threadIdx.x] = v;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
    __syncthreads();
  }
  if (threadIdx.x == 0) out[(idx / s) * ldo + idx % s] = red[0];
}

// Wide variant for the single-reduce step (up to 2 * TS_MAXS columns) on the
// FP64 matrix cores: each wave owns TS_WCHUNK rows and accumulates the
// a x s partial Gram matrix as ceil(a/16) tiles of v_mfma_f64_16x16x4f64
// (lane l supplies X(row k + l/16, column l%16) as A and W(row k + l/16,
// column l%16) as B; result register q of lane l is tile row l/16 + 4q,
// column l%16), so the sum over rows needs no cross-lane reduction.  The
// per-wave partials are summed in two deterministic stages (fixed partition
// and order).
constexpr int TS_WCHUNK = 256;     // rows per wave
constexpr int TS_WMAXS = 2 * TS_MAXS;
constexpr int TS_WSPLIT = 64;      // first-stage splits of the partial sums
typedef double gram_f64x4 __attribute__((ext_vector_type(4)));

template <int NT>
__global__ __launch_bounds__(256) void k_gram_part_wide(int64_t N, const double *__restrict__ X,
                                                        int64_t ldx, int a,
                                                        const double *__restrict__ W,
                                                        int64_t ldw, int s, int64_t nchunk,
                                                        int vec4, double *__restrict__ part) {
  const int lane = threadIdx.x & 63, m = lane & 15, g = lane >> 4;
  const int64_t chunk = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (chunk >= nchunk) return;        // whole wave; no barriers below
  const int64_t rb = chunk * TS_WCHUNK + g;
  gram_f64x4 acc[NT];
  const double *xc[NT];
  bool xok[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    acc[t] = gram_f64x4{0.0, 0.0, 0.0, 0.0};
    const int col = t * 16 + m;
    xok[t] = col < a;
    xc[t] = X + (int64_t)(xok[t] ? col : 0) * ldx;
  }
  const bool wok = m < s;
  const double *wc = W + (int64_t)(wok ? m : 0) * ldw;
  if (vec4 && (chunk + 1) * TS_WCHUNK <= N) {
    // full chunk, 32-byte aligned columns: lane group g loads rows
    // 16kk + 4g .. 16kk + 4g + 3 at once and feeds them to four products
    // (k-slot g of product q is row 16kk + 4g + q)
    const int64_t rv = chunk * TS_WCHUNK + 4 * g;
    const gram_f64x4 z4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
    for (int kk = 0; kk < TS_WCHUNK / 16; ++kk) {
      const int64_t r = rv + 16 * kk;
      const gram_f64x4 bw = wok ? *(const gram_f64x4 *)(wc + r) : z4;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const gram_f64x4 ax = xok[t] ? *(const gram_f64x4 *)(xc[t] + r) : z4;
        acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(ax[0], bw[0], acc[t], 0, 0, 0);
        acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(ax[1], bw[1], acc[t], 0, 0, 0);
        acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(ax[2], bw[2], acc[t], 0, 0, 0);
        acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(ax[3], bw[3], acc[t], 0, 0, 0);
      }
    }
  } else {
#pragma unroll 4
    for (int k = 0; k < TS_WCHUNK / 4; ++k) {
      const int64_t r = rb + 4 * k;
      const bool in = r < N;
      const double bw = (in && wok) ? wc[r] : 0.0;
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const double ax = (in && xok[t]) ? xc[t][r] : 0.0;
        acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(ax, bw, acc[t], 0, 0, 0);
      }
    }
  }
  double *outp = part + chunk * a * s;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int i = t * 16 + g + 4 * q;
      if (i < a && wok) outp[(int64_t)i * s + m] = acc[t][q];
    }
}

// Stage 1: workgroup (x, y) sums chunks [y*nchunk/S, (y+1)*nchunk/S) of the
// 64 outputs from x*64 (one wave per quarter of the range, then in order).
__global__ __launch_bounds__(256) void k_gram_reduce_s1(const double *__restrict__ part,
                                                        int64_t nchunk, int n,
                                                        double *__restrict__ part2) {
  __shared__ double red[4][64];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int idx = blockIdx.x * 64 + lane;
  const int64_t c0 = nchunk * blockIdx.y / gridDim.y, c1 = nchunk * (blockIdx.y + 1) / gridDim.y;
  const int64_t q0 = c0 + (c1 - c0) * wid / 4, q1 = c0 + (c1 - c0) * (wid + 1) / 4;
  double v = 0.0;
  if (idx < n)
    for (int64_t c = q0; c < q1; ++c) v += part[c * n + idx];
  red[wid][lane] = v;
  __syncthreads();
  if (wid == 0 && idx < n)
    part2[(int64_t)blockIdx.y * n + idx] = (red[0][lane] + red[1][lane]) +
                                           (red[2][lane] + red[3][lane]);
}

// Stage 2: out = sum over the splits, in order.
__global__ __launch_bounds__(64) void k_gram_reduce_s2(const double *__restrict__ part2,
                                                       int nsplit, int n, int s,
                                                       double *__restrict__ out, int ldo) {
  const int idx = blockIdx.x * 64 + threadIdx.x;
  if (idx >= n) return;
  double v = 0.0;
  for (int y = 0; y < nsplit; ++y) v += part2[(int64_t)y * n + idx];
  out[(idx / s) * ldo + idx % s] = v;
}

int64_t gram_wide_part_elems(int64_t N, int a, int s) {
  return (cdiv(N, TS_WCHUNK) + TS_WSPLIT) * a * s;
}

int launch_gram_wide(int64_t N, const double *X, int64_t ldx, int a, const double *W,
                     int64_t ldw, int s, double *part, double *out, int ldo, hipStream_t st) {
  if (a <= 0 || s <= 0 || N <= 0) return SPAND_OK;
  if (s > TS_WMAXS || a > TS_MAXA) {
    set_error("wide Gram matrix: %d x %d exceeds %d x %d", a, s, TS_MAXA, TS_WMAXS);
    return SPAND_EINVAL;
  }
  const int64_t nchunk = cdiv(N, TS_WCHUNK);
  const dim3 g1((unsigned)cdiv(nchunk, 4));
  // every column start 32-byte aligned: four-row vector loads
  const int vec4 = (ldx % 4 == 0) && (ldw % 4 == 0) && (uintptr_t(X) % 32 == 0) &&
                   (uintptr_t(W) % 32 == 0);
  switch (int(cdiv(a, 16))) {
#define GRAM_NT(nt)                                                                          \
  case nt:                                                                                   \
    hipLaunchKernelGGL(k_gram_part_wide<nt>, g1, dim3(256), 0, st, N, X, ldx, a, W, ldw, s, \
                       nchunk, vec4, part);                                                  \
    break;
    GRAM_NT(1) GRAM_NT(2) GRAM_NT(3) GRAM_NT(4) GRAM_NT(5)
    GRAM_NT(6) GRAM_NT(7) GRAM_NT(8) GRAM_NT(9) GRAM_NT(10)
#undef GRAM_NT
    default:
      set_error("wide Gram matrix: %d rows", a);
      return SPAND_EINVAL;
  }
  SP_HIP(hipGetLastError());
  const int n = a * s;
  double *part2 = part + nchunk * n;
  const int nsplit = int(std::min<int64_t>(TS_WSPLIT, nchunk));
  hipLaunchKernelGGL(k_gram_reduce_s1, dim3(unsigned(cdiv(n, 64)), unsigned(nsplit)), dim3(256),
                     0, st, part, nchunk, n, part2);
  SP_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_gram_reduce_s2, dim3(unsigned(cdiv(n, 64))), dim3(64), 0, st, part2,
                     nsplit, n, s, out, ldo);
  SP_HIP(hipGetLastError());
  return SPAND_OK;
}

// One pass over the rows for a single-reduce step, Q_old = Q[:, 0:a] read
// once per row: the pending block P = Q[:, a:a+sp] <- (P - Q_old R1) T^{-1}
// (its second pass) and the new block W = Q[:, a+sp:a+sp+sw] <-
// (W - Q_old C_old - Phat C_P) RV^{-1} (its first pass), coefficients from
// the single-reduce kernel.  bad = 1: nothing; bad = 2: P only.
__global__ __launch_bounds__(256) void k_ts_lag_update(int64_t N, double *__restrict__ Q,
                                                       int64_t ldq, int a, int sp, int sw, int s,
                                                       const KrylovDev *__restrict__ K) {
  __shared__ double RP[TS_MAXA * TS_MAXS];    // R1, ld TS_MAXS
  __shared__ double RW[TS_MAXA * TS_MAXS];    // C_old, ld TS_MAXS
  __shared__ double Ts[TS_MAXS * TS_MAXS], CP[TS_MAXS * TS_MAXS], RV[TS_MAXS * TS_MAXS];
  const int bad = K->bad;
  if (bad == 1) return;
  const int ww = (bad == 0) ? sw : 0;
  if (sp + ww == 0) return;
  for (int idx = threadIdx.x; idx < a * TS_MAXS; idx += 256) {
    const int i = idx / TS_MAXS, c = idx % TS_MAXS;
    RP[idx] = c < sp ? K->Lr1[i * s + c] : 0.0;
    RW[idx] = c < ww ? K->Pra[i * s + c] : 0.0;
  }
  for (int idx = threadIdx.x; idx < TS_MAXS * TS_MAXS; idx += 256) {
    const int r = idx / TS_MAXS, c = idx % TS_MAXS;
    const bool in = r < s && c < s;
    Ts[idx] = in && sp ? K->Lt[r * s + c] : 0.0;
    CP[idx] = in && sp && ww ? K->Pra[(a + r) * s + c] : 0.0;
    RV[idx] = in && ww ? K->Prb[r * s + c] : 0.0;
  }
  __syncthreads();
  // one row per thread (a grid-stride loop would let the compiler keep the
  // triangular factors in registers and spill)
  const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (r < N) {
    double ap[TS_MAXS], aw[TS_MAXS];
#pragma unroll
    for (int c = 0; c < TS_MAXS; ++c) ap[c] = aw[c] = 0.0;
#pragma unroll 2
    for (int i = 0; i < a; ++i) {
      const double xv = Q[(int64_t)i * ldq + r];
#pragma unroll
      for (int c = 0; c < TS_MAXS; ++c) {
        if (c < sp) ap[c] += xv * RP[i * TS_MAXS + c];
        if (c < ww) aw[c] += xv * RW[i * TS_MAXS + c];
      }
    }
    double p[TS_MAXS];
#pragma unroll
    for (int c = 0; c < TS_MAXS; ++c) {
      p[c] = 0.0;
      if (c < sp) {
        double v = Q[(int64_t)(a + c) * ldq + r] - ap[c];
#pragma unroll
        for (int q = 0; q < TS_MAXS; ++q)
          if (q < c) v -= p[q] * Ts[q * TS_MAXS + c];
        p[c] = v / Ts[c * TS_MAXS + c];
        Q[(int64_t)(a + c) * ldq + r] = p[c];
      }
    }
    if (ww) {
      double w[TS_MAXS];
#pragma unroll
      for (int c = 0; c < TS_MAXS; ++c) {
        w[c] = 0.0;
        if (c < ww) {
          double v = Q[(int64_t)(a + sp + c) * ldq + r] - aw[c];
#pragma unroll
          for (int q = 0; q < TS_MAXS; ++q)
            if (q < sp) v -= p[q] * CP[q * TS_MAXS + c];
#pragma unroll
          for (int q = 0; q < TS_MAXS; ++q)
            if (q < c) v -= w[q] * RV[q * TS_MAXS + c];
          w[c] = v / RV[c * TS_MAXS + c];
          Q[(int64_t)(a + sp + c) * ldq + r] = w[c];
        }
      }
    }
  }
}

int launch_ts_lag_update(int64_t N, double *Q, int64_t ldq, int a, int sp, int sw, int s,
                         const KrylovDev *K, hipStream_t st) {
  if (N <= 0 || sp + sw == 0) return SPAND_OK;
  if (a > TS_MAXA || s > TS_MAXS || (sp && sp != s) || (sw && sw != s)) {
    set_error("single-reduce update: a = %d, s = %d out of range", a, s);
    return SPAND_EINVAL;
  }
  hipLaunchKernelGGL(k_ts_lag_update, dim3(unsigned(cdiv(N, 256))), dim3(256), 0, st, N, Q, ldq,
                     a, sp, sw, s, K);
  SP_HIP(hipGetLastError());
  return SPAND_OK;
}

int launch_gram(int64_t N, const double *X, int64_t ldx, int a, const double *W, int64_t ldw,
                int s, double *part, double *out, int ldo, hipStream_t st) {
  if (a <= 0 || s <= 0) return SPAND_OK;
  const int nchunk = int(cdiv(N, TS_CHUNK));
  hipLaunchKernelGGL(k_gram_part, dim3(nchunk), dim3(256), 0, st, N, X, ldx, a, W, ldw, s, part);
  SP_HIP(hipGetLastError());
  hipLaunchKernelGGL(k_gram_reduce, dim3(a * s), dim3(256), 0, st, part, nchunk, a, s, out, ldo);
  SP_HIP(hipGetLastError());
  return SPAND_OK;
}

// W[:, j] -= sum_i X[:, i] R[i*ldr + j]
__global__ __launch_bounds__(256) void k_ts_update(int64_t N, const double *__restrict__ X,
                                                   int64_t ldx, int a,
                                                   const double *__restrict__ R, int ldr,
                                                   double *__restrict__ W, int64_t ldw, int s) {
  __shared__ double Rs[TS_MAXA * TS_MAXS];
  for (int idx = threadIdx.x; idx < a * s; idx += 256) Rs[idx] = R[(idx / s) * ldr + idx % s];
  __syncthreads();
  for (int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x; r < N;
       r += (int64_t)gridDim.x * 256) {
    double acc[TS_MAXS];
#pragma unroll
    for (int j = 0; j < TS_MAXS; ++j) acc[j] = 0.0;
    for (int i = 0; i < a; ++i) {
      const double xv = X[(int64_t)i * ldx + r];
#pragma unroll
      for (int j = 0; j < TS_MAXS; ++j)
        if (j < s) acc[j] += xv * Rs[i * s + j];
    }
#pragma unroll
    for (int j = 0; j < TS_MAXS; ++j)
      if (j < s) W[(int64_t)j * ldw + r] -= acc[j];
  }
}

int launch_ts_update(int64_t N, const double *X, int64_t ldx, int a, const double *R, int ldr,
                     double *W, int64_t ldw, int s, hipStream_t st) {
  if (a <= 0 || s <= 0 || N <= 0) return SPAND_OK;
  const unsigned g = (unsigned)std::min<int64_t>(8192, cdiv(N, 256));
  hipLaunchKernelGGL(k_ts_update, dim3(g), dim3(256), 0, st, N, X, ldx, a, R, ldr, W, ldw, s);
  SP_HIP(hipGetLastError());
  return SPAND_OK;
}

// W <- W T^{-1}, T upper triangular s x s (row-major, ld s); skip if *bad
__global__ __launch_bounds__(256) void k_ts_trsm(int64_t N, double *__restrict__ W, int64_t ldw,
                                                 int s, const double *__restrict__ T,
                                                 const int *__restrict__ bad) {
  if (*bad) return;
  __shared__ double Ts[TS_MAXS * TS_MAXS];
  for (int idx = threadIdx.x; idx < s * s; idx += 256) Ts[idx] = T[idx];
  __syncthreads();
  for (int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x; r < N;
       r += (int64_t)gridDim.x * 256) {
    double x[TS_MAXS];
#pragma unroll
    for (int j = 0; j < TS_MAXS; ++j) {
      if (j < s) {
        double v = W[(int64_t)j * ldw + r];
#pragma unroll
        for (int i = 0; i < TS_MAXS; ++i)
          if (i < j) v -= x[i] * Ts[i * s + j];
        x[j] = v / Ts[j * s + j];
      }
    }
#pragma unroll
    for (int j = 0; j < TS_MAXS; ++j)
      if (j < s) W[(int64_t)j * ldw + r] = x[j];
  }
}

int launch_ts_trsm(int64_t N, double *W, int64_t ldw, int s, const double *T, const int *bad,
                   hipStream_t st) {
  if (N <= 0 || s <= 0) return SPAND_OK;
  const unsigned g = (unsigned)std::min<int64_t>(8192, cdiv(N, 256));
  hipLaunchKernelGGL(k_ts_trsm, dim3(g), dim3(256), 0, st, N, W, ldw, s, T, bad);
  SP_HIP(hipGetLastError());
  return SPAND_OK;
}

// y = X[:, 0:k] c   (c on device)
__global__ __launch_bounds__(256) void k_ts_gemv(int64_t N, const double *__restrict__ X,
                                                 int64_t ldx, int k, const double *__restrict__ c,
                                                 double *__restrict__ y) {
  __shared__ double cs[TS_MAXA];
  for (int i = threadIdx.x; i < k; i += 256) cs[i] = c[i];
  __syncthreads();
  for (int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x; r < N;
       r += (int64_t)gridDim.x * 256) {
    double v = 0.0;
    for (int i = 0; i < k; ++i) v += X[(int64_t)i * ldx + r] * cs[i];
    y[r] = v;
  }
}

int launch_ts_gemv(int64_t N, const double *X, int64_t ldx, int k, const double *c, double *y,
                   hipStream_t st) {
  if (N <= 0) return SPAND_OK;
  const unsigned g = (unsigned)std::min<int64_t>(8192, cdiv(N, 256));
  hipLaunchKernelGGL(k_ts_gemv, dim3(g), dim3(256), 0, st, N, X, ldx, k, c, y);
  SP_HIP(hipGetLastError());
  return SPAND_OK;
}

}  // namespace spand
