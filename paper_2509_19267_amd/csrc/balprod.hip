// Sparse CG products over a block's entries, balanced by nonzeros (gfx950).
//
// With a fixed number of lanes per segment, rows of uneven length leave a wave
// waiting for its longest one: with power-law rows (mean 10, up to 2000; 1M x
// 500K, half of the columns) such a product of 5M entries took 103 us, 20 of
// them in a launch for the long rows.  Here a workgroup has the rows that
// begin in BP_CH consecutive nonzeros of A, and all their entries.  Once per
// projection bal_fill copies those on the block to the front of the
// workgroup's span of A; every CG step then streams them (coalesced, all
// loads of a tile in flight), leaves the products in LDS, and sums each row
// there, one thread per row.  A row longer than a tile is carried on.  The
// order of every sum is fixed.
// What bounds a product is the gather of the vector (4 clocks per lane and
// compute unit, 33 us for 5M entries) and, on smaller blocks, one chain of
// dependent loads.  The four products of a step at 1M x 500K, half of the
// columns and rows, with row split -> balanced: q = A_U p 103 -> 42 us, A_U^T
// q 58 -> 45 us, A^J^T p 77 -> 44 us, A^J u 144 -> 57 us; the copies 270 ->
// 340 us per iteration.  A long row summed by the one thread (instead of a
// wave) made A^J u 101 us.
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "lanes.h"

namespace rg {

constexpr int BP_NT = 256;
constexpr int BP_MUL = 4;                      // chunks of the plan together
constexpr int BP_CH = BP_MUL * (int)MP_CH;     // nonzeros of A per workgroup
constexpr int BP_K = BP_CH / BP_NT;            // per thread
constexpr int BP_SUM = 8;                      // LDS reads in flight per row
constexpr int BP_LONG = 32;                    // rows summed by a wave, above

int64_t bal_blocks(int64_t nchunk) { return (nchunk + BP_MUL - 1) / BP_MUL; }

template <typename T>
__device__ __forceinline__ void bal_rows(const Csr<T> &A, int64_t &R0,
                                         int64_t &R1) {
  const int64_t c0 = (int64_t)blockIdx.x * BP_MUL, c1 = c0 + BP_MUL;
  R0 = A.mp_rs[c0];
  R1 = A.mp_rs[c1 < A.mp_nchunk ? c1 : A.mp_nchunk];
}

// Inclusive scans over the workgroup (sums; maxima): sh holds a value per wave.
template <bool MAX>
__device__ __forceinline__ int bal_scan(int v, int *sh) {
  const int lane = threadIdx.x & (WAVE - 1), wv = threadIdx.x / WAVE;
  for (int o = 1; o < WAVE; o <<= 1) {
    const int t = __shfl_up(v, o, WAVE);
    if (lane >= o) v = MAX ? (t > v ? t : v) : v + t;
  }
  __syncthreads();
  if (lane == WAVE - 1) sh[wv] = v;
  __syncthreads();
  for (int w = 0; w < wv; ++w) v = MAX ? (sh[w] > v ? sh[w] : v) : v + sh[w];
  return v;
}

// The block's entries of each workgroup's rows, in order, from the start of
// its span: entries of marked columns (WIDE) or of marked rows.  off[r]: where
// row r begins there, cnt[2 b]: how many workgroup b has, and from where.
template <typename T, bool WIDE>
__global__ void __launch_bounds__(BP_NT)
bal_fill(Csr<T> A, const int32_t *__restrict__ mask, int32_t *__restrict__ off,
         int64_t *__restrict__ cnt, int32_t *__restrict__ idx,
         T *__restrict__ val, Ctrl *ctrl) {
  if (ctrl_done(ctrl)) return;
  __shared__ int pre[BP_CH];         // WIDE: kept before; else first row marks
  __shared__ int sh[BP_NT / WAVE], last;
  const int tid = threadIdx.x;
  int64_t R0, R1;
  bal_rows(A, R0, R1);
  if (R0 == R1) {
    if (tid == 0) cnt[2 * blockIdx.x] = cnt[2 * blockIdx.x + 1] = 0;
    return;
  }
  const int64_t E0 = A.ptr[R0], E1 = A.ptr[R1];
  int run = 0, on = 0;               // kept so far; the row in progress is on
  for (int64_t t0 = E0; t0 < E1; t0 += BP_CH) {
    const int64_t eb = t0 + tid * BP_K;
    int32_t ix[BP_K];
    T v[BP_K];
#pragma unroll
    for (int j = 0; j < BP_K; ++j) {
      ix[j] = eb + j < E1 ? A.idx[eb + j] : -1;
      v[j] = eb + j < E1 ? A.val[eb + j] : (T)0;
    }
    int keep[BP_K], k = 0;
    if (WIDE) {
#pragma unroll
      for (int j = 0; j < BP_K; ++j) keep[j] = mask[ix[j] < 0 ? 0 : ix[j]];
#pragma unroll
      for (int j = 0; j < BP_K; ++j) {
        keep[j] = ix[j] >= 0 && keep[j] != 0;
        k += keep[j];
      }
    } else {
      // each row leaves its position and whether it is on at its first
      // entry; an entry belongs to the last such mark before it
      for (int i = tid; i < BP_CH; i += BP_NT) pre[i] = 0;
      __syncthreads();
      for (int64_t r = R0 + tid; r < R1; r += BP_NT) {
        const int64_t p = A.ptr[r];
        if (p >= t0 && p < t0 + BP_CH && A.ptr[r + 1] > p)
          pre[p - t0] = ((int)(p - t0) + 1) << 1 | (mask[r] != 0);
      }
      __syncthreads();
      int m = 0;
#pragma unroll
      for (int j = 0; j < BP_K; ++j) {
        const int q = pre[tid * BP_K + j];
        m = q > m ? q : m;
      }
      m = bal_scan<true>(m, sh);
      const int lane = tid & (WAVE - 1), wv = tid / WAVE;
      int before = __shfl_up(m, 1, WAVE);
      if (lane == 0) {
        before = 0;
        for (int w = 0; w < wv; ++w) before = sh[w] > before ? sh[w] : before;
      }
      if (before == 0) before = on;
      if (tid == BP_NT - 1) last = m ? m & 1 : on;
#pragma unroll
      for (int j = 0; j < BP_K; ++j) {
        const int q = pre[tid * BP_K + j];
        before = q ? q : before;
        keep[j] = ix[j] >= 0 && (before & 1);
        k += keep[j];
      }
      __syncthreads();
      on = last;
    }
    const int inc = bal_scan<false>(k, sh);
    int at = run + inc - k;
#pragma unroll
    for (int j = 0; j < BP_K; ++j) {
      pre[tid * BP_K + j] = at;
      if (keep[j]) {
        idx[E0 + at] = ix[j];
        val[E0 + at] = v[j];
        ++at;
      }
    }
    if (tid == BP_NT - 1) last = run + inc;
    __syncthreads();
    run = last;
    for (int64_t r = R0 + tid; r < R1; r += BP_NT) {
      const int64_t p = A.ptr[r] - t0;
      if (p >= 0 && p < BP_CH && A.ptr[r] < E1) off[r] = pre[p];
    }
    __syncthreads();
  }
  for (int64_t r = R0 + tid; r < R1; r += BP_NT)
    if (A.ptr[r] == E1) off[r] = run;              // empty rows at the end
  if (tid == 0) {
    cnt[2 * blockIdx.x] = run;
    cnt[2 * blockIdx.x + 1] = E0;
  }
}

// One product with the copy; what a row's sum becomes:
//   BP_COL_WIDE    out_r = sum; ||out||^2
//   BP_COL_NARROW  s_a -= alpha sum (a: r's place in the block); ||s||^2;
//                  z -= alpha q on the workgroup's slice
//   BP_ROW_WIDE    x_r += alpha out_r (of the step before), out_r = sum
//   BP_ROW_NARROW  out_a = sum; <out, p>
template <typename T, int EPI>
__global__ void __launch_bounds__(BP_NT)
bal_prod(Csr<T> A, const int32_t *__restrict__ off,
         const int64_t *__restrict__ cnt, const int32_t *__restrict__ idx,
         const T *__restrict__ val, const T *__restrict__ vec, T *out, T *x,
         const int32_t *__restrict__ pos, const T *__restrict__ p, int64_t m,
         double *__restrict__ part, const double *__restrict__ qpart, int nq,
         int step, Ctrl *ctrl) {
  constexpr int PH = EPI == BP_COL_WIDE || EPI == BP_COL_NARROW ? 0 : 1;
  if (ctrl_done(ctrl)) return;
  if (cg_done_at_start(ctrl, PH)) return;
  __shared__ T sp[BP_CH + BP_SUM], carry[2];
  __shared__ int32_t lrow[BP_CH / BP_LONG];
  __shared__ double sh[BP_NT / WAVE];
  const int tid = threadIdx.x;
  T alpha = (T)0;
  if (EPI == BP_COL_NARROW && nq) {   // the wide product's partials of ||q||^2
    double qq = 0.0;
    for (int b = tid; b < nq; b += BP_NT) qq += qpart[b];
    qq = block_sum<BP_NT>(qq, sh);
    if (qq == 0.0) {
      if (blockIdx.x == 0 && tid == 0) ctrl->cg_done[0] = 1;
      return;
    }
    alpha = qq > 0.0 ? (T)(ctrl->cg_rzp[0][step & 1] / qq) : (T)0;
  } else if (EPI == BP_COL_NARROW || EPI == BP_ROW_WIDE) {
    alpha = (T)ctrl->cg_alpha[PH];
  }
  int64_t R0, R1;
  bal_rows(A, R0, R1);
  const int n = (int)cnt[2 * blockIdx.x];
  const int64_t E0 = cnt[2 * blockIdx.x + 1];
  double sum = 0.0;
  // the thread's first row, loaded beside the entries
  constexpr bool NARROW = EPI == BP_COL_NARROW || EPI == BP_ROW_NARROW;
  const int64_t rf = R0 + tid < R1 ? R0 + tid : -1;
  int fs = 0, fe = 0;
  int32_t fk = -1;
  if (rf >= 0) {
    fs = off[rf];
    fe = rf + 1 < R1 ? off[rf + 1] : n;
    if (NARROW) fk = pos[rf];
  }
  if (EPI == BP_COL_NARROW) {
    const int64_t per = (m + gridDim.x - 1) / gridDim.x;
    const int64_t i0 = (int64_t)blockIdx.x * per;
    for (int64_t i = i0 + tid; i < i0 + per && i < m; i += BP_NT)
      x[i] -= alpha * vec[i];
  }
  int t0 = 0, cb = 0;
  do {
    int32_t ix[BP_K];
    T v[BP_K];
#pragma unroll
    for (int j = 0; j < BP_K; ++j) {
      const int e = t0 + tid + j * BP_NT;
      ix[j] = e < n ? idx[E0 + e] : -1;
      v[j] = e < n ? val[E0 + e] : (T)0;
    }
#pragma unroll
    for (int j = 0; j < BP_K; ++j) {
      if (t0 + (j * BP_NT) >= n) break;
      const T w = vec[ix[j] < 0 ? 0 : ix[j]];
      if (ix[j] >= 0) sp[tid + j * BP_NT] = v[j] * w;
    }
    if (tid < BP_CH / BP_LONG) lrow[tid] = -1;
    __syncthreads();
    const int t1 = t0 + BP_CH;
    // what row r's sum (its part in this tile, and what is carried) becomes
    auto finish = [&](int64_t r, int l, int32_t k, T acc) {
      if (l >= t1) {
        carry[cb ^ 1] = acc;
        return;
      }
      if constexpr (EPI == BP_COL_WIDE) {
        out[r] = acc;
        sum += (double)acc * (double)acc;
      } else if constexpr (EPI == BP_COL_NARROW) {
        if (k < 0) return;
        const T sv = out[k] - alpha * acc;
        out[k] = sv;
        sum += (double)sv * (double)sv;
      } else if constexpr (EPI == BP_ROW_WIDE) {
        if (alpha != (T)0) x[r] += alpha * out[r];
        out[r] = acc;
      } else {
        if (k < 0) return;
        out[k] = acc;
        sum += (double)acc * (double)p[k];
      }
    };
    for (int64_t r = R0 + tid; r < R1; r += BP_NT) {
      const int s = r == rf ? fs : off[r];
      const int e = r == rf ? fe : r + 1 < R1 ? off[r + 1] : n;
      // the tile that has its last entry (an empty row: the next entry)
      const int l = e > s ? e - 1 : (s < n || n == 0 ? s : n - 1);
      if ((e > s ? s : l) >= t1 || l < t0) continue;
      const int a = s < t0 ? 0 : s - t0, b = (e < t1 ? e : t1) - t0;
      if (b - a > BP_LONG) {           // each has a slot of its own
        lrow[a / BP_LONG] = (int32_t)(r - R0);
        continue;
      }
      T acc = s < t0 ? carry[cb] : (T)0;
      for (int q = a; q < b; q += BP_SUM) {
        T u[BP_SUM];
#pragma unroll
        for (int i = 0; i < BP_SUM; ++i) u[i] = sp[q + i];
#pragma unroll
        for (int i = 0; i < BP_SUM; ++i) acc = q + i < b ? acc + u[i] : acc;
      }
      finish(r, l, NARROW ? (r == rf ? fk : pos[r]) : -1, acc);
    }
    __syncthreads();
    // long rows: a wave each
    const int lane = tid & (WAVE - 1);
    for (int i = tid / WAVE; i < BP_CH / BP_LONG; i += BP_NT / WAVE) {
      if (lrow[i] < 0) continue;
      const int64_t r = R0 + lrow[i];
      const int s = off[r], e = r + 1 < R1 ? off[r + 1] : n;
      const int a = s < t0 ? 0 : s - t0, b = (e < t1 ? e : t1) - t0;
      T acc = (T)0;
      for (int q = a + lane; q < b; q += WAVE) acc += sp[q];
      acc = wave_total(acc);
      if (lane == 0)
        finish(r, e - 1, NARROW ? pos[r] : -1, (s < t0 ? carry[cb] : (T)0) + acc);
    }
    t0 = t1;
    cb ^= 1;
    if (t0 < n) __syncthreads();
  } while (t0 < n);
  if (EPI != BP_ROW_WIDE) {
    sum = block_sum<BP_NT>(sum, sh);
    if (tid == 0) part[blockIdx.x] = sum;
  }
}

template <typename T>
void launch_bal_fill(const Csr<T> &A, int wide, const int32_t *mask,
                     SubWork &w, Ctrl *ctrl, hipStream_t st) {
  const dim3 grid((unsigned)bal_blocks(A.mp_nchunk));
  int32_t *off = reinterpret_cast<int32_t *>(w.ptr);
  if (wide)
    hipLaunchKernelGGL((bal_fill<T, true>), grid, dim3(BP_NT), 0, st, A, mask,
                       off, w.cnt, w.idx, (T *)w.val, ctrl);
  else
    hipLaunchKernelGGL((bal_fill<T, false>), grid, dim3(BP_NT), 0, st, A, mask,
                       off, w.cnt, w.idx, (T *)w.val, ctrl);
}
template <typename T>
void launch_bal_prod(const Csr<T> &A, int epi, const SubWork &w, const T *vec,
                     T *out, T *x, const int32_t *pos, const T *p, int64_t m,
                     double *part, const double *qpart, int nq, int step,
                     Ctrl *ctrl, hipStream_t st) {
  const dim3 grid((unsigned)bal_blocks(A.mp_nchunk));
  const int32_t *off = reinterpret_cast<const int32_t *>(w.ptr);
#define BP_LAUNCH(E)                                                          \
  hipLaunchKernelGGL((bal_prod<T, E>), grid, dim3(BP_NT), 0, st, A, off,      \
                     (const int64_t *)w.cnt, (const int32_t *)w.idx,          \
                     (const T *)w.val, vec, out, x, pos, p, m, part, qpart,  \
                     nq, step, ctrl)
  switch (epi) {
    case BP_COL_WIDE: BP_LAUNCH(BP_COL_WIDE); break;
    case BP_COL_NARROW: BP_LAUNCH(BP_COL_NARROW); break;
    case BP_ROW_WIDE: BP_LAUNCH(BP_ROW_WIDE); break;
    default: BP_LAUNCH(BP_ROW_NARROW); break;
  }
#undef BP_LAUNCH
}

#define INST_BP(T)                                                            \
  template void launch_bal_fill<T>(const Csr<T> &, int, const int32_t *,      \
                                   SubWork &, Ctrl *, hipStream_t);           \
  template void launch_bal_prod<T>(const Csr<T> &, int, const SubWork &,      \
                                   const T *, T *, T *, const int32_t *,      \
                                   const T *, int64_t, double *,              \
                                   const double *, int, int, Ctrl *,          \
                                   hipStream_t);
INST_BP(double)
INST_BP(float)

}  // namespace rg
