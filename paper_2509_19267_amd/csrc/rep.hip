// Products of one stored sparse matrix with many right-hand sides at once
// (the replicated operator I_rep (x) A of the multi-right-hand-side solver,
// Section 6's deblurring of many images with one blur).
//
// The right-hand sides' vectors are held interleaved here -- entry j of
// right-hand side s at j * rep + s -- so that a wave takes one stored row
// and 64 right-hand sides, one per lane: the row's entries are loaded once
// by the wave and broadcast lane by lane (v_readlane), and the values the
// lanes gather for one entry are 64 contiguous elements (one 512-byte run
// in FP64).  With at most 32 right-hand sides a wave takes 2 or 4 rows, 32
// or 16 lanes each.  The right-hand-side-major layout of the rest of the
// solver would make each lane gather from a different vector, and each
// stored entry would be read once per right-hand side.
#include "common.h"
#include "kernels.h"

namespace rg {

constexpr int REP_NT = 256;            // 4 waves: 4 stored rows per workgroup
constexpr int REP_ROWS = REP_NT / WAVE;
// gathers in flight per lane (measured on the 512^2 blur, 64 right-hand
// sides: 8 gain 16% over 4 in FP32, nothing in FP64)
template <typename T> struct REP_UNR { static constexpr int n = 4; };
template <> struct REP_UNR<float> { static constexpr int n = 8; };

__device__ __forceinline__ int bcast(int v, int j) {
  return __builtin_amdgcn_readlane(v, j);
}
__device__ __forceinline__ float bcast(float v, int j) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), j));
}
__device__ __forceinline__ double bcast(double v, int j) {
  const int64_t b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffff), j);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), j);
  return __longlong_as_double(((int64_t)hi << 32) | (uint32_t)lo);
}

// One wave per stored row r, lane = right-hand side s (blockIdx.y selects
// the group of 64).  Lanes past rep gather from right-hand side 0 (in
// bounds) and store nothing.  Every lane of the wave runs the entry loop
// (row and bounds are wave-uniform), as v_readlane needs.
// RC: the right-hand-side count when fixed at compile time (64, one full
// group: the gather stride is a shift), 0 when taken from A.rep.
template <typename T, int RC>
__global__ void __launch_bounds__(REP_NT)
rep_mm_kernel(Csr<T> A, const T *__restrict__ in, T *__restrict__ out,
              double *__restrict__ part, Ctrl *ctrl, int ph,
              int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  if (ph >= 0 && cg_done_at_start(ctrl, ph)) return;
  __shared__ double sh[REP_NT / WAVE];
  const int lane = threadIdx.x & (WAVE - 1);
  const int64_t R = RC > 0 ? (int64_t)RC : A.rep;
  const int64_t s = (int64_t)blockIdx.y * WAVE + lane;
  const bool live = s < R;
  const int64_t row = (int64_t)blockIdx.x * REP_ROWS + threadIdx.x / WAVE;
  T acc = (T)0;
  if (row < A.brows) {
    const T *col = in + (live ? s : 0);
    const int64_t e0 = A.ptr[row], e1 = A.ptr[row + 1];
    for (int64_t c0 = e0; c0 < e1; c0 += WAVE) {
      const int64_t e = c0 + lane;
      int ix = 0;
      T v = (T)0;
      if (e < e1) {
        ix = A.idx[e];
        v = A.val[e];
      }
      const int nc = (int)(e1 - c0 < WAVE ? e1 - c0 : WAVE);
      int j = 0;
      // UNR gathers in flight, added in entry order
      for (; j + REP_UNR<T>::n <= nc; j += REP_UNR<T>::n) {
        T g[REP_UNR<T>::n];
#pragma unroll
        for (int u = 0; u < REP_UNR<T>::n; ++u)
          g[u] = col[(int64_t)bcast(ix, j + u) * R];
#pragma unroll
        for (int u = 0; u < REP_UNR<T>::n; ++u) acc += bcast(v, j + u) * g[u];
      }
      for (; j < nc; ++j) acc += bcast(v, j) * col[(int64_t)bcast(ix, j) * R];
    }
    if (live) out[row * R + s] = acc;
  }
  if (part) {
    const double q = (row < A.brows && live) ? (double)acc * (double)acc : 0.0;
    const double t = block_sum<REP_NT>(q, sh);
    if (threadIdx.x == 0) part[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = t;
  }
}

// ------------------------------------------------------------ row groups
// Matrices whose neighbouring rows share most of their columns (a stencil, a
// banded operator): the product above is bound by the gathers, 64 values per
// stored entry from L2 through a compute unit's one load path, while its
// multiply-adds take a quarter of that time.  So a wave takes REP_RG stored
// rows at once and gathers each column that any of them holds only once.
// The group's columns are sorted by which of the rows hold them (a mask of
// REP_RG bits), so that every multiply-add is one of a stored entry (no
// padding with zeros, which would turn an infinity in a row that does not
// hold the column into a NaN) and the loop of one mask is straight code.
// Indices and values are wave-uniform and come through the scalar cache.
// Layout, made at create: the group of rows 4g .. 4g + 3 uses the span of
// those rows in the index and value arrays; its columns of mask 1 come
// first, then mask 2, ..., ascending within a mask, with the values of the
// rows holding a column side by side; counts per mask in 16 ints.
// Taken by the rule of repgroups.h.  Measured on the 256^2 blur (15 x 15
// entries, 0.30 of the gathers left), 64 right-hand sides, a product (mean of A and A^T): FP32 184 -> 83 us; A x and A^T z with
// their transposes 482 -> 260 us in FP32, 1019 -> 466 us in FP64.
constexpr int REP_RG = 4;
constexpr int RG_MASKS = 1 << REP_RG;
// Columns gathered together (16 lengthen the waits on the values: 85 against
// 83 us in FP32; 4 in FP64: no change).
constexpr int RG_UNR = 8;

// position of column c in the sorted indices [lo, hi), -1 if absent
__device__ __forceinline__ int64_t find_col(const int32_t *idx, int64_t lo,
                                            int64_t hi, int32_t c) {
  const int64_t end = hi;
  while (lo < hi) {
    const int64_t m = (lo + hi) >> 1;
    if (idx[m] < c) lo = m + 1;
    else hi = m;
  }
  return lo < end && idx[lo] == c ? lo : -1;
}

// One wave per group.  FILL == 0: counts per mask, and the columns of all
// groups into *total; FILL == 1: indices and values in their places.
template <typename T, int FILL>
__global__ void __launch_bounds__(REP_NT)
rep_rg_build(int64_t brows, const int64_t *__restrict__ ptr,
             const int32_t *__restrict__ idx, const T *__restrict__ val,
             int32_t *__restrict__ cnt, unsigned long long *total,
             int32_t *__restrict__ gidx, T *__restrict__ gval) {
  const int lane = threadIdx.x & (WAVE - 1);
  const int64_t g = (int64_t)blockIdx.x * REP_ROWS + threadIdx.x / WAVE;
  const int64_t ngroup = (brows + REP_RG - 1) / REP_RG;
  if (g >= ngroup) return;
  int64_t e[REP_RG + 1];
#pragma unroll
  for (int r = 0; r <= REP_RG; ++r) {
    const int64_t row = g * REP_RG + r;
    e[r] = ptr[row < brows ? row : brows];
  }
  // running place of each mask: entries seen, index and value offsets
  int n[RG_MASKS];
  int64_t pi[RG_MASKS], pv[RG_MASKS];
  int64_t oi = e[0], ov = e[0];
#pragma unroll
  for (int m = 0; m < RG_MASKS; ++m) {
    n[m] = 0;
    if (FILL) {
      pi[m] = oi;
      pv[m] = ov;
      oi += cnt[g * RG_MASKS + m];
      ov += (int64_t)cnt[g * RG_MASKS + m] * __builtin_popcount(m);
    }
  }
#pragma unroll
  for (int r = 0; r < REP_RG; ++r) {
    for (int64_t c0 = e[r]; c0 < e[r + 1]; c0 += WAVE) {
      const int64_t p = c0 + lane;
      int mask = 0;
      int32_t c = 0;
      int64_t at[REP_RG];
      if (p < e[r + 1]) {
        c = idx[p];
#pragma unroll
        for (int q = 0; q < REP_RG; ++q) {
          at[q] = q == r ? p : find_col(idx, e[q], e[q + 1], c);
          if (at[q] >= 0) mask |= 1 << q;
        }
        // the lowest row holding the column places it
        if ((mask & ((1 << r) - 1)) != 0) mask = 0;
      }
#pragma unroll
      for (int m = 1; m < RG_MASKS; ++m) {
        const unsigned long long b = __ballot(mask == m);
        if (FILL && mask == m) {
          const int64_t k = n[m] + __popcll(b & ((1ull << lane) - 1));
          gidx[pi[m] + k] = c;
          int64_t o = pv[m] + k * __builtin_popcount(m);
#pragma unroll
          for (int q = 0; q < REP_RG; ++q)
            if (m >> q & 1) gval[o++] = val[at[q]];
        }
        n[m] += __popcll(b);
      }
    }
  }
  if (!FILL && lane == 0) {
    int tot = 0;
#pragma unroll
    for (int m = 0; m < RG_MASKS; ++m) {
      cnt[g * RG_MASKS + m] = n[m];
      tot += n[m];
    }
    atomicAdd(total, (unsigned long long)tot);
  }
}

// Brings n entries into L2, a lane per 64 bytes (at most 16 KB): the scalar
// loads that follow would each wait on HBM.  What is returned must have a use
// for the loads to stay, an empty statement at the sums (not a volatile one:
// after that the values no longer come through the scalar cache).
template <typename E>
__device__ __forceinline__ unsigned rg_fetch(const E *p, int64_t n, int lane) {
  constexpr int PER = 64 / (int)sizeof(E);
  unsigned x = 0;
  if (n > 4 * WAVE * PER) n = 4 * WAVE * PER;
  for (int64_t i = (int64_t)lane * PER; i < n; i += WAVE * PER)
    x ^= *reinterpret_cast<const unsigned *>(p + i);
  return x;
}

// N columns of mask M, their indices in lanes j .. of ixv: the gathers in
// flight together, then the multiply-adds.  Only the first n columns are
// this mask's: of the others, read past its end (valid columns, or the
// arrays' padding), gather and value count as zero, for either may be
// infinite.
template <int M, int N, typename T>
__device__ __forceinline__ void rg_step(T (&acc)[REP_RG], const T *in,
                                        unsigned s, int ixv, int j,
                                        const T *vx, int n, int64_t R) {
  T g[N];
#pragma unroll
  for (int u = 0; u < N; ++u) g[u] = (in + (int64_t)bcast(ixv, j + u) * R)[s];
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const T x = u < n ? g[u] : (T)0;
    int k = u * __builtin_popcount(M);
#pragma unroll
    for (int r = 0; r < REP_RG; ++r)
      if (M >> r & 1) {
        const T v = vx[k++];
        acc[r] = fma(u < n ? v : (T)0, x, acc[r]);
      }
  }
}
// The n columns of mask M.  ixv: the first 64 of them, one per lane, loaded
// while the mask before was worked on; on return the next mask's.
template <int M, typename T>
__device__ __forceinline__ void rg_mask(T (&acc)[REP_RG], const T *in,
                                        unsigned s, const int32_t *&ix,
                                        const T *&vx, int n, int lane,
                                        int &ixv, int64_t R) {
  if (n == 0) return;
  constexpr int K = __builtin_popcount(M);
  constexpr int U = RG_UNR;
  const int next = ix[n + lane];
  for (int c = 0; c < n; c += WAVE) {
    const int cv = ixv;
    if (c + WAVE < n) ixv = ix[c + WAVE + lane];
    const int m = n - c < WAVE ? n - c : WAVE;
    const T *v = vx + (int64_t)c * K;
    int j = 0;
    for (; j + U <= m; j += U)
      rg_step<M, U>(acc, in, s, cv, j, v + j * K, U, R);
    const int left = m - j;
    if (left > U / 2)
      rg_step<M, U>(acc, in, s, cv, j, v + j * K, left, R);
    else if (left > U / 4)
      rg_step<M, U / 2>(acc, in, s, cv, j, v + j * K, left, R);
    else if (left > 0)
      rg_step<M, U / 4>(acc, in, s, cv, j, v + j * K, left, R);
  }
  ixv = next;
  ix += n;
  vx += (int64_t)n * K;
}

template <typename T, int RC>
__global__ void __launch_bounds__(REP_NT)
rep_rg_kernel(int64_t brows, int64_t rep, const int64_t *__restrict__ ptr,
              const int32_t *__restrict__ gidx, const T *__restrict__ gval,
              const int32_t *__restrict__ cnt, const T *__restrict__ in,
              T *__restrict__ out, double *__restrict__ part,
              const Ctrl *ctrl, int ph, int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  if (ph >= 0 && cg_done_at_start(ctrl, ph)) return;
  __shared__ double sh[REP_NT / WAVE];
  const int lane = threadIdx.x & (WAVE - 1);
  const int64_t R = RC > 0 ? (int64_t)RC : rep;
  const int64_t s = (int64_t)blockIdx.y * WAVE + lane;
  const bool live = s < R;
  const int64_t g = (int64_t)blockIdx.x * REP_ROWS +
                    __builtin_amdgcn_readfirstlane(threadIdx.x / WAVE);
  const int64_t row = g * REP_RG;
  T acc[REP_RG];
#pragma unroll
  for (int r = 0; r < REP_RG; ++r) acc[r] = (T)0;
  double q = 0.0;
  if (row < brows) {
    const unsigned o = (unsigned)(live ? s : 0);
    const int64_t e0 = ptr[row];
    const int32_t *ix = gidx + e0;
    const T *vx = gval + e0;
    const int32_t *n = cnt + g * RG_MASKS;
    const int64_t e1 = ptr[row + REP_RG < brows ? row + REP_RG : brows];
    int ixv = ix[lane];
    asm("" : "+v"(acc[0]) : "v"(rg_fetch(vx, e1 - e0, lane)));
    rg_mask<1>(acc, in, o, ix, vx, n[1], lane, ixv, R);
    rg_mask<2>(acc, in, o, ix, vx, n[2], lane, ixv, R);
    rg_mask<3>(acc, in, o, ix, vx, n[3], lane, ixv, R);
    rg_mask<4>(acc, in, o, ix, vx, n[4], lane, ixv, R);
    rg_mask<5>(acc, in, o, ix, vx, n[5], lane, ixv, R);
    rg_mask<6>(acc, in, o, ix, vx, n[6], lane, ixv, R);
    rg_mask<7>(acc, in, o, ix, vx, n[7], lane, ixv, R);
    rg_mask<8>(acc, in, o, ix, vx, n[8], lane, ixv, R);
    rg_mask<9>(acc, in, o, ix, vx, n[9], lane, ixv, R);
    rg_mask<10>(acc, in, o, ix, vx, n[10], lane, ixv, R);
    rg_mask<11>(acc, in, o, ix, vx, n[11], lane, ixv, R);
    rg_mask<12>(acc, in, o, ix, vx, n[12], lane, ixv, R);
    rg_mask<13>(acc, in, o, ix, vx, n[13], lane, ixv, R);
    rg_mask<14>(acc, in, o, ix, vx, n[14], lane, ixv, R);
    rg_mask<15>(acc, in, o, ix, vx, n[15], lane, ixv, R);
    if (live) {
#pragma unroll
      for (int r = 0; r < REP_RG; ++r)
        if (row + r < brows) {
          out[(row + r) * R + s] = acc[r];
          q += (double)acc[r] * (double)acc[r];
        }
    }
  }
  if (part) {
    const double t = block_sum<REP_NT>(q, sh);
    if (threadIdx.x == 0) part[(int64_t)blockIdx.y * gridDim.x + blockIdx.x] = t;
  }
}

int64_t rep_rg_pad() { return WAVE * REP_RG; }
int64_t rep_rg_table(int64_t brows) {
  return (brows + REP_RG - 1) / REP_RG * RG_MASKS;
}
template <typename T>
void launch_rep_rg_build(const Csr<T> &A, int32_t *cnt,
                         unsigned long long *total, int32_t *gidx, T *gval,
                         hipStream_t st) {
  const int64_t ng = (A.brows + REP_RG - 1) / REP_RG;
  const int64_t nb = (ng + REP_ROWS - 1) / REP_ROWS;
  if (nb <= 0) return;
  if (gidx)
    hipLaunchKernelGGL((rep_rg_build<T, 1>), dim3((unsigned)nb), dim3(REP_NT),
                       0, st, A.brows, A.ptr, A.idx, A.val, cnt, total, gidx,
                       gval);
  else
    hipLaunchKernelGGL((rep_rg_build<T, 0>), dim3((unsigned)nb), dim3(REP_NT),
                       0, st, A.brows, A.ptr, A.idx, A.val, cnt, total, gidx,
                       gval);
}
template void launch_rep_rg_build<double>(const Csr<double> &, int32_t *,
                                          unsigned long long *, int32_t *,
                                          double *, hipStream_t);
template void launch_rep_rg_build<float>(const Csr<float> &, int32_t *,
                                         unsigned long long *, int32_t *,
                                         float *, hipStream_t);

// At most 32 right-hand sides: a wave takes 64/GR stored rows, GR lanes
// each (lane = right-hand side), so that few right-hand sides do not leave
// most lanes idle.  Each lane loads its row's entries itself (the lanes of
// a group read the same address) and gathers GR contiguous values per
// entry.
template <typename T, int GR>
__global__ void __launch_bounds__(REP_NT)
rep_mm_group_kernel(Csr<T> A, const T *__restrict__ in, T *__restrict__ out,
                    double *__restrict__ part, Ctrl *ctrl, int ph,
                    int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  if (ph >= 0 && cg_done_at_start(ctrl, ph)) return;
  __shared__ double sh[REP_NT / WAVE];
  constexpr int RPW = WAVE / GR;          // stored rows per wave
  const int lane = threadIdx.x & (WAVE - 1);
  const int ls = lane % GR;
  const int64_t R = A.rep;                // R <= GR
  const bool live = ls < R;
  const int64_t row = ((int64_t)blockIdx.x * REP_ROWS + threadIdx.x / WAVE) * RPW +
                      lane / GR;
  T acc = (T)0;
  if (row < A.brows) {
    const T *col = in + (live ? ls : 0);
    const int64_t e0 = A.ptr[row], e1 = A.ptr[row + 1];
    int64_t e = e0;
    for (; e + 4 <= e1; e += 4) {
      int32_t ix[4];
      T v[4], g[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        ix[u] = A.idx[e + u];
        v[u] = A.val[e + u];
      }
#pragma unroll
      for (int u = 0; u < 4; ++u) g[u] = col[(int64_t)ix[u] * R];
#pragma unroll
      for (int u = 0; u < 4; ++u) acc += v[u] * g[u];
    }
    for (; e < e1; ++e) acc += A.val[e] * col[(int64_t)A.idx[e] * R];
    if (live) out[row * R + ls] = acc;
  }
  if (part) {
    const double q = (row < A.brows && live) ? (double)acc * (double)acc : 0.0;
    const double t = block_sum<REP_NT>(q, sh);
    if (threadIdx.x == 0) part[blockIdx.x] = t;
  }
}

template <typename T>
int launch_rep_mm(const Csr<T> &A, const T *in, T *out, double *part,
                  Ctrl *ctrl, int ph, int respect_done, hipStream_t st) {
  if (A.rep <= 32) {
    const int gr = A.rep <= 16 ? 16 : 32;
    const int64_t rows_per_block = (int64_t)REP_ROWS * (WAVE / gr);
    const int64_t gx = (A.brows + rows_per_block - 1) / rows_per_block;
    if (gx <= 0) return 0;
    if (gr == 16)
      hipLaunchKernelGGL((rep_mm_group_kernel<T, 16>), dim3((unsigned)gx),
                         dim3(REP_NT), 0, st, A, in, out, part, ctrl, ph,
                         respect_done);
    else
      hipLaunchKernelGGL((rep_mm_group_kernel<T, 32>), dim3((unsigned)gx),
                         dim3(REP_NT), 0, st, A, in, out, part, ctrl, ph,
                         respect_done);
    return (int)gx;
  }
  const int64_t gy = (A.rep + WAVE - 1) / WAVE;
  if (A.rg_cnt) {
    const int64_t ng = (A.brows + REP_RG - 1) / REP_RG;
    const int64_t gx = (ng + REP_ROWS - 1) / REP_ROWS;
    if (gx <= 0 || gy <= 0) return 0;
    if (A.rep == WAVE)
      hipLaunchKernelGGL((rep_rg_kernel<T, WAVE>),
                         dim3((unsigned)gx, (unsigned)gy), dim3(REP_NT), 0, st,
                         A.brows, A.rep, A.ptr, A.rg_idx, A.rg_val, A.rg_cnt,
                         in, out, part, (const Ctrl *)ctrl, ph, respect_done);
    else
      hipLaunchKernelGGL((rep_rg_kernel<T, 0>),
                         dim3((unsigned)gx, (unsigned)gy), dim3(REP_NT), 0, st,
                         A.brows, A.rep, A.ptr, A.rg_idx, A.rg_val, A.rg_cnt,
                         in, out, part, (const Ctrl *)ctrl, ph, respect_done);
    return (int)(gx * gy);
  }
  const int64_t gx = (A.brows + REP_ROWS - 1) / REP_ROWS;
  if (gx <= 0 || gy <= 0) return 0;
  if (A.rep == WAVE)
    hipLaunchKernelGGL((rep_mm_kernel<T, WAVE>), dim3((unsigned)gx, (unsigned)gy),
                       dim3(REP_NT), 0, st, A, in, out, part, ctrl, ph,
                       respect_done);
  else
    hipLaunchKernelGGL((rep_mm_kernel<T, 0>), dim3((unsigned)gx, (unsigned)gy),
                       dim3(REP_NT), 0, st, A, in, out, part, ctrl, ph,
                       respect_done);
  return (int)(gx * gy);
}

// 64 x 64 tiles through LDS (one padding column against bank conflicts)
template <typename T>
__global__ void __launch_bounds__(REP_NT)
rep_tin_kernel(const T *__restrict__ in, T *__restrict__ out, int64_t len,
               int64_t R, Ctrl *ctrl, int ph, int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  if (ph >= 0 && cg_done_at_start(ctrl, ph)) return;
  __shared__ T tile[WAVE][WAVE + 1];
  const int64_t i0 = (int64_t)blockIdx.x * WAVE, s0 = (int64_t)blockIdx.y * WAVE;
  const int tx = threadIdx.x & (WAVE - 1), ty = threadIdx.x / WAVE;
  for (int r = ty; r < WAVE; r += REP_ROWS) {
    const int64_t s = s0 + r, i = i0 + tx;
    tile[r][tx] = (s < R && i < len) ? in[s * len + i] : (T)0;
  }
  __syncthreads();
  for (int r = ty; r < WAVE; r += REP_ROWS) {
    const int64_t i = i0 + r, s = s0 + tx;
    if (i < len && s < R) out[i * R + s] = tile[tx][r];
  }
}

template <typename T>
__global__ void __launch_bounds__(REP_NT)
rep_tout_kernel(const T *__restrict__ in, T *__restrict__ out,
                T *__restrict__ x, int64_t len, int64_t R, Ctrl *ctrl, int ph,
                int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  if (ph >= 0 && cg_done_at_start(ctrl, ph)) return;
  __shared__ T tile[WAVE][WAVE + 1];
  const double alpha = (x && ph >= 0) ? ctrl->cg_alpha[ph] : 0.0;
  const int64_t i0 = (int64_t)blockIdx.x * WAVE, s0 = (int64_t)blockIdx.y * WAVE;
  const int tx = threadIdx.x & (WAVE - 1), ty = threadIdx.x / WAVE;
  for (int r = ty; r < WAVE; r += REP_ROWS) {
    const int64_t i = i0 + r, s = s0 + tx;
    tile[r][tx] = (i < len && s < R) ? in[i * R + s] : (T)0;
  }
  __syncthreads();
  for (int r = ty; r < WAVE; r += REP_ROWS) {
    const int64_t s = s0 + r, i = i0 + tx;
    if (s < R && i < len) {
      const int64_t o = s * len + i;
      if (alpha != 0.0) x[o] += (T)alpha * out[o];
      out[o] = tile[tx][r];
    }
  }
}

template <typename T>
void launch_rep_tin(const T *in, T *out, int64_t len, int64_t rep, Ctrl *ctrl,
                    int ph, int respect_done, hipStream_t st) {
  const int64_t gx = (len + WAVE - 1) / WAVE, gy = (rep + WAVE - 1) / WAVE;
  if (gx <= 0 || gy <= 0) return;
  hipLaunchKernelGGL(rep_tin_kernel<T>, dim3((unsigned)gx, (unsigned)gy),
                     dim3(REP_NT), 0, st, in, out, len, rep, ctrl, ph,
                     respect_done);
}

template <typename T>
void launch_rep_tout(const T *in, T *out, T *x, int64_t len, int64_t rep,
                     Ctrl *ctrl, int ph, int respect_done, hipStream_t st) {
  const int64_t gx = (len + WAVE - 1) / WAVE, gy = (rep + WAVE - 1) / WAVE;
  if (gx <= 0 || gy <= 0) return;
  hipLaunchKernelGGL(rep_tout_kernel<T>, dim3((unsigned)gx, (unsigned)gy),
                     dim3(REP_NT), 0, st, in, out, x, len, rep, ctrl, ph,
                     respect_done);
}

template int launch_rep_mm<double>(const Csr<double> &, const double *,
                                   double *, double *, Ctrl *, int, int,
                                   hipStream_t);
template int launch_rep_mm<float>(const Csr<float> &, const float *, float *,
                                  double *, Ctrl *, int, int, hipStream_t);
template void launch_rep_tin<double>(const double *, double *, int64_t,
                                     int64_t, Ctrl *, int, int, hipStream_t);
template void launch_rep_tin<float>(const float *, float *, int64_t, int64_t,
                                    Ctrl *, int, int, hipStream_t);
template void launch_rep_tout<double>(const double *, double *, double *,
                                      int64_t, int64_t, Ctrl *, int, int,
                                      hipStream_t);
template void launch_rep_tout<float>(const float *, float *, float *, int64_t,
                                     int64_t, Ctrl *, int, int, hipStream_t);

}  // namespace rg
