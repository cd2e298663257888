// Block projections of RGDBEK on gfx950 (the pseudoinverse updates of the
// GDBEK rule that Algorithm 1 reuses):
//   column block: y = argmin ||A_U y - z||,  z <- z - A_U y
//   row block:    d = (A^J)^+ r^J,           x <- x + d
// The column right-hand side A_U^T z is g restricted to U, already produced
// by the column residual pass.  For the row block with independent rows,
// d = A^J^T w with (A^J A^J^T) w = r^J.
//
// Dense blocks: Gram matrix (gathered from a precomputed A^T A / A A^T, or
// formed from the listed rows), then a Cholesky in one workgroup (chol.hip)
// with an optional corrected semi-normal-equations sweep (ill-conditioned
// square row blocks), or Jacobi-preconditioned CG: in one persistent launch
// (pcg.hip) or, for blocks that do not fit the device, two launches a step.
// Sparse blocks: matrix-free CGLS (columns, z updated as the CGLS residual)
// and CGNE on A^J A^J^T (rows), over copies of the block's entries: in one
// launch (gridcg.hip), with products balanced by nonzeros (balprod.hip) or
// with a fixed number of lanes per row.
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "mfma16.h"

namespace rg {

// ------------------------------------------------------------ Gram
template <typename T>
__global__ void __launch_bounds__(256)
gram_gather_kernel(const T *__restrict__ F, int64_t ldf,
                   const int32_t *__restrict__ list,
                   const int64_t *__restrict__ cnt, int64_t cap,
                   T *__restrict__ G, Ctrl *ctrl, int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  const int64_t c = *cnt;
  const int64_t a = blockIdx.y;
  if (a >= c) return;
  const int64_t la = list[a];
  for (int64_t b = (int64_t)blockIdx.x * 256 + threadIdx.x; b < c;
       b += (int64_t)gridDim.x * 256)
    G[a * cap + b] = F[la * ldf + list[b]];
}
template <typename T>
void launch_gram_gather(const T *F, int64_t ldf, const int32_t *list,
                        const int64_t *count_dev, int64_t cap, T *G,
                        Ctrl *ctrl, int respect_done, hipStream_t st) {
  int gx = (int)((cap + 255) / 256);
  if (gx > 8) gx = 8;
  hipLaunchKernelGGL(gram_gather_kernel<T>, dim3(gx, (unsigned)cap), dim3(256),
                     0, st, F, ldf, list, count_dev, cap, G, ctrl,
                     respect_done);
}

// G[a][b] = <X_{l_a}, X_{l_b}> (list == nullptr: identity) on the matrix
// cores (MFMA 16x16x4, FP64 or FP32): one
// workgroup of 4 waves per 64 x 64 lower tile (mirrored on store), each wave
// a 32 x 32 quarter as 2 x 2 MFMA blocks.  K advances 16 at a time through
// double-buffered LDS stages stored k-major (tile[k][row]), so the 16 lanes
// that feed one MFMA row group read consecutive words; the next stage is
// loaded from global memory into registers while the current one is
// multiplied.
constexpr int SY_B = 64;             // output tile (rows = columns)
constexpr int SY_K = 16;             // k per LDS stage
constexpr int SY_P = SY_B + 16;      // LDS row pitch (k-major rows of 64)
constexpr int SY_NT = 256;

template <typename T>
__device__ __forceinline__ void sy_load(const T *__restrict__ X, int64_t ld,
                                        int64_t len,
                                        const int32_t *__restrict__ list,
                                        int64_t c, int64_t r0, int64_t k0,
                                        T (&v)[4]) {
  // thread t: row r0 + t / 4, k = k0 + 4 (t % 4) .. + 3
  const int64_t r = r0 + (threadIdx.x >> 2);
  const int64_t k = k0 + 4 * (threadIdx.x & 3);
#pragma unroll
  for (int u = 0; u < 4; ++u) v[u] = (T)0;
  if (r >= c) return;
  const T *row = X + (list ? (int64_t)list[r] : r) * ld;
#pragma unroll
  for (int u = 0; u < 4; ++u)
    if (k + u < len) v[u] = row[k + u];
}

template <typename T>
__global__ void __launch_bounds__(SY_NT)
gram_mfma_kernel(const T *__restrict__ X, int64_t ld, int64_t len,
                 const int32_t *__restrict__ list,
                 const int64_t *__restrict__ cnt, int64_t cap, int64_t ldg,
                 T *__restrict__ G, Ctrl *ctrl, int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  typedef typename Mfma16<T>::v4 v4;
  const int64_t c = cnt ? *cnt : cap;
  const int64_t ta = (int64_t)blockIdx.y * SY_B, tb = (int64_t)blockIdx.x * SY_B;
  if (ta >= c || tb >= c || tb > ta) return;   // lower tiles only
  __shared__ T sa[2][SY_K][SY_P], sb[2][SY_K][SY_P];
  const int lane = threadIdx.x & (WAVE - 1);
  const int w = threadIdx.x / WAVE;
  const int wr = (w >> 1) * 32, wc = (w & 1) * 32;
  const int li = lane & 15, lk = lane >> 4;
  const int sr = threadIdx.x >> 2, sk = 4 * (threadIdx.x & 3);
  v4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = (v4){0, 0, 0, 0};
  T va[4], vb[4];
  sy_load<T>(X, ld, len, list, c, ta, 0, va);
  sy_load<T>(X, ld, len, list, c, tb, 0, vb);
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    sa[0][sk + u][sr] = va[u];
    sb[0][sk + u][sr] = vb[u];
  }
  __syncthreads();
  const int64_t nst = (len + SY_K - 1) / SY_K;
  for (int64_t st = 0; st < nst; ++st) {
    const int cur = (int)(st & 1);
    const bool more = st + 1 < nst;
    if (more) {
      sy_load<T>(X, ld, len, list, c, ta, (st + 1) * SY_K, va);
      sy_load<T>(X, ld, len, list, c, tb, (st + 1) * SY_K, vb);
    }
#pragma unroll
    for (int kk = 0; kk < SY_K / 4; ++kk) {
      const int k = 4 * kk + lk;
      T fa[2], fb[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        fa[i] = sa[cur][k][wr + 16 * i + li];
        fb[i] = sb[cur][k][wc + 16 * i + li];
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = Mfma16<T>::mma(fa[i], fb[j], acc[i][j]);
    }
    if (more) {
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        sa[cur ^ 1][sk + u][sr] = va[u];
        sb[cur ^ 1][sk + u][sr] = vb[u];
      }
    }
    __syncthreads();
  }
  const bool diag = (ta == tb);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t gi = ta + wr + 16 * i + Mfma16<T>::row(lk, r);
        const int64_t gj = tb + wc + 16 * j + li;
        if (gi >= c || gj >= c || (diag && gj > gi)) continue;
        const T v = acc[i][j][r];
        G[gi * ldg + gj] = v;
        G[gj * ldg + gi] = v;
      }
}

// The same for blocks of few tiles.  c = 250 gives 10 tiles of 64 x 64, whose
// workgroups walk the rows' length in stages of 16 as one chain (55 us at
// length 501); here a workgroup has one 16 x 16 tile and its waves share the
// length, each with GS_DEPTH independent steps of 16 in flight, straight from
// memory (a lane reads four consecutive k of row l % 16, the inner dimension
// in the same order for both operands); their sums meet in LDS.
constexpr int GS_W = 4;              // waves per tile
constexpr int GS_DEPTH = 4;
// Whole solves with the 64 x 64 tiles / these: 500 x 250 systems 38.9 / 33.8
// ms, 2003 x 501 in blocks of 175 76.6 / 66.3, 4000 x 1000 of 350 93.3 / 76.9
// and of 600 59.9 / 51.7.  Up to 1024 rows at every length (10 row blocks of
// 512 at length 20000 23.8 / 6.9 ms, of 1000 23.7 / 18.1, at 60000 67.0 / 52.3,
// in FP32 59.4 / 37.5); blocks of 2000 read their rows too often: 13.4 / 12.0 ms
// at length 2500, but 27.2 / 29.6 at 6000.
constexpr int64_t GS_MAX = 1024;
template <typename T>
__global__ void __launch_bounds__(GS_W * WAVE)
gram_small_kernel(const T *__restrict__ X, int64_t ld, int64_t len,
                  const int32_t *__restrict__ list,
                  const int64_t *__restrict__ cnt, int64_t ldg,
                  T *__restrict__ G, Ctrl *ctrl, int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  typedef typename Mfma16<T>::v4 v4;
  const int64_t c = *cnt;
  const int64_t ta = (int64_t)blockIdx.y * 16, tb = (int64_t)blockIdx.x * 16;
  if (ta >= c || tb >= c || tb > ta) return;   // lower tiles only
  __shared__ T sh[GS_W][4][WAVE];
  const int lane = threadIdx.x & (WAVE - 1), w = threadIdx.x / WAVE;
  const int lr = lane & 15, lk = lane >> 4;
  const T *xa = X + (int64_t)list[ta + lr < c ? ta + lr : c - 1] * ld;
  const T *xb = X + (int64_t)list[tb + lr < c ? tb + lr : c - 1] * ld;
  v4 acc = (v4){0, 0, 0, 0};
  for (int64_t k0 = 16 * w; k0 < len; k0 += 16 * GS_W * GS_DEPTH) {
    v4 a[GS_DEPTH], b[GS_DEPTH];
#pragma unroll
    for (int d = 0; d < GS_DEPTH; ++d) {
      const int64_t k = k0 + (int64_t)16 * GS_W * d + 4 * lk;
      if (k + 4 <= len) {            // rows are 16-byte aligned, padded to 8
        a[d] = *reinterpret_cast<const v4 *>(xa + k);
        b[d] = *reinterpret_cast<const v4 *>(xb + k);
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          a[d][u] = k + u < len ? xa[k + u] : (T)0;
          b[d][u] = k + u < len ? xb[k + u] : (T)0;
        }
      }
    }
#pragma unroll
    for (int d = 0; d < GS_DEPTH; ++d)
#pragma unroll
      for (int u = 0; u < 4; ++u)
        acc = Mfma16<T>::mma(a[d][u], b[d][u], acc);
  }
#pragma unroll
  for (int u = 0; u < 4; ++u) sh[w][u][lane] = acc[u];
  __syncthreads();
  // wave u finishes accumulator element u
  T v = (T)0;
#pragma unroll
  for (int q = 0; q < GS_W; ++q) v += sh[q][w][lane];
  const int64_t gi = ta + Mfma16<T>::row(lk, w), gj = tb + lr;
  if (gi < c && gj < c && gj <= gi) {
    G[gi * ldg + gj] = v;
    G[gj * ldg + gi] = v;
  }
}
static_assert(GS_W == 4, "one wave per accumulator element");

template <typename T>
void launch_gram_rows(const T *X, int64_t ld, int64_t len, const int32_t *list,
                      const int64_t *count_dev, int64_t cap, T *G, Ctrl *ctrl,
                      int respect_done, hipStream_t st) {
  if (list && count_dev && cap <= GS_MAX && ld % 4 == 0) {
    const unsigned ns = (unsigned)((cap + 15) / 16);
    hipLaunchKernelGGL(gram_small_kernel<T>, dim3(ns, ns), dim3(GS_W * WAVE),
                       0, st, X, ld, len, list, count_dev, cap, G, ctrl,
                       respect_done);
    return;
  }
  const unsigned nt = (unsigned)((cap + SY_B - 1) / SY_B);
  hipLaunchKernelGGL(gram_mfma_kernel<T>, dim3(nt, nt), dim3(SY_NT), 0, st, X,
                     ld, len, list, count_dev, cap, cap, G, ctrl,
                     respect_done);
}
template <typename T>
void launch_gram_full(const T *X, int64_t ldx, int64_t rows, int64_t len,
                      T *F, hipStream_t st) {
  const unsigned nt = (unsigned)((rows + SY_B - 1) / SY_B);
  hipLaunchKernelGGL(gram_mfma_kernel<T>, dim3(nt, nt), dim3(SY_NT), 0, st, X,
                     ldx, len, (const int32_t *)nullptr,
                     (const int64_t *)nullptr, rows, rows, F, (Ctrl *)nullptr,
                     0);
}

// ------------------------------------------------------------ PCG on Gram
// Jacobi-preconditioned CG on G y = h with two fence-free launches per step.
// Scalars are never broadcast through memory within a launch: every block
// re-derives them from small arrays of per-block partials of the previous
// launch, in a fixed order, so all blocks hold identical bits.
//   step t, launch A (one wave per row of G, 4 rows per block):
//     t > 0: rz_t = sum rz partials, rr = sum rr partials; stop when
//            rr <= tol^2 rr_0 (every block reaches the same verdict);
//            beta = rz_t / rz_{t-1};  p_t = zz + beta p_{t-1}  (whole vector,
//            rebuilt in LDS by every block; block 0 stores it)
//     v = G p_t on the block's rows; partial <p_t, v>
//   step t, launch B (k/256 blocks):
//     alpha = rz_t / sum <p,v> partials; y += alpha p_t; res -= alpha v;
//     zz = res / diag(G); partials of <res, zz> and <res, res>
// p alternates between two buffers by step parity.
constexpr int PG_NT = 256;
constexpr int PG_ROWS = PG_NT / WAVE;     // rows per block in launch A
constexpr int64_t PG_LDS_MAX = 8192;      // p staged in LDS (FP64: 64 KB)

template <typename T>
__global__ void __launch_bounds__(PG_NT)
pcg_init_kernel(const T *__restrict__ G, int64_t ldg,
                const int64_t *__restrict__ cnt, const T *__restrict__ hsrc,
                const int32_t *__restrict__ hl, T *__restrict__ y,
                CgWork<T> w, Ctrl *ctrl, int ph, int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  __shared__ double sh[PG_NT / WAVE];
  const int64_t c = *cnt;
  double rz = 0.0, rr = 0.0;
  for (int64_t a = threadIdx.x; a < c; a += PG_NT) {
    const T h = hl ? hsrc[hl[a]] : hsrc[a];
    const T dg = G[a * ldg + a];
    const T zz = dg > (T)0 ? h / dg : (T)0;
    y[a] = (T)0;
    w.res[a] = h;
    w.zz[a] = zz;
    w.p[a] = zz;               // p_0 in buffer 0
    rz += (double)h * (double)zz;
    rr += (double)h * (double)h;
  }
  rz = block_sum<PG_NT>(rz, sh);
  rr = block_sum<PG_NT>(rr, sh);
  if (threadIdx.x == 0) {
    ctrl->cg_rz[ph] = rz;      // rz_0
    ctrl->cg_rz0[ph] = rr;     // ||h||^2
    ctrl->cg_done[ph] = (rr == 0.0 || c == 0) ? 1 : 0;
    ctrl->cg_steps[ph] = 0;
  }
}

template <typename T>
__global__ void __launch_bounds__(PG_NT)
pcg_step_a(const T *__restrict__ G, int64_t ldg, const int64_t *__restrict__ cnt,
           CgWork<T> w, int t, int nb_b, double tol, Ctrl *ctrl, int ph,
           int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  if (ctrl->cg_done[ph]) return;
  __shared__ T ps[PG_LDS_MAX];
  __shared__ double sh[PG_NT / WAVE];
  const int64_t c = *cnt;
  const T *pold = w.p + (int64_t)((t + 1) & 1) * w.cap;
  T *pnew = w.p + (int64_t)(t & 1) * w.cap;
  if (t > 0) {
    const double *part = w.part + (int64_t)((t - 1) & 1) * 2 * w.part_cap;
    double rz = 0.0, rr = 0.0;
    for (int b = threadIdx.x; b < nb_b; b += PG_NT) {
      rz += part[2 * b];
      rr += part[2 * b + 1];
    }
    rz = block_sum<PG_NT>(rz, sh);
    rr = block_sum<PG_NT>(rr, sh);
    const double rz_prev = w.rzs[(t - 1) & 1];
    if (rr <= tol * tol * ctrl->cg_rz0[ph] || rz_prev == 0.0) {
      if (blockIdx.x == 0 && threadIdx.x == 0) {
        ctrl->cg_done[ph] = 1;
        ctrl->cg_steps[ph] = t;
      }
      return;
    }
    const double beta = rz / rz_prev;
    for (int64_t a = threadIdx.x; a < c; a += PG_NT) {
      const T pv = w.zz[a] + (T)beta * pold[a];
      ps[a] = pv;
      if (blockIdx.x == 0) pnew[a] = pv;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) w.rzs[t & 1] = rz;
  } else {
    for (int64_t a = threadIdx.x; a < c; a += PG_NT) ps[a] = pnew[a];
    if (blockIdx.x == 0 && threadIdx.x == 0) w.rzs[0] = ctrl->cg_rz[ph];
  }
  __syncthreads();
  const int lane = threadIdx.x & (WAVE - 1);
  const int64_t row = (int64_t)blockIdx.x * PG_ROWS + threadIdx.x / WAVE;
  double pv = 0.0;
  if (row < c) {
    T s = 0;
    const T *gr = G + row * ldg;
    for (int64_t b = lane; b < c; b += WAVE) s += gr[b] * ps[b];
    s = wave_sum(s);
    if (lane == 0) {
      w.v[row] = s;
      pv = (double)s * (double)ps[row];
    }
  }
  pv = block_sum<PG_NT>(pv, sh);
  if (threadIdx.x == 0) w.pv[blockIdx.x] = pv;
}

template <typename T>
__global__ void __launch_bounds__(PG_NT)
pcg_step_b(const T *__restrict__ G, int64_t ldg, const int64_t *__restrict__ cnt,
           T *__restrict__ y, CgWork<T> w, int t, int nb_a, Ctrl *ctrl, int ph,
           int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  if (ctrl->cg_done[ph]) return;
  __shared__ double sh[PG_NT / WAVE];
  const int64_t c = *cnt;
  const T *pt = w.p + (int64_t)(t & 1) * w.cap;
  double pv = 0.0;
  for (int b = threadIdx.x; b < nb_a; b += PG_NT) pv += w.pv[b];
  pv = block_sum<PG_NT>(pv, sh);
  const double rz = w.rzs[t & 1];
  const double alpha = pv != 0.0 ? rz / pv : 0.0;
  double rzn = 0.0, rr = 0.0;
  const int64_t a = (int64_t)blockIdx.x * PG_NT + threadIdx.x;
  if (a < c) {
    y[a] += (T)alpha * pt[a];
    const T r = w.res[a] - (T)alpha * w.v[a];
    w.res[a] = r;
    const T dg = G[a * ldg + a];
    const T zz = dg > (T)0 ? r / dg : (T)0;
    w.zz[a] = zz;
    rzn = (double)r * (double)zz;
    rr = (double)r * (double)r;
  }
  rzn = block_sum<PG_NT>(rzn, sh);
  rr = block_sum<PG_NT>(rr, sh);
  if (threadIdx.x == 0) {
    double *part = w.part + (int64_t)(t & 1) * 2 * w.part_cap;
    part[2 * blockIdx.x] = rzn;
    part[2 * blockIdx.x + 1] = rr;
  }
}

template <typename T>
void launch_pcg_gram_init(const T *G, int64_t cap, const int64_t *count_dev,
                          const T *hsrc, const int32_t *hlist, T *y,
                          CgWork<T> &w, Ctrl *ctrl, int ph, int respect_done,
                          hipStream_t st) {
  hipLaunchKernelGGL(pcg_init_kernel<T>, dim3(1), dim3(PG_NT), 0, st, G, cap,
                     count_dev, hsrc, hlist, y, w, ctrl, ph, respect_done);
}
template <typename T>
void launch_pcg_gram_step(const T *G, int64_t cap, const int64_t *count_dev,
                          T *y, CgWork<T> &w, int step, double tol,
                          Ctrl *ctrl, int ph, int respect_done,
                          hipStream_t st) {
  const int nb_a = (int)((cap + PG_ROWS - 1) / PG_ROWS);
  const int nb_b = (int)((cap + PG_NT - 1) / PG_NT);
  hipLaunchKernelGGL(pcg_step_a<T>, dim3(nb_a), dim3(PG_NT), 0, st, G, cap,
                     count_dev, w, step, nb_b, tol, ctrl, ph, respect_done);
  hipLaunchKernelGGL(pcg_step_b<T>, dim3(nb_b), dim3(PG_NT), 0, st, G, cap,
                     count_dev, y, w, step, nb_a, ctrl, ph, respect_done);
}
int64_t pcg_cap_max() { return PG_LDS_MAX; }

// ------------------------------------------------------------ thin updates
// out[i] (+)= sign * sum_a coef_a * M[list_a * ldm + i]: blockIdx.y takes a
// chunk of UP_CHUNK list entries, each thread two consecutive i (one 16-byte
// load per listed row when T is double; rows are padded, so i + 1 is always
// inside the row), with UP_UNROLL rows in flight; partials are combined in a
// fixed order by upd_finish.
constexpr int UP_NT = 256;
constexpr int UP_CHUNK = 32;
constexpr int UP_UNROLL = 8;
template <typename T>
__global__ void __launch_bounds__(UP_NT)
upd_partial(const T *__restrict__ M, int64_t ldm, int64_t len,
            const int32_t *__restrict__ list, const int64_t *__restrict__ cnt,
            const T *__restrict__ coef, T *__restrict__ part, Ctrl *ctrl,
            int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  typedef T v2 __attribute__((ext_vector_type(2)));
  const int64_t c = *cnt;
  const int64_t a0 = (int64_t)blockIdx.y * UP_CHUNK;
  if (a0 >= c) return;
  const int64_t a1 = a0 + UP_CHUNK < c ? a0 + UP_CHUNK : c;
  const int64_t i = 2 * ((int64_t)blockIdx.x * UP_NT + threadIdx.x);
  if (i >= len) return;
  T s0 = 0, s1 = 0;
  int64_t a = a0;
  for (; a + UP_UNROLL <= a1; a += UP_UNROLL) {
    v2 mv[UP_UNROLL];
    T cf[UP_UNROLL];
#pragma unroll
    for (int u = 0; u < UP_UNROLL; ++u) {
      mv[u] = *reinterpret_cast<const v2 *>(M + (int64_t)list[a + u] * ldm + i);
      cf[u] = coef[a + u];
    }
#pragma unroll
    for (int u = 0; u < UP_UNROLL; ++u) {
      s0 += cf[u] * mv[u].x;
      s1 += cf[u] * mv[u].y;
    }
  }
  for (; a < a1; ++a) {
    const v2 mv = *reinterpret_cast<const v2 *>(M + (int64_t)list[a] * ldm + i);
    s0 += coef[a] * mv.x;
    s1 += coef[a] * mv.y;
  }
  T *pp = part + (int64_t)blockIdx.y * len;
  pp[i] = s0;
  if (i + 1 < len) pp[i + 1] = s1;
}
template <typename T>
__global__ void __launch_bounds__(UP_NT)
upd_finish(int64_t len, const int64_t *__restrict__ cnt, int nsplit,
           const T *__restrict__ part, T sign, T *__restrict__ out,
           Ctrl *ctrl, int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  const int64_t i = (int64_t)blockIdx.x * UP_NT + threadIdx.x;
  if (i >= len) return;
  const int64_t c = *cnt;
  int ns = (int)((c + UP_CHUNK - 1) / UP_CHUNK);
  if (ns > nsplit) ns = nsplit;
  T s = 0;
  int b = 0;
  for (; b + 8 <= ns; b += 8) {
    T v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = part[(int64_t)(b + u) * len + i];
#pragma unroll
    for (int u = 0; u < 8; ++u) s += v[u];
  }
  for (; b < ns; ++b) s += part[(int64_t)b * len + i];
  out[i] += sign * s;
}

// Few listed rows: one launch of 5 us instead of two.  A workgroup has 16
// consecutive i (a thread two of them), its 32 slots of threads share the
// list, and the slots' sums meet in LDS.  Whole solves without / with it:
// 500 x 250 systems 35.4 / 33.9 ms, 2003 x 501 in blocks of 175 67.8 / 65.8.
// Up to 256 rows and lengths of 4096, beyond which the wider rows of the split
// form pay (4000 x 1000 in blocks of 500 5.33 / 5.51 ms, 8000 x 2000 of 1000
// 7.39 / 7.96).
constexpr int US_SLOTS = UP_NT / 8;
constexpr int64_t US_MAX = 256, US_LEN = 4096;
template <typename T>
__global__ void __launch_bounds__(UP_NT)
upd_small(const T *__restrict__ M, int64_t ldm, int64_t len,
          const int32_t *__restrict__ list, const int64_t *__restrict__ cnt,
          const T *__restrict__ coef, T sign, T *__restrict__ out, Ctrl *ctrl,
          int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  typedef T v2 __attribute__((ext_vector_type(2)));
  __shared__ T sh[US_SLOTS][16 + 2];
  const int64_t c = *cnt;
  const int l = threadIdx.x & 7, slot = threadIdx.x >> 3;
  const int64_t i = 16 * (int64_t)blockIdx.x + 2 * l;
  T s0 = 0, s1 = 0;
  if (i < len) {
    for (int64_t a0 = slot; a0 < c; a0 += UP_UNROLL * US_SLOTS) {
      v2 mv[UP_UNROLL];
      T cf[UP_UNROLL];
#pragma unroll
      for (int u = 0; u < UP_UNROLL; ++u) {
        const int64_t a = a0 + (int64_t)u * US_SLOTS;
        mv[u] = (v2){0, 0};
        cf[u] = (T)0;
        if (a < c) {
          mv[u] = *reinterpret_cast<const v2 *>(M + (int64_t)list[a] * ldm + i);
          cf[u] = coef[a];
        }
      }
#pragma unroll
      for (int u = 0; u < UP_UNROLL; ++u) {
        s0 += cf[u] * mv[u].x;
        s1 += cf[u] * mv[u].y;
      }
    }
  }
  sh[slot][2 * l] = s0;
  sh[slot][2 * l + 1] = s1;
  __syncthreads();
  const int64_t j = 16 * (int64_t)blockIdx.x + threadIdx.x;
  if (threadIdx.x < 16 && j < len) {
    T s = 0;
#pragma unroll
    for (int q = 0; q < US_SLOTS; ++q) s += sh[q][threadIdx.x];
    out[j] += sign * s;
  }
}

template <typename T>
static void thin_update(const T *M, int64_t ldm, int64_t len,
                        const int32_t *list, const int64_t *cnt, int64_t cap,
                        const T *coef, T *out, T sign, T *part, Ctrl *ctrl,
                        int respect_done, hipStream_t st) {
  if (cap <= US_MAX && len <= US_LEN) {
    hipLaunchKernelGGL(upd_small<T>, dim3((unsigned)((len + 15) / 16)),
                       dim3(UP_NT), 0, st, M, ldm, len, list, cnt, coef, sign,
                       out, ctrl, respect_done);
    return;
  }
  const unsigned gx = (unsigned)((len + 2 * UP_NT - 1) / (2 * UP_NT));
  const unsigned gy = (unsigned)((cap + UP_CHUNK - 1) / UP_CHUNK);
  hipLaunchKernelGGL(upd_partial<T>, dim3(gx, gy), dim3(UP_NT), 0, st, M, ldm,
                     len, list, cnt, coef, part, ctrl, respect_done);
  const unsigned gf = (unsigned)((len + UP_NT - 1) / UP_NT);
  hipLaunchKernelGGL(upd_finish<T>, dim3(gf), dim3(UP_NT), 0, st, len, cnt,
                     (int)gy, part, sign, out, ctrl, respect_done);
}

template <typename T>
void launch_col_update(const T *Acm, int64_t ldc, int64_t m,
                       const int32_t *list, const int64_t *count_dev,
                       int64_t cap, const T *y, T *z, T *scratch, Ctrl *ctrl,
                       int respect_done, hipStream_t st) {
  thin_update<T>(Acm, ldc, m, list, count_dev, cap, y, z, (T)-1, scratch,
                 ctrl, respect_done, st);
}
template <typename T>
void launch_row_update(const T *Arm, int64_t ld, int64_t n,
                       const int32_t *list, const int64_t *count_dev,
                       int64_t cap, const T *w, T *x, T *scratch, Ctrl *ctrl,
                       int respect_done, hipStream_t st) {
  thin_update<T>(Arm, ld, n, list, count_dev, cap, w, x, (T)1, scratch, ctrl,
                 respect_done, st);
}
int64_t thin_update_scratch(int64_t len, int64_t cap) {
  return len * ((cap + UP_CHUNK - 1) / UP_CHUNK);
}

// s_a = h1[l_a] - h2[l_a] - <A_{l_a}, v>  (one wave per listed row)
template <typename T>
__global__ void __launch_bounds__(256)
list_resid_kernel(const T *__restrict__ A, int64_t ld, int64_t len,
                  const int32_t *__restrict__ list,
                  const int64_t *__restrict__ cnt, const T *__restrict__ h1,
                  const T *__restrict__ h2, const T *__restrict__ v,
                  T *__restrict__ s, Ctrl *ctrl, int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  const int lane = threadIdx.x & (WAVE - 1);
  const int64_t a = (int64_t)blockIdx.x * 4 + threadIdx.x / WAVE;
  if (a >= *cnt) return;
  const int64_t l = list[a];
  T acc = 0;
  for (int64_t t = lane; t < len; t += WAVE) acc += A[l * ld + t] * v[t];
  acc = wave_sum(acc);
  if (lane == 0) s[a] = h1[l] - (h2 ? h2[l] : (T)0) - acc;
}
template <typename T>
void launch_list_resid(const T *Arm, int64_t ld, int64_t len,
                       const int32_t *list, const int64_t *count_dev,
                       int64_t cap, const T *h1, const T *h2, const T *v,
                       T *s, Ctrl *ctrl, int respect_done, hipStream_t st) {
  hipLaunchKernelGGL(list_resid_kernel<T>, dim3((unsigned)((cap + 3) / 4)),
                     dim3(256), 0, st, Arm, ld, len, list, count_dev, h1, h2,
                     v, s, ctrl, respect_done);
}

// ------------------------------------------------------------ sparse CG
// Column block, CGLS with z as the running residual:
//   s = A_U^T z (= g_U), p = s, gam = ||s||^2
//   step: q = A phat (phat = p on U, zero elsewhere)   [wide, CSR rows]
//         alpha = gam / ||q||^2                         [last block]
//         z -= alpha q ; s -= alpha A_U^T q             [narrow + elementwise]
//         gam' = ||s||^2, p = s + (gam'/gam) p          [last block]
// Row block, CG on A^J A^J^T w = r^J with Jacobi rho_J, d accumulated:
//   step: u = A^T phat (phat = p on J)                  [wide, CSC columns]
//         x += alpha_prev u_prev (fused before u is overwritten)
//         v = A^J u, alpha = rz / <p, v>                [narrow, last block]
//         res -= alpha v, zz = res/rho, beta, p = zz + beta p
constexpr int SC_NT = 256;
constexpr unsigned SC_MAXB = 512;   // blocks of a launch that ends in a ticket
constexpr unsigned SC_WIDE_MAXB = 512;   // blocks of the columns' wide product
constexpr unsigned SC_WIDE_GRID_MIN = 8;  // slots per group above which the
                                          // wide product takes a full grid
// Partials that every block of the next launch adds up for itself (a few
// loads per thread) instead of a launch of its own.
constexpr unsigned SC_SUM_MAX = 2048;
// Larger blocks update the CG vectors with separate many-workgroup launches
// (sc_cupd, sc_rupd1/2) instead of a walk by the last workgroup.
constexpr int64_t SC_SERIAL_MAX = 16384;
constexpr int SC_UNROLL = 8;        // loads in flight in one-block list walks

// Sum of nb partials (stride st), the same in every thread and block.
__device__ __forceinline__ double sum_parts(const double *__restrict__ part,
                                            int nb, int st, double *sh) {
  double t = 0.0;
  for (int b = threadIdx.x; b < nb; b += SC_NT) t += part[(int64_t)b * st];
  return block_sum<SC_NT>(t, sh);
}

template <typename T, int G>
__global__ void __launch_bounds__(SC_NT)
sc_wide_col(Csr<T> A, const T *__restrict__ phat, T *__restrict__ q,
            double *__restrict__ part, const double *__restrict__ plong,
            int64_t nlong, Ctrl *ctrl, int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  if (cg_done_at_start(ctrl, 0)) return;
  __shared__ double sh[SC_NT / WAVE];
  constexpr int SPB = SC_NT / G;
  const int lg = threadIdx.x & (G - 1);
  double qq = 0.0;
  // grid-stride over row segments: a bounded grid keeps the final ticket
  // and the partials to reduce few
  for (int64_t slot0 = (int64_t)blockIdx.x * SPB; slot0 < A.rows;
       slot0 += (int64_t)gridDim.x * SPB) {
    const int64_t slot = slot0 + threadIdx.x / G;
    int64_t s = 0, br = 0, co = 0;
    T acc = 0;
    bool mine = slot < A.rows;
    if (mine) {
      vrow(A, slot, s, br, co);
      const T *ph = phat + co;
      const int64_t e0 = A.ptr[br], e1 = seg_end(A, br);
      if (nlong && (A.long_flag ? A.long_flag[br] != 0 : e1 - e0 > A.long_limit))
        mine = false;   // sc_long_wide
      else
        for (int64_t e = e0 + lg; e < e1; e += G) acc += A.val[e] * ph[A.idx[e]];
    }
    acc = group_sum<G>(acc);
    if (mine && lg == 0) {
      q[s] = acc;
      qq += (double)acc * (double)acc;
    }
  }
  qq = block_sum<SC_NT>(qq, sh);
  if (threadIdx.x == 0) st_agent(&part[blockIdx.x], qq);
  if (!last_block(&ctrl->ticket[3])) return;
  double tot = 0.0, tl = 0.0;
  for (int b = threadIdx.x; b < (int)gridDim.x; b += SC_NT) tot += ld_agent(&part[b]);
  for (int64_t i = threadIdx.x; i < nlong; i += SC_NT) tl += plong[i];
  tot = block_sum<SC_NT>(tot, sh);
  tot += block_sum<SC_NT>(tl, sh);
  if (threadIdx.x == 0) {
    const double gam = ctrl->cg_rz[0];
    ctrl->cg_alpha[0] = tot > 0.0 ? gam / tot : 0.0;
    if (tot == 0.0) ctrl->cg_done[0] = 1;
  }
}

// The same product over a full grid (one row slot per thread group, no
// grid-stride loop) for matrices with many rows, where a bounded grid walks
// its rows as a long chain of dependent loads; each workgroup leaves its
// partial of ||q||^2, and sc_wide_col_fin sums them (in block order, then
// the long segments) and forms alpha.
template <typename T, int G>
__global__ void __launch_bounds__(SC_NT)
sc_wide_col_grid(Csr<T> A, const T *__restrict__ phat, T *__restrict__ q,
                 double *__restrict__ part, int64_t nlong, Ctrl *ctrl,
                 int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  if (cg_done_at_start(ctrl, 0)) return;
  __shared__ double sh[SC_NT / WAVE];
  constexpr int SPB = SC_NT / G;
  const int lg = threadIdx.x & (G - 1);
  const int64_t slot = (int64_t)blockIdx.x * SPB + threadIdx.x / G;
  double qq = 0.0;
  int64_t s = 0, br = 0, co = 0;
  T acc = 0;
  bool mine = slot < A.rows;
  if (mine) {
    vrow(A, slot, s, br, co);
    const T *ph = phat + co;
    const int64_t e0 = A.ptr[br], e1 = seg_end(A, br);
    if (nlong && (A.long_flag ? A.long_flag[br] != 0 : e1 - e0 > A.long_limit))
      mine = false;   // sc_long_wide
    else
      for (int64_t e = e0 + lg; e < e1; e += G) acc += A.val[e] * ph[A.idx[e]];
  }
  acc = group_sum<G>(acc);
  if (mine && lg == 0) {
    q[s] = acc;
    qq = (double)acc * (double)acc;
  }
  qq = block_sum<SC_NT>(qq, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = qq;
}
template <typename T>
__global__ void __launch_bounds__(1024)
sc_wide_col_fin(const double *__restrict__ part, int64_t nb,
                const double *__restrict__ plong, int64_t nlong, int step,
                Ctrl *ctrl, int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  if (cg_done_at_start(ctrl, 0)) return;
  __shared__ double sh[1024 / WAVE];
  double tot = 0.0, tl = 0.0;
  for (int64_t b = threadIdx.x; b < nb; b += 1024) tot += part[b];
  for (int64_t i = threadIdx.x; i < nlong; i += 1024) tl += plong[i];
  tot = block_sum<1024>(tot, sh);
  tot += block_sum<1024>(tl, sh);
  if (threadIdx.x == 0) {
    const double gam = step >= 0 ? ctrl->cg_rzp[0][step & 1] : ctrl->cg_rz[0];
    ctrl->cg_alpha[0] = tot > 0.0 ? gam / tot : 0.0;
    if (tot == 0.0) ctrl->cg_done[0] = 1;
  }
}

// narrow: w_a = <A_(U_a), q> over listed CSC columns; s -= alpha w;
// and z -= alpha q over a slice of rows; last block: gam', beta, p, phat.
template <typename T, int G>
__global__ void __launch_bounds__(SC_NT)
sc_narrow_col(Csr<T> At, const int32_t *__restrict__ U,
              const int64_t *__restrict__ cnt, const T *__restrict__ q,
              T *__restrict__ z, int64_t m, T *__restrict__ sres,
              T *__restrict__ p, T *__restrict__ phat,
              double *__restrict__ part, const double *__restrict__ plong,
              int64_t nlong, double tol, int par,
              const T *__restrict__ pre, const double *__restrict__ qpart,
              int nq, int step, Ctrl *ctrl, int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  if (cg_done_at_start(ctrl, 0)) return;
  __shared__ double sh[SC_NT / WAVE];
  double alpha;
  if (nq) {   // the wide product's partials of ||q||^2
    const double qq = sum_parts(qpart, nq, 1, sh);
    if (qq == 0.0) {
      if (blockIdx.x == 0 && threadIdx.x == 0) ctrl->cg_done[0] = 1;
      return;
    }
    alpha = qq > 0.0 ? ctrl->cg_rzp[0][step & 1] / qq : 0.0;
  } else {
    alpha = ctrl->cg_alpha[0];
  }
  const int64_t c = *cnt;
  // elementwise part: z -= alpha q on this block's slice of rows
  const int64_t per = (m + gridDim.x - 1) / gridDim.x;
  const int64_t i0 = (int64_t)blockIdx.x * per;
  for (int64_t i = i0 + threadIdx.x; i < i0 + per && i < m; i += SC_NT)
    z[i] -= (T)alpha * q[i];
  // narrow part (grid-stride over the listed columns)
  constexpr int SPB = SC_NT / G;
  const int lg = threadIdx.x & (G - 1);
  double ss = 0.0;
  for (int64_t a0 = (int64_t)blockIdx.x * SPB; a0 < c;
       a0 += (int64_t)gridDim.x * SPB) {
    const int64_t a = a0 + threadIdx.x / G;
    T acc = 0;
    bool mine = a < c;
    if (mine) {
      int64_t bc, ro;
      gsplit(At, (int64_t)U[a], bc, ro);
      if (pre) {   // many right-hand sides: A^T q formed interleaved
        if (lg == 0) acc = pre[bc * At.rep + (int64_t)U[a] / At.brows];
      } else {
        const T *qv = q + ro;
        const int64_t e0 = At.ptr[bc], e1 = At.ptr[bc + 1];
        if (nlong && e1 - e0 > At.long_limit) mine = false;   // sc_long_narrow
        else
          for (int64_t e = e0 + lg; e < e1; e += G) acc += At.val[e] * qv[At.idx[e]];
      }
    }
    acc = group_sum<G>(acc);
    if (mine && lg == 0) {
      const T sv = sres[a] - (T)alpha * acc;
      if (par) sres[a] = sv;
      else st_agent(&sres[a], sv);   // read by the last block
      ss += (double)sv * (double)sv;
    }
  }
  ss = block_sum<SC_NT>(ss, sh);
  if (par) {   // the next launch reduces the partials
    if (threadIdx.x == 0) part[blockIdx.x] = ss;
    return;
  }
  if (threadIdx.x == 0) st_agent(&part[blockIdx.x], ss);
  if (!last_block(&ctrl->ticket[4])) return;
  double tot = 0.0, tl = 0.0;
  for (int b = threadIdx.x; b < (int)gridDim.x; b += SC_NT) tot += ld_agent(&part[b]);
  for (int64_t i = threadIdx.x; i < nlong; i += SC_NT) tl += plong[i];
  tot = block_sum<SC_NT>(tot, sh);
  tot += block_sum<SC_NT>(tl, sh);
  const double gam = ctrl->cg_rz[0];
  const double beta = gam > 0.0 ? tot / gam : 0.0;
  // one block walks the whole list: keep SC_UNROLL loads in flight
  for (int64_t k0 = threadIdx.x; k0 < c; k0 += SC_UNROLL * SC_NT) {
    T sv[SC_UNROLL], po[SC_UNROLL];
    int32_t ix[SC_UNROLL];
#pragma unroll
    for (int u = 0; u < SC_UNROLL; ++u) {
      const int64_t k = k0 + (int64_t)u * SC_NT;
      if (k < c) { sv[u] = ld_agent(&sres[k]); po[u] = p[k]; ix[u] = U[k]; }
    }
#pragma unroll
    for (int u = 0; u < SC_UNROLL; ++u) {
      const int64_t k = k0 + (int64_t)u * SC_NT;
      if (k < c) {
        const T pv = sv[u] + (T)beta * po[u];
        p[k] = pv;
        phat[ix[u]] = pv;
      }
    }
  }
  if (threadIdx.x == 0) {
    ctrl->cg_beta[0] = beta;
    ctrl->cg_rz[0] = tot;
    ctrl->cg_steps[0] += 1;
    if (tot <= tol * tol * ctrl->cg_rz0[0]) ctrl->cg_done[0] = 1;
  }
}

template <typename T>
__global__ void __launch_bounds__(SC_NT)
sc_init(const int32_t *__restrict__ list, const int64_t *__restrict__ cnt,
        const T *__restrict__ rhs_src, const double *__restrict__ jac,
        T *__restrict__ sres, T *__restrict__ zz_or_null, T *__restrict__ p,
        T *__restrict__ phat, int32_t *__restrict__ pos,
        double *__restrict__ part, int gridm, Ctrl *ctrl, int ph,
        int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  __shared__ double sh[SC_NT / WAVE];
  const int64_t c = *cnt;
  double rz = 0.0, rr = 0.0;
  for (int64_t a = (int64_t)blockIdx.x * SC_NT + threadIdx.x; a < c;
       a += (int64_t)gridDim.x * SC_NT) {
    const int64_t l = list[a];
    if (pos) pos[l] = (int32_t)a;
    const T h = rhs_src[l];
    sres[a] = h;
    T zz = h;
    if (jac) {
      const double dj = jac[l];
      zz = dj > 0.0 ? (T)((double)h / dj) : (T)0;
      zz_or_null[a] = zz;
    }
    p[a] = zz;
    phat[l] = zz;
    rz += (double)h * (double)zz;
    rr += (double)h * (double)h;
  }
  rz = block_sum<SC_NT>(rz, sh);
  rr = block_sum<SC_NT>(rr, sh);
  if (threadIdx.x == 0) {
    st_agent(&part[2 * blockIdx.x], rz);
    st_agent(&part[2 * blockIdx.x + 1], rr);
  }
  if (gridm) return;   // sc_init_fin reduces the partials
  if (!last_block(&ctrl->ticket[6])) return;
  rz = 0.0;
  rr = 0.0;
  for (int b = threadIdx.x; b < (int)gridDim.x; b += SC_NT) {
    rz += ld_agent(&part[2 * b]);
    rr += ld_agent(&part[2 * b + 1]);
  }
  rz = block_sum<SC_NT>(rz, sh);
  rr = block_sum<SC_NT>(rr, sh);
  if (threadIdx.x == 0) {
    ctrl->cg_rz[ph] = rz;
    ctrl->cg_rz0[ph] = rr;
    ctrl->cg_alpha[ph] = 0.0;
    ctrl->cg_done[ph] = (rr == 0.0 || c == 0) ? 1 : 0;
    ctrl->cg_steps[ph] = 0;
  }
}

// Starts the CG of a phase from the partials of <res, zz> and ||res||^2.
__global__ void __launch_bounds__(SC_NT)
sc_init_fin(const double *__restrict__ part, int nb,
            const int64_t *__restrict__ cnt, Ctrl *ctrl, int ph,
            int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  __shared__ double sh[SC_NT / WAVE];
  const double rz = sum_parts(part, nb, 2, sh);
  const double rr = sum_parts(part + 1, nb, 2, sh);
  if (threadIdx.x == 0) {
    ctrl->cg_rz[ph] = rz;
    ctrl->cg_rzp[ph][0] = rz;
    ctrl->cg_rz0[ph] = rr;
    ctrl->cg_alpha[ph] = 0.0;
    ctrl->cg_done[ph] = (rr == 0.0 || *cnt == 0) ? 1 : 0;
    ctrl->cg_steps[ph] = 0;
  }
}

template <typename T>
__global__ void __launch_bounds__(SC_NT)
sc_clear(const int32_t *__restrict__ list, const int64_t *__restrict__ cnt,
         int64_t cap, T *__restrict__ phat, int32_t *__restrict__ pos,
         Ctrl *ctrl, int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  const int64_t c = *cnt;
  for (int64_t a = (int64_t)blockIdx.x * SC_NT + threadIdx.x; a < c;
       a += (int64_t)gridDim.x * SC_NT) {
    phat[list[a]] = (T)0;
    if (pos) pos[list[a]] = -1;
  }
}

// Finish of a listed product launched over a full grid (large blocks, many
// listed segments): the partials in block order, then the long segments,
// give what the last workgroup of the bounded launch forms.
//   columns: gam' = ||s||^2, beta = gam'/gam, stop at gam' <= tol^2 gam_0
//   rows:    alpha = rz / <p, v>
__global__ void __launch_bounds__(1024)
sc_narrow_col_fin(const double *__restrict__ part, int64_t nb,
                  const double *__restrict__ plong, int64_t nlong, double tol,
                  int step, Ctrl *ctrl, int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  if (cg_done_at_start(ctrl, 0)) return;
  __shared__ double sh[1024 / WAVE];
  double tot = 0.0, tl = 0.0;
  for (int64_t b = threadIdx.x; b < nb; b += 1024) tot += part[b];
  for (int64_t i = threadIdx.x; i < nlong; i += 1024) tl += plong[i];
  tot = block_sum<1024>(tot, sh);
  tot += block_sum<1024>(tl, sh);
  if (threadIdx.x == 0) {
    const double gam = ctrl->cg_rzp[0][step & 1];
    ctrl->cg_beta[0] = gam > 0.0 ? tot / gam : 0.0;
    ctrl->cg_rzp[0][(step + 1) & 1] = tot;
    ctrl->cg_steps[0] = step + 1;
    if (tot <= tol * tol * ctrl->cg_rz0[0]) ctrl->cg_done[0] = 1;
  }
}
__global__ void __launch_bounds__(1024)
sc_narrow_row_fin(const double *__restrict__ part, int64_t nb,
                  const double *__restrict__ plong, int64_t nlong, int step,
                  Ctrl *ctrl, int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  if (cg_done_at_start(ctrl, 1)) return;
  __shared__ double sh[1024 / WAVE];
  double tot = 0.0, tl = 0.0;
  for (int64_t b = threadIdx.x; b < nb; b += 1024) tot += part[b];
  for (int64_t i = threadIdx.x; i < nlong; i += 1024) tl += plong[i];
  tot = block_sum<1024>(tot, sh);
  tot += block_sum<1024>(tl, sh);
  if (threadIdx.x == 0) {
    const double rz = ctrl->cg_rzp[1][step & 1];
    ctrl->cg_alpha[1] = tot != 0.0 ? rz / tot : 0.0;
    ctrl->cg_steps[1] += 1;
    if (tot == 0.0) ctrl->cg_done[1] = 1;
  }
}

// Many-workgroup finish of a CG step for large blocks (SC_SERIAL_MAX).  The
// step's scalars come from the product's partials, added up by every block
// (nb of them; the block that keeps them is block 0), or, when those are too
// many (nb == 0), from a launch in between; then each kernel runs only when
// that launch completed the step (the step counter equals step + 1), so steps
// after convergence stay no-ops.
//   columns: gam' = ||s||^2, beta = gam'/gam, stop at gam' <= tol^2 gam_0
template <typename T>
__global__ void __launch_bounds__(SC_NT)
sc_cupd(const int32_t *__restrict__ U, const int64_t *__restrict__ cnt,
        const T *__restrict__ sres, T *__restrict__ p, T *__restrict__ phat,
        const double *__restrict__ part, int nb, double tol, Ctrl *ctrl,
        int step, int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  double beta;
  if (nb) {
    if (cg_done_at_start(ctrl, 0)) return;
    __shared__ double sh[SC_NT / WAVE];
    const double tot = sum_parts(part, nb, 1, sh);
    const double gam = ctrl->cg_rzp[0][step & 1];
    beta = gam > 0.0 ? tot / gam : 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      ctrl->cg_rzp[0][(step + 1) & 1] = tot;
      ctrl->cg_steps[0] = step + 1;
      if (tot <= tol * tol * ctrl->cg_rz0[0]) ctrl->cg_done[0] = 1;
    }
  } else {
    if (ctrl->cg_steps[0] != step + 1) return;
    beta = ctrl->cg_beta[0];
  }
  const int64_t c = *cnt;
  for (int64_t a = (int64_t)blockIdx.x * SC_NT + threadIdx.x; a < c;
       a += (int64_t)gridDim.x * SC_NT) {
    const T pv = sres[a] + (T)beta * p[a];
    p[a] = pv;
    phat[U[a]] = pv;
  }
}

// rows: alpha = rz / <p, v>; res -= alpha v, zz = res / rho, partials of
// <res, zz> and ||res||^2
template <typename T>
__global__ void __launch_bounds__(SC_NT)
sc_rupd1(const int32_t *__restrict__ J, const int64_t *__restrict__ cnt,
         const double *__restrict__ rho, T *__restrict__ res,
         T *__restrict__ zz, const T *__restrict__ v,
         const double *__restrict__ ppart, int nb, double *__restrict__ part,
         Ctrl *ctrl, int step, int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  __shared__ double sh[SC_NT / WAVE];
  double alpha;
  if (nb) {
    if (cg_done_at_start(ctrl, 1)) return;
    const double tot = sum_parts(ppart, nb, 1, sh);
    alpha = tot != 0.0 ? ctrl->cg_rzp[1][step & 1] / tot : 0.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      ctrl->cg_alpha[1] = alpha;
      ctrl->cg_steps[1] = step + 1;
    }
  } else {
    if (ctrl->cg_steps[1] != step + 1) return;
    alpha = ctrl->cg_alpha[1];
  }
  const int64_t c = *cnt;
  double rz1 = 0.0, rr = 0.0;
  for (int64_t a = (int64_t)blockIdx.x * SC_NT + threadIdx.x; a < c;
       a += (int64_t)gridDim.x * SC_NT) {
    const T r = res[a] - (T)alpha * v[a];
    res[a] = r;
    const double dj = rho[J[a]];
    const T zv = dj > 0.0 ? (T)((double)r / dj) : (T)0;
    zz[a] = zv;
    rz1 += (double)r * (double)zv;
    rr += (double)r * (double)r;
  }
  rz1 = block_sum<SC_NT>(rz1, sh);
  rr = block_sum<SC_NT>(rr, sh);
  if (threadIdx.x == 0) {
    part[2 * blockIdx.x] = rz1;
    part[2 * blockIdx.x + 1] = rr;
  }
}

// rows: beta = rz'/rz from sc_rupd1's nb partials, the stopping test, and
// p = zz + beta p.  (Only block 0 raises the done flag, which no block of
// this launch reads.)
template <typename T>
__global__ void __launch_bounds__(SC_NT)
sc_rupd2(const int32_t *__restrict__ J, const int64_t *__restrict__ cnt,
         const T *__restrict__ zz, T *__restrict__ p, T *__restrict__ phat,
         const double *__restrict__ part, int nb, double tol, Ctrl *ctrl,
         int step, int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  if (ctrl->cg_steps[1] != step + 1) return;
  __shared__ double sh[SC_NT / WAVE];
  const double rz1 = sum_parts(part, nb, 2, sh);
  const double rr = sum_parts(part + 1, nb, 2, sh);
  const double rz = ctrl->cg_rzp[1][step & 1];
  const double beta = rz != 0.0 ? rz1 / rz : 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctrl->cg_rzp[1][(step + 1) & 1] = rz1;
    if (rr <= tol * tol * ctrl->cg_rz0[1] || ctrl->cg_alpha[1] == 0.0)
      ctrl->cg_done[1] = 1;
  }
  const int64_t c = *cnt;
  for (int64_t a = (int64_t)blockIdx.x * SC_NT + threadIdx.x; a < c;
       a += (int64_t)gridDim.x * SC_NT) {
    const T pn = zz[a] + (T)beta * p[a];
    p[a] = pn;
    phat[J[a]] = pn;
  }
}

// Long segments of the CG products (one replica of A, rep == 1): one
// workgroup each, so that a few power-law rows do not hold up the launch
// that walks all the short ones with G lanes per segment.  The main kernels
// skip every segment longer than the limit the long lists were built with.
// Wide products take every long segment (A.longs); listed products only
// the long segments whose position in the block list is recorded in pos
// (-1: not in the block).  Each workgroup writes its result and one
// partial (q^2 for columns' wide product, s^2 or <p, v> for the listed
// ones) that the main kernel's last block adds in index order.
template <typename T>
__global__ void __launch_bounds__(SC_NT)
sc_long_wide(Csr<T> A, const T *__restrict__ phat, T *__restrict__ out,
             T *__restrict__ x, double *__restrict__ plong, Ctrl *ctrl,
             int ph, int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  if (cg_done_at_start(ctrl, ph)) return;
  __shared__ double sh[SC_NT / WAVE];
  const int64_t r = A.longs[blockIdx.x];
  const int64_t e0 = A.ptr[r], e1 = seg_end(A, r);
  T acc = 0;
  for (int64_t e = e0 + threadIdx.x; e < e1; e += SC_NT)
    acc += A.val[e] * phat[A.idx[e]];
  const T sv = (T)block_sum<SC_NT>((double)acc, sh);
  if (threadIdx.x == 0) {
    if (x) {   // rows: this column's pending x += alpha_prev u_prev first
      const double alpha = ctrl->cg_alpha[ph];
      if (alpha != 0.0) x[r] += (T)alpha * out[r];
    }
    out[r] = sv;
    plong[blockIdx.x] = (double)sv * (double)sv;
  }
}

template <typename T>
__global__ void __launch_bounds__(SC_NT)
sc_long_narrow(Csr<T> A, const int32_t *__restrict__ pos,
               const T *__restrict__ vec, T *__restrict__ dst,
               const T *__restrict__ p, double *__restrict__ plong,
               Ctrl *ctrl, int ph, int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  if (cg_done_at_start(ctrl, ph)) return;
  __shared__ double sh[SC_NT / WAVE];
  const int64_t r = A.longs[blockIdx.x];
  const int32_t a = pos[r];
  if (a < 0) {
    if (threadIdx.x == 0) plong[blockIdx.x] = 0.0;
    return;
  }
  const int64_t e0 = A.ptr[r], e1 = A.ptr[r + 1];
  T acc = 0;
  for (int64_t e = e0 + threadIdx.x; e < e1; e += SC_NT)
    acc += A.val[e] * vec[A.idx[e]];
  const T w = (T)block_sum<SC_NT>((double)acc, sh);
  if (threadIdx.x == 0) {
    if (ph == 0) {   // columns: s_a -= alpha w
      const T sv = dst[a] - (T)ctrl->cg_alpha[0] * w;
      dst[a] = sv;
      plong[blockIdx.x] = (double)sv * (double)sv;
    } else {         // rows: v_a = w
      dst[a] = w;
      plong[blockIdx.x] = (double)w * (double)p[a];
    }
  }
}

// rows: wide product u = A^T phat over CSC columns, with the pending update
// x += alpha_prev * u_prev applied first (same column, same thread).
template <typename T, int G>
__global__ void __launch_bounds__(SC_NT)
sc_wide_row(Csr<T> At, const T *__restrict__ phat, T *__restrict__ u,
            T *__restrict__ x, int64_t nlong, Ctrl *ctrl, int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  if (cg_done_at_start(ctrl, 1)) return;
  const double alpha = ctrl->cg_alpha[1];
  constexpr int SPB = SC_NT / G;
  const int lg = threadIdx.x & (G - 1);
  const int64_t slot = (int64_t)blockIdx.x * SPB + threadIdx.x / G;
  int64_t s = 0, br = 0, co = 0;
  T acc = 0;
  bool mine = slot < At.rows;
  if (mine) {
    vrow(At, slot, s, br, co);
    const T *ph = phat + co;
    const int64_t e0 = At.ptr[br], e1 = seg_end(At, br);
    if (nlong && (At.long_flag ? At.long_flag[br] != 0 : e1 - e0 > At.long_limit))
      mine = false;   // sc_long_wide
    else
      for (int64_t e = e0 + lg; e < e1; e += G) acc += At.val[e] * ph[At.idx[e]];
  }
  acc = group_sum<G>(acc);
  if (mine && lg == 0) {
    if (alpha != 0.0) x[s] += (T)alpha * u[s];
    u[s] = acc;
  }
}

template <typename T, int G>
__global__ void __launch_bounds__(SC_NT)
sc_narrow_row(Csr<T> A, const int32_t *__restrict__ J,
              const int64_t *__restrict__ cnt, const T *__restrict__ u,
              const double *__restrict__ rho, T *__restrict__ res,
              T *__restrict__ zz, T *__restrict__ p, T *__restrict__ v,
              T *__restrict__ phat, double *__restrict__ part,
              const double *__restrict__ plong, int64_t nlong, double tol,
              int par, const T *__restrict__ pre, Ctrl *ctrl,
              int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  if (cg_done_at_start(ctrl, 1)) return;
  __shared__ double sh[SC_NT / WAVE];
  const int64_t c = *cnt;
  constexpr int SPB = SC_NT / G;
  const int lg = threadIdx.x & (G - 1);
  double pv = 0.0;
  for (int64_t a0 = (int64_t)blockIdx.x * SPB; a0 < c;
       a0 += (int64_t)gridDim.x * SPB) {
    const int64_t a = a0 + threadIdx.x / G;
    T acc = 0;
    bool mine = a < c;
    if (mine) {
      int64_t brw, co;
      gsplit(A, (int64_t)J[a], brw, co);
      if (pre) {   // many right-hand sides: A u formed interleaved
        if (lg == 0) acc = pre[brw * A.rep + (int64_t)J[a] / A.brows];
      } else {
        const T *uv = u + co;
        const int64_t e0 = A.ptr[brw], e1 = A.ptr[brw + 1];
        if (nlong && e1 - e0 > A.long_limit) mine = false;   // sc_long_narrow
        else
          for (int64_t e = e0 + lg; e < e1; e += G) acc += A.val[e] * uv[A.idx[e]];
      }
    }
    acc = group_sum<G>(acc);
    if (mine && lg == 0) {
      if (par) v[a] = acc;
      else st_agent(&v[a], acc);   // read by the last block
      pv += (double)acc * (double)p[a];
    }
  }
  pv = block_sum<SC_NT>(pv, sh);
  if (par) {   // the next launch reduces the partials
    if (threadIdx.x == 0) part[blockIdx.x] = pv;
    return;
  }
  if (threadIdx.x == 0) st_agent(&part[blockIdx.x], pv);
  if (!last_block(&ctrl->ticket[5])) return;
  double tot = 0.0, tl = 0.0;
  for (int b = threadIdx.x; b < (int)gridDim.x; b += SC_NT) tot += ld_agent(&part[b]);
  for (int64_t i = threadIdx.x; i < nlong; i += SC_NT) tl += plong[i];
  tot = block_sum<SC_NT>(tot, sh);
  tot += block_sum<SC_NT>(tl, sh);
  const double rz = ctrl->cg_rz[1];
  const double alpha = tot != 0.0 ? rz / tot : 0.0;
  double rz1 = 0.0, rr = 0.0;
  // one block walks the whole list: keep SC_UNROLL loads in flight
  for (int64_t k0 = threadIdx.x; k0 < c; k0 += SC_UNROLL * SC_NT) {
    T rv[SC_UNROLL], vv[SC_UNROLL];
    double dj[SC_UNROLL];
#pragma unroll
    for (int u = 0; u < SC_UNROLL; ++u) {
      const int64_t k = k0 + (int64_t)u * SC_NT;
      if (k < c) { rv[u] = res[k]; vv[u] = ld_agent(&v[k]); dj[u] = rho[J[k]]; }
    }
#pragma unroll
    for (int u = 0; u < SC_UNROLL; ++u) {
      const int64_t k = k0 + (int64_t)u * SC_NT;
      if (k < c) {
        const T r = rv[u] - (T)alpha * vv[u];
        res[k] = r;
        const T zv = dj[u] > 0.0 ? (T)((double)r / dj[u]) : (T)0;
        zz[k] = zv;
        rz1 += (double)r * (double)zv;
        rr += (double)r * (double)r;
      }
    }
  }
  rz1 = block_sum<SC_NT>(rz1, sh);
  rr = block_sum<SC_NT>(rr, sh);
  const double beta = rz != 0.0 ? rz1 / rz : 0.0;
  for (int64_t k0 = threadIdx.x; k0 < c; k0 += SC_UNROLL * SC_NT) {
    T zv[SC_UNROLL], po[SC_UNROLL];
    int32_t ix[SC_UNROLL];
#pragma unroll
    for (int u = 0; u < SC_UNROLL; ++u) {
      const int64_t k = k0 + (int64_t)u * SC_NT;
      if (k < c) { zv[u] = zz[k]; po[u] = p[k]; ix[u] = J[k]; }
    }
#pragma unroll
    for (int u = 0; u < SC_UNROLL; ++u) {
      const int64_t k = k0 + (int64_t)u * SC_NT;
      if (k < c) {
        const T pn = zv[u] + (T)beta * po[u];
        p[k] = pn;
        phat[ix[u]] = pn;
      }
    }
  }
  if (threadIdx.x == 0) {
    ctrl->cg_alpha[1] = alpha;
    ctrl->cg_rz[1] = rz1;
    ctrl->cg_steps[1] += 1;
    if (rr <= tol * tol * ctrl->cg_rz0[1] || tot == 0.0) ctrl->cg_done[1] = 1;
  }
}

// final pending update x += alpha u (always exactly once per row phase)
template <typename T>
__global__ void __launch_bounds__(SC_NT)
sc_row_finish(int64_t n, const T *__restrict__ u, T *__restrict__ x,
              Ctrl *ctrl, int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  const double alpha = ctrl->cg_alpha[1];
  const int64_t j = (int64_t)blockIdx.x * SC_NT + threadIdx.x;
  if (j < n && alpha != 0.0) x[j] += (T)alpha * u[j];
}

// workgroups of the elementwise launches over a block
static unsigned sc_list_blocks(int64_t cap) {
  const int64_t b = (cap + SC_NT - 1) / SC_NT;
  return (unsigned)std::max<int64_t>(1, std::min<int64_t>(b, SC_SUM_MAX));
}
int64_t sparse_cg_parts(int64_t len, int64_t cap) {
  return len / 4 + cap / 4 + 1024 + 4 * (int64_t)SC_SUM_MAX;
}

// Start of a phase's CG: for blocks finished in the last workgroup one
// launch, else the partials and their sum apart.
template <typename T>
static void sc_start(const int32_t *list, const int64_t *cnt, int64_t cap,
                     const T *rhs, const double *jac, T *zz, SparseCg<T> &w,
                     int32_t *pos, int par, Ctrl *ctrl, int ph,
                     int respect_done, hipStream_t st) {
  const unsigned nb = sc_list_blocks(cap);
  hipLaunchKernelGGL(sc_init<T>, dim3(nb), dim3(SC_NT), 0, st, list, cnt, rhs,
                     jac, w.res, zz, w.p, w.phat, pos, w.part, par, ctrl, ph,
                     respect_done);
  if (par)
    hipLaunchKernelGGL(sc_init_fin, dim3(1), dim3(SC_NT), 0, st,
                       (const double *)w.part, (int)nb, cnt, ctrl, ph,
                       respect_done);
}

template <typename T>
static unsigned seg_blocks(int64_t nseg, int G) {
  return (unsigned)((nseg + (SC_NT / G) - 1) / (SC_NT / G));
}

#define RG_SWITCH_G(GV, CALL)                 \
  switch (GV) {                               \
    case 1: { constexpr int GG = 1; CALL; } break;   \
    case 2: { constexpr int GG = 2; CALL; } break;   \
    case 4: { constexpr int GG = 4; CALL; } break;   \
    case 8: { constexpr int GG = 8; CALL; } break;   \
    case 16: { constexpr int GG = 16; CALL; } break; \
    case 32: { constexpr int GG = 32; CALL; } break; \
    default: { constexpr int GG = 64; CALL; } break; \
  }

template <typename T>
void launch_sparse_colproj(const Csr<T> &csr, const Csr<T> &csc,
                           const int32_t *U, const int64_t *count_dev,
                           int64_t cap, const T *g, T *z, SparseCg<T> &w,
                           int max_steps, double tol, Ctrl *ctrl,
                           int respect_done, hipStream_t st) {
  // long segments apart only for one replica of A (the lists are built
  // for it); a replicated operator walks every segment with G lanes
  const int64_t nlw = csr.rep == 1 && w.pos ? csr.nlong : 0;
  const int64_t nln = csc.rep == 1 && w.pos ? csc.nlong : 0;
  // many right-hand sides: both products over interleaved vectors, and the
  // listed product reads its value from them (one lane per listed column)
  const bool mm = csr.rep >= REP_MM_MIN && w.t0 != nullptr;
  const int par = (w.split || cap > SC_SERIAL_MAX || mm) ? 1 : 0;
  sc_start<T>(U, count_dev, cap, g, (const double *)nullptr, (T *)nullptr, w,
              nln ? w.pos : (int32_t *)nullptr, par, ctrl, 0, respect_done, st);
  const unsigned nbw = std::min<unsigned>(seg_blocks<T>(csr.rows, csr.group), SC_WIDE_MAXB);
  // many rows: a full grid and a separate reduction instead of a bounded
  // grid walking SC_WIDE_GRID_MIN or more row slots per thread group
  const unsigned nbg = seg_blocks<T>(csr.rows, csr.group);
  const bool wide_grid = par || (nbg >= SC_WIDE_GRID_MIN * SC_WIDE_MAXB &&
                                 (int64_t)nbg <= w.part_cap);
  const int gn = mm ? 1 : csc.group;
  // large blocks: the listed product over a full grid (no grid-stride walk,
  // no last-workgroup ticket)
  const unsigned nbn = par ? seg_blocks<T>(cap, gn)
                           : std::max(64u, std::min(seg_blocks<T>(cap, gn),
                                                    SC_MAXB));
  const unsigned nbu = sc_list_blocks(cap);
  // The step's scalars: added up from the partials by the next launch where
  // those are few, else by a launch in between (which also adds the long
  // segments').  Where the listed product
  // reads the wide one's partials, its own lie apart.
  const bool sum_n = par && !nln && nbn <= SC_SUM_MAX;
  const bool sum_w = sum_n && !mm && !nlw && nbg <= SC_SUM_MAX;
  double *pn = sum_n ? w.part + (w.part_cap - 4 * (int64_t)SC_SUM_MAX) : w.part;
  for (int s = 0; s < max_steps; ++s) {
    if (mm) {
      // q = A phat for every right-hand side, ||q||^2 -> alpha; then A^T q
      launch_rep_tin<T>(w.phat, w.t0, csr.bcols, csr.rep, ctrl, 0,
                        respect_done, st);
      const int nbm = launch_rep_mm<T>(csr, w.t0, w.t1, w.part, ctrl, 0,
                                       respect_done, st);
      hipLaunchKernelGGL(sc_wide_col_fin<T>, dim3(1), dim3(1024), 0, st,
                         (const double *)w.part, (int64_t)nbm,
                         (const double *)nullptr, (int64_t)0, s, ctrl,
                         respect_done);
      launch_rep_tout<T>(w.t1, w.wide, (T *)nullptr, csr.brows, csr.rep, ctrl,
                         0, respect_done, st);
      launch_rep_mm<T>(csc, w.t1, w.t2, (double *)nullptr, ctrl, 0,
                       respect_done, st);
    } else {
    if (nlw)
      hipLaunchKernelGGL(sc_long_wide<T>, dim3((unsigned)nlw), dim3(SC_NT), 0,
                         st, csr, w.phat, w.wide, (T *)nullptr, w.plong, ctrl,
                         0, respect_done);
    if (wide_grid) {
      RG_SWITCH_G(csr.group,
                  hipLaunchKernelGGL((sc_wide_col_grid<T, GG>), dim3(nbg),
                                     dim3(SC_NT), 0, st, csr, w.phat, w.wide,
                                     w.part, nlw, ctrl, respect_done));
      if (!sum_w)
        hipLaunchKernelGGL(sc_wide_col_fin<T>, dim3(1), dim3(1024), 0, st,
                           (const double *)w.part, (int64_t)nbg,
                           (const double *)w.plong, nlw, par ? s : -1, ctrl,
                           respect_done);
    } else {
      RG_SWITCH_G(csr.group, hipLaunchKernelGGL((sc_wide_col<T, GG>), dim3(nbw),
                                                dim3(SC_NT), 0, st, csr, w.phat,
                                                w.wide, w.part, w.plong, nlw,
                                                ctrl, respect_done));
    }
    }
    if (nln)
      hipLaunchKernelGGL(sc_long_narrow<T>, dim3((unsigned)nln), dim3(SC_NT),
                         0, st, csc, w.pos, w.wide, w.res, w.p, w.plong, ctrl,
                         0, respect_done);
    RG_SWITCH_G(gn,
                hipLaunchKernelGGL((sc_narrow_col<T, GG>), dim3(nbn),
                                   dim3(SC_NT), 0, st, csc, U, count_dev,
                                   w.wide, z, csr.rows, w.res, w.p, w.phat,
                                   pn, w.plong, nln, tol, par,
                                   mm ? (const T *)w.t2 : (const T *)nullptr,
                                   (const double *)w.part,
                                   sum_w ? (int)nbg : 0, s, ctrl,
                                   respect_done));
    if (par && !sum_n)
      hipLaunchKernelGGL(sc_narrow_col_fin, dim3(1), dim3(1024), 0, st,
                         (const double *)pn, (int64_t)nbn,
                         (const double *)w.plong, nln, tol, s, ctrl,
                         respect_done);
    if (par)
      hipLaunchKernelGGL(sc_cupd<T>, dim3(nbu), dim3(SC_NT), 0, st, U,
                         count_dev, w.res, w.p, w.phat, (const double *)pn,
                         sum_n ? (int)nbn : 0, tol, ctrl, s, respect_done);
  }
  hipLaunchKernelGGL(sc_clear<T>, dim3(nbu), dim3(SC_NT), 0, st, U, count_dev,
                     cap, w.phat, nln ? w.pos : (int32_t *)nullptr, ctrl,
                     respect_done);
}

template <typename T>
void launch_sparse_rowproj(const Csr<T> &csr, const Csr<T> &csc,
                           const int32_t *J, const int64_t *count_dev,
                           int64_t cap, const T *r, const double *rho, T *x,
                           SparseCg<T> &w, int max_steps, double tol,
                           Ctrl *ctrl, int respect_done, hipStream_t st) {
  const int64_t nlw = csc.rep == 1 && w.pos ? csc.nlong : 0;
  const int64_t nln = csr.rep == 1 && w.pos ? csr.nlong : 0;
  const unsigned nbw = seg_blocks<T>(csc.rows, csc.group);
  const bool mm = csr.rep >= REP_MM_MIN && w.t0 != nullptr;
  const int gn = mm ? 1 : csr.group;
  const int par = (w.split || cap > SC_SERIAL_MAX || mm) ? 1 : 0;
  // w.v doubles as the Jacobi-scaled residual buffer zz during steps
  sc_start<T>(J, count_dev, cap, r, rho, w.v, w,
              nln ? w.pos : (int32_t *)nullptr, par, ctrl, 1, respect_done, st);
  const unsigned nbn = par ? seg_blocks<T>(cap, gn)
                           : std::min<unsigned>(seg_blocks<T>(cap, gn), SC_MAXB);
  const unsigned nbu = sc_list_blocks(cap);
  // as for the columns: the product's partials added up by sc_rupd1 where
  // they are few; sc_rupd1's own lie apart
  const bool sum_n = par && !nln && nbn <= SC_SUM_MAX;
  double *pu = w.part + (w.part_cap - 4 * (int64_t)SC_SUM_MAX);
  for (int s = 0; s < max_steps; ++s) {
    if (mm) {
      // u = A^T phat for every right-hand side (the pending x += alpha u
      // applied as u is replaced), then A u
      launch_rep_tin<T>(w.phat, w.t0, csr.brows, csr.rep, ctrl, 1,
                        respect_done, st);
      launch_rep_mm<T>(csc, w.t0, w.t1, (double *)nullptr, ctrl, 1,
                       respect_done, st);
      launch_rep_tout<T>(w.t1, w.wide, x, csc.brows, csr.rep, ctrl, 1,
                         respect_done, st);
      launch_rep_mm<T>(csr, w.t1, w.t2, (double *)nullptr, ctrl, 1,
                       respect_done, st);
    } else {
    if (nlw)
      hipLaunchKernelGGL(sc_long_wide<T>, dim3((unsigned)nlw), dim3(SC_NT), 0,
                         st, csc, w.phat, w.wide, x, w.plong, ctrl, 1,
                         respect_done);
    RG_SWITCH_G(csc.group, hipLaunchKernelGGL((sc_wide_row<T, GG>), dim3(nbw),
                                              dim3(SC_NT), 0, st, csc, w.phat,
                                              w.wide, x, nlw, ctrl,
                                              respect_done));
    }
    if (nln)
      hipLaunchKernelGGL(sc_long_narrow<T>, dim3((unsigned)nln), dim3(SC_NT),
                         0, st, csr, w.pos, w.wide, w.v + cap, w.p, w.plong,
                         ctrl, 1, respect_done);
    RG_SWITCH_G(gn,
                hipLaunchKernelGGL((sc_narrow_row<T, GG>), dim3(nbn),
                                   dim3(SC_NT), 0, st, csr, J, count_dev,
                                   w.wide, rho, w.res, w.v, w.p,
                                   w.v + cap, w.phat, w.part, w.plong, nln,
                                   tol, par,
                                   mm ? (const T *)w.t2 : (const T *)nullptr,
                                   ctrl, respect_done));
    if (par) {
      if (!sum_n)
        hipLaunchKernelGGL(sc_narrow_row_fin, dim3(1), dim3(1024), 0, st,
                           (const double *)w.part, (int64_t)nbn,
                           (const double *)w.plong, nln, s, ctrl,
                           respect_done);
      hipLaunchKernelGGL(sc_rupd1<T>, dim3(nbu), dim3(SC_NT), 0, st, J,
                         count_dev, rho, w.res, w.v, w.v + cap,
                         (const double *)w.part, sum_n ? (int)nbn : 0, pu,
                         ctrl, s, respect_done);
      hipLaunchKernelGGL(sc_rupd2<T>, dim3(nbu), dim3(SC_NT), 0, st, J,
                         count_dev, w.v, w.p, w.phat, (const double *)pu,
                         (int)nbu, tol, ctrl, s, respect_done);
    }
  }
  hipLaunchKernelGGL(sc_row_finish<T>, dim3((unsigned)((csc.rows + SC_NT - 1) / SC_NT)),
                     dim3(SC_NT), 0, st, csc.rows, w.wide, x, ctrl,
                     respect_done);
  hipLaunchKernelGGL(sc_clear<T>, dim3(nbu), dim3(SC_NT), 0, st, J, count_dev,
                     cap, w.phat, nln ? w.pos : (int32_t *)nullptr, ctrl,
                     respect_done);
}

// ------------------------------------------------------------ small sparse
// Dense row- and column-major copies of a sparse A (one thread per row,
// repeated entries summed in storage order; the buffers come zeroed).
template <typename T>
__global__ void __launch_bounds__(256)
densify_kernel(Csr<T> A, T *__restrict__ rm, int64_t ld, T *__restrict__ cm,
               int64_t ldc) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= A.rows) return;
  for (int64_t e = A.ptr[i]; e < A.ptr[i + 1]; ++e) {
    const int64_t j = A.idx[e];
    rm[i * ld + j] += A.val[e];
    cm[j * ldc + i] += A.val[e];
  }
}

template <typename T>
__global__ void __launch_bounds__(256)
list_scatter(const int32_t *__restrict__ list, const int64_t *__restrict__ cnt,
             const T *__restrict__ coef, T *__restrict__ dst, Ctrl *ctrl,
             int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  const int64_t c = *cnt;
  for (int64_t a = (int64_t)blockIdx.x * 256 + threadIdx.x; a < c;
       a += (int64_t)gridDim.x * 256)
    dst[list[a]] = coef[a];
}

// out_i += sign * sum_e A_ie phat_(idx e), one thread per row of the view
// (small systems only), in storage order
template <typename T>
__global__ void __launch_bounds__(256)
rows_axpy(Csr<T> A, const T *__restrict__ phat, int sign, T *__restrict__ out,
          Ctrl *ctrl, int respect_done) {
  if (respect_done && ctrl_done(ctrl)) return;
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= A.rows) return;
  T acc = 0;
  bool any = false;
  for (int64_t e = A.ptr[i]; e < A.ptr[i + 1]; ++e) {
    const T v = phat[A.idx[e]];
    if (v != (T)0) {
      acc += A.val[e] * v;
      any = true;
    }
  }
  if (any) out[i] += sign > 0 ? acc : -acc;
}

template <typename T>
void launch_densify(const Csr<T> &A, T *rm, int64_t ld, T *cm, int64_t ldc,
                    hipStream_t st) {
  const unsigned nb = (unsigned)((A.rows + 255) / 256);
  hipLaunchKernelGGL(densify_kernel<T>, dim3(nb > 0 ? nb : 1), dim3(256), 0, st,
                     A, rm, ld, cm, ldc);
}

template <typename T>
void launch_sparse_block_update(const Csr<T> &A, const int32_t *list,
                                const int64_t *count_dev, int64_t cap,
                                const T *coef, int sign, T *phat, T *out,
                                Ctrl *ctrl, int respect_done, hipStream_t st) {
  const unsigned nl = (unsigned)std::max<int64_t>(1, std::min<int64_t>(
      (cap + 255) / 256, 256));
  hipLaunchKernelGGL(list_scatter<T>, dim3(nl), dim3(256), 0, st, list,
                     count_dev, coef, phat, ctrl, respect_done);
  const unsigned nr = (unsigned)((A.rows + 255) / 256);
  hipLaunchKernelGGL(rows_axpy<T>, dim3(nr > 0 ? nr : 1), dim3(256), 0, st, A,
                     phat, sign, out, ctrl, respect_done);
  hipLaunchKernelGGL(sc_clear<T>, dim3(64), dim3(SC_NT), 0, st, list,
                     count_dev, cap, phat, (int32_t *)nullptr, ctrl,
                     respect_done);
}

// ------------------------------------------------------------ instantiate
#define RG_INST(T)                                                            \
  template void launch_gram_gather<T>(const T *, int64_t, const int32_t *,   \
                                      const int64_t *, int64_t, T *, Ctrl *,  \
                                      int, hipStream_t);                      \
  template void launch_gram_rows<T>(const T *, int64_t, int64_t,             \
                                    const int32_t *, const int64_t *,        \
                                    int64_t, T *, Ctrl *, int, hipStream_t);  \
  template void launch_gram_full<T>(const T *, int64_t, int64_t, int64_t,    \
                                    T *, hipStream_t);                        \
  template void launch_pcg_gram_init<T>(const T *, int64_t, const int64_t *, \
                                        const T *, const int32_t *, T *,     \
                                        CgWork<T> &, Ctrl *, int, int,        \
                                        hipStream_t);                         \
  template void launch_pcg_gram_step<T>(const T *, int64_t, const int64_t *, \
                                        T *, CgWork<T> &, int, double,       \
                                        Ctrl *, int, int, hipStream_t);       \
  template void launch_col_update<T>(const T *, int64_t, int64_t,            \
                                     const int32_t *, const int64_t *,       \
                                     int64_t, const T *, T *, T *, Ctrl *,   \
                                     int, hipStream_t);                       \
  template void launch_row_update<T>(const T *, int64_t, int64_t,            \
                                     const int32_t *, const int64_t *,       \
                                     int64_t, const T *, T *, T *, Ctrl *,   \
                                     int, hipStream_t);                       \
  template void launch_list_resid<T>(const T *, int64_t, int64_t,            \
                                     const int32_t *, const int64_t *,       \
                                     int64_t, const T *, const T *,          \
                                     const T *, T *, Ctrl *, int,            \
                                     hipStream_t);                            \
  template void launch_sparse_colproj<T>(const Csr<T> &, const Csr<T> &,     \
                                         const int32_t *, const int64_t *,   \
                                         int64_t, const T *, T *,            \
                                         SparseCg<T> &, int, double, Ctrl *, \
                                         int, hipStream_t);                   \
  template void launch_sparse_rowproj<T>(const Csr<T> &, const Csr<T> &,     \
                                         const int32_t *, const int64_t *,   \
                                         int64_t, const T *, const double *, \
                                         T *, SparseCg<T> &, int, double,    \
                                         Ctrl *, int, hipStream_t);
RG_INST(double)
RG_INST(float)
template void launch_densify<double>(const Csr<double> &, double *, int64_t,
                                     double *, int64_t, hipStream_t);
template void launch_densify<float>(const Csr<float> &, float *, int64_t,
                                    float *, int64_t, hipStream_t);
template void launch_sparse_block_update<double>(
    const Csr<double> &, const int32_t *, const int64_t *, int64_t,
    const double *, int, double *, double *, Ctrl *, int, hipStream_t);
template void launch_sparse_block_update<float>(
    const Csr<float> &, const int32_t *, const int64_t *, int64_t,
    const float *, int, float *, float *, Ctrl *, int, hipStream_t);
#undef RG_INST

// ------------------------------------------------------------ block restriction
// The wide products of the sparse CG (columns: q = A phat over CSR rows;
// rows: u = A^T phat over CSC columns) multiply by a vector that is zero
// outside the block, so only the entries of the block's columns (rows) can
// contribute.  Once per iteration those entries are copied, in storage
// order and with their original indices, into a compact matrix of the same
// row count; every CG step then streams it instead of all of A (about the
// block's share of the nonzeros).  The long rows of A (one workgroup each
// in the CG products) stay long in the copy.  The sums drop only zero terms
// and stay deterministic; their grouping across lanes differs from the full
// pass's, so the two agree to rounding.
// One stored matrix: the copy keeps A's row starts ("gapped"), so one pass
// suffices:
//   mark:   mask[list_a] = 1
//   fill:   each row's marked entries, in order, from A.ptr_r (ballot
//           ranks); end_r = A.ptr_r + their count
//   unmark: mask[list_a] = 0
// For the replicated operator I_rep (x) A of a few right-hand sides the copy
// is a compact matrix over the virtual rows and columns (each right-hand
// side keeps the entries of its own block; the capacity is the k longest
// columns' entries per right-hand side, not A's):
//   mark
//   count:  cnt_r = #{e in row r : mask[idx_e]}            (G lanes per row)
//   scan:   ptr = exclusive prefix sum of cnt             (three launches)
//   fill:   each row's marked entries, in order, to ptr_r
//   unmark
constexpr int SB_NT = 256;
constexpr int SB_TILE = 2048;          // scan elements per workgroup

__global__ void __launch_bounds__(SB_NT)
sub_mark(const int32_t *__restrict__ list, const int64_t *__restrict__ cnt,
         int32_t *__restrict__ mask, int32_t v, Ctrl *ctrl) {
  if (ctrl_done(ctrl)) return;
  const int64_t c = *cnt;
  for (int64_t a = (int64_t)blockIdx.x * SB_NT + threadIdx.x; a < c;
       a += (int64_t)gridDim.x * SB_NT)
    mask[list[a]] = v;
}

template <typename T, int G>
__global__ void __launch_bounds__(SB_NT)
sub_count(Csr<T> A, const int32_t *__restrict__ mask, int64_t *__restrict__ cnt,
          const uint8_t *__restrict__ long_flag, Ctrl *ctrl) {
  if (ctrl_done(ctrl)) return;
  constexpr int SPB = SB_NT / G;
  const int lg = threadIdx.x & (G - 1);
  const int64_t r = (int64_t)blockIdx.x * SPB + threadIdx.x / G;
  int64_t k = 0;
  const bool mine = r < A.rows && !(long_flag && long_flag[r]);   // sub_count_long
  if (mine) {
    int64_t br, co;      // stored row and column offset (replicated A)
    gsplit(A, r, br, co);
    const int32_t *mk = mask + co;
    const int64_t e0 = A.ptr[br], e1 = A.ptr[br + 1];
    for (int64_t e = e0 + lg; e < e1; e += G) k += mk[A.idx[e]] ? 1 : 0;
  }
  k = group_sum<G>(k);
  if (mine && lg == 0) cnt[r] = k;
  if (r == A.rows && lg == 0) cnt[r] = 0;   // sentinel: ptr[rows] = total
}

// exclusive scan of n int64 values: per-tile sums, scan of the tile sums in
// one workgroup, then per-tile scans with the tile offset
__global__ void __launch_bounds__(SB_NT)
sub_scan_a(const int64_t *__restrict__ v, int64_t n,
           int64_t *__restrict__ tile, Ctrl *ctrl) {
  if (ctrl_done(ctrl)) return;
  __shared__ int64_t sh[SB_NT / WAVE];
  const int64_t i0 = (int64_t)blockIdx.x * SB_TILE;
  int64_t s = 0;
  for (int64_t i = i0 + threadIdx.x; i < i0 + SB_TILE && i < n; i += SB_NT)
    s += v[i];
  s = block_sum_i64<SB_NT>(s, sh);
  if (threadIdx.x == 0) tile[blockIdx.x] = s;
}
__global__ void __launch_bounds__(1024)
sub_scan_b(int64_t *__restrict__ tile, int64_t ntile, Ctrl *ctrl) {
  if (ctrl_done(ctrl)) return;
  __shared__ int64_t sh[1024];
  int64_t carry = 0;
  for (int64_t b0 = 0; b0 < ntile; b0 += 1024) {
    const int64_t b = b0 + threadIdx.x;
    const int64_t v = b < ntile ? tile[b] : 0;
    sh[threadIdx.x] = v;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
      const int64_t t = threadIdx.x >= o ? sh[threadIdx.x - o] : 0;
      __syncthreads();
      sh[threadIdx.x] += t;
      __syncthreads();
    }
    if (b < ntile) tile[b] = carry + sh[threadIdx.x] - v;   // exclusive
    const int64_t tot = sh[1023];
    __syncthreads();
    carry += tot;
  }
}
__global__ void __launch_bounds__(SB_NT)
sub_scan_c(const int64_t *__restrict__ v, int64_t n,
           const int64_t *__restrict__ tile, int64_t *__restrict__ out,
           Ctrl *ctrl) {
  if (ctrl_done(ctrl)) return;
  constexpr int PER = SB_TILE / SB_NT;   // consecutive elements per thread
  __shared__ int64_t sh[SB_NT];
  const int64_t i0 = (int64_t)blockIdx.x * SB_TILE + (int64_t)threadIdx.x * PER;
  int64_t loc[PER];
  int64_t s = 0;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int64_t i = i0 + u;
    loc[u] = s;
    s += i < n ? v[i] : 0;
  }
  sh[threadIdx.x] = s;
  __syncthreads();
  for (int o = 1; o < SB_NT; o <<= 1) {
    const int64_t t = threadIdx.x >= o ? sh[threadIdx.x - o] : 0;
    __syncthreads();
    sh[threadIdx.x] += t;
    __syncthreads();
  }
  const int64_t base = tile[blockIdx.x] + sh[threadIdx.x] - s;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const int64_t i = i0 + u;
    if (i < n) out[i] = base + loc[u];
  }
}

// ptr == nullptr: the gapped copy of one stored matrix -- row r's entries
// start at A.ptr[r] and end[r] receives their end (no count or scan)
template <typename T, int G>
__global__ void __launch_bounds__(SB_NT)
sub_fill(Csr<T> A, const int32_t *__restrict__ mask,
         const int64_t *__restrict__ ptr, int32_t *__restrict__ idx,
         T *__restrict__ val, const uint8_t *__restrict__ long_flag,
         int64_t *__restrict__ end, Ctrl *ctrl) {
  if (ctrl_done(ctrl)) return;
  constexpr int SPB = SB_NT / G;
  const int lane = threadIdx.x & (WAVE - 1);
  const int lg = threadIdx.x & (G - 1);
  const int gbase = lane & ~(G - 1);          // first lane of the group
  const int64_t r = (int64_t)blockIdx.x * SPB + threadIdx.x / G;
  const bool live = r < A.rows && !(long_flag && long_flag[r]);  // sub_fill_long
  int64_t br = 0, co = 0;   // stored row and column offset (replicated A)
  if (live) gsplit(A, r, br, co);
  const int64_t e0 = live ? A.ptr[br] : 0, e1 = live ? A.ptr[br + 1] : 0;
  int64_t pos = live ? (ptr ? ptr[r] : e0) : 0;
  // every lane of a wave runs the same trip count (ballots need the whole
  // wave): the longest segment of the wave's groups
  int64_t len = e1 - e0;
  for (int o = 32; o > 0; o >>= 1) {
    const int64_t t = __shfl_xor(len, o, WAVE);
    len = t > len ? t : len;
  }
  const unsigned long long gmask =
      (G == 64) ? ~0ull : (((1ull << G) - 1ull) << gbase);
  for (int64_t c = 0; c < len; c += G) {
    const int64_t e = e0 + c + lg;
    const bool in = e < e1;
    const int32_t j = in ? (int32_t)(co + A.idx[e]) : 0;
    const bool take = in && mask[j] != 0;
    const unsigned long long bal = __ballot(take);
    const unsigned long long mine = bal & gmask;
    const unsigned long long below = mine & ((1ull << lane) - 1ull);
    if (take) {
      const int64_t o = pos + __popcll(below);
      idx[o] = j;
      val[o] = A.val[e];
    }
    pos += __popcll(mine);
  }
  if (!ptr && live && lg == 0) end[r] = pos;
}

// long rows (A.longs): one workgroup each, in storage order
template <typename T>
__global__ void __launch_bounds__(SB_NT)
sub_count_long(Csr<T> A, const int32_t *__restrict__ mask,
               int64_t *__restrict__ cnt, Ctrl *ctrl) {
  if (ctrl_done(ctrl)) return;
  __shared__ int64_t sh[SB_NT / WAVE];
  const int64_t r = A.longs[blockIdx.x];
  const int64_t e0 = A.ptr[r], e1 = A.ptr[r + 1];
  int64_t k = 0;
  for (int64_t e = e0 + threadIdx.x; e < e1; e += SB_NT)
    k += mask[A.idx[e]] ? 1 : 0;
  k = block_sum_i64<SB_NT>(k, sh);
  if (threadIdx.x == 0) cnt[r] = k;
}
template <typename T>
__global__ void __launch_bounds__(SB_NT)
sub_fill_long(Csr<T> A, const int32_t *__restrict__ mask,
              const int64_t *__restrict__ ptr, int32_t *__restrict__ idx,
              T *__restrict__ val, int64_t *__restrict__ end, Ctrl *ctrl) {
  if (ctrl_done(ctrl)) return;
  __shared__ int64_t wsum[SB_NT / WAVE];
  const int lane = threadIdx.x & (WAVE - 1);
  const int w = threadIdx.x / WAVE;
  const int64_t r = A.longs[blockIdx.x];
  const int64_t e0 = A.ptr[r], e1 = A.ptr[r + 1];
  int64_t pos = ptr ? ptr[r] : e0;
  for (int64_t c = e0; c < e1; c += SB_NT) {
    const int64_t e = c + threadIdx.x;
    const bool in = e < e1;
    const int32_t j = in ? A.idx[e] : 0;
    const bool take = in && mask[j] != 0;
    const unsigned long long bal = __ballot(take);
    if (lane == 0) wsum[w] = __popcll(bal);
    __syncthreads();
    int64_t before = 0, tot = 0;
    for (int i = 0; i < SB_NT / WAVE; ++i) {
      before += i < w ? wsum[i] : 0;
      tot += wsum[i];
    }
    if (take) {
      const int64_t o = pos + before + __popcll(bal & ((1ull << lane) - 1ull));
      idx[o] = j;
      val[o] = A.val[e];
    }
    pos += tot;
    __syncthreads();
  }
  if (!ptr && threadIdx.x == 0) end[r] = pos;
}

int64_t sub_scan_tiles(int64_t n) { return (n + SB_TILE - 1) / SB_TILE; }

template <typename T>
__global__ void __launch_bounds__(SB_NT)
mark_long_kernel(Csr<T> A, uint8_t *__restrict__ flag) {
  const int64_t r = (int64_t)blockIdx.x * SB_NT + threadIdx.x;
  if (r < A.rows)
    flag[r] = (A.long_limit > 0 && A.ptr[r + 1] - A.ptr[r] > A.long_limit) ? 1 : 0;
}
template <typename T>
void launch_mark_long(const Csr<T> &A, uint8_t *flag, hipStream_t st) {
  hipLaunchKernelGGL(mark_long_kernel<T>, dim3((unsigned)((A.rows + SB_NT - 1) / SB_NT)),
                     dim3(SB_NT), 0, st, A, flag);
}
template void launch_mark_long<double>(const Csr<double> &, uint8_t *, hipStream_t);
template void launch_mark_long<float>(const Csr<float> &, uint8_t *, hipStream_t);

template <typename T>
Csr<T> launch_sub_matrix(const Csr<T> &A, const int32_t *list,
                         const int64_t *count_dev, int64_t list_cap,
                         SubWork &w, int unmark, Ctrl *ctrl, hipStream_t st) {
  const unsigned gm = (unsigned)std::min<int64_t>(
      std::max<int64_t>((list_cap + SB_NT - 1) / SB_NT, 1), 1024);
  hipLaunchKernelGGL(sub_mark, dim3(gm), dim3(SB_NT), 0, st, list, count_dev,
                     w.mask, 1, ctrl);
  const int64_t rows = A.rows;
  const int G = A.group;
  const unsigned nb = (unsigned)((rows + 1 + SB_NT / G - 1) / (SB_NT / G));
  const uint8_t *lf = (A.nlong && A.rep == 1) ? w.long_flag : nullptr;
  if (A.rep == 1) {
    // one stored matrix: the gapped copy, each row's block entries at the
    // start of its own span of A (row ends in w.cnt), in one pass
    RG_SWITCH_G(G, hipLaunchKernelGGL((sub_fill<T, GG>), dim3(nb), dim3(SB_NT),
                                      0, st, A, w.mask, (const int64_t *)nullptr,
                                      w.idx, (T *)w.val, lf, w.cnt, ctrl));
    if (lf)
      hipLaunchKernelGGL(sub_fill_long<T>, dim3((unsigned)A.nlong), dim3(SB_NT),
                         0, st, A, w.mask, (const int64_t *)nullptr, w.idx,
                         (T *)w.val, w.cnt, ctrl);
    if (unmark)
      hipLaunchKernelGGL(sub_mark, dim3(gm), dim3(SB_NT), 0, st, list,
                         count_dev, w.mask, 0, ctrl);
    Csr<T> B = A;
    B.idx = w.idx;
    B.val = (const T *)w.val;
    B.pend = w.cnt;
    B.group = w.group;
    // A's long rows stay long segments (one workgroup each) in the copy
    B.long_flag = w.long_flag;
    B.mp_rs = nullptr;     // no merge plan: row-split passes only
    B.mp_nchunk = 0;
    return B;
  }
  RG_SWITCH_G(G, hipLaunchKernelGGL((sub_count<T, GG>), dim3(nb), dim3(SB_NT),
                                    0, st, A, w.mask, w.cnt, lf, ctrl));
  if (lf)
    hipLaunchKernelGGL(sub_count_long<T>, dim3((unsigned)A.nlong), dim3(SB_NT),
                       0, st, A, w.mask, w.cnt, ctrl);
  const int64_t nt = sub_scan_tiles(rows + 1);
  hipLaunchKernelGGL(sub_scan_a, dim3((unsigned)nt), dim3(SB_NT), 0, st, w.cnt,
                     rows + 1, w.tile, ctrl);
  hipLaunchKernelGGL(sub_scan_b, dim3(1), dim3(1024), 0, st, w.tile, nt, ctrl);
  hipLaunchKernelGGL(sub_scan_c, dim3((unsigned)nt), dim3(SB_NT), 0, st, w.cnt,
                     rows + 1, w.tile, w.ptr, ctrl);
  RG_SWITCH_G(G, hipLaunchKernelGGL((sub_fill<T, GG>), dim3(nb), dim3(SB_NT),
                                    0, st, A, w.mask, (const int64_t *)w.ptr,
                                    w.idx, (T *)w.val, lf, (int64_t *)nullptr,
                                    ctrl));
  if (lf)
    hipLaunchKernelGGL(sub_fill_long<T>, dim3((unsigned)A.nlong), dim3(SB_NT),
                       0, st, A, w.mask, (const int64_t *)w.ptr, w.idx,
                       (T *)w.val, (int64_t *)nullptr, ctrl);
  hipLaunchKernelGGL(sub_mark, dim3(gm), dim3(SB_NT), 0, st, list, count_dev,
                     w.mask, 0, ctrl);
  Csr<T> B = A;
  B.ptr = w.ptr;
  B.idx = w.idx;
  B.val = (const T *)w.val;
  B.nnz = w.cap;
  B.group = w.group;
  // the replicated operator I_rep (x) A: the copy is a plain matrix over
  // the virtual rows and columns (column indices already offset)
  B.rep = 1;
  B.brows = A.rows;
  B.bcols = A.cols;
  B.longs = nullptr;
  B.nlong = 0;
  B.long_limit = 0;
  B.long_flag = nullptr;
  B.mp_rs = nullptr;     // no merge plan: row-split passes only
  B.mp_nchunk = 0;
  return B;
}
// ------------------------------------------------------------ balanced CG
// The block projections of one stored matrix with products balanced by
// nonzeros.  wr and wc hold the block's entries by rows and by columns.
//
// Taken where a block has more than BAL_MIN_CAP indices, because it was
// faster over all of its range on power-law rows (8 iterations, row split /
// balanced, ms): 10000 x 5000 at 1 % blocks 2.19 / 2.14 and at 50 % 4.13 /
// 3.08, 100000 x 50000 at 10 % 4.83 / 3.24, 1M x 500K at 10 % 13.4 / 11.3 and
// at 50 % 32.1 / 20.9; on 96 grid systems 272 / 253.  Below that the visit of
// all rows costs more than the block (3000 x 1500 at 1 %: 1.90 / 1.96).  Not
// for even rows of 64 entries and more (no long segments), where a wave per
// row is already balanced (40000 x 20000, 1 % dense: 208 / 219), nor where a
// workgroup would get many thousand (empty) rows, which are not spread, nor
// with longer rows or columns than BAL_MAX_LEN: one workgroup walks such a one
// tile by tile, while the row split has a workgroup without tiles for it (50 %
// blocks of 100000 x 100000 with 4 long rows, row split / balanced, ms: of
// 4000 entries 5.37 / 4.93, of 16000 7.5 / 7.7, of 100000 21.6 / 28.6; with
// 200 long rows of 4000 6.2 / 5.9, of 8000 8.0 / 8.3).
constexpr int64_t BAL_MIN_CAP = 32;
constexpr int64_t BAL_MAX_LEN = 4096;
constexpr int64_t BAL_MAX_ROWS = 1024;         // of one chunk of the plan
template <typename T>
bool balanced_cg_takes(const Csr<T> &csr, const Csr<T> &csc, int64_t cap,
                       int64_t part_cap) {
  if (csr.rep != 1 || !csr.mp_rs || !csc.mp_rs || cap <= BAL_MIN_CAP)
    return false;
  if (csr.group == 64 && csc.group == 64 && !csr.nlong && !csc.nlong)
    return false;
  if (std::max(csr.mp_maxrows, csc.mp_maxrows) > BAL_MAX_ROWS) return false;
  if (std::max(csr.mp_maxlen, csc.mp_maxlen) > BAL_MAX_LEN) return false;
  // the copies' and the partials' room
  const int64_t nb = bal_blocks(std::max(csr.mp_nchunk, csc.mp_nchunk));
  return nb + 4 * (int64_t)SC_SUM_MAX <= part_cap &&
         2 * nb <= std::min(csr.rows, csc.rows);
}
template <typename T>
static void bal_copies(const Csr<T> &wide, SubWork &ww, const Csr<T> &narrow,
                       SubWork &wn, int32_t *mask, const int32_t *list,
                       const int64_t *count_dev, int64_t cap, Ctrl *ctrl,
                       hipStream_t st) {
  const unsigned gm = (unsigned)std::min<int64_t>(
      std::max<int64_t>((cap + SB_NT - 1) / SB_NT, 1), 1024);
  hipLaunchKernelGGL(sub_mark, dim3(gm), dim3(SB_NT), 0, st, list, count_dev,
                     mask, 1, ctrl);
  launch_bal_fill<T>(wide, 1, mask, ww, ctrl, st);
  launch_bal_fill<T>(narrow, 0, mask, wn, ctrl, st);
  hipLaunchKernelGGL(sub_mark, dim3(gm), dim3(SB_NT), 0, st, list, count_dev,
                     mask, 0, ctrl);
}
template <typename T>
void launch_balanced_colproj(const Csr<T> &csr, const Csr<T> &csc,
                             SubWork &wr, SubWork &wc, int32_t *mask,
                             const int32_t *U, const int64_t *count_dev,
                             int64_t cap, const T *g, T *z, SparseCg<T> &w,
                             int max_steps, double tol, Ctrl *ctrl,
                             hipStream_t st) {
  bal_copies<T>(csr, wr, csc, wc, mask, U, count_dev, cap, ctrl, st);
  sc_start<T>(U, count_dev, cap, g, (const double *)nullptr, (T *)nullptr, w,
              w.pos, 1, ctrl, 0, 1, st);
  const int64_t nw = bal_blocks(csr.mp_nchunk), nn = bal_blocks(csc.mp_nchunk);
  // partials added up by the next launch where they are few, as above
  const bool sum_w = nw <= SC_SUM_MAX, sum_n = nn <= SC_SUM_MAX;
  double *pn = sum_n ? w.part + (w.part_cap - 4 * (int64_t)SC_SUM_MAX) : w.part;
  if (!sum_n && sum_w) pn = w.part + SC_SUM_MAX;
  const unsigned nbu = sc_list_blocks(cap);
  for (int s = 0; s < max_steps; ++s) {
    launch_bal_prod<T>(csr, BP_COL_WIDE, wr, w.phat, w.wide, (T *)nullptr,
                       nullptr, (const T *)nullptr, 0, w.part, nullptr, 0, s,
                       ctrl, st);
    if (!sum_w)
      hipLaunchKernelGGL(sc_wide_col_fin<T>, dim3(1), dim3(1024), 0, st,
                         (const double *)w.part, nw, (const double *)nullptr,
                         (int64_t)0, s, ctrl, 1);
    launch_bal_prod<T>(csc, BP_COL_NARROW, wc, w.wide, w.res, z, w.pos,
                       (const T *)nullptr, csr.rows, pn, w.part,
                       sum_w ? (int)nw : 0, s, ctrl, st);
    if (!sum_n)
      hipLaunchKernelGGL(sc_narrow_col_fin, dim3(1), dim3(1024), 0, st,
                         (const double *)pn, nn, (const double *)nullptr,
                         (int64_t)0, tol, s, ctrl, 1);
    hipLaunchKernelGGL(sc_cupd<T>, dim3(nbu), dim3(SC_NT), 0, st, U, count_dev,
                       w.res, w.p, w.phat, (const double *)pn,
                       sum_n ? (int)nn : 0, tol, ctrl, s, 1);
  }
  hipLaunchKernelGGL(sc_clear<T>, dim3(nbu), dim3(SC_NT), 0, st, U, count_dev,
                     cap, w.phat, w.pos, ctrl, 1);
}
template <typename T>
void launch_balanced_rowproj(const Csr<T> &csr, const Csr<T> &csc,
                             SubWork &wr, SubWork &wc, int32_t *mask,
                             const int32_t *J, const int64_t *count_dev,
                             int64_t cap, const T *r, const double *rho, T *x,
                             SparseCg<T> &w, int max_steps, double tol,
                             Ctrl *ctrl, hipStream_t st) {
  bal_copies<T>(csc, wc, csr, wr, mask, J, count_dev, cap, ctrl, st);
  sc_start<T>(J, count_dev, cap, r, rho, w.v, w, w.pos, 1, ctrl, 1, 1, st);
  const int64_t nn = bal_blocks(csr.mp_nchunk);
  const bool sum_n = nn <= SC_SUM_MAX;
  double *pu = w.part + (w.part_cap - 4 * (int64_t)SC_SUM_MAX);
  const unsigned nbu = sc_list_blocks(cap);
  for (int s = 0; s < max_steps; ++s) {
    launch_bal_prod<T>(csc, BP_ROW_WIDE, wc, w.phat, w.wide, x, nullptr,
                       (const T *)nullptr, 0, (double *)nullptr, nullptr, 0, s,
                       ctrl, st);
    launch_bal_prod<T>(csr, BP_ROW_NARROW, wr, w.wide, w.v + cap, (T *)nullptr,
                       w.pos, w.p, 0, w.part, nullptr, 0, s, ctrl, st);
    if (!sum_n)
      hipLaunchKernelGGL(sc_narrow_row_fin, dim3(1), dim3(1024), 0, st,
                         (const double *)w.part, nn, (const double *)nullptr,
                         (int64_t)0, s, ctrl, 1);
    hipLaunchKernelGGL(sc_rupd1<T>, dim3(nbu), dim3(SC_NT), 0, st, J,
                       count_dev, rho, w.res, w.v, w.v + cap,
                       (const double *)w.part, sum_n ? (int)nn : 0, pu, ctrl,
                       s, 1);
    hipLaunchKernelGGL(sc_rupd2<T>, dim3(nbu), dim3(SC_NT), 0, st, J,
                       count_dev, w.v, w.p, w.phat, (const double *)pu,
                       (int)nbu, tol, ctrl, s, 1);
  }
  hipLaunchKernelGGL(sc_row_finish<T>,
                     dim3((unsigned)((csc.rows + SC_NT - 1) / SC_NT)),
                     dim3(SC_NT), 0, st, csc.rows, w.wide, x, ctrl, 1);
  hipLaunchKernelGGL(sc_clear<T>, dim3(nbu), dim3(SC_NT), 0, st, J, count_dev,
                     cap, w.phat, w.pos, ctrl, 1);
}
#define INST_BAL(T)                                                           \
  template bool balanced_cg_takes<T>(const Csr<T> &, const Csr<T> &, int64_t, \
                                     int64_t);                                \
  template void launch_balanced_colproj<T>(                                   \
      const Csr<T> &, const Csr<T> &, SubWork &, SubWork &, int32_t *,        \
      const int32_t *, const int64_t *, int64_t, const T *, T *,              \
      SparseCg<T> &, int, double, Ctrl *, hipStream_t);                       \
  template void launch_balanced_rowproj<T>(                                   \
      const Csr<T> &, const Csr<T> &, SubWork &, SubWork &, int32_t *,        \
      const int32_t *, const int64_t *, int64_t, const T *, const double *,   \
      T *, SparseCg<T> &, int, double, Ctrl *, hipStream_t);
INST_BAL(double)
INST_BAL(float)

template Csr<double> launch_sub_matrix<double>(const Csr<double> &, const int32_t *, const int64_t *, int64_t, SubWork &, int, Ctrl *, hipStream_t);
template Csr<float> launch_sub_matrix<float>(const Csr<float> &, const int32_t *, const int64_t *, int64_t, SubWork &, int, Ctrl *, hipStream_t);

// ------------------------------------------------------------ tall row blocks
// A row block with more rows than A has columns (k_row > n) is in general
// inconsistent: r^J need not lie in range(A^J), and CG on A^J A^J^T does not
// reach the pseudoinverse update there.  Such blocks are projected by CGLS on
// min ||A^J d - r^J|| started at d = 0, whose limit is the minimum-norm
// least-squares solution (A^J)^+ r^J (for independent columns,
// (A^J^T A^J)^-1 A^J^T r^J):
//   res = r^J, s = A^J^T res, p = s, gam = ||s||^2
//   step: q = A^J p; alpha = gam / ||q||^2; d += alpha p; res -= alpha q;
//         s = A^J^T res; gam' = ||s||^2 (stop when gam' <= tol^2 gam_0);
//         p = s + (gam'/gam) p
//   x += d
// The vector recurrences and their norms run in one workgroup (fixed
// order); the products are listed-row dots and the thin row update (dense),
// or listed CSR segment dots and a CSC pass over the residual scattered
// onto the block's rows (sparse).  Ctrl::cg_rz[1] holds gam, cg_rz0[1] gam_0.
constexpr int TL_NT = 1024;

// d = 0, s = 0 (n); rhat = 0 (m); CG flags of the row phase reset
template <typename T>
__global__ void __launch_bounds__(256)
tall_init(int64_t n, int64_t m, T *__restrict__ d, T *__restrict__ s,
          T *__restrict__ rhat, Ctrl *ctrl) {
  if (ctrl_done(ctrl)) return;
  const int64_t stride = (int64_t)gridDim.x * 256;
  const int64_t i0 = (int64_t)blockIdx.x * 256 + threadIdx.x;
  for (int64_t i = i0; i < n; i += stride) { d[i] = (T)0; s[i] = (T)0; }
  if (rhat)
    for (int64_t i = i0; i < m; i += stride) rhat[i] = (T)0;
  if (i0 == 0) { ctrl->cg_done[1] = 0; ctrl->cg_steps[1] = 0; }
}

// res_a = r[J_a] (and rhat[J_a] = res_a)
template <typename T>
__global__ void __launch_bounds__(256)
tall_load(const int32_t *__restrict__ J, const int64_t *__restrict__ cnt,
          const T *__restrict__ r, T *__restrict__ res, T *__restrict__ rhat,
          Ctrl *ctrl) {
  if (ctrl_done(ctrl)) return;
  const int64_t c = *cnt;
  for (int64_t a = (int64_t)blockIdx.x * 256 + threadIdx.x; a < c;
       a += (int64_t)gridDim.x * 256) {
    const T v = r[J[a]];
    res[a] = v;
    if (rhat) rhat[J[a]] = v;
  }
}

// gam = gam_0 = ||s||^2, p = s
template <typename T>
__global__ void __launch_bounds__(TL_NT)
tall_start(int64_t n, const T *__restrict__ s, T *__restrict__ p, Ctrl *ctrl) {
  if (ctrl_done(ctrl)) return;
  __shared__ double sh[TL_NT / WAVE];
  double g = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += TL_NT) {
    const T v = s[i];
    p[i] = v;
    g += (double)v * (double)v;
  }
  g = block_sum<TL_NT>(g, sh);
  if (threadIdx.x == 0) {
    ctrl->cg_rz[1] = g;
    ctrl->cg_rz0[1] = g;
    if (!(g > 0.0)) ctrl->cg_done[1] = 1;
  }
}

// dense q_a = <A_{J_a}, p>: one wave per listed row
template <typename T>
__global__ void __launch_bounds__(256)
tall_rowdot(const T *__restrict__ A, int64_t ld, int64_t n,
            const int32_t *__restrict__ J, const int64_t *__restrict__ cnt,
            const T *__restrict__ p, T *__restrict__ q, Ctrl *ctrl) {
  if (ctrl_done(ctrl) || ctrl->cg_done[1]) return;
  const int lane = threadIdx.x & (WAVE - 1);
  const int64_t a = (int64_t)blockIdx.x * 4 + threadIdx.x / WAVE;
  if (a >= *cnt) return;
  const T *row = A + (int64_t)J[a] * ld;
  T acc = (T)0;
  for (int64_t t = lane; t < n; t += WAVE) acc += row[t] * p[t];
  acc = wave_sum(acc);
  if (lane == 0) q[a] = acc;
}

// alpha = gam / ||q||^2; d += alpha p; res -= alpha q; then the input of the
// next transpose product: s = 0 (dense, accumulated into) or rhat[J_a] = res_a
template <typename T>
__global__ void __launch_bounds__(TL_NT)
tall_mid(int64_t n, const int32_t *__restrict__ J,
         const int64_t *__restrict__ cnt, const T *__restrict__ p,
         const T *__restrict__ q, T *__restrict__ d, T *__restrict__ res,
         T *__restrict__ s, T *__restrict__ rhat, Ctrl *ctrl) {
  if (ctrl_done(ctrl) || ctrl->cg_done[1]) return;
  __shared__ double sh[TL_NT / WAVE];
  const int64_t c = *cnt;
  double qq = 0.0;
  for (int64_t a = threadIdx.x; a < c; a += TL_NT)
    qq += (double)q[a] * (double)q[a];
  qq = block_sum<TL_NT>(qq, sh);
  const double gam = ctrl->cg_rz[1];
  if (!(qq > 0.0)) {
    if (threadIdx.x == 0) ctrl->cg_done[1] = 1;
    return;
  }
  const T alpha = (T)(gam / qq);
  for (int64_t i = threadIdx.x; i < n; i += TL_NT) {
    d[i] += alpha * p[i];
    if (!rhat) s[i] = (T)0;
  }
  for (int64_t a = threadIdx.x; a < c; a += TL_NT) {
    const T v = res[a] - alpha * q[a];
    res[a] = v;
    if (rhat) rhat[J[a]] = v;
  }
}

// gam' = ||s||^2; stop at gam' <= tol^2 gam_0; p = s + (gam'/gam) p
template <typename T>
__global__ void __launch_bounds__(TL_NT)
tall_end(int64_t n, const T *__restrict__ s, T *__restrict__ p, double tol,
         int max_steps, Ctrl *ctrl) {
  if (ctrl_done(ctrl) || ctrl->cg_done[1]) return;
  __shared__ double sh[TL_NT / WAVE];
  double g = 0.0;
  for (int64_t i = threadIdx.x; i < n; i += TL_NT)
    g += (double)s[i] * (double)s[i];
  g = block_sum<TL_NT>(g, sh);
  const double gam = ctrl->cg_rz[1];
  const int steps = ctrl->cg_steps[1] + 1;
  const bool stop = g <= tol * tol * ctrl->cg_rz0[1] || steps >= max_steps ||
                    !(gam > 0.0);
  if (!stop) {
    const T beta = (T)(g / gam);
    for (int64_t i = threadIdx.x; i < n; i += TL_NT) p[i] = s[i] + beta * p[i];
  }
  __syncthreads();   // every thread has read gam before it is replaced
  if (threadIdx.x == 0) {
    ctrl->cg_rz[1] = g;
    ctrl->cg_steps[1] = steps;
    if (stop) ctrl->cg_done[1] = 1;
  }
}

// x += d
template <typename T>
__global__ void __launch_bounds__(256)
tall_finish(int64_t n, const T *__restrict__ d, T *__restrict__ x, Ctrl *ctrl) {
  if (ctrl_done(ctrl)) return;
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * 256)
    x[i] += d[i];
}

static unsigned tall_grid(int64_t len) {
  int64_t g = (len + 255) / 256;
  if (g > 1024) g = 1024;
  return (unsigned)(g < 1 ? 1 : g);
}

template <typename T>
void launch_tall_rowproj_dense(const Dense<T> &A, const int32_t *J,
                               const int64_t *count_dev, int64_t cap,
                               const T *r, T *x, TallWork<T> &w, T *upd,
                               int max_steps, double tol, Ctrl *ctrl,
                               hipStream_t st) {
  const int64_t n = A.cols;
  hipLaunchKernelGGL(tall_init<T>, dim3(tall_grid(n)), dim3(256), 0, st, n,
                     (int64_t)0, w.d, w.s, (T *)nullptr, ctrl);
  hipLaunchKernelGGL(tall_load<T>, dim3(tall_grid(cap)), dim3(256), 0, st, J,
                     count_dev, r, w.res, (T *)nullptr, ctrl);
  thin_update<T>(A.a, A.ld, n, J, count_dev, cap, w.res, w.s, (T)1, upd, ctrl,
                 1, st);
  hipLaunchKernelGGL(tall_start<T>, dim3(1), dim3(TL_NT), 0, st, n,
                     (const T *)w.s, w.p, ctrl);
  const unsigned gq = (unsigned)((cap + 3) / 4);
  for (int k = 0; k < max_steps; ++k) {
    hipLaunchKernelGGL(tall_rowdot<T>, dim3(gq), dim3(256), 0, st, A.a, A.ld,
                       n, J, count_dev, (const T *)w.p, w.q, ctrl);
    hipLaunchKernelGGL(tall_mid<T>, dim3(1), dim3(TL_NT), 0, st, n, J,
                       count_dev, (const T *)w.p, (const T *)w.q, w.d, w.res,
                       w.s, (T *)nullptr, ctrl);
    thin_update<T>(A.a, A.ld, n, J, count_dev, cap, w.res, w.s, (T)1, upd,
                   ctrl, 1, st);
    hipLaunchKernelGGL(tall_end<T>, dim3(1), dim3(TL_NT), 0, st, n,
                       (const T *)w.s, w.p, tol, max_steps, ctrl);
  }
  hipLaunchKernelGGL(tall_finish<T>, dim3(tall_grid(n)), dim3(256), 0, st, n,
                     (const T *)w.d, x, ctrl);
}

template <typename T>
void launch_tall_rowproj_sparse(const Csr<T> &csr, const Csr<T> &csc,
                                const int32_t *J, const int64_t *count_dev,
                                int64_t cap, const T *r, T *x, TallWork<T> &w,
                                int max_steps, double tol, Ctrl *ctrl,
                                hipStream_t st) {
  const int64_t n = csr.cols, m = csr.rows;
  hipLaunchKernelGGL(tall_init<T>, dim3(tall_grid(std::max(n, m))), dim3(256),
                     0, st, n, m, w.d, w.s, w.rhat, ctrl);
  hipLaunchKernelGGL(tall_load<T>, dim3(tall_grid(cap)), dim3(256), 0, st, J,
                     count_dev, r, w.res, w.rhat, ctrl);
  SegArgs<T> tp;            // s = A^T rhat over the CSC
  tp.v = w.rhat;
  tp.out = w.s;
  launch_segdot<T>(csc, EPI_STORE, tp, ctrl, 1, st);
  hipLaunchKernelGGL(tall_start<T>, dim3(1), dim3(TL_NT), 0, st, n,
                     (const T *)w.s, w.p, ctrl);
  SegArgs<T> lp;            // q = A^J p over the listed CSR rows
  lp.v = w.p;
  lp.out = w.q;
  lp.list = J;
  lp.count_dev = count_dev;
  lp.list_cap = cap;
  for (int k = 0; k < max_steps; ++k) {
    launch_segdot<T>(csr, EPI_LIST_STORE, lp, ctrl, 1, st);
    hipLaunchKernelGGL(tall_mid<T>, dim3(1), dim3(TL_NT), 0, st, n, J,
                       count_dev, (const T *)w.p, (const T *)w.q, w.d, w.res,
                       w.s, w.rhat, ctrl);
    launch_segdot<T>(csc, EPI_STORE, tp, ctrl, 1, st);
    hipLaunchKernelGGL(tall_end<T>, dim3(1), dim3(TL_NT), 0, st, n,
                       (const T *)w.s, w.p, tol, max_steps, ctrl);
  }
  hipLaunchKernelGGL(tall_finish<T>, dim3(tall_grid(n)), dim3(256), 0, st, n,
                     (const T *)w.d, x, ctrl);
}

template void launch_tall_rowproj_dense<double>(const Dense<double> &, const int32_t *, const int64_t *, int64_t, const double *, double *, TallWork<double> &, double *, int, double, Ctrl *, hipStream_t);
template void launch_tall_rowproj_dense<float>(const Dense<float> &, const int32_t *, const int64_t *, int64_t, const float *, float *, TallWork<float> &, float *, int, double, Ctrl *, hipStream_t);
template void launch_tall_rowproj_sparse<double>(const Csr<double> &, const Csr<double> &, const int32_t *, const int64_t *, int64_t, const double *, double *, TallWork<double> &, int, double, Ctrl *, hipStream_t);
template void launch_tall_rowproj_sparse<float>(const Csr<float> &, const Csr<float> &, const int32_t *, const int64_t *, int64_t, const float *, float *, TallWork<float> &, int, double, Ctrl *, hipStream_t);

}  // namespace rg
