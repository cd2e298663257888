// Cholesky solve of a small Gram block (up to CHOL_MAX) in one workgroup:
// L L^T = G, then L L^T y = h.
//
// A factorisation this small is bound by its serial chain (one pivot after
// the other), not by its k^3/3 flops, so everything that is not on the chain
// is taken off it.  Panels of 16 columns; a pivot below 1e-13 of the largest
// diagonal marks the column as dependent (its unknown is set to zero), which
// keeps the projection onto the span of the block exact for rank-deficient
// blocks.
//
// Blocks up to 256 (every block the solver chooses by itself): the whole
// lower triangle stays in the registers of 15 waves, as 16 x 16 tiles in the
// accumulator layout of the matrix cores (136 tiles, 10 per wave).  Per
// panel, wave 0 factors the diagonal tile in registers (a row per lane,
// broadcasts by DPP) together with its inverse, while the other waves take
// the previous panel's product from their tiles; then the tiles below it are
// multiplied by the inverse, and one more product completes the next panel,
// both on the matrix cores with operands exchanged through LDS.  The two
// triangular solves use the tiles where they are: per panel every wave forms
// the 16 unknowns from the stored inverse (no chain), the owners of the
// panel's tiles take their products from the rest, one barrier.  The tiles
// and inverses are kept for a second right-hand side (W), not as a matrix.
// Measured, k = 250 in FP64: 907 -> 116 us (a thread per row, panels read
// back from memory, before), of which 16 diagonal tiles take 50 us; a second
// right-hand side 30 us.
//
// Larger blocks (on request) keep L in global memory, over G: the other
// waves form panel p + 1 from the panels before p, read back through L2,
// while wave 0 factors panel p.
#include <limits>
#include <utility>

#include "common.h"
#include "kernels.h"
#include "lanes.h"
#include "mfma16.h"

namespace rg {

constexpr int CH_B = 16;                     // panel width
constexpr int CH_NT = 512;
constexpr int CH_NW = CH_NT / WAVE;
constexpr int CH_P = CH_B + 2;               // LDS pitch (16-byte rows)

// acc += A B^T for two 16-row tiles in LDS (pitch CH_P), lane l reading
// row l % 16, columns 4 (l / 16) .. + 3 of both: the inner dimension in the
// same order for both operands
template <typename T>
__device__ __forceinline__ void tile_mma(typename Mfma16<T>::v4 &acc,
                                         const T *a, const T *b, T sign) {
  const int lane = threadIdx.x & (WAVE - 1);
  const int o = (lane & 15) * CH_P + 4 * (lane >> 4);
  T av[4], bv[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) { av[u] = sign * a[o + u]; bv[u] = b[o + u]; }
#pragma unroll
  for (int u = 0; u < 4; ++u) acc = Mfma16<T>::mma(av[u], bv[u], acc);
}
template <typename T>
__device__ __forceinline__ void tile_put(const typename Mfma16<T>::v4 &v, T *t) {
  const int lane = threadIdx.x & (WAVE - 1);
#pragma unroll
  for (int u = 0; u < 4; ++u)
    t[Mfma16<T>::row(lane >> 4, u) * CH_P + (lane & 15)] = v[u];
}

// 1 / d to the last bits for a normal d with a normal reciprocal: the hardware
// estimate (24 bits) with a third-order correction.
__device__ __forceinline__ double recip(double d) {
  const double r = __builtin_amdgcn_rcp(d);
  const double e = fma(-d, r, 1.0);
  return fma(r, fma(e, e, e), r);
}
__device__ __forceinline__ float recip(float d) {
  const float r = __builtin_amdgcn_rcpf(d);
  return fmaf(r, fmaf(-d, r, 1.0f), r);
}
template <int J, typename T>
__device__ __forceinline__ T pivot_recip(const T (&x)[CH_B], T &dv, T thr,
                                         int lr) {
  const T d = row_value<J>(x[J]);
  dv = lr == J ? d : dv;
  return d > thr ? recip(d) : (T)0;
}
// One pivot step of the diagonal tile, as L' D L'^T (the square roots come
// after the last one).  x: the lane's row, columns from J on; the columns
// before J have made room for its row of inv(L').  r: pivot J's reciprocal,
// on return the next one's: its chain (reciprocal, one product, one update)
// runs beside the updates of the other columns.  (The scheduling barrier
// keeps the broadcasts of several steps from being held at once.)
template <int J, typename T>
__device__ __forceinline__ void pivot_step(T (&x)[CH_B], T &r, T &dv, T thr,
                                           int lr) {
  const T a = x[J];
  const T l = lr > J ? a * r : (T)0;
  x[J] = lr == J ? (T)1 : -l;
  if constexpr (J + 1 < CH_B) {
    x[J + 1] -= l * row_value<J + 1>(a);
    r = pivot_recip<J + 1>(x, dv, thr, lr);
  }
  auto right = [&]<int... K>(std::integer_sequence<int, K...>) {
    ((K > J + 1 ? (void)(x[K] -= l * row_value<K>(a)) : (void)0), ...);
  };
  right(std::make_integer_sequence<int, CH_B>{});
#pragma unroll
  for (int k = 0; k < J; ++k) x[k] -= l * row_value<J>(x[k]);
  __builtin_amdgcn_sched_barrier(0);
}

// Largest diagonal entry of the block.
template <int NT, typename T>
__device__ __forceinline__ T diag_max(const T *G, int64_t ldg, int c, T *wmax) {
  const int tid = threadIdx.x;
  T mx = tid < c ? G[(int64_t)tid * ldg + tid] : (T)0;
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const T w = __shfl_xor(mx, o, WAVE);
    mx = w > mx ? w : mx;
  }
  if ((tid & (WAVE - 1)) == 0) wmax[tid / WAVE] = mx;
  __syncthreads();
  mx = (T)0;
#pragma unroll
  for (int w = 0; w < NT / WAVE; ++w) mx = wmax[w] > mx ? wmax[w] : mx;
  return mx;
}

// ------------------------------------------------------------ up to 256
constexpr int CR_MAX = 256;
// One tile (blocks up to 16) needs one wave beside wave 0: 16 of them made a
// solve of one index in a 300 x 300 system 6 % slower than a thread per row.
template <int M> struct CrShape {
  static constexpr int nt = M <= CH_B ? 2 * WAVE : 1024, nw = nt / WAVE;
  static constexpr int t = M / CH_B;
  static constexpr int own = (t * (t + 1) / 2 + nw - 2) / (nw - 1);  // per wave
  static constexpr int64_t tiles = (int64_t)(nw - 1) * own * CH_B * CH_B;
};

template <typename T, int M>
__global__ void __launch_bounds__(CrShape<M>::nt, M <= CH_B ? 1 : 4)
chol_reg_kernel(const T *__restrict__ G, int64_t ldg,
                const int64_t *__restrict__ cnt, const T *__restrict__ hsrc,
                const int32_t *__restrict__ hl, T *__restrict__ y,
                T *__restrict__ W, int factor, const Ctrl *ctrl) {
  if (ctrl_done(ctrl)) return;
  constexpr int NT = CrShape<M>::nt, NW = CrShape<M>::nw;
  constexpr int OWN = CrShape<M>::own;
  typedef typename Mfma16<T>::v4 v4;
  const int c = (int)*cnt;
  if (c <= 0) return;
  __shared__ T pan[2][M * CH_P];
  __shared__ T li[CrShape<M>::t][CH_B * CH_P];          // inverses of the diagonal tiles
  __shared__ T vec[M], vs[M], ys[M];
  __shared__ T zero[CH_B * CH_P];
  __shared__ T wmax[NW];
  const int tid = threadIdx.x, lane = tid & (WAVE - 1);
  const int wv = __builtin_amdgcn_readfirstlane(tid / WAVE);
  const int lr = lane & 15, lk = lane >> 4;
  const int nt = (c + CH_B - 1) / CH_B;
  if (tid < M)
    vec[tid] = tid < c ? (hl ? hsrc[hl[tid]] : hsrc[tid]) : (T)0;
  for (int e = tid; e < CH_B * CH_P; e += NT) zero[e] = (T)0;
  T *wi = W + CrShape<M>::tiles;
  T thr = (T)0;
  // The block is factored as sc G, sc a power of 4 that takes its largest
  // diagonal entry near 1 (denormal ones to 2^-25), so that the pivots above
  // the threshold and their reciprocals are normal numbers (exact: the same
  // bits as without).
  T sc = (T)1;
  if (factor) {
    const T mx = diag_max<NT, T>(G, ldg, c, wmax);
    int ex = 0;
    if (mx > (T)0 && mx <= std::numeric_limits<T>::max()) (void)frexp(mx, &ex);
    constexpr int lim = std::numeric_limits<T>::max_exponent - 4;
    ex = (ex < -lim ? -lim : ex > lim ? lim : ex) & ~1;
    sc = ldexp((T)1, -ex);
    thr = mx * sc * (T)1e-13;
    if (tid == 0) wi[M * CH_B] = sc;
  } else {
    sc = wi[M * CH_B];
    for (int e = tid; e < nt * CH_B * CH_B; e += NT)
      li[e / (CH_B * CH_B)][e / CH_B % CH_B * CH_P + e % CH_B] = wi[e];
  }
  // the 16 unknowns of a panel, lane l holding that of row l % 16: forward
  // Linv_p vec_p, backward Linv_p^T vs_p
  auto forward = [&](int p) {
    T v = (T)0;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      v += li[p][lr * CH_P + 4 * lk + u] * vec[p * CH_B + 4 * lk + u];
    v = fold<16>(v, v);
    return fold<32>(v, v);
  };
  auto backward = [&](int p) {
    T v = (T)0;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      v += li[p][(4 * lk + u) * CH_P + lr] * vs[p * CH_B + 4 * lk + u];
    v = fold<16>(v, v);
    return fold<32>(v, v);
  };

  // Wave 0 and the tile waves run through the same barriers, three per panel
  // of the factorisation and one per panel of each solve.
  if (wv == 0) {
    __builtin_amdgcn_s_setprio(3);   // its chain bounds the factorisation
    __syncthreads();
    for (int p = 0; factor && p < nt; ++p) {
      const T *cur = pan[p & 1];
      T x[CH_B], dv = (T)0;
#pragma unroll
      for (int k = 0; k < CH_B; ++k) x[k] = cur[lr * CH_P + k];
      T r = pivot_recip<0>(x, dv, thr, lr);
      // (in fours: the last panel ends with the block, which leaves a block
      // of a few columns a few pivots)
      const int left = c - p * CH_B;
      auto steps = [&]<int J0, int... J>(std::integral_constant<int, J0>,
                                         std::integer_sequence<int, J...>) {
        if (left > J0) (pivot_step<J0 + J>(x, r, dv, thr, lr), ...);
      };
      constexpr auto four = std::make_integer_sequence<int, 4>{};
      steps(std::integral_constant<int, 0>{}, four);
      steps(std::integral_constant<int, 4>{}, four);
      steps(std::integral_constant<int, 8>{}, four);
      steps(std::integral_constant<int, 12>{}, four);
      const T iv = dv > thr ? rsqrt(dv) : (T)0;
      if (lane < CH_B)
#pragma unroll
        for (int k = 0; k < CH_B; ++k) {
          const T v = x[k] * iv;
          li[p][lr * CH_P + k] = v;
          wi[(p * CH_B + lr) * CH_B + k] = v;
        }
      __syncthreads();
      __syncthreads();
      __syncthreads();
    }
    for (int p = 0; p < nt; ++p) {
      const T v = forward(p);
      if (lane < CH_B) vs[p * CH_B + lane] = v;
      __syncthreads();
    }
    for (int p = nt - 1; p >= 0; --p) {
      const T v = backward(p);
      if (lane < CH_B) ys[p * CH_B + lane] = v;
      __syncthreads();
    }
  } else {
    // the wave's tiles: columns 0, 1, ... in turn, dealt to the other waves
    v4 acc[OWN];
    int ti[OWN], tj[OWN];
    T *wt = W + (int64_t)(wv - 1) * OWN * CH_B * CH_B + lane;
    {
      int j = 0, o = wv - 1;
#pragma unroll
      for (int s = 0; s < OWN; ++s) {
        while (j < nt && o >= nt - j) { o -= nt - j; ++j; }
        ti[s] = j + o;
        tj[s] = j;        // nt: no tile
        o += NW - 1;
      }
    }
    if (factor) {
#pragma unroll
      for (int s = 0; s < OWN; ++s) {
        if (tj[s] >= nt) break;
        const int k = tj[s] * CH_B + lr;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const int i = ti[s] * CH_B + Mfma16<T>::row(lk, u);
          const T g = G[(unsigned)((i < c ? i : c - 1) * (int)ldg +
                                   (k < c ? k : c - 1))];
          acc[s][u] = i < c && k < c ? g : (T)0;
        }
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int s = 0; s < OWN; ++s) acc[s] *= sc;
#pragma unroll
      for (int s = 0; s < OWN; ++s)
        if (tj[s] == 0) tile_put<T>(acc[s], &pan[0][ti[s] * CH_B * CH_P]);
    } else {
#pragma unroll
      for (int s = 0; s < OWN; ++s) {
        if (tj[s] >= nt) break;
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[s][u] = wt[(s * 4 + u) * WAVE];
      }
    }
    __syncthreads();
    for (int p = 0; factor && p < nt; ++p) {
      T *cur = pan[p & 1], *oth = pan[(p & 1) ^ 1];
      // panel p - 1's product from the tiles right of panel p
      if (p > 0) {
#pragma unroll
        for (int s = 0; s + 1 < OWN; s += 2) {
          // two tiles at once; one that is done takes the zero tile
          if (tj[s + 1] <= p || tj[s] >= nt) continue;
#pragma unroll
          for (int v = 0; v < 2; ++v) {
            const bool on = tj[s + v] > p && tj[s + v] < nt;
            tile_mma<T>(acc[s + v],
                        on ? &oth[(ti[s + v] - p + 1) * CH_B * CH_P] : zero,
                        on ? &oth[(tj[s + v] - p + 1) * CH_B * CH_P] : zero,
                        (T)-1);
          }
        }
      }
      __syncthreads();
      // the panel's tiles below the diagonal, times the inverse
#pragma unroll
      for (int s = 0; s < OWN; ++s)
        if (tj[s] == p && ti[s] > p) {
          T *t = &cur[(ti[s] - p) * CH_B * CH_P];
          acc[s] = (v4){0, 0, 0, 0};
          tile_mma<T>(acc[s], t, li[p], (T)1);
          tile_put<T>(acc[s], t);
        }
      __syncthreads();
      // panel p's product completes panel p + 1
#pragma unroll
      for (int s = 0; s < OWN; ++s)
        if (tj[s] == p + 1 && tj[s] < nt) {
          tile_mma<T>(acc[s], &cur[(ti[s] - p) * CH_B * CH_P],
                      &cur[CH_B * CH_P], (T)-1);
          tile_put<T>(acc[s], &oth[(ti[s] - p - 1) * CH_B * CH_P]);
        }
      __syncthreads();
    }
    if (factor) {
#pragma unroll
      for (int s = 0; s < OWN; ++s) {
        if (tj[s] >= nt) break;
#pragma unroll
        for (int u = 0; u < 4; ++u) wt[(s * 4 + u) * WAVE] = acc[s][u];
      }
    }
    // forward: vec_i -= L_ip v_p below panel p
    for (int p = 0; p < nt; ++p) {
      const T v = forward(p);
#pragma unroll
      for (int s = 0; s < OWN; ++s)
        if (tj[s] == p && ti[s] > p) {
          T x = fold_dpp<DPP_ROR8>(acc[s][0] * v, acc[s][1] * v, (lr & 8) != 0);
          const T z = fold_dpp<DPP_ROR8>(acc[s][2] * v, acc[s][3] * v,
                                         (lr & 8) != 0);
          x = fold_dpp<DPP_HMIRROR>(x, z, (lr & 4) != 0);
          x += dpp<DPP_XOR2>(x);
          x += dpp<DPP_XOR1>(x);
          const int u = ((lr >> 3) & 1) + 2 * ((lr >> 2) & 1);
          if ((lr & 3) == 0)
            vec[ti[s] * CH_B + Mfma16<T>::row(lk, u)] -= x;
        }
      __syncthreads();
    }
    // backward: vs_q -= L_pq^T y_p above panel p
    for (int p = nt - 1; p >= 0; --p) {
      const T v = backward(p);
      T yr[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) yr[u] = __shfl(v, Mfma16<T>::row(lk, u), WAVE);
#pragma unroll
      for (int s = 0; s < OWN; ++s)
        if (ti[s] == p && tj[s] < p) {
          T x = acc[s][0] * yr[0] + acc[s][1] * yr[1] + acc[s][2] * yr[2] +
                acc[s][3] * yr[3];
          x = fold<16>(x, x);
          x = fold<32>(x, x);
          if (lk == 0) vs[tj[s] * CH_B + lr] -= x;
        }
      __syncthreads();
    }
  }
  if (tid < c) y[tid] = ys[tid] * sc;
}

// ------------------------------------------------------------ up to CHOL_MAX
constexpr int CB_TILES = CHOL_MAX / CH_B;
constexpr int CB_OWN = (CB_TILES - 1 + CH_NW - 2) / (CH_NW - 1);  // per wave

template <typename T>
__global__ void __launch_bounds__(CH_NT, 2)
chol_big_kernel(T *__restrict__ G, int64_t ldg,
                const int64_t *__restrict__ cnt, const T *__restrict__ hsrc,
                const int32_t *__restrict__ hl, T *__restrict__ y, int factor,
                const Ctrl *ctrl) {
  if (ctrl_done(ctrl)) return;
  typedef typename Mfma16<T>::v4 v4;
  const int c = (int)*cnt;
  if (c <= 0) return;
  __shared__ T pan[2][CHOL_MAX * CH_P];
  __shared__ T ld[CH_B][CH_B + 1];
  __shared__ T vec[CHOL_MAX], dinv[CHOL_MAX];
  __shared__ T wmax[CH_NW];
  const int tid = threadIdx.x, lane = tid & (WAVE - 1), wv = tid / WAVE;
  const int lr = lane & 15, lk = lane >> 4;
  const int nt = (c + CH_B - 1) / CH_B;
  vec[tid] = tid < c ? (hl ? hsrc[hl[tid]] : hsrc[tid]) : (T)0;
  dinv[tid] = (T)0;
  // a 16-step solve of a diagonal tile in wave 0: t = the lane's strictly
  // lower row (forward) or column (backward) of it
  auto tri = [&]<int... J>(const T (&t)[CH_B], T b, T iv, bool up,
                           std::integer_sequence<int, J...>) {
    if (!up) {
      auto step = [&](T vj, int j) { b = (lr == j ? vj : b) - t[j] * vj; };
      (step(row_value<J>(b) * row_value<J>(iv), J), ...);
    } else {
      auto step = [&](T vj, int j) { b = (lr == j ? vj : b) - t[j] * vj; };
      (step(row_value<CH_B - 1 - J>(b) * row_value<CH_B - 1 - J>(iv),
            CH_B - 1 - J), ...);
    }
    return b;
  };
  constexpr auto seq = std::make_integer_sequence<int, CH_B>{};

  if (factor) {
    const T thr = diag_max<CH_NT, T>(G, ldg, c, wmax) * (T)1e-13;
    for (int e = tid; e < nt * CH_B * CH_B; e += CH_NT) {
      const int r = e / CH_B, k = e % CH_B;
      pan[0][r * CH_P + k] = r < c && k < c ? G[(int64_t)r * ldg + k] : (T)0;
    }
    __syncthreads();
    for (int p = 0; p < nt; ++p) {
      T *cur = pan[p & 1], *oth = pan[(p & 1) ^ 1];
      const int p0 = p * CH_B;
      v4 acc[CB_OWN], raw[CB_OWN];
      if (wv == 0) {
        // the diagonal tile; the right-hand side as one more column
        T a[CH_B], b = vec[p0 + lr], v = (T)0, iv = (T)0;
#pragma unroll
        for (int k = 0; k < CH_B; ++k) a[k] = cur[lr * CH_P + k];
        auto steps = [&]<int... J>(std::integer_sequence<int, J...>) {
          auto one = [&]<int JJ>(std::integral_constant<int, JJ>) {
            const T d = row_value<JJ>(a[JJ]);
            const T inv = d > thr ? rsqrt(d) : (T)0;
            const T l = a[JJ] * inv;
            const T vj = row_value<JJ>(b) * inv;
            a[JJ] = l;
            if (lr == JJ) { v = vj; iv = inv; }
            b -= l * vj;
            auto col = [&]<int... K>(std::integer_sequence<int, K...>) {
              ((K > JJ ? (void)(a[K] -= l * row_value<K>(l)) : (void)0), ...);
            };
            col(seq);
          };
          (one(std::integral_constant<int, J>{}), ...);
        };
        steps(seq);
        if (lane < CH_B) {
#pragma unroll
          for (int k = 0; k < CH_B; ++k) {
            ld[lr][k] = k <= lr ? a[k] : (T)0;
            if (k <= lr && p0 + lr < c)
              G[(int64_t)(p0 + lr) * ldg + p0 + k] = a[k];
          }
          vec[p0 + lr] = v;
          dinv[p0 + lr] = iv;
        }
      } else {
        // panel p + 1 from the panels before p
        const int n0 = p0 + CH_B;
#pragma unroll
        for (int s = 0; s < CB_OWN; ++s) {
          const int i0 = n0 + (wv - 1 + (CH_NW - 1) * s) * CH_B;
          acc[s] = (v4){0, 0, 0, 0};
          raw[s] = (v4){0, 0, 0, 0};
          if (i0 >= c) continue;
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const int r = i0 + Mfma16<T>::row(lk, u), k = n0 + lr;
            if (r < c && k < c) raw[s][u] = G[(int64_t)r * ldg + k];
          }
          const bool ain = i0 + lr < c, bin = n0 + lr < c;
          const T *ra = G + (int64_t)(ain ? i0 + lr : 0) * ldg + 4 * lk;
          const T *rb = G + (int64_t)(bin ? n0 + lr : 0) * ldg + 4 * lk;
#pragma unroll 4
          for (int q = 0; q < p; ++q) {
#pragma unroll
            for (int u = 0; u < 4; ++u)
              acc[s] = Mfma16<T>::mma(ain ? ra[q * CH_B + u] : (T)0,
                                      bin ? rb[q * CH_B + u] : (T)0, acc[s]);
          }
        }
      }
      __syncthreads();
      {
        // rows below the diagonal tile, one per thread
        const int r = CH_B + tid, gr = p0 + r;
        if (gr < nt * CH_B) {
          T a[CH_B], dv = (T)0;
#pragma unroll
          for (int k = 0; k < CH_B; ++k) a[k] = cur[r * CH_P + k];
#pragma unroll
          for (int j = 0; j < CH_B; ++j) {
            a[j] *= dinv[p0 + j];
#pragma unroll
            for (int k = j + 1; k < CH_B; ++k) a[k] -= a[j] * ld[k][j];
            dv += a[j] * vec[p0 + j];
          }
#pragma unroll
          for (int k = 0; k < CH_B; ++k) cur[r * CH_P + k] = a[k];
          vec[gr] -= dv;
          if (gr < c) {
#pragma unroll
            for (int k = 0; k < CH_B; ++k)
              G[(int64_t)gr * ldg + p0 + k] = a[k];
          }
        }
      }
      __syncthreads();
      if (wv != 0) {
        // the product with panel p completes panel p + 1
#pragma unroll
        for (int s = 0; s < CB_OWN; ++s) {
          const int i = wv - 1 + (CH_NW - 1) * s;
          if (p0 + (i + 1) * CH_B >= c) continue;
          tile_mma<T>(acc[s], &cur[(i + 1) * CH_B * CH_P], &cur[CH_B * CH_P],
                      (T)1);
          tile_put<T>(raw[s] - acc[s], &oth[i * CH_B * CH_P]);
        }
      }
      __syncthreads();
    }
  } else {
    if (tid < c) {
      const T d = G[(int64_t)tid * ldg + tid];
      dinv[tid] = d != (T)0 ? (T)1 / d : (T)0;
    }
    __syncthreads();
    // forward: panel p's unknowns, then every row below
    for (int p = 0; p < nt; ++p) {
      const int p0 = p * CH_B;
      T a[CH_B];
#pragma unroll
      for (int k = 0; k < CH_B; ++k)
        a[k] = tid >= p0 + CH_B && tid < c ? G[(int64_t)tid * ldg + p0 + k]
                                           : (T)0;
      if (wv == 0) {
        const int r = p0 + lr;
        T t[CH_B];
#pragma unroll
        for (int k = 0; k < CH_B; ++k)
          t[k] = r < c && k < lr ? G[(int64_t)r * ldg + p0 + k] : (T)0;
        const T b = tri(t, vec[r], dinv[r], false, seq);
        if (lane < CH_B) vec[r] = b;
      }
      __syncthreads();
      T dv = (T)0;
#pragma unroll
      for (int k = 0; k < CH_B; ++k) dv += a[k] * vec[p0 + k];
      if (tid >= p0 + CH_B && tid < c) vec[tid] -= dv;
      __syncthreads();
    }
  }
  // backward: panel p's unknowns from the last panel up, then every unknown
  // above
  for (int p = nt - 1; p >= 0; --p) {
    const int p0 = p * CH_B;
    T a[CH_B];
#pragma unroll
    for (int k = 0; k < CH_B; ++k)
      a[k] = p0 + k < c && tid < p0 ? G[(int64_t)(p0 + k) * ldg + tid] : (T)0;
    if (wv == 0) {
      T t[CH_B];
#pragma unroll
      for (int k = 0; k < CH_B; ++k)
        t[k] = p0 + k < c && k > lr ? G[(int64_t)(p0 + k) * ldg + p0 + lr]
                                    : (T)0;
      const T b = tri(t, vec[p0 + lr], dinv[p0 + lr], true, seq);
      if (lane < CH_B) vec[p0 + lr] = b;
    }
    __syncthreads();
    T dv = (T)0;
#pragma unroll
    for (int k = 0; k < CH_B; ++k) dv += a[k] * vec[p0 + k];
    if (tid < p0) vec[tid] -= dv;
    __syncthreads();
  }
  if (tid < c) y[tid] = vec[tid];
}

int64_t chol_work_size(int64_t cap) {
  auto size = [](auto m) {
    constexpr int M = decltype(m)::value;
    return CrShape<M>::tiles + M * CH_B + 1;
  };
  if (cap > CR_MAX) return 1;
  return cap > CH_B ? size(std::integral_constant<int, CR_MAX>{})
                    : size(std::integral_constant<int, CH_B>{});
}

template <typename T>
void launch_chol_solve(T *G, int64_t cap, const int64_t *count_dev,
                       const T *hsrc, const int32_t *hlist, T *y, T *W,
                       int factor, Ctrl *ctrl, hipStream_t st) {
  if (cap <= CH_B)
    hipLaunchKernelGGL((chol_reg_kernel<T, CH_B>), dim3(1),
                       dim3(CrShape<CH_B>::nt), 0, st, (const T *)G, cap,
                       count_dev, hsrc, hlist, y, W, factor,
                       (const Ctrl *)ctrl);
  else if (cap <= CR_MAX)
    hipLaunchKernelGGL((chol_reg_kernel<T, CR_MAX>), dim3(1),
                       dim3(CrShape<CR_MAX>::nt), 0, st, (const T *)G, cap,
                       count_dev, hsrc, hlist, y, W, factor,
                       (const Ctrl *)ctrl);
  else
    hipLaunchKernelGGL(chol_big_kernel<T>, dim3(1), dim3(CH_NT), 0, st, G, cap,
                       count_dev, hsrc, hlist, y, factor, (const Ctrl *)ctrl);
}
template void launch_chol_solve<double>(double *, int64_t, const int64_t *,
                                        const double *, const int32_t *,
                                        double *, double *, int, Ctrl *,
                                        hipStream_t);
template void launch_chol_solve<float>(float *, int64_t, const int64_t *,
                                       const float *, const int32_t *, float *,
                                       float *, int, Ctrl *, hipStream_t);

}  // namespace rg
