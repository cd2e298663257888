// Sparse block projections in one launch (gfx950): the CGLS of a column block
// (min ||A_U y - z||, z its running residual), the CG of a row block on
// A^J A^J^T, and the CGLS of a row block taller than A is wide
// (min ||A^J d - r^J||), each over the block's own entries.
//
// A CG step spread over launches costs three to five of them, 4-5 us each for
// a chain of dependent loads and a launch, and 1.3 us for each one left over
// in a captured graph once the CG has met its tolerance.  Here up to one
// workgroup per compute unit stays for the whole CG; a step is two (CG on
// rows: three) phases between grid-wide sums.  A lane group keeps the first
// entries of its segments and what its thread owns of the vectors in
// registers, so that a phase is one round of gathers, a lane reduction and a
// store.  Vectors that others gather are written and read at agent scope (past
// the caches, so no cache is flushed).  What bounds a phase is latency: a
// gather from beyond the L2 caches, and two hops of the grid-wide sum.
//
// Measured, one launch / launches per CG phase: 30 iterations of 8000 x 500,
// 1 % dense, with tall row blocks 4.3 / 12.8 ms, of 24000 x 3000 7.9 / 25.5
// ms; 10 iterations of 12000 x 6000 11.3 / 24.8 ms; grid systems of 12 and 24
// grids in FP32 117 / 136 ms and 146 / 167 ms.  Of that (FP32, 12 grids): the
// second and third entry kept 14 ms, sums in two levels 9 ms, pairs 3 ms.
#include <algorithm>

#include "common.h"
#include "kernels.h"
#include "lanes.h"
#include "team.h"

namespace rg {

constexpr int GC_NT = 512;
constexpr int GC_NODE = 64;
constexpr int GC_KEEP = 2;     // segments of a lane group kept in registers
constexpr int GC_ENT = 3;      // entries of each kept in registers by a lane
constexpr unsigned long long GC_EMPTY = 0x7FF4A5C35A3C1E87ull;
constexpr int GC_SEGS = 8;     // segments per lane group a block may have

template <typename T>
struct GcSeg {
  int e0, e1;                  // the lane's first entry, the segment's end
  int32_t ix[GC_ENT];          // indices of its first entries (-1: none)
  T v[GC_ENT];
};

// One product over the segments of A (listed, or all): which segments this
// lane group has in its workgroup's share, and (FULL) the entries it keeps.
template <typename T, bool FULL>
struct GcProd {
  const Csr<T> *A;
  const int32_t *list;
  int nseg, lg, grp, ngrp, l;
  GcSeg<T> keep[GC_KEEP];

  __device__ __forceinline__ GcSeg<T> load(int s) const {
    GcSeg<T> k;
    k.e0 = k.e1 = 0;
    if (s < nseg) {
      const int64_t r = list ? (int64_t)list[s] : (int64_t)s;
      k.e0 = (int)A->ptr[r] + l;
      k.e1 = (int)seg_end(*A, r);
    }
#pragma unroll
    for (int j = 0; j < GC_ENT; ++j) {
      const int e = k.e0 + (j << lg);
      k.ix[j] = e < k.e1 ? A->idx[e] : -1;
      k.v[j] = e < k.e1 ? A->val[e] : (T)0;
    }
    return k;
  }
  __device__ __forceinline__ void init(const Csr<T> &M, const int32_t *li,
                                       int n, int lanes_log2) {
    A = &M;
    list = li;
    nseg = n;
    lg = lanes_log2;
    l = threadIdx.x & ((1 << lg) - 1);
    ngrp = ((int)gridDim.x * GC_NT) >> lg;
    share((int)blockIdx.x);
    if constexpr (FULL) {
#pragma unroll
      for (int u = 0; u < GC_KEEP; ++u) keep[u] = load(grp + u * ngrp);
    }
  }
  __device__ __forceinline__ void share(int b) {
    grp = (b * GC_NT + (int)threadIdx.x) >> lg;
  }
  // the kept entries: gathers without branches, all in flight together (a
  // lane without an entry reads the first element and leaves it out)
  template <typename G>
  __device__ __forceinline__ T head(const GcSeg<T> &k, G &&at) const {
    T acc = (T)0;
#pragma unroll
    for (int j = 0; j < GC_ENT; ++j) {
      const T x = at(k.ix[j] < 0 ? 0 : k.ix[j]);
      acc += k.ix[j] < 0 ? (T)0 : k.v[j] * x;
    }
    return acc;
  }
  template <typename G>
  __device__ __forceinline__ T rest(const GcSeg<T> &k, T acc, G &&at) const {
    for (int e = k.e0 + (GC_ENT << lg); e < k.e1; e += 1 << lg)
      acc += A->val[e] * at(A->idx[e]);
    for (int o = 1 << lg >> 1; o > 0; o >>= 1) acc += __shfl_xor(acc, o, WAVE);
    return acc;
  }
  // done(u, s, y) in the first lane of each segment's group, u the slot of a
  // kept segment or -1
  template <typename G, typename D>
  __device__ __forceinline__ void run(G &&at, D &&done) const {
    if constexpr (FULL) {
      T y[GC_KEEP];
#pragma unroll
      for (int u = 0; u < GC_KEEP; ++u) y[u] = (T)0;
      // a second segment only where the first round did not reach all
      if (nseg > ngrp) {
#pragma unroll
        for (int u = 0; u < GC_KEEP; ++u) y[u] = head(keep[u], at);
      } else {
        y[0] = head(keep[0], at);
      }
#pragma unroll
      for (int u = 0; u < GC_KEEP; ++u) {
        if (u > 0 && nseg <= u * ngrp) break;
        const int s = grp + u * ngrp;
        y[u] = rest(keep[u], y[u], at);
        if (s < nseg && l == 0) done(u, s, y[u]);
      }
    }
    for (int s = grp + (FULL ? GC_KEEP : 0) * ngrp; s < nseg; s += ngrp) {
      const GcSeg<T> k = load(s);
      const T t = rest(k, head(k, at), at);
      if (l == 0) done(-1, s, t);
    }
  }
  // the segments of this lane group, in its first lane: f(u, s)
  template <typename F>
  __device__ __forceinline__ void own(F &&f) const {
    if (l != 0) return;
    if constexpr (FULL) {
#pragma unroll
      for (int u = 0; u < GC_KEEP; ++u)
        if (grp + u * ngrp < nseg) f(u, grp + u * ngrp);
    }
    for (int s = grp + (FULL ? GC_KEEP : 0) * ngrp; s < nseg; s += ngrp)
      f(-1, s);
  }
};

// The workgroups that are on the device together (team.h) take the shares of
// those that are not (share b of rank b mod size), with the same sums in the
// same order, so that the results do not depend on it.

// What the workgroups exchange between two phases: two partial sums per
// share, which are also the barrier.  A workgroup publishes its own once all
// its stores have landed (vmcnt in every wave); a slot holds a signalling NaN
// (no sum is one) until then.  The first workgroup of GC_NODE shares adds up
// theirs and publishes that, every workgroup polls these totals (all polling
// all: 65536 polls a phase with 256 workgroups, 9 % slower).  Three sets of
// slots rotate: with phase f read, everybody has read phase f - 1, and the
// slots of that one are emptied, which lands before f + 1 is published,
// without which nobody publishes f + 2.  Waits are bounded (Ctrl::sync_fail).
template <bool FULL>
struct GcEx {
  Ctrl *c;
  unsigned long long *slots;     // 3 sets of 2 values per share and per node
  unsigned *seqp;
  unsigned seq;
  int ph;
  Team tm;

  __device__ __forceinline__ void init(Ctrl *ctrl, int phase, double *part,
                                       unsigned *sq, const Team &team) {
    c = ctrl;
    ph = phase;
    slots = reinterpret_cast<unsigned long long *>(part);
    seqp = sq;
    seq = ld_agent(sq);
    tm = team;
  }
  // f(b) for the shares of this workgroup
  template <typename F>
  __device__ __forceinline__ void each(F &&f) const {
    if constexpr (FULL) {
      f((int)blockIdx.x);
    } else {
      for (int b = tm.rank; b < (int)gridDim.x; b += tm.size) f(b);
    }
  }
  // f(b, a) for the shares of this workgroup, and the total of the a that
  // its threads leave, over all shares; false after a timed-out wait
  template <typename F>
  __device__ __forceinline__ bool phase(double &a, F &&f) {
    double none = 0.0;
    return phase2<1>(a, none, [&](int b, double &x, double &) { f(b, x); });
  }
  template <int N = 2, typename F>
  __device__ __forceinline__ bool phase2(double &a, double &b, F &&f) {
    __shared__ double sh[2][GC_NT / WAVE], tot[2];
    __shared__ int s_fail;
    const int tid = threadIdx.x, lane = tid & (WAVE - 1), wv = tid / WAVE;
    const int P = (int)gridDim.x, Q = (P + GC_NODE - 1) / GC_NODE;
    const int span = 2 * (P + Q);
    unsigned long long *s = slots + (size_t)(seq % 3) * span, *sq = s + 2 * P;
    each([&](int k) {
      a = 0.0;
      b = 0.0;
      f(k, a, b);
      a = wave_total(a);
      if (N > 1) b = wave_total(b);
      if (!FULL) __syncthreads();        // sh of the share before
      if (lane == 0) { sh[0][wv] = a; sh[1][wv] = b; }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if (tid < N) {
        double t = 0.0;
#pragma unroll
        for (int w = 0; w < GC_NT / WAVE; ++w) t += sh[tid][w];
        st_agent(&s[tid * P + k],
                 (unsigned long long)__double_as_longlong(t));
      }
    });
    if (wv == 0) {
      bool ok = true;
      if (Q > 1)
        each([&](int k) {
          if (k % GC_NODE != 0) return;
          ok = poll<N>(s, P, k + lane, k + lane < P, a, b) && ok;
          a = wave_total(a);
          if (N > 1) b = wave_total(b);
          if (lane < N)
            st_agent(&sq[lane * Q + k / GC_NODE],
                     (unsigned long long)__double_as_longlong(lane ? b : a));
        });
      if (Q > 1) ok = poll<N>(sq, Q, lane, lane < Q, a, b) && ok;
      else ok = poll<N>(s, P, lane, lane < P, a, b) && ok;
      a = wave_total(a);
      if (N > 1) b = wave_total(b);
      ok = __all(ok);
      if (lane == 0) { tot[0] = a; tot[1] = b; s_fail = !ok; }
      unsigned long long *o = slots + (size_t)((seq + 2) % 3) * span;
      each([&](int k) {
        if (lane >= 2) return;
        st_agent(&o[lane * P + k], GC_EMPTY);
        if (k % GC_NODE == 0)
          st_agent(&o[2 * P + lane * Q + k / GC_NODE], GC_EMPTY);
      });
    }
    __syncthreads();
    if (s_fail) return false;
    a = tot[0];
    b = tot[1];
    ++seq;
    return true;
  }
  template <int N>
  __device__ __forceinline__ bool poll(const unsigned long long *s, int P,
                                       int i, bool mine, double &a, double &b) {
    a = 0.0;
    b = 0.0;
    bool ok = true;
    if (mine) {
      unsigned long long u, v;
      int64_t spins = 0;
      while (true) {
        u = ld_agent(&s[i]);
        v = N > 1 ? ld_agent(&s[P + i]) : 0;
        if (u != GC_EMPTY && v != GC_EMPTY) break;
        if (++spins > GRID_SPIN_MAX ||
            ((spins & 63) == 0 && ld_agent(&c->sync_fail) != 0)) {
          st_agent(&c->sync_fail, 1);
          ok = false;
          break;
        }
      }
      a = __longlong_as_double((long long)u);
      b = __longlong_as_double((long long)v);
    }
    return ok;
  }
  __device__ __forceinline__ void leave(int steps) {
    if (tm.rank == 0 && threadIdx.x == 0) {
      *seqp = seq;
      c->cg_steps[ph] = steps;
      c->cg_done[ph] = 1;
    }
  }
};

__global__ void __launch_bounds__(256)
gc_clear_kernel(double *part, int64_t n, unsigned *seq,
                unsigned long long *team, int32_t *cmask, int64_t cols,
                int32_t *rmask, int64_t rows) {
  unsigned long long *x = reinterpret_cast<unsigned long long *>(part);
  const int64_t i0 = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t step = (int64_t)gridDim.x * 256;
  for (int64_t i = i0; i < n; i += step) x[i] = GC_EMPTY;
  for (int64_t i = i0; i < cols; i += step) cmask[i] = 0;
  for (int64_t i = i0; i < rows; i += step) rmask[i] = 0;
  if (i0 < 2) seq[i0] = 0;
  if (i0 < 4) team[i0] = 0;
}

// Two numbers that are gathered together: at agent scope in one access.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t gc_rsrc(void *p) {
  return __builtin_amdgcn_make_buffer_rsrc(p, 0, 0xFFFFFFFF, 0x00020000);
}
constexpr int GC_AGENT = 1 << 4;           // sc1
template <typename T>
struct GcPairs {
  T *p;
  __device__ __forceinline__ void get(int i, T &x, T &y) const {
    if constexpr (sizeof(T) == 8) {
      typedef unsigned int u4 __attribute__((ext_vector_type(4)));
      const u4 w = __builtin_amdgcn_raw_buffer_load_b128(
          gc_rsrc(p), (int)((unsigned)i * 16u), 0, GC_AGENT);
      x = __hiloint2double((int)w.y, (int)w.x);
      y = __hiloint2double((int)w.w, (int)w.z);
    } else {
      const unsigned long long w =
          ld_agent(reinterpret_cast<const unsigned long long *>(p) + i);
      x = __uint_as_float((unsigned)w);
      y = __uint_as_float((unsigned)(w >> 32));
    }
  }
  __device__ __forceinline__ void put(int i, T x, T y) const {
    if constexpr (sizeof(T) == 8) {
      typedef unsigned int u4 __attribute__((ext_vector_type(4)));
      const u4 w = {(unsigned)__double2loint(x), (unsigned)__double2hiint(x),
                    (unsigned)__double2loint(y), (unsigned)__double2hiint(y)};
      __builtin_amdgcn_raw_buffer_store_b128(
          w, gc_rsrc(p), (int)((unsigned)i * 16u), 0, GC_AGENT);
    } else {
      st_agent(reinterpret_cast<unsigned long long *>(p) + i,
               (unsigned long long)__float_as_uint(x) |
                   (unsigned long long)__float_as_uint(y) << 32);
    }
  }
};

// In the kernels below the first lane of a lane group owns what belongs to
// its segments: for the kept ones (slot k >= 0) in registers, for others in
// memory.  A direction p = s + beta p_old is never stored as such: where it
// is gathered it is formed from the pair (s, p_old), which its owner replaces
// by (s_new, p) in the phase in which nobody gathers it.
// ------------------------------------------------------------ columns
// W: the block's entries by rows (indices: columns of A); At: all columns;
// mask: the block's marks that W was copied with, cleared here.
//   phase 1: q = A_U p;  phase 2: z -= alpha q, s -= alpha A_U^T q
template <typename T, bool FULL>
__device__ __forceinline__ void
gc_col(const Team &team, const Csr<T> &W, int lgw, const Csr<T> &At, int lgt,
       const int32_t *__restrict__ U, int c, int32_t *__restrict__ mask,
       const T *__restrict__ g, T *__restrict__ z, T *q, T *sp, double *part,
       unsigned *seq, int max_steps, double tol, Ctrl *ctrl) {
  GcEx<FULL> ex;
  ex.init(ctrl, 0, part, seq, team);
  GcProd<T, FULL> pw, pt;
  pw.init(W, nullptr, (int)W.rows, lgw);
  pt.init(At, U, c, lgt);
  const GcPairs<T> SP{sp};
  int32_t uk[GC_KEEP];                    // columns: index, s, p
  T sk[GC_KEEP], pk[GC_KEEP];
  T zk[GC_KEEP], qk[GC_KEEP];             // rows: z, q
  double rr0;
  if (!ex.phase(rr0, [&](int b, double &rr) {
        pt.share(b);
        pt.own([&](int k, int a) {
          const int32_t u = U[a];
          const T h = g[u];
          if (k >= 0) { uk[k] = u; sk[k] = h; pk[k] = (T)0; }
          SP.put(u, h, (T)0);
          mask[u] = 0;
          rr += (double)h * (double)h;
        });
        pw.own([&](int k, int i) { if (k >= 0) zk[k] = z[i]; });
      }))
    return;
  double gam = rr0, beta = 0.0;
  int t = 0;
  const bool run = rr0 != 0.0 && c > 0;
  while (run && t < max_steps) {
    auto dir = [&](int32_t i) {
      T s, po;
      SP.get(i, s, po);
      return s + (T)beta * po;
    };
    double qq;
    if (!ex.phase(qq, [&](int b, double &acc) {
          pw.share(b);
          pw.run(dir, [&](int k, int i, T y) {
            if (k >= 0) qk[k] = y;
            st_agent(&q[i], y);
            acc += (double)y * (double)y;
          });
          pt.own([&](int k, int) {
            if (k >= 0) pk[k] = sk[k] + (T)beta * pk[k];
          });
        }))
      return;
    if (qq == 0.0) break;
    const double alpha = qq > 0.0 ? gam / qq : 0.0;   // (not for a NaN)
    double ss;
    if (!ex.phase(ss, [&](int b, double &acc) {
          pw.share(b);
          pt.share(b);
          pt.run([&](int32_t i) { return ld_agent(&q[i]); },
                 [&](int k, int a, T y) {
                   const int32_t u = k >= 0 ? uk[k] : U[a];
                   T sv, pv;
                   if (k >= 0) { sv = sk[k]; pv = pk[k]; }
                   else { SP.get(u, sv, pv); pv = sv + (T)beta * pv; }
                   sv -= (T)alpha * y;
                   if (k >= 0) sk[k] = sv;
                   SP.put(u, sv, pv);
                   acc += (double)sv * (double)sv;
                 });
          pw.own([&](int k, int i) {
            if (k >= 0) zk[k] -= (T)alpha * qk[k];
            else z[i] -= (T)alpha * ld_agent(&q[i]);
          });
        }))
      return;
    ++t;
    if (ss <= tol * tol * rr0) break;
    beta = gam > 0.0 ? ss / gam : 0.0;
    gam = ss;
  }
  pw.own([&](int k, int i) { if (k >= 0) z[i] = zk[k]; });
  ex.leave(t);
}
template <typename T>
__global__ void __launch_bounds__(GC_NT)
gc_col_kernel(Csr<T> W, int lgw, Csr<T> At, int lgt, const int32_t *U,
              const int64_t *cnt, int32_t *mask, const T *g, T *z, T *q,
              T *sp, double *part, unsigned *seq, unsigned long long *team,
              int max_steps, double tol, Ctrl *ctrl) {
  if (ctrl_done(ctrl)) return;
  Team tm;
  __shared__ unsigned long long s_old;
  tm.enter(team, &s_old);
  if (!tm.settle(team, &s_old, ctrl)) return;
  if (tm.size == (int)gridDim.x)
    gc_col<T, true>(tm, W, lgw, At, lgt, U, (int)*cnt, mask, g, z, q, sp, part,
                    seq, max_steps, tol, ctrl);
  else
    gc_col<T, false>(tm, W, lgw, At, lgt, U, (int)*cnt, mask, g, z, q, sp, part,
                     seq, max_steps, tol, ctrl);
}

// ------------------------------------------------------------ rows
// W: the block's entries by columns (indices: rows of A); A: all rows.
//   phase 1: u = A^J^T p;  phase 2: v = A^J u, <p, v>, <p, rho p>;
//   phase 3: x += alpha u, res -= alpha v, zz = res / rho
template <typename T, bool FULL>
__device__ __forceinline__ void
gc_row(const Team &team, const Csr<T> &W, int lgw, const Csr<T> &A, int lga,
       const int32_t *__restrict__ J, int c, int32_t *__restrict__ mask,
       const T *__restrict__ r, const double *__restrict__ rho,
       T *__restrict__ x, T *u, T *zp, T *__restrict__ res, T *__restrict__ v, double *part, unsigned *seq,
       int max_steps, double tol, Ctrl *ctrl) {
  GcEx<FULL> ex;
  ex.init(ctrl, 1, part, seq, team);
  GcProd<T, FULL> pw, pa;
  pw.init(W, nullptr, (int)W.rows, lgw);
  pa.init(A, J, c, lga);
  const GcPairs<T> ZP{zp};
  int32_t jk[GC_KEEP];                    // rows: index, rho, res, zz, p, v
  double dk[GC_KEEP];
  T rk[GC_KEEP], zk[GC_KEEP], pk[GC_KEEP], vk[GC_KEEP];
  T xk[GC_KEEP], uk[GC_KEEP];             // columns: x, u
  auto scale = [](T h, double dj) {
    return dj > 0.0 ? (T)((double)h / dj) : (T)0;
  };
  double rz, rr0;
  if (!ex.phase2(rz, rr0, [&](int b, double &a0, double &a1) {
        pa.share(b);
        pa.own([&](int k, int a) {
          const int32_t i = J[a];
          const T h = r[i];
          const double dj = rho[i];
          const T zz = scale(h, dj);
          if (k >= 0) {
            jk[k] = i; dk[k] = dj; rk[k] = h; zk[k] = zz; pk[k] = (T)0;
          } else {
            res[a] = h;
          }
          ZP.put(i, zz, (T)0);
          mask[i] = 0;
          a0 += (double)h * (double)zz;
          a1 += (double)h * (double)h;
        });
        pw.own([&](int k, int j) { if (k >= 0) xk[k] = x[j]; });
      }))
    return;
  // A block of dependent rows that contradict each other leaves a residual
  // that A^J^T does not see; the direction turns into it, and <p, A A^T p> into
  // the square of a rounding error.  Below this part of its bound no step is
  // taken and the CG ends.  (A zero there, which ended it before, depends on
  // the order of the sums: with each of 5 rows 4 times, 10 iterations, 4 of 60
  // solves ended in infinity.)
  constexpr double GC_NULL = sizeof(T) == 8 ? 0x1p-98 : 0x1p-44;
  double beta = 0.0;
  int t = 0;
  const bool run = rr0 != 0.0 && c > 0;
  while (run && t < max_steps) {
    auto dir = [&](int32_t i) {
      T s, po;
      ZP.get(i, s, po);
      return s + (T)beta * po;
    };
    double pv;
    if (!ex.phase(pv, [&](int b, double &) {
          pw.share(b);
          pw.run(dir, [&](int k, int j, T y) {
            if (k >= 0) uk[k] = y;
            st_agent(&u[j], y);
          });
          pa.own([&](int k, int) {
            if (k >= 0) pk[k] = zk[k] + (T)beta * pk[k];
          });
        }))
      return;
    double pp;
    if (!ex.phase2(pv, pp, [&](int b, double &a0, double &a1) {
          pa.share(b);
          pa.run([&](int32_t i) { return ld_agent(&u[i]); },
                 [&](int k, int a, T y) {
                   if (k >= 0) vk[k] = y;
                   else v[a] = y;
                   const double pa = (double)(k >= 0 ? pk[k] : dir(J[a]));
                   a0 += (double)y * pa;
                   a1 += (k >= 0 ? dk[k] : rho[J[a]]) * pa * pa;
                 });
        }))
      return;
    // a direction that the rows do not see beyond rounding (the residual of a
    if (pv <= GC_NULL * pp) pv = 0.0;
    const double alpha = pv != 0.0 ? rz / pv : 0.0;
    double rz1, rr;
    if (!ex.phase2(rz1, rr, [&](int b, double &a0, double &a1) {
          pw.share(b);
          pa.share(b);
          pa.own([&](int k, int a) {
            const int32_t i = k >= 0 ? jk[k] : J[a];
            const T rv =
                k >= 0 ? rk[k] - (T)alpha * vk[k] : res[a] - (T)alpha * v[a];
            const T zz = scale(rv, k >= 0 ? dk[k] : rho[i]);
            T p;
            if (k >= 0) { rk[k] = rv; zk[k] = zz; p = pk[k]; }
            else { res[a] = rv; p = dir(i); }
            ZP.put(i, zz, p);
            a0 += (double)rv * (double)zz;
            a1 += (double)rv * (double)rv;
          });
          pw.own([&](int k, int j) {
            if (alpha == 0.0) return;
            if (k >= 0) xk[k] += (T)alpha * uk[k];
            else x[j] += (T)alpha * ld_agent(&u[j]);
          });
        }))
      return;
    ++t;
    if (rr <= tol * tol * rr0 || pv == 0.0) break;
    beta = rz != 0.0 ? rz1 / rz : 0.0;
    rz = rz1;
  }
  pw.own([&](int k, int j) { if (k >= 0) x[j] = xk[k]; });
  ex.leave(t);
}
template <typename T>
__global__ void __launch_bounds__(GC_NT)
gc_row_kernel(Csr<T> W, int lgw, Csr<T> A, int lga, const int32_t *J,
              const int64_t *cnt, int32_t *mask, const T *r,
              const double *rho, T *x, T *u, T *zp, T *res, T *v, double *part, unsigned *seq,
              unsigned long long *team, int max_steps, double tol,
              Ctrl *ctrl) {
  if (ctrl_done(ctrl)) return;
  Team tm;
  __shared__ unsigned long long s_old;
  tm.enter(team, &s_old);
  if (!tm.settle(team, &s_old, ctrl)) return;
  if (tm.size == (int)gridDim.x)
    gc_row<T, true>(tm, W, lgw, A, lga, J, (int)*cnt, mask, r, rho, x, u, zp,
                    res, v, part, seq, max_steps, tol, ctrl);
  else
    gc_row<T, false>(tm, W, lgw, A, lga, J, (int)*cnt, mask, r, rho, x, u, zp,
                     res, v, part, seq, max_steps, tol, ctrl);
}

// ------------------------------------------------------------ tall rows
// A: all rows; At: all columns.  rq: pairs (residual, q) of all m rows, zero
// off the block; the residual r - alpha q is formed where it is gathered.
//   phase 1: q = A^J p;  phase 2: d += alpha p, s = A^T (r - alpha q)
template <typename T, bool FULL>
__device__ __forceinline__ void
gc_tall(const Team &team, const Csr<T> &A, int lga, const Csr<T> &At,
        int lgt, const int32_t *__restrict__ J, int c,
        const T *__restrict__ r, T *__restrict__ x, T *__restrict__ d, T *rq,
        T *sp, double *part, unsigned *seq, int max_steps, double tol,
        Ctrl *ctrl) {
  const int m = (int)A.rows, n = (int)At.rows;
  GcEx<FULL> ex;
  ex.init(ctrl, 1, part, seq, team);
  GcProd<T, FULL> pa, pt;
  pa.init(A, J, c, lga);
  pt.init(At, nullptr, n, lgt);
  const GcPairs<T> SP{sp}, RQ{rq};
  int32_t jk[GC_KEEP];                    // rows: index, residual, q
  T rk[GC_KEEP], qk[GC_KEEP];
  T sk[GC_KEEP], pk[GC_KEEP], dk[GC_KEEP];   // columns: s, p, d
  double g;
  if (!ex.phase(g, [&](int b, double &) {
        for (int i = b * GC_NT + (int)threadIdx.x; i < m;
             i += (int)gridDim.x * GC_NT)
          RQ.put(i, (T)0, (T)0);
      }))
    return;
  if (!ex.phase(g, [&](int b, double &) {
        pa.share(b);
        pa.own([&](int k, int a) {
          const int32_t i = J[a];
          const T h = r[i];
          if (k >= 0) { jk[k] = i; rk[k] = h; }
          RQ.put(i, h, (T)0);
        });
      }))
    return;
  T alpha = (T)0, beta = (T)0;
  auto resid = [&](int32_t i) {
    T rv, qv;
    RQ.get(i, rv, qv);
    return rv - alpha * qv;
  };
  auto dir = [&](int32_t i) {
    T s, po;
    SP.get(i, s, po);
    return s + beta * po;
  };
  if (!ex.phase(g, [&](int b, double &acc) {
        pt.share(b);
        pt.run(resid, [&](int k, int j, T y) {
          if (k >= 0) { sk[k] = y; pk[k] = (T)0; dk[k] = (T)0; }
          else d[j] = (T)0;
          SP.put(j, y, (T)0);
          acc += (double)y * (double)y;
        });
      }))
    return;
  const double gam0 = g;
  double gam = gam0;
  int t = 0;
  const bool run = gam0 > 0.0;
  while (run && t < max_steps) {
    double qq;
    if (!ex.phase(qq, [&](int b, double &acc) {
          pa.share(b);
          pa.run(dir, [&](int k, int a, T y) {
            const int32_t i = k >= 0 ? jk[k] : J[a];
            RQ.put(i, k >= 0 ? rk[k] : resid(i), y);
            if (k >= 0) qk[k] = y;
            acc += (double)y * (double)y;
          });
          pt.own([&](int k, int) {
            if (k >= 0) pk[k] = sk[k] + beta * pk[k];
          });
        }))
      return;
    if (!(qq > 0.0)) break;
    alpha = (T)(gam / qq);
    if (!ex.phase(g, [&](int b, double &acc) {
          pt.share(b);
          pa.own([&](int k, int) { if (k >= 0) rk[k] -= alpha * qk[k]; });
          pt.run(resid, [&](int k, int j, T y) {
            const T p = k >= 0 ? pk[k] : dir(j);
            if (k >= 0) { sk[k] = y; dk[k] += alpha * p; }
            else d[j] += alpha * p;
            SP.put(j, y, p);
            acc += (double)y * (double)y;
          });
        }))
      return;
    ++t;
    if (g <= tol * tol * gam0 || !(gam > 0.0)) break;
    beta = (T)(g / gam);
    gam = g;
  }
  ex.each([&](int b) {
    pt.share(b);
    pt.own([&](int k, int j) { x[j] += k >= 0 ? dk[k] : d[j]; });
  });
  ex.leave(t);
}
template <typename T>
__global__ void __launch_bounds__(GC_NT)
gc_tall_kernel(Csr<T> A, int lga, Csr<T> At, int lgt, const int32_t *J,
               const int64_t *cnt, const T *r, T *x, T *d, T *rq, T *sp,
               double *part, unsigned *seq, unsigned long long *team,
               int max_steps, double tol, Ctrl *ctrl) {
  if (ctrl_done(ctrl)) return;
  Team tm;
  __shared__ unsigned long long s_old;
  tm.enter(team, &s_old);
  if (!tm.settle(team, &s_old, ctrl)) return;
  if (tm.size == (int)gridDim.x)
    gc_tall<T, true>(tm, A, lga, At, lgt, J, (int)*cnt, r, x, d, rq, sp, part,
                     seq, max_steps, tol, ctrl);
  else
    gc_tall<T, false>(tm, A, lga, At, lgt, J, (int)*cnt, r, x, d, rq, sp, part,
                      seq, max_steps, tol, ctrl);
}

// ------------------------------------------------------------ launchers
static int gc_log2(int g) {
  int l = 0;
  while ((1 << l) < g) ++l;
  return l;
}
// Workgroups for two products of so many lanes: a segment per lane group
// where the compute units allow it.
static int gc_grid(int64_t lanes1, int64_t lanes2, int ncu) {
  const int64_t b = (std::max(lanes1, lanes2) + GC_NT - 1) / GC_NT;
  return (int)std::max<int64_t>(1, std::min<int64_t>(b, ncu));
}
// Up to GC_SEGS segments per lane group if every compute unit has a
// workgroup: there the one launch is 14 % faster on grid systems (24 grids,
// FP64, 122 / 142 ms), at twice that 6 % (48 grids, 172 / 184; in FP32 216 /
// 217), at four times 3 % slower (96 grids, 278 / 270).  Long segments have
// launches of their own; several right-hand sides fill the device as it is.
template <typename T>
bool grid_cg_takes(const Csr<T> &A, const Csr<T> &At, int ncu) {
  const int64_t most = (int64_t)GC_SEGS * GC_NT * ncu;
  return A.rep == 1 && A.nlong == 0 && At.nlong == 0 && ncu <= GC_NT &&
         A.rows * A.group <= most && At.rows * At.group <= most;
}
template <typename T>
void launch_grid_clear(GridCg<T> &w, int ncu, int32_t *cmask, int64_t cols,
                       int32_t *rmask, int64_t rows, hipStream_t st) {
  const int64_t n = 24 * (int64_t)ncu;
  const int64_t b = (std::max({n, cols, rows}) + 255) / 256;
  hipLaunchKernelGGL(gc_clear_kernel, dim3((unsigned)std::min<int64_t>(b, 1024)),
                     dim3(256), 0, st, w.part, n, w.seq, w.team, cmask, cols,
                     rmask, rows);
}
template <typename T>
void launch_grid_colproj(const Csr<T> &W, const Csr<T> &At, const int32_t *U,
                         const int64_t *cnt, int64_t cap, int32_t *mask,
                         const T *g, T *z,
                         GridCg<T> &w, int ncu, int max_steps, double tol,
                         Ctrl *ctrl, hipStream_t st) {
  const int grid = gc_grid(W.rows * W.group, cap * At.group, ncu);
  hipLaunchKernelGGL(gc_col_kernel<T>, dim3(grid), dim3(GC_NT), 0, st, W,
                     gc_log2(W.group), At, gc_log2(At.group), U, cnt, mask, g, z,
                     w.q, w.sp, w.part, w.seq, w.team, max_steps, tol, ctrl);
}
template <typename T>
void launch_grid_rowproj(const Csr<T> &W, const Csr<T> &A, const int32_t *J,
                         const int64_t *cnt, int64_t cap, int32_t *mask,
                         const T *r,
                         const double *rho, T *x, GridCg<T> &w, T *res, T *v,
                         int ncu, int max_steps, double tol, Ctrl *ctrl,
                         hipStream_t st) {
  const int grid = gc_grid(W.rows * W.group, cap * A.group, ncu);
  hipLaunchKernelGGL(gc_row_kernel<T>, dim3(grid), dim3(GC_NT), 0, st, W,
                     gc_log2(W.group), A, gc_log2(A.group), J, cnt, mask, r, rho, x,
                     w.q, w.sp, res, v, w.part + 12 * ncu,
                     w.seq + 1, w.team + 2, max_steps, tol, ctrl);
}
template <typename T>
void launch_grid_tall(const Csr<T> &A, const Csr<T> &At, const int32_t *J,
                      const int64_t *cnt, int64_t cap, const T *r, T *x,
                      GridCg<T> &w, TallWork<T> &tw, int ncu, int max_steps,
                      double tol, Ctrl *ctrl, hipStream_t st) {
  const int grid = gc_grid(cap * A.group, At.rows * At.group, ncu);
  hipLaunchKernelGGL(gc_tall_kernel<T>, dim3(grid), dim3(GC_NT), 0, st, A,
                     gc_log2(A.group), At, gc_log2(At.group), J, cnt, r, x,
                     tw.d, w.rq, w.sp,
                     w.part + 12 * ncu, w.seq + 1, w.team + 2, max_steps, tol, ctrl);
}

#define INST_GC(T)                                                            \
  template void launch_grid_clear<T>(GridCg<T> &, int, int32_t *, int64_t,     \
                                     int32_t *, int64_t, hipStream_t);        \
  template bool grid_cg_takes<T>(const Csr<T> &, const Csr<T> &, int);        \
  template void launch_grid_colproj<T>(                                       \
      const Csr<T> &, const Csr<T> &, const int32_t *, const int64_t *,       \
      int64_t, int32_t *, const T *, T *, GridCg<T> &, int, int, double,      \
      Ctrl *, hipStream_t);                                                   \
  template void launch_grid_rowproj<T>(                                       \
      const Csr<T> &, const Csr<T> &, const int32_t *, const int64_t *,       \
      int64_t, int32_t *, const T *, const double *, T *, GridCg<T> &, T *,   \
      T *, int, int, double, Ctrl *, hipStream_t);                                      \
  template void launch_grid_tall<T>(                                          \
      const Csr<T> &, const Csr<T> &, const int32_t *, const int64_t *,       \
      int64_t, const T *, T *, GridCg<T> &, TallWork<T> &, int, int, double,  \
      Ctrl *, hipStream_t);
INST_GC(double)
INST_GC(float)

}  // namespace rg
