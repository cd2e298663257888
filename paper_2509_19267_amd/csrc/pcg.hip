// Persistent Jacobi-preconditioned CG on a gathered Gram block (gfx950): the
// whole CG of one block projection (Section 2's pseudoinverse updates) in
// one launch of at most one workgroup per compute unit.
//
// The workgroups need not all be on the device: those that are (team.h) deal
// the block's rows among themselves, with the same bits whatever their number
// (fewer hold more rows, streamed from G where registers and LDS are full).
// Counting them costs 2-3 us a launch: 2003 x 501 layer 43.5 -> 45.1 ms.
// Workgroup w owns rows [w rpw, (w+1) rpw) of the block G; thread t of every
// workgroup owns columns t, t + 512, ... of it.  What bounds a CG step is
// not the product but the exchange between the workgroups, and reading the
// block again: so
//  - the block stays on the chip.  Each thread keeps its columns of the
//    workgroup's first RR rows in registers and of the next RL in LDS (512
//    KB of registers and 160 KB of LDS per compute unit: a 4000 x 4000 FP64
//    block is 128 MB, the chip's registers and LDS 168 MB).  Only rows past
//    RR + RL are stored packed to global memory and read again every step
//    (from the same compute unit, through L2).  With a precomputed Gram F of
//    all columns (rows) the block's entries come straight from it, once;
//  - direction, residual and inverse diagonal live in registers at the
//    thread's own columns (every workgroup updates the whole vectors, with
//    identical bits), so the product needs no broadcast of the direction;
//  - the row sums are reduced across lanes by halving: v_permlane32_swap and
//    v_permlane16_swap fold two rows per add, then DPP inside 16 lanes;
//  - the workgroups exchange only v = G p, and the data is its own flag:
//    every entry is one agent-scope store into a buffer that holds a
//    signalling NaN until then (no arithmetic result is one), and a reader
//    polls the entries themselves.  No atomics, fences, barrier counter or
//    separate <p, v> partials: one store and one load latency per step.
// Three exchange buffers rotate: a workgroup that has read all of step s
// knows that everybody has finished reading step s - 1, and clears its share
// of that buffer then; the clear has landed (vmcnt wait) before the same
// wave publishes step s + 1, without which nobody reads step s + 2.  That
// holds because every workgroup that reads also publishes: those without a
// row leave at once (pcgshare.h).  The rotation goes on across launches (seq,
// read before the first publish and written after the last).  Polls are
// bounded: a timed-out wait raises Ctrl::sync_fail, which ends the other
// waits, so the launch always drains.
// Measured per launch, against the same CG with the block re-read from
// memory each step and a counter barrier between the workgroups: FP64 4000
// (mean of column and row blocks, 5 and 8 steps) 328 -> 150 us, most of it
// now the gather of the block from the full Gram; FP64 301 (about 40 steps)
// 319 -> 106 us, 2.5 us per step; FP64 750 (exact) 111 us.
#include "common.h"
#include "kernels.h"
#include "lanes.h"
#include "pcgshare.h"
#include "team.h"

namespace rg {

constexpr int PQ_NT = 512;
constexpr int PQ_NW = PQ_NT / WAVE;
constexpr int PQ_RMAX = 256;   // rows of one workgroup
// Rows per workgroup while the grid allows: fewer rows shorten the lane
// reductions, more workgroups lengthen the exchange (2003 x 501 layer: 54.6
// ms at 4 rows, 51.1 at 8, 53.5 at 16).
constexpr int PQ_RPW = 8;

template <typename T> struct PqBits;
template <> struct PqBits<double> {
  using type = unsigned long long;
  static constexpr type empty = 0x7FF4A5C35A3C1E87ull;   // signalling NaNs
};
template <> struct PqBits<float> {
  using type = unsigned;
  static constexpr type empty = 0x7FA5C3E7u;
};

template <typename T>
struct PqArgs {
  T *G;                 // packed block (cap x cap), or its unread storage
  const T *F;           // full Gram to gather from (nullable)
  int64_t ldg, ldf;
  const int64_t *cnt;
  const T *hsrc;
  const int32_t *hl;
  const double *nrm;    // diagonal of the full Gram
  T *y;
  T *xch;               // 3 x cap exchange buffers
  unsigned *seq;        // steps exchanged since the buffers were cleared
  unsigned long long *team;   // workgroups counted in, team size
  int cap, max_steps;
  double tol;
  Ctrl *ctrl;
  int ph;
};

// One group of N row sums: rows k0 .. k0+N-1 of the workgroup into
// part[wave][row].
template <int N, typename T>
__device__ __forceinline__ void put_rows(T (&acc)[N], int k0, T *part, int lane,
                                         int wv) {
  const T s = wave_totals<N>(acc, lane);
  if ((lane & (WAVE / N - 1)) == 0)
    part[wv * PQ_RMAX + k0 + lane / (WAVE / N)] = s;
}

template <typename T, int NC, int RR, int RL>
__global__ void __launch_bounds__(PQ_NT, 2)
pcg_persist_kernel(const PqArgs<T> a) {
  Ctrl *ctrl = a.ctrl;
  if (ctrl_done(ctrl)) return;
  using B = typename PqBits<T>::type;
  constexpr B EMPTY = PqBits<T>::empty;
  constexpr int R8 = RR / 8 * 8, RX = RR - R8;   // rows by eight, the rest
  static_assert(RX == 0 || RX == 2 || RX == 4, "");
  static_assert(RL % 2 == 0, "");
  __shared__ T gl[RL > 0 ? RL * NC * PQ_NT : 1];
  __shared__ T part[PQ_NW * PQ_RMAX];
  __shared__ T ys[PQ_RMAX];
  __shared__ double sh[3][PQ_NW];
  __shared__ int s_fail;
  const int tid = threadIdx.x, lane = tid & (WAVE - 1), wv = tid / WAVE;
  const int c = (int)*a.cnt;
  Team team;
  __shared__ unsigned long long s_old;
  int me, per, r0, nr;
  const int ph = a.ph;
  if (tid == 0) s_fail = 0;
  for (int k = tid; k < PQ_RMAX; k += PQ_NT) ys[k] = (T)0;

  // the thread's columns: block index, and where their entries are in a row
  // of the source
  T p[NC], r[NC], di[NC];
  T g[RR][NC];
  double rz = 0.0, rr = 0.0;
  {
    int32_t off[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const int col = tid + j * PQ_NT;
      off[j] = col < c ? a.hl[col] : 0;
    }
    team.enter(a.team, &s_old);
    T d[NC];
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const bool in = tid + j * PQ_NT < c;
      r[j] = in ? a.hsrc[off[j]] : (T)0;
      d[j] = in ? (T)a.nrm[off[j]] : (T)0;
    }
    if (!a.F) {
#pragma unroll
      for (int j = 0; j < NC; ++j) off[j] = tid + j * PQ_NT;
    }
    auto row = [&](int k) -> const T * {
      return a.F ? a.F + (int64_t)a.hl[r0 + k] * a.ldf
                 : a.G + (int64_t)(r0 + k) * a.ldg;
    };
    // who is there, and this workgroup's share
    if (!team.settle(a.team, &s_old, ctrl, (a.cap + PQ_RMAX - 1) / PQ_RMAX))
      return;
    const PqShare share = pq_share(c, a.cap, team.size);
    me = team.size == (int)gridDim.x ? (int)blockIdx.x : team.rank;
    per = share.per;
    if (me >= share.active) return;
    r0 = me * share.rpw;
    nr = c - r0 < share.rpw ? (c - r0 > 0 ? c - r0 : 0) : share.rpw;
#pragma unroll
    for (int k = 0; k < RR; ++k) {
      if (k < nr) {
        const T *gr = row(k);
#pragma unroll
        for (int j = 0; j < NC; ++j)
          g[k][j] = tid + j * PQ_NT < c ? gr[off[j]] : (T)0;
      } else {
#pragma unroll
        for (int j = 0; j < NC; ++j) g[k][j] = (T)0;
      }
    }
    if constexpr (RL > 0) {
#pragma unroll
      for (int k = 0; k < RL; ++k) {
        if (RR + k < nr) {
          const T *gr = row(RR + k);
#pragma unroll
          for (int j = 0; j < NC; ++j)
            gl[(k * NC + j) * PQ_NT + tid] =
                tid + j * PQ_NT < c ? gr[off[j]] : (T)0;
        }
      }
    }
    if (a.F) {
      for (int k = RR + RL; k < nr; ++k) {
        const T *gr = row(k);
        T *gw = a.G + (int64_t)(r0 + k) * a.ldg;
        T v[NC];
#pragma unroll
        for (int j = 0; j < NC; ++j)
          v[j] = tid + j * PQ_NT < c ? gr[off[j]] : (T)0;
#pragma unroll
        for (int j = 0; j < NC; ++j)
          if (tid + j * PQ_NT < c) gw[tid + j * PQ_NT] = v[j];
      }
    }
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      di[j] = d[j] > (T)0 ? (T)1 / d[j] : (T)0;
      p[j] = r[j] * di[j];
      rz += (double)r[j] * (double)p[j];
      rr += (double)r[j] * (double)r[j];
    }
  }
  rz = wave_total(rz);
  rr = wave_total(rr);
  if (lane == 0) { sh[1][wv] = rz; sh[2][wv] = rr; }
  __syncthreads();
  rz = 0.0;
  rr = 0.0;
#pragma unroll
  for (int w = 0; w < PQ_NW; ++w) { rz += sh[1][w]; rr += sh[2][w]; }
  const double rr0 = rr;
  const unsigned seq = ld_agent(a.seq);
  __syncthreads();   // sh[1], sh[2] are written again in the first step

  int t = 0;
  const bool run = !(rr0 == 0.0 || c == 0);
  while (run && t < a.max_steps) {
    const unsigned s = seq + (unsigned)t;
    B *xb = reinterpret_cast<B *>(a.xch) + (int64_t)(s % 3) * a.cap;
    // v = G p on the workgroup's rows
    for (int k = RR + RL; k < nr; k += 2) {
      T acc[2] = {(T)0, (T)0};
      const T *g0 = a.G + (int64_t)(r0 + k) * a.ldg;
      const bool two = k + 1 < nr;
      const T *g1 = two ? g0 + a.ldg : g0;
#pragma unroll
      for (int j = 0; j < NC; ++j) {
        const int col = tid + j * PQ_NT;
        if (col < c) {
          acc[0] += g0[col] * p[j];
          acc[1] += g1[col] * p[j];
        }
      }
      put_rows<2>(acc, k, part, lane, wv);
    }
#pragma unroll
    for (int k0 = 0; k0 < R8; k0 += 8) {
      if (k0 < nr) {
        T acc[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          acc[k] = (T)0;
#pragma unroll
          for (int j = 0; j < NC; ++j) acc[k] += g[k0 + k][j] * p[j];
        }
        put_rows<8>(acc, k0, part, lane, wv);
      }
    }
    if constexpr (RX > 0) {
      if (R8 < nr) {
        T acc[RX];
#pragma unroll
        for (int k = 0; k < RX; ++k) {
          acc[k] = (T)0;
#pragma unroll
          for (int j = 0; j < NC; ++j) acc[k] += g[R8 + k][j] * p[j];
        }
        put_rows<RX>(acc, R8, part, lane, wv);
      }
    }
    if constexpr (RL > 0) {
#pragma unroll
      for (int k0 = 0; k0 < RL; k0 += 2) {
        if (RR + k0 < nr) {
          T acc[2];
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            acc[k] = (T)0;
#pragma unroll
            for (int j = 0; j < NC; ++j)
              acc[k] += gl[((k0 + k) * NC + j) * PQ_NT + tid] * p[j];
          }
          put_rows<2>(acc, RR + k0, part, lane, wv);
        }
      }
    }
    __syncthreads();
    // publish; the clears of the previous step by this wave have landed
    if (wv == 0) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      for (int k = lane; k < nr; k += WAVE) {
        T v = (T)0;
#pragma unroll
        for (int w = 0; w < PQ_NW; ++w) v += part[w * PQ_RMAX + k];
        B bits;
        __builtin_memcpy(&bits, &v, sizeof(T));
        st_agent(&xb[r0 + k], bits);
      }
    }
    // collect v at the thread's columns
    T v[NC];
    {
      int64_t spins = 0;
      while (true) {
        bool ok = true;
        B bits[NC];
#pragma unroll
        for (int j = 0; j < NC; ++j)
          bits[j] = tid + j * PQ_NT < c ? ld_agent(&xb[tid + j * PQ_NT]) : (B)0;
#pragma unroll
        for (int j = 0; j < NC; ++j) {
          ok = ok && bits[j] != EMPTY;
          __builtin_memcpy(&v[j], &bits[j], sizeof(T));
        }
        if (ok) break;
        __builtin_amdgcn_s_sleep(1);
        if (++spins > GRID_SPIN_MAX ||
            ((spins & 63) == 0 && ld_agent(&ctrl->sync_fail) != 0)) {
          st_agent(&ctrl->sync_fail, 1);
          s_fail = 1;
          break;
        }
      }
    }
    double pv = 0.0;
#pragma unroll
    for (int j = 0; j < NC; ++j) pv += (double)p[j] * (double)v[j];
    pv = wave_total(pv);
    if (lane == 0) sh[0][wv] = pv;
    __syncthreads();
    if (s_fail) return;
    // everybody has read the previous step: clear this workgroup's share
    if (wv == 0) {
      B *xp = reinterpret_cast<B *>(a.xch) + (int64_t)((s + 2) % 3) * a.cap;
      const int i0 = me * per;
      const int i1 = i0 + per < a.cap ? i0 + per : a.cap;
      for (int i = i0 + lane; i < i1; i += WAVE)
        st_agent(&xp[i], EMPTY);
    }
    pv = 0.0;
#pragma unroll
    for (int w = 0; w < PQ_NW; ++w) pv += sh[0][w];
    const double alpha = pv != 0.0 ? rz / pv : 0.0;
    double rz1 = 0.0;
    rr = 0.0;
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const int k = tid + j * PQ_NT - r0;
      if (k >= 0 && k < nr) ys[k] += (T)alpha * p[j];
      r[j] -= (T)alpha * v[j];
      rz1 += (double)r[j] * (double)(r[j] * di[j]);
      rr += (double)r[j] * (double)r[j];
    }
    rz1 = wave_total(rz1);
    rr = wave_total(rr);
    if (lane == 0) { sh[1][wv] = rz1; sh[2][wv] = rr; }
    __syncthreads();
    rz1 = 0.0;
    rr = 0.0;
#pragma unroll
    for (int w = 0; w < PQ_NW; ++w) { rz1 += sh[1][w]; rr += sh[2][w]; }
    ++t;
    if (rr <= a.tol * a.tol * rr0 || rz == 0.0 || pv == 0.0) break;
    const double beta = rz1 / rz;
    rz = rz1;
#pragma unroll
    for (int j = 0; j < NC; ++j) p[j] = r[j] * di[j] + (T)beta * p[j];
  }
  __syncthreads();
  for (int k = tid; k < nr; k += PQ_NT) a.y[r0 + k] = ys[k];
  if (me == 0 && tid == 0) {
    *a.seq = seq + (unsigned)t;
    ctrl->cg_steps[ph] = t;
    ctrl->cg_done[ph] = 1;
  }
}

template <typename T>
__global__ void __launch_bounds__(256)
pcg_clear_kernel(T *xch, int64_t n, unsigned *seq, unsigned long long *team) {
  using B = typename PqBits<T>::type;
  B *x = reinterpret_cast<B *>(xch);
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) x[i] = PqBits<T>::empty;
  if (i == 0) *seq = 0;
  if (i < 2) team[i] = 0;
}

static int64_t pcg_persist_cap(bool f64) { return f64 ? 4096 : 8192; }

// Eight rows per workgroup while that leaves compute units over, else all
// compute units.
int pcg_persist_grid(int64_t cap, int ncu) {
  int64_t p = (cap + PQ_RPW - 1) / PQ_RPW;
  if (p > ncu) p = ncu;
  return (int)(p < 1 ? 1 : p);
}
bool pcg_persist_fits(int64_t cap, int ncu, bool f64) {
  const int p = pcg_persist_grid(cap, ncu);
  return cap <= pcg_persist_cap(f64) && (cap + p - 1) / p <= PQ_RMAX;
}

template <typename T>
void launch_pcg_clear(CgWork<T> &w, hipStream_t st) {
  const int64_t n = 3 * w.cap;
  hipLaunchKernelGGL(pcg_clear_kernel<T>, dim3((unsigned)((n + 255) / 256)),
                     dim3(256), 0, st, w.xch, n, w.seq, w.team);
}

template <typename T>
void launch_pcg_persist(T *G, int64_t cap, const int64_t *count_dev,
                        const T *hsrc, const int32_t *hlist, const double *nrm,
                        T *y, CgWork<T> &w, int grid, int max_steps,
                        double tol, Ctrl *ctrl, int ph, hipStream_t st,
                        const T *F, int64_t ldf) {
  // columns per thread and rows kept in registers and LDS, by block size:
  // what 256 registers per thread hold beside the vectors
#define RG_PQ(NC, RR, RL)                                                    \
  hipLaunchKernelGGL((pcg_persist_kernel<T, NC, RR, RL>), dim3(grid),        \
                     dim3(PQ_NT), 0, st,                                     \
                     (PqArgs<T>{G, F, cap, ldf, count_dev, hsrc, hlist,  \
                                    nrm, y, w.xch, w.seq, w.team, (int)cap,  \
                                    max_steps, tol, ctrl, ph}))
  if (cap <= 1 * PQ_NT) RG_PQ(1, 16, 0);
  else if (cap <= 2 * PQ_NT) RG_PQ(2, 16, 0);
  else if (cap <= 4 * PQ_NT) RG_PQ(4, 16, 0);
  else if constexpr (sizeof(T) == 8) {
    if (cap <= 6 * PQ_NT) RG_PQ(6, 12, 4);
    else RG_PQ(8, 8, 4);
  } else {
    if (cap <= 8 * PQ_NT) RG_PQ(8, 16, 4);
    else if (cap <= 10 * PQ_NT) RG_PQ(10, 12, 6);
    else RG_PQ(16, 4, 4);
  }
#undef RG_PQ
}

#define INST_PQ(T)                                                           \
  template void launch_pcg_clear<T>(CgWork<T> &, hipStream_t);               \
  template void launch_pcg_persist<T>(T *, int64_t, const int64_t *,         \
                                      const T *, const int32_t *,            \
                                      const double *, T *, CgWork<T> &, int, \
                                      int, double, Ctrl *, int, hipStream_t, \
                                      const T *, int64_t);
INST_PQ(double)
INST_PQ(float)

}  // namespace rg
