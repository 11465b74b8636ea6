// Several Newton-Leja terms per launch as a pipeline of waves.
//
// A block owns one run of rows of one strip (kPipeCols own columns of a wave
// strip, two columns per lane).  Wave 0 loads: one input row per tick, a few
// ticks ahead in registers, the face averages of kxx and kyy formed once, into
// LDS.  Wave t = 1 .. nst computes stage t: one row per tick, two rows behind
// stage t - 1, its vertical windows in registers.  A tick is one block barrier:
// in it every stage takes one row of y_{t-1} and p_{t-1} from its predecessor
// and of the coefficients from the loader, and hands on one row of y_t and
// p_t.  The last stage stores y and p.  One pass over memory (56 B per point in
// FP64) then covers nst terms; a row of 128 points costs a wave 44 FP64 and 8
// shift instructions.
//
// What bounds it: at 4096^2 a launch of seven terms takes 206 - 225 us by HIP
// events (939.5 MB needed, 1010 MB moved by the counters: 193 us at the rate of
// a copy) where the three-term staged kernel took 183 us for three; the rest is
// LDS traffic, 7 KB a row and stage (coefficients, y, p), and issue, two blocks of
// eight waves a CU.  Up to 1024^2 the latency of rows + 21
// ticks of 0.35 - 0.45 us bounds it (512^2: 16 us a launch of seven terms, where
// four terms in LDS took 15.4).  Two rows a tick or two stages a wave gain 7 % at
// 4096^2 but lose 20 - 80 % up to 1024^2 (longer ticks); 3 rows in flight a wave
// suffice (4 take the same time).
//
// The stencil in flux form:
//   Fx(i+1/2) = kf (u_{i+1} - u_i),  Fy(j+1/2) = kf (u_{j+1} - u_j)
//   H_j = kxy_j (u_{i+1} - u_{i-1}), G_i = kxy_i (u_{j+1} - u_{j-1})
//   A u = dFx + dFy + (G_{i+1} - G_{i-1}) + (H_{j+1} - H_{j-1}) + advection
// so a row's differences serve the rows below it too, and the x-neighbours'
// Fx and G come by DPP shifts.
//
// Ticks.  With a0 = J0 - nst, wave 0 puts at tick m the coefficients of index m
// (kxy of row a0 + m, the kxx faces of row a0 + m - 1 and the kyy faces above
// it), y_0 of row a0 + m - 1 and p_0 of row a0 + m - 2.  At tick n stage t takes
// y_{t-1} of row e = a0 + n - 2t and works on row e - 1 with the coefficients of
// index e - a0, which it read during tick n - 1 (so that a tick starts with two
// LDS reads to wait for, not five).  Its first complete row is that of tick
// 3t + 1; it takes y from tick 3t - 1 on and ends with tick R + 2 nst + t.  The
// hand-overs alternate between two LDS rows by the tick's parity (p is held
// back one tick in registers); the coefficients of an index are read last
// 2 nst - 1 ticks after they were put, so 2 nst slots are kept.
//
// Every wave executes the same number of barriers.
#pragma once

#include <climits>

#include "decide.h"
#include "pipe.h"
#include "tile.h"

namespace adl {

constexpr int kPipeRow = kWave * 2;  // doubles of an LDS row


__device__ __forceinline__ void pipe_put(double* row, const double (&c)[2]) {
  typedef double d2 __attribute__((ext_vector_type(2)));
  d2 v;
  v.x = c[0];
  v.y = c[1];
  *reinterpret_cast<d2*>(row) = v;
}
__device__ __forceinline__ void pipe_get(const double* row, double (&c)[2]) {
  typedef double d2 __attribute__((ext_vector_type(2)));
  const d2 v = *reinterpret_cast<const d2*>(row);
  c[0] = v.x;
  c[1] = v.y;
}

// Buffer resources: base address in scalar registers, the row's byte offset as
// the scalar offset, the lane's column as a 32-bit vector offset, so a load
// takes no address arithmetic.  Arrays are limited to 2 GiB (launch_pipe).
typedef __amdgpu_buffer_rsrc_t PipeRsrc;
// (a null array has no records: its loads give zero)
__device__ __forceinline__ PipeRsrc pipe_rsrc(const void* p) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, p ? 0x7fffffff : 0, 0x00020000);
}
constexpr int kPipeDrop = (int)0x80000000u;  // a vector offset past every array: the store is dropped

// a lane's part of a row as stored
template <typename T>
struct PipeRaw {
  T c[2];
};
// PAIR: nx even and 16-byte aligned vectors: a lane's two columns are adjacent
// in memory whenever one of them is in the grid (its first column is even);
// col: the lane's columns to load
template <bool PAIR, bool NT, typename T>
__device__ __forceinline__ void pipe_load(PipeRsrc r, const int (&col)[2], int soff, PipeRaw<T>& o) {
  constexpr int aux = NT ? 2 : 0;
  typedef double d2 __attribute__((ext_vector_type(2)));
  typedef float f2 __attribute__((ext_vector_type(2)));
  if constexpr (PAIR && sizeof(T) == 8) {
    const d2 v = __builtin_bit_cast(d2, __builtin_amdgcn_raw_buffer_load_b128(r, col[0] * 8, soff, aux));
    o.c[0] = v.x;
    o.c[1] = v.y;
  } else if constexpr (PAIR) {
    const f2 v = __builtin_bit_cast(f2, __builtin_amdgcn_raw_buffer_load_b64(r, col[0] * 4, soff, aux));
    o.c[0] = v.x;
    o.c[1] = v.y;
  } else {
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      if constexpr (sizeof(T) == 8)
        o.c[v] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, col[v] * 8, soff, aux));
      else
        o.c[v] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, col[v] * 4, soff, aux));
    }
  }
}
// col: the lane's own columns, kPipeDrop / 8 where it stores nothing
template <bool PAIR, bool NT, typename T>
__device__ __forceinline__ void pipe_store(PipeRsrc r, const int (&col)[2], int soff, const double (&c)[2]) {
  constexpr int aux = NT ? 2 : 0;
  typedef unsigned u2 __attribute__((ext_vector_type(2)));
  typedef unsigned u4 __attribute__((ext_vector_type(4)));
  typedef double d2 __attribute__((ext_vector_type(2)));
  typedef float f2 __attribute__((ext_vector_type(2)));
  if constexpr (PAIR && sizeof(T) == 8) {
    d2 v;
    v.x = c[0];
    v.y = c[1];
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), r, col[0] * 8, soff, aux);
  } else if constexpr (PAIR) {
    f2 v;
    v.x = (float)c[0];
    v.y = (float)c[1];
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), r, col[0] * 4, soff, aux);
  } else {
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      if constexpr (sizeof(T) == 8)
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, c[v]), r, col[v] * 8, soff, aux);
      else
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, (float)c[v]), r, col[v] * 4, soff, aux);
    }
  }
}

constexpr int kPipeAhead = 3;  // rows in flight ahead of the row being put
template <bool ADVF>
constexpr int kPipeCoef = ADVF ? 5 : 3;
constexpr int kPipeThreads = kWave * (1 + kPipeMax);
// LDS of a block, in rows: the coefficient ring (2 nst slots of kxy, kxx faces,
// kyy faces (, ax', ay')), y and p handed to each stage (two rows each), the
// added row (two)
inline size_t pipe_lds_bytes(int nst, bool advf, bool src) {
  const size_t rows = (size_t)(advf ? 5 : 3) * 2 * nst + 4 * nst + (src ? 2 : 0);
  const size_t need = sizeof(double) * kPipeRow * rows;
  return need < sizeof(double) * kDecideLds ? sizeof(double) * kDecideLds : need;
}

// the coefficients of one index, at a lane's two columns
struct PipeCoef {
  double m[2], kx[2], ky[2], ax[2], ay[2];
};
// a stage's windows: its input rows C (the row worked on) and S below it, and
// what the ticks before computed: C's east neighbour, the x difference of C,
// the y flux between S and C, H of C and of S
struct PipeWin {
  double C[2], S[2], CE, dEC[2], FyS[2], HC[2], HS[2];
};

// A u at row C from the new row u above it (and the windows), which
// then slide up one row; cN, cC, cS: the coefficients of the rows' indices
template <bool ADVF>
__device__ __forceinline__ void pipe_row(PipeWin& w, const double (&u)[2], const PipeCoef& cN, const PipeCoef& cC,
                                         const PipeCoef& cS, double axc, double ayc, double (&a)[2],
                                         double (&centre)[2]) {
  const double dx0 = w.C[1] - w.C[0], dx1 = w.CE - w.C[1], Fx0 = cN.kx[0] * dx0;
  const double uW = dpp_f64_any<kDppWaveShr1>(u[1]), uE = dpp_f64_any<kDppWaveShl1>(u[0]);
  const double dE[2] = {u[1] - uW, uE - u[0]};
  double G[2], dv[2], dy[2];
#pragma unroll
  for (int v = 0; v < 2; ++v) {
    dy[v] = u[v] - w.C[v];
    dv[v] = u[v] - w.S[v];
    G[v] = cC.m[v] * dv[v];
  }
  // (the west neighbour's x flux and G in one shift)
  const double BW = dpp_f64_any<kDppWaveShr1>(__builtin_fma(cN.kx[1], dx1, G[1]));
  const double GE = dpp_f64_any<kDppWaveShl1>(G[0]);
  double Fy[2], H[2];
#pragma unroll
  for (int v = 0; v < 2; ++v) {
    Fy[v] = cN.ky[v] * dy[v];
    H[v] = cN.m[v] * dE[v];
  }
  a[0] = ((Fx0 + G[1]) - BW) + ((Fy[0] - w.FyS[0]) + (H[0] - w.HS[0]));
  a[1] = (__builtin_fma(cN.kx[1], dx1, -Fx0) + __builtin_fma(-cC.m[0], dv[0], GE)) +
         ((Fy[1] - w.FyS[1]) + (H[1] - w.HS[1]));
  if constexpr (ADVF) {
    // ax'_E u_E - ax'_W u_W, and ay'_N u_N - ay'_S u_S
    const double Q0 = cN.ax[0] * w.C[0], Q1 = cN.ax[1] * w.C[1];
    const double QW = dpp_f64_any<kDppWaveShr1>(Q1), QE = dpp_f64_any<kDppWaveShl1>(Q0);
    const double Qx[2] = {Q1 - QW, QE - Q0};
#pragma unroll
    for (int v = 0; v < 2; ++v) a[v] += Qx[v] + __builtin_fma(cN.ay[v], u[v], -(cS.ay[v] * w.S[v]));
  } else {
#pragma unroll
    for (int v = 0; v < 2; ++v) a[v] += __builtin_fma(axc, w.dEC[v], ayc * dv[v]);
  }
#pragma unroll
  for (int v = 0; v < 2; ++v) {
    centre[v] = w.C[v];
    w.S[v] = w.C[v];
    w.C[v] = u[v];
    w.HS[v] = w.HC[v];
    w.HC[v] = H[v];
    w.dEC[v] = dE[v];
    w.FyS[v] = Fy[v];
  }
  w.CE = uE;
}

// What every wave of a block knows of its run.
struct PipeRun {
  int nst, J0, J1, a0, i0, nticks;
  // a row r needs the rim's care (a Dirichlet grid's ghost rows or columns)
  // where (unsigned)(r + rimb) >= riml: never on a periodic grid, in every row
  // of a strip with ghost columns
  int rimb;
  unsigned riml;
  int col0;  // the lane's first column
};
template <class Args>
__device__ __forceinline__ PipeRun pipe_run(const FieldView& F, const Args& A, int b) {
  PipeRun r;
  const int cb = b % A.ncb, run = b / A.ncb;
  r.nst = A.nst;
  r.J0 = run * A.rows;
  r.J1 = min(r.J0 + A.rows, F.ny);
  r.a0 = r.J0 - r.nst;
  r.i0 = cb * kPipeCols - 2 * kPipeFrame;
  const int puts = r.J1 - r.J0 + 2 * r.nst + 1;  // (in whole groups of kPipeAhead)
  r.nticks = max(r.J1 - r.J0 + 3 * r.nst + 1, (puts + kPipeAhead - 1) / kPipeAhead * kPipeAhead);
  const bool per = F.bc == BC_PERIODIC;
  r.rimb = per ? 1 << 30 : 0;
  r.riml = per ? 0xffffffffu : (r.i0 < 0 || r.i0 + kPipeRow > F.nx) ? 0u : (unsigned)F.ny;
  r.col0 = r.i0 + (int)(threadIdx.x & (kWave - 1)) * 2;
  return r;
}
// whether the lane's columns lie in the grid, and whether it is left of it
// (recomputed where it is needed, on the rim: as loop invariants the masks
// would take scalar registers)
__device__ __forceinline__ void pipe_inside(const FieldView& F, const PipeRun& r, bool (&in)[2], bool& left) {
  int c = r.col0, nx = F.nx;
  __asm__ volatile("" : "+v"(c), "+s"(nx));
#pragma unroll
  for (int v = 0; v < 2; ++v) in[v] = c + v >= 0 && c + v < nx;
  left = c < 0;
}

// The stop flag as one wave read it, the same for the whole block, which its
// barriers need (an LDS word that the first puts overwrite).
__device__ __forceinline__ bool pipe_stopped(double* lds, int flag, bool mine) {
  int* const word = reinterpret_cast<int*>(lds);
  if (mine) *word = flag;
  __syncthreads();
  const int stop = __builtin_amdgcn_readfirstlane(*word);
  __syncthreads();
  return stop != 0;
}

// Wave 0: the rows a0 .. J1 - 1 + nst into LDS.  stop: the sweep's stop flag, or
// null; it is read ahead of the first rows, whose loads are in flight while the
// block waits for it (read before them it cost 1 us a launch).
template <typename TF, typename TYI, bool ADVF, bool PAIR, bool NT, int MODE, class Args>
__device__ __forceinline__ void pipe_loader(const FieldView& F, const Args& A, double* lds, const PipeRun& r,
                                            const int* stop) {
  int flag = 0;
  if (stop) flag = __hip_atomic_load(stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int lane = threadIdx.x & (kWave - 1);
  const bool per = F.bc == BC_PERIODIC;
  constexpr int NC = kPipeCoef<ADVF>;
  const int ring = 2 * r.nst * NC * kPipeRow;
  double* const fld = lds + lane * 2;
  double* const yb = fld + ring;
  double* const pb = yb + 2 * r.nst * kPipeRow;
  double* const wb = pb + 2 * r.nst * kPipeRow;
  // the columns to load: wrapped, or clamped to the edge
  int cl[2];
#pragma unroll
  for (int v = 0; v < 2; ++v) {
    const int c = r.col0 + v;
    cl[v] = per ? wrap_col(c, F.nx) : min(max(c, 0), F.nx - 1);
  }
  if constexpr (PAIR) cl[0] &= ~1;  // (a clamped pair starts on the even column)
  const PipeRsrc rm = pipe_rsrc(F.kxy), rk = pipe_rsrc(F.kxx), rg = pipe_rsrc(F.kyy), ry = pipe_rsrc(A.yin);
  const PipeRsrc rax = pipe_rsrc(ADVF ? F.ax : F.kxx), ray = pipe_rsrc(ADVF ? F.ay : F.kyy);
  const PipeRsrc rp = pipe_rsrc((MODE & PIPE_SRC) ? (const void*)A.src : (const void*)A.pin);
  // the row to load next: running (rr), after the boundary rule (rw), and the
  // two before it (rows past the last one needed, which no stage reads, repeat
  // it); offsets in elements
  int left_to_load = r.J1 - r.J0 + 2 * r.nst, rr = r.a0, rw = rr;
  const int rlow = per ? INT_MIN : 0, rtop = per ? 0 : F.ny - 1;
  if (per) {
    rw %= F.ny;
    if (rw < 0) rw += F.ny;
  } else {
    rw = min(max(rw, 0), F.ny - 1);
  }
  int o1 = rw * F.nx, o2 = o1;  // (no stage reads the rows below a0)
  struct Set {
    PipeRaw<TF> m, k, g, ax, ay;
    PipeRaw<TYI> y;
    PipeRaw<double> p;
  };
  Set set[kPipeAhead];
  constexpr int SF = sizeof(TF), SY = sizeof(TYI);
  auto load = [&](Set& s) {
    const int o = rw * F.nx;
    pipe_load<PAIR, false>(rm, cl, o * SF, s.m);
    pipe_load<PAIR, false>(rg, cl, o * SF, s.g);
    pipe_load<PAIR, false>(rk, cl, o1 * SF, s.k);
    if constexpr (ADVF) {
      pipe_load<PAIR, false>(rax, cl, o1 * SF, s.ax);
      pipe_load<PAIR, false>(ray, cl, o * SF, s.ay);
    }
    pipe_load<PAIR, false>(ry, cl, o1 * SY, s.y);
    if constexpr (MODE == PIPE_LATER || (MODE & PIPE_SRC)) pipe_load<PAIR, NT>(rp, cl, o2 * 8, s.p);
    o2 = o1;
    o1 = o;
    const int step = left_to_load > 0 ? 1 : 0;
    --left_to_load;
    rr += step;
    rw += step;
    rw = rr <= rlow ? 0 : rw;
    rw = rw == F.ny ? rtop : rw;
  };
#pragma unroll
  for (int i = 0; i < kPipeAhead; ++i) load(set[i]);
  if (stop && pipe_stopped(lds, flag, lane == 0)) return;
  double gp[2] = {0.0, 0.0}, yp[2] = {0.0, 0.0};  // kyy and y of the row before
  int row = r.a0, slot = 0;  // the row to put, where its coefficients go
  auto put = [&](Set& s, int par) {
    // the row moves to fresh registers and its set is loaded again at once
    // (without the copies the compiler moves sets in flight between registers
    // at the loop's back edge, waiting for every load)
    double y[2], m[2], k[2], g[2], ax[2] = {}, ay[2] = {}, p[2] = {};
#pragma unroll
    for (int v = 0; v < 2; ++v) {
      m[v] = (double)vcopy(s.m.c[v]);
      g[v] = (double)vcopy(s.g.c[v]);
      k[v] = (double)vcopy(s.k.c[v]);
      if constexpr (ADVF) {
        ax[v] = (double)vcopy(s.ax.c[v]);
        ay[v] = (double)vcopy(s.ay.c[v]);
      }
      y[v] = (double)vcopy(s.y.c[v]);
      if constexpr (MODE == PIPE_LATER || (MODE & PIPE_SRC)) p[v] = vcopy(s.p.c[v]);
    }
    load(s);
    if ((unsigned)(row + r.rimb) >= r.riml || (unsigned)(row - 1 + r.rimb) >= r.riml) {
      // outside a Dirichlet grid: the edge column's kxx and kyy (a pair outside
      // on the left was loaded as columns 0, 1, on the right as the last two;
      // the rows are the edge row's already), zero for the rest
      bool in[2], left;
      pipe_inside(F, r, in, left);
      const bool inr = row >= 0 && row < F.ny, iny = row - 1 >= 0 && row - 1 < F.ny;
      if constexpr (PAIR) {
        const double ke = left ? k[0] : k[1], ge = left ? g[0] : g[1];
#pragma unroll
        for (int v = 0; v < 2; ++v) {
          k[v] = in[v] ? k[v] : ke;
          g[v] = in[v] ? g[v] : ge;
        }
      }
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        y[v] = iny && in[v] ? y[v] : 0.0;
        m[v] = inr && in[v] ? m[v] : 0.0;
        ax[v] = in[v] ? ax[v] : 0.0;
        ay[v] = inr && in[v] ? ay[v] : 0.0;
      }
    }
    ++row;
    const double kE = dpp_f64_any<kDppWaveShl1>(k[0]);
    const double fx[2] = {0.5 * (k[0] + k[1]), 0.5 * (k[1] + kE)};
    const double fy[2] = {0.5 * (gp[0] + g[0]), 0.5 * (gp[1] + g[1])};
    double* const f = fld + slot;
    slot += NC * kPipeRow;
    slot = slot == ring ? 0 : slot;
#pragma unroll
    for (int v = 0; v < 2; ++v) gp[v] = g[v];
    pipe_put(f, m);
    pipe_put(f + kPipeRow, fx);
    pipe_put(f + 2 * kPipeRow, fy);
    if constexpr (ADVF) {
      pipe_put(f + 3 * kPipeRow, ax);
      pipe_put(f + 4 * kPipeRow, ay);
    }
    pipe_put(yb + par, y);
    if constexpr ((MODE & PIPE_SRC) != 0) pipe_put(wb + par, p);
    if constexpr (MODE != PIPE_LATER) {
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        p[v] = A.d0 * yp[v];
        yp[v] = y[v];
      }
    }
    pipe_put(pb + par, p);
  };
  const int puts = r.J1 - r.J0 + 2 * r.nst + 1;
  int m = 0, par = 0;
#pragma unroll 1
  for (; m < puts; m += kPipeAhead) {
#pragma unroll
    for (int i = 0; i < kPipeAhead; ++i) {
      put(set[i], par);
      par = kPipeRow - par;
      __syncthreads();
    }
  }
#pragma unroll 1
  for (; m < r.nticks; ++m) __syncthreads();
}

// Wave t: stage t of the run's rows (MODE PIPE_LATER: any but a first launch's
// stage 1, which takes the added row, forms the stage vector and whether y_0 is zero).
template <typename TY, bool ADVF, bool PAIR, bool NT, int MODE, class Args>
__device__ __forceinline__ void pipe_stage(const FieldView& F, const Args& A, double* lds, const PipeRun& r, int t,
                                           int b, const int* stop) {
  if (stop && pipe_stopped(lds, 0, false)) return;
  const int lane = threadIdx.x & (kWave - 1);
  constexpr int NC = kPipeCoef<ADVF>;
  const int nst = r.nst, ring = 2 * nst * NC * kPipeRow;
  double* const fld = lds + lane * 2;
  double* const yb = fld + ring;
  double* const pb = yb + 2 * nst * kPipeRow;
  const double* const wb = pb + 2 * nst * kPipeRow;
  double* const yr = yb + 2 * (t - 1) * kPipeRow;
  double* const pr = pb + 2 * (t - 1) * kPipeRow;
  int cs[2];  // the columns to store
#pragma unroll
  for (int v = 0; v < 2; ++v) {
    const int c = r.col0 + v;
    cs[v] = c >= 0 && c < F.nx && lane >= kPipeFrame && lane < kWave - kPipeFrame ? c : kPipeDrop / 8;
  }
  const double ig = A.invg;
  const double shift = A.shift_of(t), dk = A.dk_of(t);
  constexpr bool wants_max = MODE != PIPE_LATER, has_src = (MODE & PIPE_SRC) != 0, stagevec = (MODE & PIPE_STAGE) != 0;
  const double srcc = has_src ? A.srcc : 0.0;
  const double axc = F.axc, ayc = F.ayc;
  // what the stage stores
  double* pout = A.p_of(t);
  void* yout = t == nst ? A.yout : nullptr;
  __asm__ volatile("" : "+s"(yout), "+s"(pout));  // (held, not loaded again at every store)
  const int flags = __builtin_amdgcn_readfirstlane((t < nst ? 1 : 0) | (yout || pout ? 2 : 0));
  PipeWin win{};
  PipeCoef c1{}, c2{}, nx{};  // indices e - 1, e - 2; the next tick's e
  double hold[2] = {};        // p of the last row
  double yn2[2] = {}, pn2[2] = {};
  unsigned some[2] = {};  // bits of the y_0 (and src) seen, without their signs
  // first tick (an even one, maybe a tick before the rows are there: the
  // windows are whole again by the first complete row), last tick with work
  const int n0 = (3 * t - 1) & ~1, n1 = r.J1 - r.J0 + 2 * nst + t;
  int row = r.a0 + n0 - 2 * t - 1;  // the row worked on
  int slot = (n0 - 2 * t + 2 * nst) % (2 * nst) * NC * kPipeRow;
  const unsigned R = r.J1 - r.J0;
  auto fetch = [&]() {
    const double* const f = fld + slot;
    pipe_get(f, nx.m);
    pipe_get(f + kPipeRow, nx.kx);
    pipe_get(f + 2 * kPipeRow, nx.ky);
    if constexpr (ADVF) {
      pipe_get(f + 3 * kPipeRow, nx.ax);
      pipe_get(f + 4 * kPipeRow, nx.ay);
    }
    slot += NC * kPipeRow;
    slot = slot == ring ? 0 : slot;
  };
  auto tick = [&](int rd, int wr) {
    int fl = flags;
    __asm__ volatile("" : "+s"(fl));  // (opaque: the compiler would make a copy of the loop per case)
    double u[2], p[2], s[2] = {}, a[2], cc[2], y[2], pn[2];
    pipe_get(yr + rd, u);
    pipe_get(pr + rd, p);
    if (has_src) pipe_get(wb + rd, s);
    const PipeCoef cE = nx;
    fetch();
    pipe_row<ADVF>(win, u, cE, c1, c2, axc, ayc, a, cc);
    if (stagevec) {
      // the stage vector A u + s
#pragma unroll
      for (int v = 0; v < 2; ++v) y[v] = a[v] + s[v];
    } else {
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        if (has_src) a[v] = __builtin_fma(srcc, s[v], a[v]);
        y[v] = __builtin_fma(-shift, cc[v], a[v]) * ig;
      }
    }
    if ((unsigned)(row + r.rimb) >= r.riml) {
      // rows and columns outside a Dirichlet grid hold zero at every stage
      bool in[2], left;
      pipe_inside(F, r, in, left);
      const bool out = row < 0 || row >= F.ny;
#pragma unroll
      for (int v = 0; v < 2; ++v) y[v] = out || !in[v] ? 0.0 : y[v];
    }
    if (fl & 1) {
      if constexpr (sizeof(TY) == 4) {
        // (stages read y in its storage type's rounding, as a one-term launch
        // reads it back from memory, a stage vector in FP64; p and the norms
        // take it unrounded)
        double z[2];
#pragma unroll
        for (int v = 0; v < 2; ++v) z[v] = stagevec ? y[v] : storage_round<TY>(y[v]);
        pipe_put(yr + 2 * kPipeRow + wr, z);
      } else {
        pipe_put(yr + 2 * kPipeRow + wr, y);
      }
      pipe_put(pr + 2 * kPipeRow + wr, hold);
    }
#pragma unroll
    for (int v = 0; v < 2; ++v) pn[v] = __builtin_fma(dk, y[v], p[v]);
    if ((unsigned)(row - r.J0) < R) {
      // norms (on every lane of the strip; the frame's are dropped at the end)
      // and stores of the run's own rows.  (y^2 is summed and scaled by d^2 once:
      // a product d y per point made every pipeline case 2 % slower, 4096^2
      // steps 5353 -> 5461 us.  The host sees to a y^2 that overflows.)
#pragma unroll
      for (int v = 0; v < 2; ++v) {
        yn2[v] = __builtin_fma(y[v], y[v], yn2[v]);
        pn2[v] = __builtin_fma(pn[v], pn[v], pn2[v]);
        if constexpr (wants_max) {
          const double a0 = stagevec ? y[v] : cc[v];
          some[v] |= (unsigned)__double2hiint(a0) << 1 | (unsigned)__double2loint(a0);
          if (has_src && !stagevec) some[v] |= (unsigned)__double2hiint(s[v]) << 1 | (unsigned)__double2loint(s[v]);
        }
      }
      if (fl & 2) {
        const int o = row * F.nx;
        if (yout) pipe_store<PAIR, NT, TY>(pipe_rsrc(yout), cs, o * (int)sizeof(TY), y);
        if (pout) pipe_store<PAIR, NT, double>(pipe_rsrc(pout), cs, o * 8, pn);
      }
    }
#pragma unroll
    for (int v = 0; v < 2; ++v) hold[v] = pn[v];
    c2 = c1;
    c1 = cE;
    ++row;
    __syncthreads();
  };
#pragma unroll 1
  for (int n = 1; n < n0; ++n) __syncthreads();
  fetch();
  __syncthreads();
  int n = n0;
  constexpr int P = kPipeRow;
#pragma unroll 1
  while (true) {
    tick(P, 0);
    if (n++ == n1) break;
    tick(0, P);
    if (n++ == n1) break;
    tick(P, 0);
    if (n++ == n1) break;
    tick(0, P);
    if (n++ == n1) break;
  }
#pragma unroll 1
  for (; n < r.nticks; ++n) __syncthreads();
  if (A.replay) return;

  // the stage's partials: term t of the launch at rows 3t, 3t + 1; row 2 of a
  // first launch: whether any y_0 or src is not zero (the test needs no more)
  double acc[3] = {0.0, 0.0, 0.0};
#pragma unroll
  for (int v = 0; v < 2; ++v) {
    if (cs[v] < 0) continue;  // (not an own column)
    acc[0] += yn2[v];
    acc[1] += pn2[v];
    if (some[v]) acc[2] = 1.0;
  }
#pragma unroll
  for (int o = kWave / 2; o > 0; o >>= 1) {
    acc[0] += __shfl_xor(acc[0], o);
    acc[1] += __shfl_xor(acc[1], o);
    if constexpr (MODE != PIPE_LATER) acc[2] = fmax(acc[2], __shfl_xor(acc[2], o));
  }
  if (lane == 0) {
    double* const part = A.partials + (long)A.slot * A.slot_stride;
    const long nb = A.nblocks;
    const int term = t - 1 - A.stage;
    if (term >= 0) {
      part[3L * term * nb + b] = acc[0] * dk * dk;
      part[(3L * term + 1) * nb + b] = acc[1];
    }
    if (wants_max) part[2 * nb + b] = acc[2];
  }
}

template <typename TF, typename TY, bool ADVF, bool PAIR, bool NT, int MODE>
__global__ __launch_bounds__(kPipeThreads, ADVF ? 2 : 4) void pipe_kernel(FieldView F, PipeArgs A) {
  extern __shared__ __attribute__((aligned(16))) double lds[];
  // XCD-contiguous logical blocks: neighbouring strips, which share lines at
  // their common edge, run on one XCD
  const int L = xcd_contiguous(blockIdx.x, gridDim.x);
  if (L == 0) {
    if constexpr (MODE != PIPE_LATER) {
      // a new sweep: clear the control block (no block of this launch reads it)
      if (!A.replay && threadIdx.x == 0) {
        Ctl c{};
        *A.ctl = c;
      }
    } else {
      if (!A.replay && A.nterms_prev > 0) leja_decide<true>(A, lds);
    }
    return;
  }
  const int* const stop = MODE == PIPE_LATER && !A.replay ? &A.ctl->stop : nullptr;
  const PipeRun r = pipe_run(F, A, L - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  using TYI = std::conditional_t<MODE == PIPE_LATER, TY, double>;
  if (wave == 0) pipe_loader<TF, TYI, ADVF, PAIR, NT, MODE>(F, A, lds, r, stop);
  else if (MODE != PIPE_LATER && wave == 1) pipe_stage<TY, ADVF, PAIR, NT, MODE>(F, A, lds, r, 1, L - 1, stop);
  else pipe_stage<TY, ADVF, PAIR, NT, PIPE_LATER>(F, A, lds, r, wave, L - 1, stop);
}

template <typename TF, typename TY, bool ADVF, bool PAIR, bool NT, int MODE>
static hipError_t pipe_go(const FieldView& f, const PipeArgs& a, hipStream_t st) {
  const dim3 grid(a.nblocks + 1), blk(kWave * (1 + a.nst));
  const size_t lds = pipe_lds_bytes(a.nst, ADVF, (MODE & PIPE_SRC) != 0);
  auto* k = pipe_kernel<TF, TY, ADVF, PAIR, NT, MODE>;
  if (a.ev_start) hipExtLaunchKernelGGL(k, grid, blk, lds, st, a.ev_start, a.ev_stop, 0, f, a);
  else hipLaunchKernelGGL(k, grid, blk, lds, st, f, a);
  return hipGetLastError();
}

template <typename TF, typename TY, bool ADVF, int MODE>
static hipError_t pipe_vectors(const FieldView& f, const PipeArgs& a, hipStream_t st) {
  if (!a.pair) return pipe_go<TF, TY, ADVF, false, false, MODE>(f, a, st);
  if (a.stream) return pipe_go<TF, TY, ADVF, true, true, MODE>(f, a, st);
  return pipe_go<TF, TY, ADVF, true, false, MODE>(f, a, st);
}

template <typename TF, typename TY, bool ADVF>
static hipError_t pipe_mode(const FieldView& f, const PipeArgs& a, hipStream_t st) {
  if (!a.first) return pipe_vectors<TF, TY, ADVF, PIPE_LATER>(f, a, st);
  if (a.stage) {
    if (a.src) return pipe_vectors<TF, TY, ADVF, PIPE_FIRST | PIPE_STAGE | PIPE_SRC>(f, a, st);
    return pipe_vectors<TF, TY, ADVF, PIPE_FIRST | PIPE_STAGE>(f, a, st);
  }
  if (a.src) return pipe_vectors<TF, TY, ADVF, PIPE_FIRST | PIPE_SRC>(f, a, st);
  return pipe_vectors<TF, TY, ADVF, PIPE_FIRST>(f, a, st);
}

template <typename TF>
hipError_t launch_pipe_fields(const FieldView& f, const PipeArgs& a, hipStream_t st) {
  if constexpr (sizeof(TF) == 4) {
    if (a.f32y) return f.ax ? pipe_mode<TF, float, true>(f, a, st) : pipe_mode<TF, float, false>(f, a, st);
  }
  return f.ax ? pipe_mode<TF, double, true>(f, a, st) : pipe_mode<TF, double, false>(f, a, st);
}

}  // namespace adl
