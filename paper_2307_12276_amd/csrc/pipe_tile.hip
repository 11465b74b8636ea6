// Small grids: up to kPipeMax Newton terms per launch on tiles held in
// registers.
//
// A block owns kTileCols x kTileRows points and computes a frame of kPipeMax
// more on every side (each stage's outermost ring is one ring less valid): 64
// columns, a lane each, and 24 rows, three per wave, with y, p and the
// coefficients of the wave's rows in registers through all stages.  A stage
// exchanges only the edge rows of neighbouring waves through LDS (y, and the
// kxy differences H that the rows above and below need), one barrier a stage,
// where the pipeline needs one per row and stage and fills and drains over 21
// ticks.  The points computed are three times the points owned, so larger grids,
// which fill the chip, take the pipeline (pipe_geometry).
//
// Bound by the latency of a stage (three rows of 25 FP64 and 8 shift
// instructions a wave, the exchange) and of the loads, which are all in flight at
// once.  A launch of seven terms, 256^2: 12.4 us on the
// pipeline, 9.7 us here, of which about 3 are the launch (phi_0 by 98 sweeps:
// 27.4 -> 20.5 ms).
#include <type_traits>

#include <hip/hip_ext.h>

#include "decide.h"
#include "pipe.h"
#include "tile.h"

namespace adl {

constexpr int kTileK = 3, kTileWaves = 8, kTileThreads = kWave * kTileWaves;
static_assert(kTileK * kTileWaves == kTileRows + 2 * kPipeMax && kWave == kTileCols + 2 * kPipeMax, "frame");
constexpr int kTileSums = 2 * kPipeMax + 1;  // norms of a launch, and whether y_0 is not zero

template <typename TF, typename TY, bool ADVF, int MODE>
__global__ __launch_bounds__(kTileThreads, 4) void tile_kernel(FieldView F, PipeArgs A) {
  // edge rows [stage parity][wave][bottom y, H, top y, H], then the norms
  __shared__ double lds[kTileSums * kTileThreads + 1];
  static_assert(kTileSums * kTileThreads >= 2 * kTileWaves * 4 * kWave && kTileSums * kTileThreads >= kDecideLds, "");
  const int L = xcd_contiguous(blockIdx.x, gridDim.x);
  if (L == 0) {
    if constexpr (MODE != PIPE_LATER) {
      if (!A.replay && threadIdx.x == 0) {
        Ctl c{};
        *A.ctl = c;
      }
    } else {
      if (!A.replay && A.nterms_prev > 0) leja_decide<true>(A, lds);
    }
    return;
  }
  // the stop flag, one read for the whole block, which its barriers need: in
  // flight ahead of the rows, and passed on at the first stage's barrier
  int* const word = reinterpret_cast<int*>(lds + kTileSums * kTileThreads);
  int flag = 0;
  if constexpr (MODE == PIPE_LATER) {
    if (!A.replay && threadIdx.x == 0) flag = __hip_atomic_load(&A.ctl->stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  using TYI = std::conditional_t<MODE == PIPE_LATER, TY, double>;
  constexpr bool SRC = (MODE & PIPE_SRC) != 0, STAGE = (MODE & PIPE_STAGE) != 0;
  constexpr int K = kTileK;
  const int b = L - 1, lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  const int cb = b % A.ncb, run = b / A.ncb, nst = A.nst;
  const bool per = F.bc == BC_PERIODIC;
  const int J0 = run * kTileRows, J1 = min(J0 + kTileRows, F.ny);
  const int c = cb * kTileCols - kPipeMax + lane, j0 = J0 - kPipeMax + wave * K;
  const bool incol = per || (c >= 0 && c < F.nx);
  const bool own = lane >= kPipeMax && lane < kWave - kPipeMax && c < F.nx;
  const int cl = per ? wrap_col(c, F.nx) : min(max(c, 0), F.nx - 1);
  // the tile's rows j0 - 1 .. j0 + K after the boundary rule, as offsets
  int ro[K + 2];
  bool inrow[K + 2];
#pragma unroll
  for (int i = 0; i < K + 2; ++i) {
    const int j = j0 - 1 + i;
    inrow[i] = per || (j >= 0 && j < F.ny);
    ro[i] = (per ? wrap_col(j, F.ny) : min(max(j, 0), F.ny - 1)) * F.nx;
  }
  const TF* const kxx = reinterpret_cast<const TF*>(F.kxx) + cl;
  const TF* const kxy = reinterpret_cast<const TF*>(F.kxy) + cl;
  const TF* const kyy = reinterpret_cast<const TF*>(F.kyy) + cl;
  const TF* const fax = ADVF ? reinterpret_cast<const TF*>(F.ax) + cl : nullptr;
  const TF* const fay = ADVF ? reinterpret_cast<const TF*>(F.ay) + cl : nullptr;
  const TYI* const yin = reinterpret_cast<const TYI*>(A.yin) + cl;
  double u[K], p[K], m[K], kx[K], g[K + 2], ax[K], ay[K], s[K];
#pragma unroll
  for (int i = 0; i < K + 2; ++i) g[i] = (double)kyy[ro[i]];
#pragma unroll
  for (int i = 0; i < K; ++i) {
    u[i] = (double)yin[ro[i + 1]];
    kx[i] = (double)kxx[ro[i + 1]];
    m[i] = (double)kxy[ro[i + 1]];
    if constexpr (ADVF) {
      ax[i] = (double)fax[ro[i + 1]];
      ay[i] = (double)fay[ro[i + 1]];
    }
    if constexpr (MODE == PIPE_LATER) p[i] = A.pin[ro[i + 1] + cl];
    if constexpr (SRC) s[i] = A.src[ro[i + 1] + cl];
  }
  double ky[K + 1];  // faces below row j0, and above each row
#pragma unroll
  for (int i = 0; i <= K; ++i) ky[i] = 0.5 * (g[i] + g[i + 1]);
#pragma unroll
  for (int i = 0; i < K; ++i) {
    kx[i] = 0.5 * (kx[i] + dpp_f64_any<kDppWaveShl1>(kx[i]));
    const bool in = incol && inrow[i + 1];  // (outside a Dirichlet grid: zero)
    u[i] = in ? u[i] : 0.0;
    m[i] = in ? m[i] : 0.0;
    if constexpr (ADVF) {
      ax[i] = in ? ax[i] : 0.0;
      ay[i] = in ? ay[i] : 0.0;
    }
    if constexpr (MODE != PIPE_LATER) p[i] = A.d0 * u[i];
  }
  const double axc = F.axc, ayc = F.ayc, ig = A.invg;
  double tn[kPipeMax], pn[kPipeMax];
  unsigned some = 0;
#pragma unroll
  for (int t = 0; t < kPipeMax; ++t) tn[t] = pn[t] = 0.0;

#pragma unroll
  for (int t = 1; t <= kPipeMax; ++t) {
    if (t > nst) break;
    // x differences; H = kxy (u_E - u_W) (+ ay u), which the neighbours' rows need
    double dE[K], H[K];
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const double uW = dpp_f64_any<kDppWaveShr1>(u[i]), uE = dpp_f64_any<kDppWaveShl1>(u[i]);
      dE[i] = uE - uW;
      H[i] = m[i] * dE[i];
      if constexpr (ADVF) H[i] = __builtin_fma(ay[i], u[i], H[i]);
    }
    double* const ex = lds + (t & 1) * (kTileWaves * 4 * kWave) + lane;
    double* const mine = ex + wave * 4 * kWave;
    mine[0] = u[0];
    mine[kWave] = H[0];
    mine[2 * kWave] = u[K - 1];
    mine[3 * kWave] = H[K - 1];
    if (MODE == PIPE_LATER && t == 1 && threadIdx.x == 0) *word = flag;
    __syncthreads();
    if constexpr (MODE == PIPE_LATER) {
      if (t == 1 && __builtin_amdgcn_readfirstlane(*word)) return;
    }
    // (the outermost waves' outer rows are frame: any value does)
    const double* const lo = ex + max(wave - 1, 0) * 4 * kWave;
    const double* const hi = ex + min(wave + 1, kTileWaves - 1) * 4 * kWave;
    double uS = lo[2 * kWave], HS = lo[3 * kWave];
    const double uT = hi[0], HT = hi[kWave];
    const double shift = A.shift[t - 1], dk = A.dk[t - 1];
    double* const pout = A.pst[t - 1];
    const bool first = MODE != PIPE_LATER && t == 1;
    double FyS = ky[0] * (u[0] - uS);
#pragma unroll
    for (int i = 0; i < K; ++i) {
      const double uN = i + 1 < K ? u[i + 1 < K ? i + 1 : 0] : uT, HN = i + 1 < K ? H[i + 1 < K ? i + 1 : 0] : HT;
      const double uC = u[i];
      const double Fx = kx[i] * (dpp_f64_any<kDppWaveShl1>(uC) - uC);
      const double dv = uN - uS;
      double G = m[i] * dv;
      if constexpr (ADVF) G = __builtin_fma(ax[i], uC, G);
      const double GE = dpp_f64_any<kDppWaveShl1>(G), BW = dpp_f64_any<kDppWaveShr1>(Fx + G);
      const double FyN = ky[i + 1] * (uN - uC);
      double a = ((Fx + GE) - BW) + ((FyN - FyS) + (HN - HS));
      if constexpr (!ADVF) a += __builtin_fma(axc, dE[i], ayc * dv);
      double y;
      if (STAGE && first) {
        y = a;
        if constexpr (SRC) y += s[i];
      } else {
        if constexpr (SRC) {
          if (first) a = __builtin_fma(A.srcc, s[i], a);
        }
        y = __builtin_fma(-shift, uC, a) * ig;
      }
      if (!per) y = incol && inrow[i + 1] ? y : 0.0;
      p[i] = __builtin_fma(dk, y, p[i]);
      const int j = j0 + i;
      if (j >= J0 && j < J1) {
        // (on every lane; the frame's are dropped at the end)
        tn[t - 1] = __builtin_fma(y, y, tn[t - 1]);
        pn[t - 1] = __builtin_fma(p[i], p[i], pn[t - 1]);
        if (first) {
          const double a0 = STAGE ? y : uC;
          some |= (unsigned)__double2hiint(a0) << 1 | (unsigned)__double2loint(a0);
          if (SRC && !STAGE) some |= (unsigned)__double2hiint(s[i]) << 1 | (unsigned)__double2loint(s[i]);
        }
        if (own) {
          if (pout) pout[ro[i + 1] + cl] = p[i];
          if (t == nst && A.yout) reinterpret_cast<TY*>(A.yout)[ro[i + 1] + cl] = (TY)y;
        }
      }
      uS = uC;
      HS = H[i];
      FyS = FyN;
      // (stages read y as it is stored, a stage vector in FP64)
      u[i] = STAGE && first ? y : storage_round<TY>(y);
    }
  }
  if (A.replay) return;

  // the block's partials: term t at rows 3t, 3t + 1; row 2 of a first launch:
  // whether any y_0 or src is not zero
  __syncthreads();
#pragma unroll
  for (int t = 0; t < kPipeMax; ++t) {
    lds[2 * t * kTileThreads + threadIdx.x] = own ? tn[t] : 0.0;
    lds[(2 * t + 1) * kTileThreads + threadIdx.x] = own ? pn[t] : 0.0;
  }
  if constexpr (MODE != PIPE_LATER) lds[2 * kPipeMax * kTileThreads + threadIdx.x] = own && some ? 1.0 : 0.0;
  __syncthreads();
  double* const part = A.partials + (long)A.slot * A.slot_stride;
  const long nb = A.nblocks;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int v = wave + q * kTileWaves, t = v / 2, term = t - A.stage;
    if (v >= kTileSums || (MODE == PIPE_LATER && v == kTileSums - 1)) continue;
    double r = 0.0;
#pragma unroll
    for (int w = 0; w < kTileWaves; ++w) r += lds[v * kTileThreads + w * kWave + lane];
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) r += __shfl_xor(r, o);
    if (lane != 0) continue;
    if (v == kTileSums - 1) {
      part[2 * nb + b] = r;
    } else if (t < nst && term >= 0) {
      const double d = A.dk[t];
      part[(3L * term + (v & 1)) * nb + b] = (v & 1) ? r : r * d * d;
    }
  }
}

template <typename TF, typename TY, bool ADVF, int MODE>
static hipError_t tile_go(const FieldView& f, const PipeArgs& a, hipStream_t st) {
  const dim3 grid(a.nblocks + 1), blk(kTileThreads);
  auto* k = tile_kernel<TF, TY, ADVF, MODE>;
  if (a.ev_start) hipExtLaunchKernelGGL(k, grid, blk, 0, st, a.ev_start, a.ev_stop, 0, f, a);
  else hipLaunchKernelGGL(k, grid, blk, 0, st, f, a);
  return hipGetLastError();
}

template <typename TF, typename TY, bool ADVF>
static hipError_t tile_mode(const FieldView& f, const PipeArgs& a, hipStream_t st) {
  if (!a.first) return tile_go<TF, TY, ADVF, PIPE_LATER>(f, a, st);
  if (a.stage) {
    if (a.src) return tile_go<TF, TY, ADVF, PIPE_FIRST | PIPE_STAGE | PIPE_SRC>(f, a, st);
    return tile_go<TF, TY, ADVF, PIPE_FIRST | PIPE_STAGE>(f, a, st);
  }
  if (a.src) return tile_go<TF, TY, ADVF, PIPE_FIRST | PIPE_SRC>(f, a, st);
  return tile_go<TF, TY, ADVF, PIPE_FIRST>(f, a, st);
}

hipError_t launch_tile(const FieldView& f, const PipeArgs& a, hipStream_t st) {
  if (f.f32) {
    if (a.f32y) return f.ax ? tile_mode<float, float, true>(f, a, st) : tile_mode<float, float, false>(f, a, st);
    return f.ax ? tile_mode<float, double, true>(f, a, st) : tile_mode<float, double, false>(f, a, st);
  }
  return f.ax ? tile_mode<double, double, true>(f, a, st) : tile_mode<double, double, false>(f, a, st);
}

}  // namespace adl
