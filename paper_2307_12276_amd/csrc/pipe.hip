// The pipeline kernels' launch geometry and launcher.
#include <type_traits>

#include <hip/hip_ext.h>

#include "pipe_kernel.h"

namespace adl {

// The tile kernel where its blocks are at most one per CU: a sweep of 89 terms,
// us, on the pipeline / tiles: 256^2 159 / 148, 320^2 162 / 149 (224 tiles), 384^2
// 180 / 190 (312 tiles), 512^2 202 / 258, 1024^2 350 / 610; 64^2 146 / 146.
constexpr long kTileBlocks = 255;
// Else the pipeline.  One block per CU where that leaves a block at most kPipeRows1 rows, else two:
// two share a CU's issue slots but halve the rows, and a launch takes rows + 21
// ticks.  A sweep of 89 terms, us, with 255 / 511 blocks: 256^2 173 / 199, 512^2
// 213 / 233, 896^2 (29 rows) 313 / 321, 2048 x 512 (40 rows) 365 / 362, 1024^2
// (41 rows) 369 / 371, 1280^2 466 / 457, 4096^2 step 7430 / 5834.  With
// advection fields two blocks' LDS (98 KB each) does not fit a CU: 1001 x 777
// step 486 / 664.
void pipe_geometry(int nx, int ny, bool advf, PipeArgs& a) {
  const long tiles = (long)((nx + kTileCols - 1) / kTileCols) * ((ny + kTileRows - 1) / kTileRows);
  a.tile = tiles <= kTileBlocks;
  if (a.tile) {
    a.ncb = (nx + kTileCols - 1) / kTileCols;
    a.rows = kTileRows;
    a.nblocks = (int)tiles;
    return;
  }
  a.ncb = (nx + kPipeCols - 1) / kPipeCols;
  auto rows = [&](int blocks) {
    int runs = blocks / a.ncb;
    if (runs < 1) runs = 1;
    if (runs > ny) runs = ny;
    return (ny + runs - 1) / runs;
  };
  a.rows = rows(kPipeBlocks1);
  if (a.rows > kPipeRows1 && !advf) a.rows = rows(kPipeBlocks2);
  a.nblocks = a.ncb * ((ny + a.rows - 1) / a.rows);
}

hipError_t launch_pipe(const FieldView& f, const PipeArgs& a, hipStream_t st) {
  // (float Newton vectors come with float fields)
  if ((long)f.nx * f.ny >= kPipePoints || (a.f32y && !f.f32)) return hipErrorInvalidValue;
  if (a.nst < 1 || a.nst > kPipeMax || a.rows < 1 || a.ncb * (a.tile ? kTileCols : kPipeCols) < f.nx ||
      (a.tile && a.rows != kTileRows) ||
      a.nblocks != a.ncb * ((f.ny + a.rows - 1) / a.rows))
    return hipErrorInvalidValue;
  // (a replay writes no partials)
  if (!a.replay && 3L * a.nst * a.nblocks > a.slot_stride) return hipErrorInvalidValue;
  // a first launch forms its p_0, a later one reads it; the added row and the
  // stage vector belong to first launches
  if (a.first ? a.pin != nullptr : (a.pin == nullptr || a.src || a.stage)) return hipErrorInvalidValue;
  // what is read and what is stored are distinct vectors
  if (a.yin == nullptr || a.yin == a.yout) return hipErrorInvalidValue;
  bool any = false;
  for (int t = 0; t < kPipeMax; ++t) {
    if (!a.pst[t]) continue;
    any = true;
    if (t >= a.nst || a.pst[t] == a.pin || a.pst[t] == a.yin || a.pst[t] == a.yout || a.pst[t] == a.src)
      return hipErrorInvalidValue;
    for (int i = 0; i < t; ++i)
      if (a.pst[i] == a.pst[t]) return hipErrorInvalidValue;
  }
  if (!any) return hipErrorInvalidValue;
  if (a.tile) return launch_tile(f, a, st);
  return f.f32 ? launch_pipe_fields<float>(f, a, st) : launch_pipe_fields<double>(f, a, st);
}

// The decision that closes a chunk, which the host waits for: one block of 16
// waves, a wave per row of partials (15 rows at seven terms).
__global__ __launch_bounds__(16 * kWave) void decide_kernel(LejaArgs A) {
  leja_decide(A);
  if (A.hctl && threadIdx.x == 0) publish_outcome(A);
}
hipError_t launch_decide(const LejaArgs& a, hipStream_t st) {
  decide_kernel<<<1, 16 * kWave, 0, st>>>(a);
  return hipGetLastError();
}

// (bound by memory: 24 B a point, 62 us at 4096^2)
__global__ __launch_bounds__(kBlock) void pipe_update_kernel(PipeUpdate A) {
  const int m = A.ctl->degree;
  if (!A.ctl->stop || A.ctl->status != 1 || m == 0) return;
  const int L = m <= A.lead ? 0 : 1 + (m - A.lead - 1) / kPipeMax;
  const int last = min(A.lead + L * kPipeMax, A.maxdeg);
  const double* p = m == A.mark[0] ? A.markp[0] : m == A.mark[1] ? A.markp[1] : m == last ? A.pbuf[L % 3] : nullptr;
  if (!p) return;
  double* __restrict__ u = A.u;
  const double* __restrict__ q = p;
  const long step = (long)gridDim.x * blockDim.x;
#pragma unroll 4
  for (long i = (long)blockIdx.x * blockDim.x + threadIdx.x; i < A.n; i += step) u[i] = u[i] + A.h * q[i];
}
hipError_t launch_pipe_update(const PipeUpdate& a, hipStream_t st) {
  const long nb = (a.n + kBlock - 1) / kBlock;
  pipe_update_kernel<<<nb < 8192 ? nb : 8192, kBlock, 0, st>>>(a);
  return hipGetLastError();
}

// One wave per iteration's sum, then the tests in order: iteration j stops the
// method where lambda_j differs from lambda_{j-1} (0 before the first) by at most
// rtol lambda_j, and (status 4) where lambda_j or the norm it is taken from is
// zero, not finite or so far from 1 that sums of squares lose digits.
constexpr double kPowerLow = 1e-150, kPowerHigh = 1e150, kPowerLow2 = 1e-200, kPowerHigh2 = 1e200;
constexpr int kPowerIters = 8 * kPipeMax;  // most iterations of a chunk
__global__ __launch_bounds__(16 * kWave) void power_decide_kernel(PowerDecide A) {
  __shared__ double n2[kPowerIters + 1];
  const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  for (int j = wave; j <= A.iters; j += 16) {
    // (j = 0: the chunk's start vector)
    const double* p = j == 0 ? A.init : A.partials + (3L * kPipeMax * ((j - 1) / kPipeMax) + 3 * ((j - 1) % kPipeMax)) * A.nb;
    const int n = j == 0 ? (A.init ? A.ninit : 0) : A.nb;
    double v = 0.0;
#pragma unroll 8
    for (int i = lane; i < n; i += kWave) v += p[i];
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
    if (lane == 0) n2[j] = j == 0 && !A.init ? A.ctl->tn2 : v;
  }
  __syncthreads();
  if (threadIdx.x != 0) return;
  Ctl* c = A.ctl;
  double lam = c->lam, lam_prev = c->lam_prev;  // (zero in the first chunk)
  int stop = 0, status = 0, k = A.k;
  for (int j = 1; j <= A.iters && !stop; ++j) {
    ++k;
    lam_prev = lam;
    lam = n2[j] == 0.0 ? 0.0 : A.scale * sqrt(n2[j] / n2[j - 1]);
    if (!(lam > kPowerLow && lam < kPowerHigh && n2[j] > kPowerLow2 && n2[j] < kPowerHigh2)) {
      stop = 1; status = 4;
    } else if (fabs(lam - lam_prev) <= A.rtol * lam) {
      stop = 1; status = 1;
    } else if (k >= A.max_iter) {
      stop = 1; status = 3;
    }
  }
  c->tn2 = n2[A.iters];
  c->lam = lam;
  c->lam_prev = lam_prev;
  c->iters = k;
  c->status = status;
  c->stop = stop;
}
hipError_t launch_power_decide(const PowerDecide& a, hipStream_t st) {
  if (a.iters < 1 || a.iters > kPowerIters) return hipErrorInvalidValue;
  power_decide_kernel<<<1, 16 * kWave, 0, st>>>(a);
  return hipGetLastError();
}

}  // namespace adl
