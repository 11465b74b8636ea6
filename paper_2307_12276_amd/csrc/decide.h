// The stopping decision of a Newton-Leja launch, taken by one block of the
// next launch, and the block-wide reductions it and the kernels use.
#pragma once

#include "device.h"

namespace adl {

// ---------------------------------------------------------------------------
// Block-wide fixed-order reduction (sums for k < NS, NaN-propagating max for
// the rest); every thread receives the totals.
// ---------------------------------------------------------------------------
template <int NA, int NS>
__device__ __forceinline__ void block_allreduce_at(double (&v)[NA], double* sh) {
#pragma unroll
  for (int k = 0; k < NA; ++k) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const double t = __shfl_xor(v[k], o);
      v[k] = (k < NS) ? v[k] + t : nanmax(v[k], t);
    }
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < NA; ++k) sh[wave * NA + k] = v[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NA; ++k) {
    double s = sh[k];
    for (int w = 1; w < nw; ++w) s = (k < NS) ? s + sh[w * NA + k] : nanmax(s, sh[w * NA + k]);
    v[k] = s;
  }
}
// the same with a static LDS array (sh: NA * 16 doubles)
template <int NA, int NS>
__device__ __forceinline__ void block_allreduce(double (&v)[NA]) {
  __shared__ double sh[NA * 16];
  block_allreduce_at<NA, NS>(v, sh);
}

// Stopping test of the terms of the previous launch (k_prev+1 ..
// k_prev+nterms_prev, in order) from its block partials, taken by one block
// and recorded in the control block by thread 0 unless an earlier launch has
// already stopped the sweep.  Args: LejaArgs or PipeArgs.
//
// Term t's partials are rows 3t (||d y||^2) and 3t + 1 (||p||^2) of the slot;
// row 2 of a sweep's first launch is max(|y_0|, |w2|), or 1 where either is not
// zero (only zero is told from the rest).  A wave takes one
// segment of a row at a time (fixed order: lanes, shuffle tree, segments), so
// that the rows' loads and shuffles run side by side: the decision closing a
// chunk is on the host's critical path.
// (dsh: a kernel's dynamic LDS for the segment totals, kDecideLds doubles,
// or null for a static array; the four-term staged and the pipeline kernels
// pass their rings)
constexpr int kDecideTerms = 8;   // most terms of a launch
constexpr int kDecideSegs = 16;   // most segments of a row
constexpr int kDecideLds = (2 * kDecideTerms + 1) * kDecideSegs;
template <bool DYN = false, class Args>
__device__ __forceinline__ void leja_decide(const Args& A, double* dsh = nullptr) {
  double* sh = dsh;
  if constexpr (!DYN) {
    __shared__ double st[kDecideLds];
    sh = st;
  }
  const double* part = A.partials + (long)A.slot_prev * A.slot_stride;
  const int nb = A.nb_prev, nt = A.nterms_prev;
  const int lane = threadIdx.x & (kWave - 1), nw = blockDim.x / kWave;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
  // (in flight beside the partials)
  const int stopped = __hip_atomic_load(&A.ctl->stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int done = A.ctl->degree;
  // norms of the terms before the decided ones (the window of the test)
  double hist[kStopHist];
#pragma unroll
  for (int i = 0; i < kStopHist; ++i) hist[i] = A.ctl->hist[i];
  const int rows = 2 * nt + 1;  // the last one: row 2, a maximum
  const int segs = min(kDecideSegs, (nb + 1023) / 1024), len = (nb + segs - 1) / segs;
  for (int task = wave; task < rows * segs; task += nw) {
    const int r = task / segs, s = task - r * segs;
    const bool mx = r == 2 * nt;
    const double* p = part + (long)(mx ? 2 : 3 * (r / 2) + (r & 1)) * nb;
    const int i1 = min((s + 1) * len, nb);
    double v = 0.0;
    if (mx) {
      for (int i = s * len + lane; i < i1; i += kWave) v = nanmax(v, p[i]);
    } else {
#pragma unroll 8
      for (int i = s * len + lane; i < i1; i += kWave) v += p[i];
    }
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) {
      const double t = __shfl_xor(v, o);
      v = mx ? nanmax(v, t) : v + t;
    }
    if (lane == 0) sh[task] = v;
  }
  __syncthreads();
  if (threadIdx.x != 0 || stopped) return;  // (stopped: decided by an earlier launch)
  // Terms up to `done` were decided already: a chunk's closing decision
  // launch decides the chunk's last launch, and the first launch of the next
  // chunk is handed the same launch.  Each term enters the window once.
  if (A.k_prev + nt <= done) return;
  int stop = 0, status = 0, degree = A.k_prev + nt;
  double tn2 = 0.0, pn2 = 0.0;
  for (int t = 0; t < nt && !stop; ++t) {
    const int deg = A.k_prev + t + 1;
    if (deg <= done) continue;
    tn2 = pn2 = 0.0;
    for (int s = 0; s < segs; ++s) {
      tn2 += sh[2 * t * segs + s];
      pn2 += sh[(2 * t + 1) * segs + s];
    }
    double m0 = 0.0;
    for (int s = 0; s < segs; ++s) m0 = nanmax(m0, sh[2 * nt * segs + s]);
    if (!isfinite(tn2) || !isfinite(pn2)) {
      stop = 1; status = 2; degree = deg;
    } else if (deg == 1 && m0 == 0.0) {
      stop = 1; status = 1; degree = 0;
    } else if (window_stop(hist, deg, sqrt(tn2), pn2, A.tol)) {
      stop = 1; status = 1; degree = deg;
    } else if (deg >= A.max_degree) {
      stop = 1; status = 3; degree = deg;
    }
  }
  Ctl* c = A.ctl;
  c->tn2 = tn2;
  c->pn2 = pn2;
#pragma unroll
  for (int i = 0; i < kStopHist; ++i) c->hist[i] = hist[i];
  c->degree = degree;
  c->status = status;
  __hip_atomic_store(&c->stop, stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The sweep's outcome for the host (thread 0 of the decision launch, after
// leja_decide): the control block's fields (written by this thread, or by an
// earlier launch), then the sequence number with a system-scope release, so
// that a host that sees the number sees the fields too.
__device__ __forceinline__ void publish_outcome(const LejaArgs& A) {
  HostCtl* h = A.hctl;
  const Ctl* c = A.ctl;
  h->stop = __hip_atomic_load(&c->stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  h->status = c->status;
  h->degree = c->degree;
  __hip_atomic_store(&h->seq, A.hseq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The sweep's stop flag, read once per block (thread 0) and broadcast, so that
// a concurrent update of the flag cannot split a block.
__device__ __forceinline__ bool block_stopped(const Ctl* ctl) {
  __shared__ int s_stop;
  if (threadIdx.x == 0) s_stop = __hip_atomic_load(&ctl->stop, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  return s_stop != 0;
}

}  // namespace adl
