// Up to kPipeMax applications of A per launch as a pipeline of waves: the
// launch arguments and the launcher (pipe_kernel.h holds the kernel).
#pragma once

#include "internal.h"

namespace adl {

// stages of a launch: Newton terms, or (first launch of a midpoint step) the
// stage vector and then terms
constexpr int kPipeMax = 7;
// A strip is one wave wide at two columns per lane; each stage loses one
// column at either end, so kPipeFrame lanes a side are the frame (8 columns
// for up to 8 stages), and 112 columns are the strip's own: rows of seven
// whole 128-byte lines, so that no line is written by two blocks
constexpr int kPipeFrame = 4;
constexpr int kPipeCols = (kWave - 2 * kPipeFrame) * 2;
// worker blocks of a launch, in one round over the chip's 256 CUs less the
// deciding block: one per CU, or two (70 KB of LDS each): pipe_geometry
constexpr int kPipeBlocks1 = 255, kPipeBlocks2 = 511, kPipeRows1 = 40;

// grids of fewer points: every byte offset of an FP64 vector below 2^31
constexpr long kPipePoints = 1L << 28;

// a launch's MODE: a later one, or a first one (p_0 = d0 y_0), maybe with an
// added row (src) and with the stage vector as its first stage
enum { PIPE_LATER = 0, PIPE_FIRST = 1, PIPE_SRC = 2, PIPE_STAGE = 4 };

// the points a block of the tile kernel owns (pipe_tile.hip)
constexpr int kTileCols = kWave - 2 * kPipeMax, kTileRows = 24 - 2 * kPipeMax;

// One launch: stages 1 .. nst on y_0 = yin.  Stage t computes
//   y_t = ((A y_{t-1} + srcc src) - shift[t-1] y_{t-1}) invg,
//   p_t = p_{t-1} + dk[t-1] y_t
// (src enters stage 1 only); with `stage`, stage 1 is y_1 = A y_0 + src.
struct PipeArgs {
  const void* yin;   // y_0 of the launch
  const double* pin; // p_0 (later launches)
  const double* src; // first launches: added to A y_0 in stage 1, or null
  double srcc;
  double d0;         // first launches: p_0 = d0 y_0
  void* yout;        // y_nst, or null: not stored
  double* pst[kPipeMax];  // p_t of stage t, or null: not stored
  double shift[kPipeMax], dk[kPipeMax];
  double invg;       // 1 / gamma
  int nst;
  int first;         // y_0 = v in FP64, p_0 = d0 y_0; no decision
  int stage;         // stage 1 forms the stage vector (its y stays FP64 and is y_0 of the sweep)
  int replay;        // no stop flag, no decision, no partials
  int f32y;          // Newton vectors stored as float
  int stream;        // non-temporal hints on p_0 and the stored vectors
  int pair;          // rows readable two columns at a time (nx even, 16-byte aligned vectors)
  int tile;          // the tile kernel's launch
  int rows;          // rows per run
  int ncb, nblocks;  // strips, worker blocks
  // the decision of the previous launch (leja_decide) and this launch's partials
  double* partials;
  long slot_stride;
  int slot;
  int nb_prev, k_prev, nterms_prev, slot_prev;
  double tol;
  int max_degree;
  Ctl* ctl;
  hipEvent_t ev_start, ev_stop;
  // stage t's shift, d and p array
  __host__ __device__ double shift_of(int t) const { return shift[t - 1]; }
  __host__ __device__ double dk_of(int t) const { return dk[t - 1]; }
  __host__ __device__ double* p_of(int t) const { return pst[t - 1]; }
};
// tile, rows, ncb and nblocks of a launch on an nx x ny grid
void pipe_geometry(int nx, int ny, bool advf, PipeArgs& a);
// a launch's block partials take 3 x nst x nblocks values of its slot
hipError_t launch_pipe(const FieldView& f, const PipeArgs& a, hipStream_t st);
// (launch_pipe's, for a.tile)
hipError_t launch_tile(const FieldView& f, const PipeArgs& a, hipStream_t st);
// u += h p of a sweep that stopped (status 1) at a degree whose p was stored: a
// marked one, or the last term of launch L (in pbuf[L mod 3]), launches being of
// `lead` terms, then kPipeMax each, up to maxdeg.
struct PipeUpdate {
  double* u;
  double h;
  long n;
  const Ctl* ctl;
  int mark[2];
  const double* markp[2];
  const double* pbuf[3];
  int lead, maxdeg;
};
hipError_t launch_pipe_update(const PipeUpdate& a, hipStream_t st);
// The power method's tests of iterations k + 1 .. k + iters: launch i of the
// chunk (kPipeMax iterations, the last one maybe fewer) left its partials at
// partials + 3 kPipeMax nb i, ||y_0||^2 of the first chunk is the sum of
// init[0 .. ninit) (else ctl->tn2).  lambda_j = scale ||y_j|| / ||y_{j-1}||.
// Status 4: a norm out of range.
struct PowerDecide {
  const double* partials;
  const double* init;
  int ninit, nb;
  int k, iters;
  double scale, rtol;
  int max_iter;
  Ctl* ctl;
};
hipError_t launch_power_decide(const PowerDecide& a, hipStream_t st);
// the decision of launch slot_prev alone, published to the host mirror if hctl is set
hipError_t launch_decide(const LejaArgs& a, hipStream_t st);

}  // namespace adl
