// Internal interface between the C ABI (api.cpp) and the HIP kernels.
#pragma once

#include <hip/hip_runtime_api.h>

#include <cstdint>

#include "collide_d3q27.hpp"   // Rates<R>

namespace cmlbm {

struct Geom {
  int nx, ny, nz;
  uint32_t nxy;
  uint64_t N;   // nodes
};

// The launch's map from a block's linear index to its row segment: rows
// r = z*ny + y of nx nodes are cut into nseg segments of one block each, so
// block L works on row L / nseg, segment L % nseg, and row r is (y, z) =
// (r % ny, r / ny).  The dividers are set up on the host (Divider), which keeps
// these divisions on the scalar unit.  Filled by the launchers.
struct RowMap {
  uint32_t nseg;
  Divider seg, ny;
};

// Body force: a uniform vector (already multiplied by the time scale) or a
// field [3][nz][ny][nx] times `scale`.
template <typename FT>
struct ForceArgs {
  FT uni[3];
  const FT* field;
  FT scale;
};

template <typename R>
struct StepArgs {
  Geom g;
  const void* fin;
  void* fout;
  const uint8_t* mask;
  ForceArgs<R> force;
  Rates<R> rates;
  // Optional FP64 totals of the input state, fused into the step: per-block
  // partials [step_blocks(g)][4], a second-stage buffer [kReduceChunks][4] and
  // the device output [4].  All null for a plain step.
  double* partials;
  double* stage;
  double* totals;
  RowMap rm;
};

// Tiles of the two-steps-in-one-pass kernel, in each run of zlen planes along z:
// `main` tiles over the first nbx blocks of 64 nodes along x, and `tail` tiles
// of tail_rows rows over a short last block.
struct Tiles2 {
  uint32_t nbx, main, tail, tail_rows, zlen;
  Divider bx, all, tail_width;   // by nbx, by main + tail, by the tail's columns with its halo
};

template <typename R>
struct AuxArgs {
  Geom g;
  const void* in0;
  void* out0;
  void* out1;
  const uint8_t* mask;
  ForceArgs<R> force;
};

template <typename R>
struct AdjArgs {
  Geom g;
  const void* fpost;      // forward post-collision state of step n (storage type)
  const R* lam_next;      // dL/dfbar^{n+1} (compute type)
  R* lam;                 // dL/dfbar^n (compute type)
  double* dLdF;           // [3][N], accumulated (force field mode)
  const uint8_t* mask;
  ForceArgs<R> force;
  Rates<R> rates;
};

// prec: 0 FP64, 1 FP32, 2 FP32 compute / FP16 deviation storage, 3 BF16 deviations.
hipError_t launch_step(int q, int prec, const StepArgs<double>& a64, const StepArgs<float>& a32, hipStream_t st);
// Two steps from a.fin to a.fout in one pass (no totals), the same populations as
// two launch_step calls, by the tiles that step2_plan (step2_plan.hpp) makes.
hipError_t launch_step2(int q, int prec, const StepArgs<double>& a64, const StepArgs<float>& a32, const Tiles2& t,
                        hipStream_t st);
hipError_t launch_gather(int q, int prec, const AuxArgs<double>& a64, const AuxArgs<float>& a32, hipStream_t st);
// Population buffer (blocked layout) <-> full populations in compute type,
// structure of arrays [Q][N]; to_soa selects the direction.
hipError_t launch_convert(int q, int prec, const Geom& g, const void* in, void* out, bool to_soa, hipStream_t st);
// pre: the buffer holds pre-collision populations (phase 0 of the in-place
// step) and is read in place instead of pulled.
hipError_t launch_macro(int q, int prec, const AuxArgs<double>& a64, const AuxArgs<float>& a32, bool pre,
                        hipStream_t st);
hipError_t launch_totals(int q, int prec, const AuxArgs<double>& a64, const AuxArgs<float>& a32, bool pre,
                         double* partials, int nblk, double* out4, hipStream_t st);
// One in-place step on the buffer a.fout (a.fin unused); parity = phase of the
// buffer on entry (0 or 1).
hipError_t launch_step_inplace(int q, int prec, const StepArgs<double>& a64, const StepArgs<float>& a32, int parity,
                               hipStream_t st);
// fpost == nullptr: fpre is an in-place buffer in phase 0 (storage type, blocked rows).
hipError_t launch_init(int q, int prec, const Geom& g, const void* rho0, const void* u0, const ForceArgs<double>& f64,
                       const ForceArgs<float>& f32, const uint8_t* mask, void* fpre, void* fpost, hipStream_t st);
hipError_t launch_adjoint(int q, int prec, const AdjArgs<double>& a64, const AdjArgs<float>& a32, double* partials,
                          int nblk, double* dLdomega, double* dLdF_uniform, hipStream_t st);

// Wall-layout sensitivity of one step (fpost, lam_next, mask, force, rates of
// the AdjArgs; lam and dLdF unused): accumulates into dLdphi[N] (FP64).
// post = false: fpost is the step's input state and the collision is
// recomputed (FP64 atomics); post = true: fpost is the collided state the
// streaming moves, and each node gathers its own terms.
hipError_t launch_wall_sensitivity(int q, int prec, const AdjArgs<double>& a64, const AdjArgs<float>& a32,
                                   double* dLdphi, bool post, hipStream_t st);

hipError_t launch_ke_sum(int q, int prec, const Geom& g, const void* fpre, const uint8_t* mask,
                         const ForceArgs<double>& f64, const ForceArgs<float>& f32, double* partials, int nblk,
                         double* out, hipStream_t st);
hipError_t launch_ke_seed(int q, int prec, const Geom& g, const void* fpre, const uint8_t* mask,
                          const ForceArgs<double>& f64, const ForceArgs<float>& f32, double scale, void* lam,
                          double* dLdF, double* partials, int nblk, hipStream_t st);
hipError_t launch_init_adjoint(int q, int prec, const Geom& g, const void* u0, const void* lam0,
                               const uint8_t* mask, const ForceArgs<double>& f64, const ForceArgs<float>& f32,
                               double* dLdF, double* partials, int nblk, hipStream_t st);

// Whether a step takes the nodes in a row, whatever rows of the lattice they are in
// (k_step_thin), by the bytes of a stored population.  Measured against the row kernel,
// as a ratio of its time:
//   * nx <= 8, every kind: 0.53 to 1.01 from 1296 rows (1.3 at 135 rows, where a step is
//     all latency);
//   * nx = 9 to 16, where a row is a large part of a wavefront: with walls 0.52 to 1.08
//     from 4096 rows; without, D3Q27 FP64 0.49 to 1.00 from there, but FP32 0.90 to 1.24
//     at 4970 rows and 0.95 to 1.11 at 7140, 0.73 to 0.95 at 10920, D3Q15 FP32 0.72 to 1.21
//     at 9506, 0.73 to 0.99 at 19740; D3Q27 16-bit 0.82 to 1.08 up to 7140, 0.73 to 0.98
//     from 8190; D3Q15 16-bit 0.63 to 1.08, D3Q15 FP64 0.72 to 1.12 up to 7140, 0.52 to
//     0.98 from 8190;
//   * nx = 17 to 32, 16-bit storage: 0.74 to 1.14 at 8100 to 12100 rows, 0.50 to 1.06
//     from 16384.  (The wider types are at the memory's rate in rows: 1.03 at 32 x
//     400 x 400, and a run takes two steps per pass.)
// From nx = 40 the row kernel is ahead.
inline bool thin_pays(int q, int bytes, bool walls, const Geom& g) {
  if (g.nx > 32 || g.N >= (uint64_t(1) << 31)) return false;
  const uint64_t rows = uint64_t(g.ny) * uint64_t(g.nz);
  if (g.nx <= 8) return rows >= 1536;
  if (g.nx > 16) return bytes == 2 && rows >= 16384;
  if (walls) return rows >= 4096;
  if (bytes == 4) return rows >= (q == 27 ? 10240 : 16384);
  return rows >= ((q == 27) == (bytes == 8) ? 4096 : 8192);
}

// Threads of a block that takes segments of rows of nx nodes, at most `most`: as
// few segments as blocks of `most` give, of about the same number of wavefronts (nx
// = 320: 192 + 128, not 256 + 64 with three of eight wavefronts idle).  The adjoint
// of D3Q27 FP32 at 320 x 320 x 256: 2388 -> 2072 us, with an obstacle 2853 -> 2268.
inline int even_block(int nx, int most) {
  const int nseg = (nx + most - 1) / most, each = (nx + nseg - 1) / nseg;
  return (each + 63) / 64 * 64;
}

// Blocks of the adjoint launch: a multiple of 8 (one share per XCD), each block
// visiting at most kAdjItems row segments (each thread that many nodes).
constexpr uint64_t kAdjItems = 8;
inline int adjoint_blocks(const Geom& g) {
  const uint64_t items = uint64_t((g.nx + 255) / 256) * uint64_t(g.ny) * uint64_t(g.nz);
  uint64_t nb = (items + kAdjItems - 1) / kAdjItems;
  nb = ((nb + 7) / 8) * 8;
  return int(nb);
}
// Segments of equal size where the stride of a block's items (its XCD's blocks) is
// a multiple of a row's segments: a thread's chain of multiply-adds then stays in one
// segment, and has the same nodes in it as with segments of 256.  Elsewhere it would
// have others, and the gradients other roundings.
inline int adjoint_block(const Geom& g) {
  const int nseg = (g.nx + 255) / 256;
  return nseg == 1 || adjoint_blocks(g) / 8 % nseg == 0 ? even_block(g.nx, 256) : 256;
}

// Whether the adjoint takes the form with a wavefront per row segment (k_adjoint's
// SPLIT) on a lattice, and the rows of partial sums that its blocks leave.  The
// factors of D3Q27 take 100 KB of LDS (148 in FP64), one block on a CU: the form wins while
// there are a few blocks per CU (640 blocks, 96 x 50 x 50: 33 against 65 us; 2304,
// 96^3: 96 against 87), in FP64 likewise (43 against 76; 2048, 256 x 64 x 64: 201
// against 163).  D3Q15's take 51 KB in FP32 (2304 blocks: 46 against 57 us; 4096,
// 128^3: 106 against 121).
inline bool adjoint_split(int q, bool wide, const Geom& g) {
  return adjoint_blocks(g) * (adjoint_block(g) / 64) <= (q == 15 && !wide ? 4096 : 1024);
}
inline int adjoint_rows(int q, bool wide, const Geom& g) {
  return adjoint_blocks(g) * (adjoint_split(q, wide, g) ? adjoint_block(g) / 64 : 1);
}

constexpr int kTotalsBlocks = 2048;
constexpr int kReduceChunks = 256;

// Blocks of one launch of the step with totals (one per segment of a row, at most
// CMLBM_STEP_BLOCK nodes wide).
uint64_t step_blocks(const Geom& g);

// Static device scratch of the allocation-free fused-totals step: room for the
// per-block partials of at most kStaticStepBlocks step blocks and the
// second-stage sums, kStaticScratchDoubles doubles (16 MiB + 8 KiB) per device,
// held until the process ends.
constexpr uint64_t kStaticStepBlocks = uint64_t(1) << 19;
constexpr uint64_t kStaticScratchDoubles = 4 * (kStaticStepBlocks + kReduceChunks);

// Device address of that scratch on the current device, looked up once per
// device (hipGetSymbolAddress) and cached; *out is null on failure.
hipError_t static_scratch(double** out);

// Work-items of the largest grid the lattice's launches use (the step and the
// adjoint cover whole row segments rounded up to 64 lanes); a dispatch counts
// its work-items in 32 bits.
uint64_t max_work_items(const Geom& g);

}  // namespace cmlbm
