// Tiles of the two-steps-in-one-pass kernel (step2.hip), and where it is the faster
// way.  Host code.
#pragma once

#include <cstdint>

#include "kernels.hpp"

namespace cmlbm {

constexpr uint32_t kSlots = 256;      // blocks at work at a time: one on a CU

// Rows of a tile.  (wide: FP64 storage, whose waiting populations are in LDS.)
constexpr int tile2_rows(int q, bool wide, bool walls) { return wide && (q == 27 || walls) ? 4 : 8; }

// Rows of a tail tile beside main ones: each row is cache lines of its own in
// every load, so that a tile of 130 rows of 2 nodes holds up the launch (130 x
// 130 x 70 D3Q27 FP32, two steps: 160 us at 130 rows, 82 at 40, 81 at 24, 89 at 12;
// one step at a time 109 us).
constexpr uint32_t kTailRows = 24;

// Planes per block.  A block's time is its planes and about three more (two
// planes of halo, filling the pipeline), and the launch's that of a block times
// the rounds of kSlots blocks.  For a number of rounds the best is the most runs
// along z that fit in them, so only those are tried, until the rounds alone cost more
// than the best (65535 planes: 164 us for every number of planes, 2 at most so).
inline uint32_t run_length(uint32_t tiles, uint32_t nz) {
  uint64_t best = ~uint64_t(0);
  uint32_t arg = nz;
  for (uint64_t rounds = (uint64_t(tiles) + kSlots - 1) / kSlots; uint64_t(tiles) * nz + 3 * kSlots * rounds < best * kSlots; ++rounds) {
    const uint64_t fit = rounds * kSlots / tiles, runs = fit < nz ? fit : nz;
    const uint32_t zlen = uint32_t((nz + runs - 1) / runs);
    const uint64_t cost = rounds * (zlen + 3);
    if (cost < best) {
      best = cost;
      arg = zlen;
    }
    if (runs == nz) break;
  }
  return arg;
}

inline Tiles2 step2_tiles(int q, bool wide, bool walls, const Geom& g) {
  const uint32_t rows = uint32_t(tile2_rows(q, wide, walls)), plane = 66 * (rows + 2), waves = rows + 3;
  const uint32_t nx = uint32_t(g.nx), ny = uint32_t(g.ny), nz = uint32_t(g.nz);
  Tiles2 t{};
  t.nbx = (nx + 63) / 64;
  // A short last block of the rows takes more rows, packed over the threads,
  // where that is less work: collisions of both steps by all wavefronts for
  // tail_rows rows, against rows + 3 and rows by wavefront for `rows` rows.
  const uint32_t len = nx & 63u;
  if (len) {
    uint32_t r = plane / (len + 2) - 2;
    if (wide && r * len > rows * 64) r = rows * 64 / len;
    if (t.nbx > 1 && r > kTailRows) r = kTailRows;
    if (r > ny) r = ny;
    const uint32_t busy = ((len + 2) * (r + 2) + 63) / 64;
    if (2 * busy * ((ny + r - 1) / r) < (waves + rows) * ((ny + rows - 1) / rows)) {
      t.nbx -= 1;
      t.tail_rows = r;
      t.tail = (ny + r - 1) / r;
      t.tail_width = Divider::of(len + 2);
    }
  }
  t.main = t.nbx * ((ny + rows - 1) / rows);
  t.zlen = run_length(t.main + t.tail, nz);
  t.bx = Divider::of(t.nbx);
  t.all = Divider::of(t.main + t.tail);
  return t;
}

// What two steps in one pass and two single ones take, fitted to the times of both at
// 380 lattices of each kind (2^17 to 2^25 nodes, thin in any direction, ragged, long):
//   pass: rounds of kSlots blocks x turns of a block (zlen + 2) x
//         (turn + wave W + row r), in ns: W the wavefronts of collisions in the two
//         steps of a turn, r the rows of a tail tile (lines of their own in each load);
//   step: call + nodes (node + narrow / nx), in ns and ps, the last term for the
//         step that takes nodes in a row (nx <= 16).
// The standard deviations from the times are 7 to 13% and 8 to 11%.
struct Step2Cost {
  float turn, wave, row, call, node, narrow;
};
inline Step2Cost step2_cost(int q, bool wide, bool walls) {
  if (q == 27) {
    if (wide) return walls ? Step2Cost{2540, 412, 15, 1400, 91.6f, 122} : Step2Cost{1135, 429, 16, 2760, 81, 86};
    return walls ? Step2Cost{1970, 241, 15, 3340, 48, 134} : Step2Cost{1340, 207, 14, 3250, 40.4f, 121};
  }
  if (wide) return walls ? Step2Cost{1080, 265, 0, 2590, 48.5f, 59} : Step2Cost{940, 224, 0, 2790, 43.9f, 56};
  return walls ? Step2Cost{1020, 163, 6, 3380, 25.1f, 62} : Step2Cost{610, 129, 6, 2440, 22.7f, 57};
}

// Where two steps in one pass are the faster way, and its tiles: FP64 and FP32
// storage (16-bit storage is bound by the collisions, of which this way has more)
// where the costs above say so.  They do not where a block's halo is most of its
// work: D3Q27 FP32, one pass against two single steps, 512 x 1 x 515 48 against 28 us,
// 100 x 1 x 2700 70 against 30, 4 x 4 x 16384 161 against 36, 8 x 8 x 8192 97 against 55;
// but 512 x 4 x 512 63 against 86, 64^3 20 against 26.  Of 2760 lattices and kinds, 533
// took 1.02 to 9 times as long as single steps without the costs, and 19 do with
// them (16 by 2-7%, 8 x 12 x 2953 by 20%); 174 that would gain 3% or more keep single
// steps.  (On lattices that are thin in a direction the costs scatter most, and the
// margin is 4%.)
// The costs do not know that
//   * one plane has three different ones to collide in its turn (512 x 515 x 1 38.6
//     against 28.0 us, 2048 x 2048 x 1 409 against 320);
//   * rows of one node in FP64 D3Q27 are 8 bytes of every line (1 x 512 x 513 1.7
//     times two single steps, 1 x 6291 x 140 1.5);
//   * below 2^18 nodes neither way's launch is filled (56^3 0.92-0.98, with walls
//     1.03-1.13, 32^3 1.3-1.4; D3Q15 FP32 with walls, the lightest, 1.12 at 64^3, 1.02
//     at 64 x 96 x 64, 0.84 at 128 x 64 x 64), unless rows that fill their last block
//     badly leave lanes of the single steps idle (56 x 200 x 200 0.71-0.89).
// (The kernel's offsets within a plane of population rows have 32 bits.)
inline bool step2_plan(int q, int prec, const Geom& g, bool walls, Tiles2& t) {
  if (prec > 1 || g.nz == 1) return false;
  const bool wide = prec == 0;
  if (uint64_t(g.nxy) * uint64_t(q) * (wide ? 8 : 4) >= (uint64_t(1) << 32)) return false;
  if (g.nx == 1 && wide && q == 27) return false;
  const uint64_t lanes = uint64_t((g.nx + 63) / 64) * 64 * uint64_t(g.ny) * uint64_t(g.nz);
  const bool light = q == 15 && !wide && walls;
  if (g.N < (uint64_t(1) << (light ? 19 : 18)) && (lanes < (uint64_t(1) << 20) || g.nx <= 8)) return false;

  t = step2_tiles(q, wide, walls, g);
  const Step2Cost c = step2_cost(q, wide, walls);
  const uint32_t rows = uint32_t(tile2_rows(q, wide, walls)), tiles = t.main + t.tail;
  const uint32_t blocks = tiles * ((uint32_t(g.nz) + t.zlen - 1) / t.zlen);
  uint32_t waves = t.main ? 2 * (uint32_t(g.ny) < rows ? uint32_t(g.ny) : rows) + 3 : 0;
  if (t.tail) {
    const uint32_t busy = 2 * ((((uint32_t(g.nx) & 63u) + 2) * (t.tail_rows + 2) + 63) / 64);
    if (busy > waves) waves = busy;
  }
  const double turn = double(c.turn) + double(c.wave) * waves + double(c.row) * t.tail_rows;
  const double pass = double((blocks + kSlots - 1) / kSlots) * double(t.zlen + 2) * turn;
  const double step = double(c.call) + 1e-3 * double(g.N) * (double(c.node) + (g.nx <= 16 ? double(c.narrow) / g.nx : 0.0));
  const bool thin = g.nx <= 16 || g.ny < 16 || g.nz < 16;
  return pass <= (thin ? 0.96 : 1.0) * 2 * step;
}

}  // namespace cmlbm
