// Host build of the library's launch rules, for the tests: which lattices take
// two steps in one pass and by what tiles, which take their nodes in a row, and the
// adjoint's launch form.
#include <cstdint>

#include "step2_plan.hpp"

namespace {

cmlbm::Geom geom(int nx, int ny, int nz) {
  cmlbm::Geom g{};
  g.nx = nx;
  g.ny = ny;
  g.nz = nz;
  g.nxy = uint32_t(nx) * uint32_t(ny);
  g.N = uint64_t(g.nxy) * uint64_t(nz);
  return g;
}

}  // namespace

extern "C" {

// Whether cmlbm_run takes two steps per pass; out: main tiles, tail tiles, rows
// of a tail tile, planes per block.
int hp_step2_plan(int q, int prec, int nx, int ny, int nz, int walls, uint32_t* out) {
  cmlbm::Tiles2 t{};
  const bool pays = cmlbm::step2_plan(q, prec, geom(nx, ny, nz), walls != 0, t);
  out[0] = t.main;
  out[1] = t.tail;
  out[2] = t.tail_rows;
  out[3] = t.zlen;
  return pays ? 1 : 0;
}

uint32_t hp_run_length(uint32_t tiles, uint32_t nz) { return cmlbm::run_length(tiles, nz); }

// Whether a step without totals takes the nodes in a row.
int hp_thin(int q, int bytes, int nx, int ny, int nz, int walls) {
  return cmlbm::thin_pays(q, bytes, walls != 0, geom(nx, ny, nz)) ? 1 : 0;
}

// The adjoint step's launch; out: blocks, nodes of a row segment, 1 in the form
// with a wavefront per segment.
void hp_adjoint(int q, int prec, int nx, int ny, int nz, int* out) {
  const cmlbm::Geom g = geom(nx, ny, nz);
  out[0] = cmlbm::adjoint_blocks(g);
  out[1] = cmlbm::adjoint_block(g);
  out[2] = cmlbm::adjoint_split(q, prec == 0, g) ? 1 : 0;
}

}  // extern "C"
