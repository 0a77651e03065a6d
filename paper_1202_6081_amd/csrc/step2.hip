// Two time steps in one pass over the populations.
//
// A single step reads and writes every population once and is bound by that
// traffic (profiles of k_step: 70-77% of the HBM peak with the vector units 40%
// busy), so two steps as two passes move twice the bytes that their outcome
// needs.  k_step2 keeps the state between the two in the CU:
//
//   * a block owns a tile of 64 nodes along x (one 64-node block of the
//     population layout) by ROWS rows along y and walks it along z.  One
//     wavefront has each row of the tile and of its halo (rows y0 - 1 and
//     y0 + ROWS), and one more the two halo columns x0 - 1 and x0 + 64;
//   * at plane z every thread pulls its node and collides it (the first step of
//     tile and halo), hands the populations that move in x or y to the tile
//     through LDS, and the tile's threads collect the populations of their
//     column: those with e_z = -1 complete plane z - 1, whose second step is then
//     collided and stored; those with e_z = 0 and 1 wait in registers (FP64: in
//     LDS) for the next two planes;
//   * the loads of plane z + 1 are in flight while plane z is collided.  They
//     are waited for ahead of the stores: behind them the wait would cover the
//     stores as well, which share its counter.
//
// The arithmetic is that of k_step on the same stored values (16-bit formats
// would round between the steps as the buffer does), so the outcome is
// k_step's bit for bit.
//
// What bounds it: 512^3 D3Q27 FP32 (force field): 17.3 GB read (1.07 of one
// step's: halo rows mostly come from the XCD's L2) and 14.5 GB written, 6.5 ms
// for two steps against 10.9 ms; the same traffic with no collisions takes
// 6.0 ms, the collisions with no traffic 4.8 ms (19 collisions per 16 nodes).
// FP64 13.4 against 20.6 ms; D3Q15 FP32 3.4 against 5.3 ms, FP64 6.3 against
// 10.7 ms.  16-bit storage halves the traffic but not the collisions (5.2 against
// 5.2 ms): it keeps the single steps.
//
// Tile and registers: 8 rows are 11 wavefronts, 3 per SIMD, whose 168
// registers hold the node, the next plane's loads and the waiting populations;
// 12 rows (4 per SIMD, 128 registers) spill and, in D3Q15, where they fit, are
// 1% slower; 4 rows collide 11 nodes per 8 and are 5-18% slower.  FP64 D3Q27 has
// room for 4 rows in LDS.  With the exchange plane twice in LDS one barrier per
// plane is enough (3% faster than one plane and two barriers).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "kernels.hpp"
#include "node.hpp"
#include "step2_plan.hpp"

namespace cmlbm {
namespace {

// Directions with e_z = z, and how many of them precede a.
template <int Q>
constexpr int z_slot(int a, int z) {
  int n = 0;
  for (int b = 0; b < a; ++b) n += Lattice<Q>::e(b).z == z ? 1 : 0;
  return n;
}
template <int Q>
constexpr int z_count(int z) {
  return z_slot<Q>(Q, z);
}

// Directions that leave their column (the exchanged ones), likewise.
template <int Q>
constexpr bool moves_xy(int a) {
  return Lattice<Q>::e(a).x != 0 || Lattice<Q>::e(a).y != 0;
}
template <int Q>
constexpr int xy_slot(int a) {
  int n = 0;
  for (int b = 0; b < a; ++b) n += moves_xy<Q>(b) ? 1 : 0;
  return n;
}

// Rows of a tile and where the waiting populations are kept.
template <int Q, class ST, bool MASK>
struct Tile2 {
  static constexpr bool wide = sizeof(typename ST::T) == 8;
  static constexpr int rows = tile2_rows(Q, wide, MASK);
  static constexpr bool in_lds = wide;      // and the exchange plane once instead of twice
  static constexpr int threads = 64 * (rows + 3);
};

// FULL: nx is a multiple of 64.  FIELD: the force is a field.
template <int Q, class ST, bool MASK, bool FULL, bool FIELD>
__global__ __launch_bounds__((Tile2<Q, ST, MASK>::threads)) void k_step2(StepArgs<typename ST::R> args, Tiles2 tl) {
  using R = typename ST::R;
  using T = typename ST::T;
  constexpr uint32_t sz = uint32_t(sizeof(T)), rz = uint32_t(sizeof(R));
  constexpr int ROWS = Tile2<Q, ST, MASK>::rows;
  constexpr bool IN_LDS = Tile2<Q, ST, MASK>::in_lds;
  constexpr int kW = 66, kPlane = kW * (ROWS + 2);          // the exchange plane: tile and halo
  constexpr int kXY = xy_slot<Q>(Q), kMid = z_count<Q>(0), kUp = z_count<Q>(1);
  __shared__ T plane[IN_LDS ? 1 : 2][kXY * kPlane];
  // waiting populations (IN_LDS): e_z = 0, e_z = 1 of two planes and, with
  // walls, the node's own e_z = 1 of the plane before
  __shared__ T wait[IN_LDS ? kMid + (MASK ? 3 : 2) * kUp : 1][ROWS * 64];

  const Geom g = args.g;
  const uint32_t nx = uint32_t(g.nx), ny = uint32_t(g.ny), nz = uint32_t(g.nz);
  const uint32_t L = step_block_id();
  const uint32_t c = tl.all.div(L), t = L - c * (tl.main + tl.tail);
  const bool packed = t >= tl.main;
  const uint32_t ty = packed ? t - tl.main : tl.bx.div(t);
  const uint32_t b0 = (packed ? tl.nbx : t - ty * tl.nbx) * 64u, y0 = ty * (packed ? tl.tail_rows : uint32_t(ROWS));
  const uint32_t z0 = c * tl.zlen, zn = min(tl.zlen, nz - z0);
  const uint32_t len = min(64u, nx - b0), rows = min(packed ? tl.tail_rows : uint32_t(ROWS), ny - y0);
  // This thread's column is (xi, r) of the tile with its halo: xi 0 and len + 1
  // beside the block, r 0 and rows + 1 beside the rows; `width` columns a row in
  // the exchange plane.
  const uint32_t width = packed ? len + 2 : uint32_t(kW);
  const uint32_t lane = threadIdx.x & 63u, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint32_t r, xi;
  bool active, inner;
  if (packed) {
    r = tl.tail_width.div(threadIdx.x);
    xi = threadIdx.x - r * width;
    active = r < rows + 2;
    inner = active && r >= 1 && r <= rows && xi >= 1 && xi <= len;
  } else {
    const bool edge = wave == uint32_t(ROWS + 2);
    r = edge ? lane >> 1 : wave;
    xi = edge ? ((lane & 1u) ? len + 1 : 0u) : lane + 1;
    active = r < rows + 2 && (edge || lane < len);
    inner = !edge && active && r >= 1 && r <= rows;
  }
  const uint32_t x = xi == 0 ? (b0 == 0 ? nx - 1 : b0 - 1) : (b0 + xi - 1 >= nx ? b0 + xi - 1 - nx : b0 + xi - 1);
  const uint32_t y = r == 0 ? (y0 == 0 ? ny - 1 : y0 - 1) : (y0 + r - 1 >= ny ? y0 + r - 1 - ny : y0 + r - 1);
  // x - e_x and y - e_y, indexed [e + 1]; their byte offsets in a plane of
  // population rows (direction 0), and the direction stride there
  const uint32_t xs[3] = {x == nx - 1 ? 0 : x + 1, x, x == 0 ? nx - 1 : x - 1};
  const uint32_t ys[3] = {y == ny - 1 ? 0 : y + 1, y, y == 0 ? ny - 1 : y - 1};
  const uint32_t rowB = nx * uint32_t(Q) * sz;
  uint32_t xo[3], xl[3], yo[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    const uint32_t bb = xs[i] & ~63u;
    xo[i] = (bb * uint32_t(Q) + (xs[i] - bb)) * sz;
    xl[i] = min(64u, nx - bb) * sz;
    yo[i] = ys[i] * rowB;
  }
  const uint64_t planeB = uint64_t(rowB) * ny;              // below 2^32, as the launch checks
  const char* const fin = static_cast<const char*>(args.fin);
  auto above = [&](uint32_t z) { return z == nz - 1 ? 0u : z + 1; };
  auto below = [&](uint32_t z) { return z == 0 ? nz - 1 : z - 1; };

  // Walls: nine bits of a plane, one for each (x - e_x, y - e_y); a word of
  // three consecutive planes has the bit of direction a at wall_bit(a), for the
  // node of its middle plane.  The bytes of a plane are on their way
  // while the plane two before it is collided.
  auto wall_bit = [](int a) { return (1 - Lattice<Q>::e(a).z) * 9 + (Lattice<Q>::e(a).x + 1) * 3 + Lattice<Q>::e(a).y + 1; };
  auto load_walls = [&](uint32_t z, uint32_t(&m)[9]) {
    const __amdgpu_buffer_rsrc_t rs = array_rsrc(args.mask + uint64_t(z) * g.nxy, g.nxy);
#pragma unroll
    for (int i = 0; i < 9; ++i) m[i] = __builtin_amdgcn_raw_buffer_load_b8(rs, ys[i % 3] * nx + xs[i / 3], 0, 0);
  };
  auto wall_bits = [&](const uint32_t(&m)[9]) {
    uint32_t w = 0;
#pragma unroll
    for (int i = 0; i < 9; ++i) w |= uint32_t(m[i] != 0) << i;
    return w;
  };

  // The node's populations and force of plane z, as loaded.  solid: the wall
  // word around z.
  T raw[Q];
  R rF[3] = {R(0), R(0), R(0)};
#pragma unroll
  for (int a = 0; a < Q; ++a) raw[a] = T(0);
  auto load = [&](uint32_t z, uint32_t solid) {
    const char* const pl[3] = {fin + above(z) * planeB, fin + z * planeB, fin + below(z) * planeB};
    auto offset = [&](int ex, int ey, int a) {
      return yo[ey + 1] + xo[ex + 1] + (FULL ? 0u : uint32_t(a) * xl[ex + 1]);
    };
    if constexpr (!FULL) {
      // (27 offsets would not fit the registers over the loop)
#pragma unroll
      for (int i = 0; i < 3; ++i) asm volatile("" : "+v"(xl[i]));
    }
    auto pulled = [&](int a) {
      const Vel e = Lattice<Q>::e(a);
      return buf_load<T>(array_rsrc(pl[e.z + 1], uint32_t(planeB)), offset(e.x, e.y, a), FULL ? uint32_t(a) * 64u * sz : 0u);
    };
    if (MASK && __builtin_amdgcn_ballot_w64(solid != 0)) {
      // Wavefronts beside a wall choose the address lane by lane, with no branch
      // in the direction loop.  Nodes of the wall load nothing.  (Kept over the
      // loop, the 2 Q 64-bit offsets would not fit the registers.)
#pragma unroll
      for (int i = 0; i < 3; ++i) asm volatile("" : "+v"(xo[i]));
      if (!((solid >> wall_bit(0)) & 1u)) {
#pragma unroll
        for (int a = 0; a < Q; ++a) {
          const Vel e = Lattice<Q>::e(a);
          const int ab = opposite<Q>(a);
          const char* from = pl[e.z + 1] + (offset(e.x, e.y, a) + (FULL ? uint32_t(a) * 64u * sz : 0u));
          const char* back = pl[1] + (offset(0, 0, ab) + (FULL ? uint32_t(ab) * 64u * sz : 0u));
          raw[a] = *reinterpret_cast<const T*>(a > 0 && ((solid >> wall_bit(a)) & 1u) ? back : from);
        }
      }
    } else {
#pragma unroll
      for (int a = 0; a < Q; ++a) raw[a] = pulled(a);
    }
    if constexpr (FIELD) {
      const R* Ff = args.force.field + uint64_t(z) * g.nxy;
#pragma unroll
      for (int i = 0; i < 3; ++i) rF[i] = buf_load<R>(array_rsrc(Ff + i * g.N, g.nxy * rz), (y * nx + x) * rz, 0u);
    }
  };

  // Waiting populations of the column: of the last plane, from the one before
  // it (up0) and its own (mid), and of the next plane from the last (up1).
  R up0[Q], mid[Q], up1[Q], Fp[3] = {R(0), R(0), R(0)};
#pragma unroll
  for (int a = 0; a < Q; ++a) up0[a] = mid[a] = up1[a] = R(0);
  T own_up = T(0);                                        // (0, 0, 1) of the last plane
  const uint32_t column = (r - 1) * len + xi - 1;         // in wait (tile threads only)
  const uint32_t here = r * width + xi;                   // in the exchange plane
  uint32_t z = below(z0);
  uint32_t walls = 0, walls_next = 0;                     // words around z - 1 and z + 1
  if constexpr (MASK) {
    if (active) {
      uint32_t m[4][9];
      load_walls(below(z), m[0]);
      load_walls(z, m[1]);
      load_walls(above(z), m[2]);
      load_walls(above(above(z)), m[3]);
      const uint32_t w = wall_bits(m[0]) | (wall_bits(m[1]) << 9) | (wall_bits(m[2]) << 18);
      walls = (w << 9) & 0x7ffffffu;
      walls_next = (w >> 9) | (wall_bits(m[3]) << 18);
      load(z, w);
    }
  } else {
    if (active) load(z, 0u);
  }
  for (uint32_t p = 0; p < zn + 2; ++p) {
    // first step of plane z; the loads of the next plane are on their way
    R f[Q], F[3];
#pragma unroll
    for (int a = 0; a < Q; ++a) f[a] = decode<ST, Q>(raw[a], a);
#pragma unroll
    for (int i = 0; i < 3; ++i) F[i] = FIELD ? R(args.force.scale) * rF[i] : R(args.force.uni[i]);
    const uint32_t zx = above(z);
    const uint32_t walls_here = walls >> 9;               // planes z - 1 and z, from bit 0
    const uint32_t walls_last = walls;
    uint32_t mb[9] = {};
    if (MASK && active) load_walls(above(above(zx)), mb);
    if (active && p + 1 < zn + 2) load(zx, walls_next);
    __builtin_amdgcn_sched_barrier(0);
    collide<Q>(f, F[0], F[1], F[2], args.rates);
    T v[Q];
    encode_all<ST, Q>(f, v);
    pin_all<ST, Q>(v);
    if constexpr (MASK) {
      walls = walls_here | (((walls_next >> 9) & 511u) << 18);
      walls_next = (walls_next >> 9) | (wall_bits(mb) << 18);
    }
    T* const out = plane[IN_LDS ? 0 : p & 1u] + here;
    if constexpr (IN_LDS) __syncthreads();
    if (active) {
#pragma unroll
      for (int a = 0; a < Q; ++a)
        if (moves_xy<Q>(a)) out[xy_slot<Q>(a) * kPlane] = v[a];
    }
    __syncthreads();
    // fbar~_a of plane z from the node that direction a comes from
    auto arrive = [&](int a) {
      return moves_xy<Q>(a) ? out[xy_slot<Q>(a) * kPlane - Lattice<Q>::e(a).y * int(width) - Lattice<Q>::e(a).x] : v[a];
    };
    auto own = [&](int a) { return moves_xy<Q>(a) ? out[xy_slot<Q>(a) * kPlane] : v[a]; };
    const bool bounce = MASK && __builtin_amdgcn_ballot_w64(inner && walls_last != 0);
    // second step of the last plane
    R h[Q];
    const bool done = inner && p >= 2 && !(MASK && ((walls_last >> wall_bit(0)) & 1u));
    if (done) {
#pragma unroll
      for (int a = 0; a < Q; ++a) {
        const int ez = Lattice<Q>::e(a).z;
        if (ez < 0) {
          T w = arrive(a);
          if (MASK && bounce) {
            // from a wall: the node's own reversed population, of the last plane
            constexpr int kOwn = kMid + 2 * kUp;
            const int ab = opposite<Q>(a);
            T back;
            if constexpr (IN_LDS)
              back = wait[kOwn + z_slot<Q>(ab, 1)][column];
            else
              back = moves_xy<Q>(ab) ? plane[(p + 1) & 1u][here + xy_slot<Q>(ab) * kPlane] : own_up;
            w = ((walls_last >> wall_bit(a)) & 1u) ? back : w;
          }
          h[a] = decode<ST, Q>(w, a);
        } else if constexpr (IN_LDS) {
          h[a] = decode<ST, Q>(wait[ez == 0 ? z_slot<Q>(a, 0) : kMid + z_slot<Q>(a, 1) + int(p & 1u) * kUp][column], a);
        } else {
          h[a] = ez == 0 ? mid[a] : up0[a];
        }
      }
      collide<Q>(h, Fp[0], Fp[1], Fp[2], args.rates);
    }
    // the next plane's loads have to be here now, ahead of the stores
#pragma unroll
    for (int a = 0; a < Q; ++a) asm volatile("" : "+v"(raw[a]));
    if constexpr (FIELD) {
#pragma unroll
      for (int i = 0; i < 3; ++i) asm volatile("" : "+v"(rF[i]));
    }
    __builtin_amdgcn_sched_barrier(0);
    if (done) {
      T w[Q];
      encode_all<ST, Q>(h, w);
      const __amdgpu_buffer_rsrc_t rs = array_rsrc(static_cast<char*>(args.fout) + below(z) * planeB, uint32_t(planeB));
#pragma unroll
      for (int a = 0; a < Q; ++a) buf_store(w[a], rs, yo[1] + xo[1], uint32_t(a) * len * sz);
    }
    if (inner) {
#pragma unroll
      for (int a = 0; a < Q; ++a) {
        const int ez = Lattice<Q>::e(a).z, ab = opposite<Q>(a);
        if (ez < 0) continue;
        T w = arrive(a);
        if constexpr (IN_LDS) {
          if (ez == 0) {
            if (MASK && bounce) w = ((walls_last >> (18 + wall_bit(a) - 9)) & 1u) ? own(ab) : w;
            wait[z_slot<Q>(a, 0)][column] = w;
          } else {
            const int s = kMid + z_slot<Q>(a, 1);
            // this plane's population from a wall below
            if (MASK && bounce && ((walls_last >> (9 + wall_bit(a))) & 1u)) wait[s + int((p + 1) & 1u) * kUp][column] = own(ab);
            wait[s + int(p & 1u) * kUp][column] = w;
            if constexpr (MASK) wait[s + 2 * kUp][column] = own(a);
          }
        } else {
          if (ez == 0) {
            if (MASK && bounce) w = ((walls_last >> (18 + wall_bit(a) - 9)) & 1u) ? own(ab) : w;
            mid[a] = decode<ST, Q>(w, a);
          } else {
            up0[a] = up1[a];
            if (MASK && bounce) up0[a] = ((walls_last >> (9 + wall_bit(a))) & 1u) ? decode<ST, Q>(own(ab), a) : up0[a];
            up1[a] = decode<ST, Q>(w, a);
          }
        }
        if (MASK && !moves_xy<Q>(a) && ez > 0) own_up = v[a];
      }
    }
#pragma unroll
    for (int i = 0; i < 3; ++i) Fp[i] = F[i];
    z = zx;
  }
}

template <int Q, class ST, bool MASK, bool FULL>
void launch_tiles(const StepArgs<typename ST::R>& a, const Tiles2& t, dim3 grid, hipStream_t st) {
  const dim3 block(Tile2<Q, ST, MASK>::threads);
  if (a.force.field)
    hipLaunchKernelGGL((k_step2<Q, ST, MASK, FULL, true>), grid, block, 0, st, a, t);
  else
    hipLaunchKernelGGL((k_step2<Q, ST, MASK, FULL, false>), grid, block, 0, st, a, t);
}

template <int Q, class ST, bool MASK>
hipError_t step2_impl(const StepArgs<typename ST::R>& a, const Tiles2& t, hipStream_t st) {
  const uint32_t len = uint32_t(a.g.nx) & 63u, nz = uint32_t(a.g.nz);
  const dim3 grid((t.main + t.tail) * ((nz + t.zlen - 1) / t.zlen));
  if (len == 0)
    launch_tiles<Q, ST, MASK, true>(a, t, grid, st);
  else
    launch_tiles<Q, ST, MASK, false>(a, t, grid, st);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_step2(int q, int prec, const StepArgs<double>& a64, const StepArgs<float>& a32, const Tiles2& t,
                        hipStream_t st) {
  if (prec == 0) {
    if (q == 27) return a64.mask ? step2_impl<27, StF64, true>(a64, t, st) : step2_impl<27, StF64, false>(a64, t, st);
    return a64.mask ? step2_impl<15, StF64, true>(a64, t, st) : step2_impl<15, StF64, false>(a64, t, st);
  }
  if (q == 27) return a32.mask ? step2_impl<27, StF32, true>(a32, t, st) : step2_impl<27, StF32, false>(a32, t, st);
  return a32.mask ? step2_impl<15, StF32, true>(a32, t, st) : step2_impl<15, StF32, false>(a32, t, st);
}

}  // namespace cmlbm
