// Per-node device code that the step, in-place, read-out and adjoint kernels
// share: storage formats, lattice geometry, the pull, the collision call and
// the blocked-row store.  (The population layout and the pull are described in
// kernels.hip.)
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "collide_d3q15.hpp"
#include "collide_d3q27.hpp"
#include "kernels.hpp"

namespace cmlbm {

// ---------------------------------------------------------------------------
// Storage policies
// ---------------------------------------------------------------------------
struct StF64 {
  using T = double;
  using R = double;
  static constexpr bool dev = false;
};
struct StF32 {
  using T = float;
  using R = float;
  static constexpr bool dev = false;
};
struct StF16 {
  using T = _Float16;
  using R = float;
  static constexpr bool dev = true;
};
struct StBF16 {
  using T = __bf16;
  using R = float;
  static constexpr bool dev = true;
};

template <class ST, int Q>
__device__ __forceinline__ typename ST::R decode(typename ST::T v, int a) {
  using R = typename ST::R;
  if constexpr (ST::dev)
    return R(weight<Q>(a)) + static_cast<R>(v);
  else
    return v;
}

template <class ST, int Q>
__device__ __forceinline__ typename ST::T encode(typename ST::R v, int a) {
  using R = typename ST::R;
  if constexpr (ST::dev)
    return static_cast<typename ST::T>(v - R(weight<Q>(a)));
  else
    return v;
}

// All Q stored values of one node (the hot paths): as encode, with FP16
// deviations converted two at a time by the packed conversion (the same
// round-to-nearest-even of each FP32 value; measured as fast as or faster than
// the mixed-precision multiply-add-and-round the compiler otherwise forms).
template <class ST, int Q>
__device__ __forceinline__ void encode_all(const typename ST::R (&f)[Q], typename ST::T (&v)[Q]) {
  using R = typename ST::R;
  if constexpr (ST::dev && __is_same(typename ST::T, _Float16)) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
#pragma unroll
    for (int a = 0; a + 1 < Q; a += 2) {
      const f16x2 h = __builtin_convertvector((f32x2){f[a] - R(weight<Q>(a)), f[a + 1] - R(weight<Q>(a + 1))}, f16x2);
      v[a] = h.x;
      v[a + 1] = h.y;
    }
    if constexpr (Q & 1) v[Q - 1] = encode<ST, Q>(f[Q - 1], Q - 1);
  } else {
#pragma unroll
    for (int a = 0; a < Q; ++a) v[a] = encode<ST, Q>(f[a], a);
  }
}

// Marks the encoded populations as computed here (an empty statement per
// register: no instruction is emitted), so that the compiler does not sink the
// end of the collision into later branches, where it would fuse its multiplies
// and adds differently.  FP16 deviations are pinned in the pairs that the
// packed conversion writes, so that they stay packed.
template <class ST, int Q>
__device__ __forceinline__ void pin_all(typename ST::T (&v)[Q]) {
  using T = typename ST::T;
  if constexpr (ST::dev && __is_same(T, _Float16)) {
#pragma unroll
    for (int a = 0; a + 1 < Q; a += 2) {
      uint32_t p = uint32_t(__builtin_bit_cast(uint16_t, v[a])) | (uint32_t(__builtin_bit_cast(uint16_t, v[a + 1])) << 16);
      asm volatile("" : "+v"(p));
      v[a] = __builtin_bit_cast(T, uint16_t(p));
      v[a + 1] = __builtin_bit_cast(T, uint16_t(p >> 16));
    }
    if constexpr (Q & 1) asm volatile("" : "+v"(v[Q - 1]));
  } else {
#pragma unroll
    for (int a = 0; a < Q; ++a) asm volatile("" : "+v"(v[a]));
  }
}

// Element idx of an array whose byte size fits in 32 bits: a uniform base
// pointer plus a 32-bit byte offset, which maps onto the scalar-base form of
// the global load instructions.
template <typename T>
__device__ __forceinline__ T ld32(const T* base, uint32_t idx) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + idx * uint32_t(sizeof(T)));
}

// ---------------------------------------------------------------------------
// Geometry
// ---------------------------------------------------------------------------
struct Coord {
  int x, y, z;
};

// Node x of row `row` (row = z*ny + y).
__device__ __forceinline__ Coord row_coord(const RowMap& rm, const Geom& g, uint32_t row, uint32_t x) {
  const uint32_t z = rm.ny.div(row);
  return {int(x), int(row - z * uint32_t(g.ny)), int(z)};
}

__device__ __forceinline__ Coord coord_of(const Geom& g, uint32_t n) {
  const uint32_t z = n / g.nxy;
  const uint32_t r = n - z * g.nxy;
  const uint32_t y = r / uint32_t(g.nx);
  return {int(r - y * uint32_t(g.nx)), int(y), int(z)};
}

// Offset of (a, x) inside a row of the blocked population layout.
template <int Q>
__device__ __forceinline__ uint32_t in_row(uint32_t nx, int a, uint32_t x) {
  const uint32_t b0 = x & ~63u;
  const uint32_t len = min(64u, nx - b0);
  return b0 * uint32_t(Q) + uint32_t(a) * len + (x - b0);
}

// Source rows and x positions of the pull (s = +1: x - e) or of the reverse
// gather (s = -1: x + e), periodic.
struct Stencil {
  uint32_t row[3][3];   // row index (z - s*ez)*ny + (y - s*ey), indexed [ey+1][ez+1]
  uint32_t xs[3];       // x - s*ex, indexed [ex+1]
  __device__ __forceinline__ Stencil(const Geom& g, Coord c, int s) {
    const int xm = c.x == 0 ? g.nx - 1 : c.x - 1, xp = c.x == g.nx - 1 ? 0 : c.x + 1;
    const int ym = c.y == 0 ? g.ny - 1 : c.y - 1, yp = c.y == g.ny - 1 ? 0 : c.y + 1;
    const int zm = c.z == 0 ? g.nz - 1 : c.z - 1, zp = c.z == g.nz - 1 ? 0 : c.z + 1;
    const int X[3] = {s > 0 ? xp : xm, c.x, s > 0 ? xm : xp};
    const int Y[3] = {s > 0 ? yp : ym, c.y, s > 0 ? ym : yp};
    const int Z[3] = {s > 0 ? zp : zm, c.z, s > 0 ? zm : zp};
#pragma unroll
    for (int i = 0; i < 3; ++i) xs[i] = uint32_t(X[i]);
#pragma unroll
    for (int j = 0; j < 3; ++j)
#pragma unroll
      for (int k = 0; k < 3; ++k) row[j][k] = uint32_t(Z[k]) * uint32_t(g.ny) + uint32_t(Y[j]);
  }
  __device__ __forceinline__ uint32_t node(Vel e, uint32_t nx) const {
    return row[e.y + 1][e.z + 1] * nx + xs[e.x + 1];
  }
};

// Raw buffer access: a resource over one row (base in SGPRs, size bound) plus a
// 32-bit byte offset.  Stores past the bound are dropped by the hardware.
// Word 3 = 0x00020000 is the raw-buffer descriptor of the gfx9 family.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t array_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, int(bytes), 0x00020000);
}

// Load through a buffer resource: base in scalar registers, 32-bit per-lane
// and wave-uniform byte offsets, so that no 64-bit per-lane address is formed
// (with plain pointers the compiler factors the per-lane offset out of a group
// of loads and adds each uniform part back with a 64-bit vector add).
template <typename T>
__device__ __forceinline__ T buf_load(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  if constexpr (sizeof(T) == 4) {
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
  } else if constexpr (sizeof(T) == 8) {
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, voff, soff, 0));
  } else {
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b16(r, voff, soff, 0));
  }
}

// Element of a byte offset from a uniform base (scalar-base load form).
template <typename T>
__device__ __forceinline__ T ldb(const void* base, uint32_t byte_off) {
  return *reinterpret_cast<const T*>(static_cast<const char*>(base) + byte_off);
}

// Pull the pre-collision populations of node (row0, x) from the blocked
// post-collision buffer `fin`.  With MASK, a link whose source is solid takes
// the node's own reversed population (half-way bounce-back).
//
// WAVE: the caller guarantees that a wavefront covers one 64-node block of
// one row (block size a multiple of 64, one row per block).  Then the block
// start and length of the node's own x are wave-uniform, and the byte offset
// of direction a splits into a per-lane part and a scalar part a*len, folded
// into the base pointer; only the x-neighbour directions keep a per-lane
// multiply-add.  BUF: load through buffer resources over the source rows
// (where the caller's register pressure makes the compiler rebuild 64-bit
// per-lane addresses for the plain loads).
template <int Q, class ST, bool MASK, bool WAVE = false, bool BUF = false>
__device__ __forceinline__ void pull(const typename ST::T* __restrict__ fin, const Geom& g, const uint8_t* mask,
                                     const Stencil& st, uint32_t row0, uint32_t x, typename ST::R (&f)[Q]) {
  using T = typename ST::T;
  const uint64_t rowQ = uint64_t(g.nx) * Q;
  if constexpr (WAVE) {
    constexpr uint32_t sz = uint32_t(sizeof(T));
    const uint32_t nx = uint32_t(g.nx);
    const uint32_t b0 = __builtin_amdgcn_readfirstlane(x & ~63u);
    const uint32_t lenB = min(64u, nx - b0) * sz;            // wave-uniform
    const uint32_t cbase = (b0 * uint32_t(Q) + (x - b0)) * sz;
    uint32_t nbase[3], nlen[3];
#pragma unroll
    for (int i = 0; i < 3; i += 2) {
      const uint32_t xs = st.xs[i];
      const uint32_t bb = xs & ~63u;
      nbase[i] = (bb * uint32_t(Q) + (xs - bb)) * sz;
      nlen[i] = min(64u, nx - bb) * sz;
    }
    const T* own = fin + uint64_t(row0) * rowQ;
    // bit a: x - e_a solid.  One round of mask loads ahead of the population
    // loads, which then issue back to back (a mask byte tested per direction
    // made each population load wait for its own mask load).  Direction 0
    // reads the node's own slot 0 either way.
    uint32_t solid = 0;
    if constexpr (MASK) {
#pragma unroll
      for (int a = 1; a < Q; ++a) solid |= uint32_t(mask[st.node(Lattice<Q>::e(a), nx)] != 0) << a;
    }
    // When every block of a row is full (nx a multiple of 64), the blocks of
    // the x-neighbours have the same direction stride lenB, and that part of
    // their offsets is wave-uniform too.
    auto gather = [&](auto full) {
#pragma unroll
      for (int a = 0; a < Q; ++a) {
        const Vel e = Lattice<Q>::e(a);
        const T* rp = fin + uint64_t(st.row[e.y + 1][e.z + 1]) * rowQ;
        T v;
        if constexpr (BUF) {
          static_assert(!MASK, "a per-lane choice of row must not select the descriptor");
          const uint32_t rowB = uint32_t(rowQ) * sz;
          if (e.x == 0)
            v = buf_load<T>(array_rsrc(rp, rowB), cbase, uint32_t(a) * lenB);
          else if constexpr (decltype(full)::value)
            v = buf_load<T>(array_rsrc(rp, rowB), nbase[e.x + 1], uint32_t(a) * lenB);
          else
            v = buf_load<T>(array_rsrc(rp, rowB), nbase[e.x + 1] + uint32_t(a) * nlen[e.x + 1], 0u);
        } else {
          if (MASK && ((solid >> a) & 1u))
            v = ldb<T>(reinterpret_cast<const char*>(own) + uint32_t(opposite<Q>(a)) * lenB, cbase);
          else if (e.x == 0)
            v = ldb<T>(reinterpret_cast<const char*>(rp) + uint32_t(a) * lenB, cbase);
          else if constexpr (decltype(full)::value)
            v = ldb<T>(reinterpret_cast<const char*>(rp) + uint32_t(a) * lenB, nbase[e.x + 1]);
          else
            v = ldb<T>(rp, nbase[e.x + 1] + uint32_t(a) * nlen[e.x + 1]);
        }
        f[a] = decode<ST, Q>(v, a);
      }
    };
    if ((nx & 63u) == 0)
      gather(std::true_type{});
    else
      gather(std::false_type{});
  } else {
    uint32_t solid = 0;   // bit a: x - e_a solid, as above
    if constexpr (MASK) {
#pragma unroll
      for (int a = 1; a < Q; ++a) solid |= uint32_t(mask[st.node(Lattice<Q>::e(a), uint32_t(g.nx))] != 0) << a;
    }
#pragma unroll
    for (int a = 0; a < Q; ++a) {
      const Vel e = Lattice<Q>::e(a);
      const T* rp = fin + uint64_t(st.row[e.y + 1][e.z + 1]) * rowQ;
      T v;
      if constexpr (MASK) {
        if ((solid >> a) & 1u)
          v = ld32(fin + uint64_t(row0) * rowQ, in_row<Q>(uint32_t(g.nx), opposite<Q>(a), x));
        else
          v = ld32(rp, in_row<Q>(uint32_t(g.nx), a, st.xs[e.x + 1]));
      } else {
        v = ld32(rp, in_row<Q>(uint32_t(g.nx), a, st.xs[e.x + 1]));
      }
      f[a] = decode<ST, Q>(v, a);
    }
  }
}

template <typename R, typename FT>
__device__ __forceinline__ void force_at(const ForceArgs<FT>& F, uint64_t N, uint32_t node, R& Fx, R& Fy, R& Fz) {
  if (F.field) {
    Fx = R(F.scale) * R(F.field[node]);
    Fy = R(F.scale) * R(F.field[N + node]);
    Fz = R(F.scale) * R(F.field[2 * N + node]);
  } else {
    Fx = R(F.uni[0]);
    Fy = R(F.uni[1]);
    Fz = R(F.uni[2]);
  }
}

template <int Q, typename R>
__device__ __forceinline__ void collide(R (&f)[Q], R Fx, R Fy, R Fz, const Rates<R>& p) {
  if constexpr (Q == 27) {
    R m[27];
#pragma unroll
    for (int a = 0; a < 27; ++a) m[cube27(a)] = f[a];
    collide27(m, Fx, Fy, Fz, p);
#pragma unroll
    for (int a = 0; a < 27; ++a) f[a] = m[cube27(a)];
  } else {
    collide15(f, Fx, Fy, Fz, p);
  }
}

// ---------------------------------------------------------------------------
// The fused pull-stream + collide + force step
// ---------------------------------------------------------------------------
// Launch shape: one block covers up to CMLBM_STEP_BLOCK consecutive x of one row, so
// every row base is uniform across the block.  Hardware hands consecutive
// block ids to the eight XCDs in turn; with CMLBM_XCD_REMAP the block id is
// permuted so that each XCD receives a contiguous run of rows, keeping a row's
// segments and their shared edge cache lines in one XCD's L2.
#ifndef CMLBM_STEP_BLOCK
#define CMLBM_STEP_BLOCK 256
#endif
#ifndef CMLBM_XCD_REMAP
#define CMLBM_XCD_REMAP 1
#endif
#ifndef CMLBM_NT_STORE
#define CMLBM_NT_STORE 1
#endif
// In-place scatter phase without walls: 0 = shifted stores, 1 = aligned stores
// for 16-bit storage only (measured: 16-bit 2-5% faster aligned, FP32 2% slower
// from the block barrier, FP64 even), 2 = aligned stores always.
#ifndef CMLBM_ALIGNED_SCATTER
#define CMLBM_ALIGNED_SCATTER 1
#endif

__device__ __forceinline__ uint32_t step_block_id() {
  uint32_t L = blockIdx.x;
#if CMLBM_XCD_REMAP
  const uint32_t G = gridDim.x, per = G >> 3;
  if (L < (per << 3)) L = (L & 7u) * per + (L >> 3);
#endif
  return L;
}

constexpr int kStoreAux = CMLBM_NT_STORE ? 2 : 0;   // 2: nontemporal (streaming) store
// A per-lane byte offset past every row's bound: the raw buffer store drops it.
constexpr uint32_t kDropOffset = 0x80000000u;

// voff: per-lane byte offset; soff: wave-uniform byte offset; AUX: cache
// policy bits (kStoreAux streams past the caches; 0 keeps the line).
template <int AUX = kStoreAux, typename T>
__device__ __forceinline__ void buf_store(T v, __amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  if constexpr (sizeof(T) == 4) {
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, voff, soff, AUX);
  } else if constexpr (sizeof(T) == 8) {
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u32x2, v), r, voff, soff, AUX);
  } else {
    __builtin_amdgcn_raw_buffer_store_b16(__builtin_bit_cast(uint16_t, v), r, voff, soff, AUX);
  }
}

// FP64 mass and momentum of one node's pre-collision populations, rho u
// including F/2 (Eqs. densitycalculation, velocitycalculation).
template <int Q, typename R>
__device__ __forceinline__ void add_node_totals(const R (&f)[Q], R Fx, R Fy, R Fz, double (&acc)[4]) {
  double rho = 0, jx = 0.5 * double(Fx), jy = 0.5 * double(Fy), jz = 0.5 * double(Fz);
#pragma unroll
  for (int a = 0; a < Q; ++a) {
    const Vel e = Lattice<Q>::e(a);
    const double v = double(f[a]);
    rho += v;
    if (e.x > 0) jx += v;
    if (e.x < 0) jx -= v;
    if (e.y > 0) jy += v;
    if (e.y < 0) jy -= v;
    if (e.z > 0) jz += v;
    if (e.z < 0) jz -= v;
  }
  acc[0] += rho;
  acc[1] += jx;
  acc[2] += jy;
  acc[3] += jz;
}

template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double* sh /* [NV][8] */);

// Body force at node (row, x), row = z*ny + y uniform across the wavefront.
template <typename R>
__device__ __forceinline__ void force_row(const StepArgs<R>& args, const Geom& g, uint32_t row, uint32_t x, R& Fx,
                                          R& Fy, R& Fz) {
  if (args.force.field) {
    const R* Ff = args.force.field + uint64_t(row) * uint32_t(g.nx);
    const R sc = R(args.force.scale);
    Fx = sc * ld32(Ff, x);
    Fy = sc * ld32(Ff + g.N, x);
    Fz = sc * ld32(Ff + 2 * g.N, x);
  } else {
    Fx = R(args.force.uni[0]);
    Fy = R(args.force.uni[1]);
    Fz = R(args.force.uni[2]);
  }
}

// The two ends of one node's update: pull + force, and the store.
template <int Q, class ST, bool MASK>
__device__ __forceinline__ void load_node(const StepArgs<typename ST::R>& args, const Geom& g, uint32_t row,
                                          uint32_t x, typename ST::R (&f)[Q], typename ST::R& Fx,
                                          typename ST::R& Fy, typename ST::R& Fz) {
  const Coord c = row_coord(args.rm, g, row, x);
  const Stencil st(g, c, +1);
  pull<Q, ST, MASK, true>(static_cast<const typename ST::T*>(args.fin), g, args.mask, st, row, x, f);
  force_row(args, g, row, x, Fx, Fy, Fz);
}

// Store of node (row, x); a wavefront covers one 64-node block of the row, so
// the direction stride of the blocked layout is wave-uniform (scalar offset).
template <int Q, class ST>
__device__ __forceinline__ void store_node(const StepArgs<typename ST::R>& args, const Geom& g, uint32_t row,
                                           uint32_t x, const typename ST::R (&f)[Q]) {
  using T = typename ST::T;
  constexpr uint32_t sz = uint32_t(sizeof(T));
  const uint32_t nx = uint32_t(g.nx);
  const uint32_t rowQ = nx * uint32_t(Q);
  const __amdgpu_buffer_rsrc_t rs = array_rsrc(static_cast<T*>(args.fout) + uint64_t(row) * rowQ, rowQ * sz);
  const uint32_t b0 = __builtin_amdgcn_readfirstlane(x & ~63u);
  const uint32_t lenB = min(64u, nx - b0) * sz;
  const uint32_t cbase = (b0 * uint32_t(Q) + (x - b0)) * sz;
  T v[Q];
  encode_all<ST, Q>(f, v);
#pragma unroll
  for (int a = 0; a < Q; ++a) buf_store(v[a], rs, cbase, uint32_t(a) * lenB);
}

}  // namespace cmlbm
