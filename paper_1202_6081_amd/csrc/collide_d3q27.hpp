// D3Q27 central-moment collision with forcing, and its hand-written adjoint.
//
// The cascaded collision of Premnath & Banerjee (arXiv:1202.6081, Sec. 7 and
// Sec. 8) produces post-collision populations whose central moments about the
// local velocity u are the pre-collision ones relaxed toward the factorized
// attractors.  On D3Q27 the central moments of all 27 monomials
// (e_x-u_x)^a (e_y-u_y)^b (e_z-u_z)^c, a, b, c in {0, 1, 2}, factorize per axis,
// so the raw-moment sums of Appendix B followed by the binomial shift of Sec. 6
// become three passes of 3-point transforms over a 3x3x3 cube, and the return
// to populations (the K g + S rows of Sec. 8) becomes three inverse passes.
//
// Source term (Sec. 5, Eq. discretecentralsources): S changes only the three
// first-order central moments, by F.  Adding S to fbar therefore sets the
// first central moments to -F/2 + F = F/2, which the collision conserves; the
// velocity includes F/2 (Eq. velocitycalculation).
//
// Cube layout: m[a*9 + b*3 + c] holds the population with e = (a-1, b-1, c-1)
// before the forward passes and the central moment with exponents (a, b, c)
// after them.
#pragma once

#include <type_traits>
#include <utility>

#include "lattice.hpp"

namespace cmlbm {

constexpr int K3(int a, int b, int c) { return a * 9 + b * 3 + c; }

// Relaxation rates indexed by the paper's kernel number b = 4..26 (entries
// 0..3 unused): w[b] = omega_b and wc[b] = 1 - omega_b.
template <typename R>
struct Rates {
  R w[27];
  R wc[27];
  // 0: factorized attractors as the literal products of post-collision
  // second moments (kxx kyy, kxx kyy kzz); 1: per unit mass, rho (kxx/rho)
  // (kyy/rho) and rho (kxx/rho)(kyy/rho)(kzz/rho).
  int per_mass;
};

// In a function that starts with this, the multiply-adds are those written
// (fma_r) and no others.  Several sums of the collision and of its adjoint have two
// products of which either could be fused; left to the compiler, the choice, and with it
// the rounding, depends on the code around them, and the kernels that run the collision (two
// buffers, in place, two steps in one pass) or the adjoint (with running sums or with
// their factors kept) would not agree bit for bit.
#define CMLBM_FMA_AS_WRITTEN _Pragma("clang fp contract(off)")

template <int I>
using Ic = std::integral_constant<int, I>;

template <class Fn, int... I>
CMLBM_HD void unroll_impl(Fn&& fn, std::integer_sequence<int, I...>) {
  (fn(Ic<I>{}), ...);
}

// fn(Ic<0>{}), ..., fn(Ic<N-1>{}): the index is a compile-time constant.
template <int N, class Fn>
CMLBM_HD void unroll(Fn&& fn) {
  unroll_impl(fn, std::make_integer_sequence<int, N>{});
}

// -- 3-point transforms along one axis --------------------------------------
// Populations (p_-, p_0, p_+) -> central moments (k0, k1, k2) about u:
// k_n = sum_e p_e (e - u)^n.
template <typename R>
CMLBM_HD void fwd_line(R& a, R& b, R& c, R u) {
  CMLBM_FMA_AS_WRITTEN
  const R k0 = a + b + c;
  const R d = c - a;
  const R k1 = fma_r(-u, k0, d);
  const R k2 = fma_r(-u, d + k1, c + a);
  a = k0;
  b = k1;
  c = k2;
}

// Central moments (m0, m1, m2) about u -> populations (p_-, p_0, p_+).
// (p_+ is formed as (r2 + r1)/2: the shorter p_- + r1 measured ten times the
// FP32 error on a steady duct flow, 2.1e-3 against 1.8e-4 relative L2 after
// 4e5 steps, the rounding errors of a steady state repeating every step.)
// With HALVE = false, p_- and p_+ come out doubled (r2 -+ r1): the caller
// applies the power-of-two factors of all passes at once (exact, so the
// result is the same bit for bit).
template <bool HALVE = true, typename R>
CMLBM_HD void inv_line(R& a, R& b, R& c, R u) {
  const R m0 = a, m1 = b, m2 = c;
  const R r1 = m1 + u * m0;              // raw first moment
  const R r2 = m2 + u * (m1 + r1);       // raw second moment
  if constexpr (HALVE) {
    a = R(0.5) * (r2 - r1);
    c = R(0.5) * (r2 + r1);
  } else {
    a = r2 - r1;
    c = r2 + r1;
  }
  b = m0 - r2;
}

// inv_line with its multiply-adds as written.
template <bool HALVE, typename R>
CMLBM_HD void inv_line_as_written(R& a, R& b, R& c, R u) {
  CMLBM_FMA_AS_WRITTEN
  const R m0 = a, m1 = b, m2 = c;
  const R r1 = fma_r(u, m0, m1);
  const R r2 = fma_r(u, m1 + r1, m2);
  a = HALVE ? R(0.5) * (r2 - r1) : r2 - r1;
  b = m0 - r2;
  c = HALVE ? R(0.5) * (r2 + r1) : r2 + r1;
}

// Adjoint of inv_line: (m0, r1) are the forward input and the raw first moment, m1r1 =
// m1 + r1, (ga, gb, gc) hold the adjoints of the outputs on entry and of the
// inputs on exit; adds to gu.
template <typename R>
CMLBM_HD void inv_line_adj(R m0, R m1r1, R u, R& ga, R& gb, R& gc, R& gu) {
  CMLBM_FMA_AS_WRITTEN
  const R pa = ga, pb = gb, pc = gc;
  const R gr2 = fma_r(R(0.5), pa + pc, -pb);
  const R gr1 = fma_r(R(0.5), pc - pa, gr2 * u);
  gu = fma_r(gr2, m1r1, gu);
  gu = fma_r(gr1, m0, gu);
  ga = fma_r(gr1, u, pb);
  gb = fma_r(gr2, u, gr1);
  gc = gr2;
}

// The forward transform of the step in two halves: raw moments first, one
// axis at a time, (p_-, p_0, p_+) -> (sum, p_+ - p_-, p_+ + p_-) (3 operations
// per line), then the binomial shift to central moments about u, one axis at a
// time (the shifts along different axes act on different exponents and
// commute).  Density and momentum are then the raw moments 000, 100, 010, 001.
template <typename R>
CMLBM_HD void raw_line(R& a, R& b, R& c) {
  const R s2 = c + a, s1 = c - a;
  a = s2 + b;
  b = s1;
  c = s2;
}

// Raw (r0, r1, r2) along an axis -> central (r0, r1 - u r0, r2 - 2 u r1 + u^2 r0).
template <typename R>
CMLBM_HD void shift_line(R a, R& b, R& c, R u) {
  CMLBM_FMA_AS_WRITTEN
  const R k1 = fma_r(-u, a, b);
  c = fma_r(-u, b + k1, c);
  b = k1;
}

// Inverse of shift_line: central (k0, k1, k2) about u -> raw (r0, r1, r2).
template <typename R>
CMLBM_HD void unshift_line(R a, R& b, R& c, R u) {
  CMLBM_FMA_AS_WRITTEN
  const R r1 = fma_r(u, a, b);
  c = fma_r(u, r1 + b, c);
  b = r1;
}

// Adjoint of shift_line from its output (k0, k1): (g0, g1, g2) hold the
// adjoints of (k0, k1, k2) on entry and of (r0, r1, r2) on exit; with
// k1 = r1 - u r0 and k2 = r2 - u (r1 + k1), dk2/du = -2 k1 and dk1/du = -k0.
// SECOND: which of the two products is fused.
template <bool SECOND, typename R>
CMLBM_HD void shift_line_adj(R k0, R k1, R u, R& g0, R& g1, R g2, R& gu) {
  CMLBM_FMA_AS_WRITTEN
  const R k2 = R(2) * k1;
  gu -= SECOND ? fma_r(k2, g2, k0 * g1) : fma_r(k0, g1, k2 * g2);
  const R t = fma_r(-u, g2, g1);
  g0 = fma_r(-u, t, g0);
  g1 = fma_r(-u, g2, t);
}

// Adjoint of raw_line (a linear map): (ga, gb, gc) hold the adjoints of
// (sum, p_+ - p_-, p_+ + p_-) on entry and of (p_-, p_0, p_+) on exit.
template <typename R>
CMLBM_HD void raw_line_adj(R& ga, R& gb, R& gc) {
  const R g0 = ga, g1 = gb, g2 = gc;
  const R t = g0 + g2;
  ga = t - g1;
  gb = g0;
  gc = t + g1;
}

// Base index and stride of line l (0..8) along an axis (0 = x, 1 = y, 2 = z).
template <int AXIS>
CMLBM_HDC int line_base(int l) {
  return AXIS == 2 ? (l / 3) * 9 + (l % 3) * 3 : AXIS == 1 ? (l / 3) * 9 + (l % 3) : l;
}
template <int AXIS>
CMLBM_HDC int line_stride() {
  return AXIS == 0 ? 9 : AXIS == 1 ? 3 : 1;
}

template <int AXIS, typename R>
CMLBM_HD void fwd_pass(R (&m)[27], R u) {
  constexpr int S = line_stride<AXIS>();
#pragma unroll
  for (int l = 0; l < 9; ++l) {
    const int o = line_base<AXIS>(l);
    fwd_line(m[o], m[o + S], m[o + 2 * S], u);
  }
}

template <int AXIS, typename R>
CMLBM_HD void raw_pass(R (&m)[27]) {
  constexpr int S = line_stride<AXIS>();
#pragma unroll
  for (int l = 0; l < 9; ++l) {
    const int o = line_base<AXIS>(l);
    raw_line(m[o], m[o + S], m[o + 2 * S]);
  }
}

template <int AXIS, typename R>
CMLBM_HD void shift_pass(R (&m)[27], R u) {
  constexpr int S = line_stride<AXIS>();
#pragma unroll
  for (int l = 0; l < 9; ++l) {
    const int o = line_base<AXIS>(l);
    shift_line(m[o], m[o + S], m[o + 2 * S], u);
  }
}

template <int AXIS, typename R>
CMLBM_HD void unshift_pass(R (&m)[27], R u) {
  constexpr int S = line_stride<AXIS>();
#pragma unroll
  for (int l = 0; l < 9; ++l) {
    const int o = line_base<AXIS>(l);
    unshift_line(m[o], m[o + S], m[o + 2 * S], u);
  }
}

// m: the output of shift_pass<AXIS> (central moments along AXIS).  The sum for gu has
// two products a line, neither of them needed elsewhere: which one is fused is free, and
// fixed by the bits of SECOND (from the first line up) so that results keep their bits.
template <int AXIS, typename R>
CMLBM_HD void shift_pass_adj(const R (&m)[27], R u, R (&g)[27], R& gu) {
  constexpr int S = line_stride<AXIS>();
  constexpr unsigned SECOND = AXIS == 2 ? 0xbe : AXIS == 1 ? 0x9e : 0xb0;
  unroll<9>([&](auto l) {
    constexpr int o = line_base<AXIS>(decltype(l)::value);
    shift_line_adj<(SECOND >> decltype(l)::value & 1) != 0>(m[o], m[o + S], u, g[o], g[o + S], g[o + 2 * S], gu);
  });
}

template <int AXIS, typename R>
CMLBM_HD void raw_pass_adj(R (&g)[27]) {
  constexpr int S = line_stride<AXIS>();
#pragma unroll
  for (int l = 0; l < 9; ++l) {
    const int o = line_base<AXIS>(l);
    raw_line_adj(g[o], g[o + S], g[o + 2 * S]);
  }
}

template <int AXIS, bool HALVE = true, typename R>
CMLBM_HD void inv_pass(R (&m)[27], R u) {
  constexpr int S = line_stride<AXIS>();
#pragma unroll
  for (int l = 0; l < 9; ++l) {
    const int o = line_base<AXIS>(l);
    inv_line<HALVE>(m[o], m[o + S], m[o + 2 * S], u);
  }
}

template <int AXIS, bool HALVE = true, typename R>
CMLBM_HD void inv_pass_as_written(R (&m)[27], R u) {
  constexpr int S = line_stride<AXIS>();
#pragma unroll
  for (int l = 0; l < 9; ++l) {
    const int o = line_base<AXIS>(l);
    inv_line_as_written<HALVE>(m[o], m[o + S], m[o + 2 * S], u);
  }
}

// m: the input of the inverse pass.
template <int AXIS, typename R>
CMLBM_HD void inv_pass_adj(const R (&m)[27], R u, R (&g)[27], R& gu) {
  CMLBM_FMA_AS_WRITTEN
  constexpr int S = line_stride<AXIS>();
#pragma unroll
  for (int l = 0; l < 9; ++l) {
    const int o = line_base<AXIS>(l);
    // (the z pass, lines with e_y = -1: with both roundings, as the raw first moment is
    // a halved sum there)
    const R m1 = m[o + S], r1 = AXIS == 2 && l % 3 == 0 ? m1 + u * m[o] : fma_r(u, m[o], m1);
    inv_line_adj(m[o], m1 + r1, u, g[o], g[o + S], g[o + 2 * S], gu);
  }
}

// The diagonal second moments: their combinations D1 = xx - yy, D2 = xx + yy - 2 zz and
// T = xx + yy + zz (g7, g8 relaxed toward 0, g9 toward rho), and the relaxed ones, kxx =
// X/6, kyy = Y/6, kzz = Z/3.
template <typename R>
struct Diagonal27 {
  R D1, D2, T, X, Y, Z, kxx, kyy, kzz;
  CMLBM_HD Diagonal27(R xx, R yy, R zz, R rho, const Rates<R>& p) {
    CMLBM_FMA_AS_WRITTEN
    const R xy2 = xx + yy;
    D1 = xx - yy;
    D2 = fma_r(R(-2), zz, xy2);
    T = xy2 + zz;
    const R t = fma_r(p.w[9], rho, p.wc[9] * T);
    const R d1 = p.wc[7] * D1, td = fma_r(p.wc[8], D2, t + t);
    X = fma_r(d1, R(3), td);
    Y = fma_r(d1, R(-3), td);
    Z = fma_r(-p.wc[8], D2, t);
    kxx = X * R(1.0 / 6.0);
    kyy = Y * R(1.0 / 6.0);
    kzz = Z * R(1.0 / 3.0);
  }
};

// The attractors' sums and differences, axy = kxx kyy (over rho: per_mass) etc.: axy + axz
// + ayz, axy + axz - 2 ayz and axy - axz.  PM: attractor form, 0 literal, 1 per unit mass.
template <int PM, typename R>
struct Attractors27 {
  R axy, axz, ayz, a1, a2, a3;
  CMLBM_HD Attractors27(const Diagonal27<R>& k, R sm) {
    CMLBM_FMA_AS_WRITTEN
    const R xy = k.kxx * k.kyy, xz = k.kxx * k.kzz, yz = k.kyy * k.kzz;
    R xy_xz;
    if constexpr (PM) {
      axy = xy * sm;
      axz = xz * sm;
      ayz = yz * sm;
      xy_xz = fma_r(xy, sm, axz);
      a1 = fma_r(yz, sm, xy_xz);
      a3 = fma_r(xy, sm, -axz);
    } else {
      axy = xy;
      axz = xz;
      ayz = yz;
      xy_xz = fma_r(k.kxx, k.kzz, xy);
      a1 = fma_r(k.kyy, k.kzz, xy_xz);
      a3 = fma_r(-k.kxx, k.kzz, xy);
    }
    a2 = fma_r(R(-2), ayz, xy_xz);
  }
};

// Third order pairs relaxed, xyy + xzz (g10) with xyy - xzz (g13) and the y, z
// analogues: twice the moments.
template <typename R>
CMLBM_HD void relax_pairs27(R (&m)[27], const Rates<R>& p) {
  auto pair = [&](int i, int j, int bs, int bd) {
    CMLBM_FMA_AS_WRITTEN
    const R s = m[i] + m[j], d = p.wc[bd] * (m[i] - m[j]);
    m[i] = fma_r(p.wc[bs], s, d);
    m[j] = fma_r(p.wc[bs], s, -d);
  };
  pair(K3(1, 2, 0), K3(1, 0, 2), 10, 13);
  pair(K3(2, 1, 0), K3(0, 1, 2), 11, 14);
  pair(K3(2, 0, 1), K3(0, 2, 1), 12, 15);
}

// The inverse pass along x from relaxed moments, of which m still holds the unrelaxed
// ones that are only multiplied by a factor, and twice the third order pairs: the factors
// are fused into the sums that use the moments.  k: the diagonal second order, m220 and
// m202 of the fourth, and its m022 = T/3; m222.  HALVE as in inv_line.
template <bool HALVE, typename R>
CMLBM_HD void unshift_x27(R (&m)[27], R rho, R ux, R Fx, R Fy, R Fz, const Rates<R>& p, R kxx, R kyy, R kzz, R Y, R Z,
                          R m220, R m202, R T, R m222) {
  CMLBM_FMA_AS_WRITTEN
  constexpr R third = R(1.0 / 3.0), sixth = R(1.0 / 6.0), half = R(0.5);
  // the lines along x: (raw first moment, raw second, rest) -> (p_-, p_0, p_+)
  auto line = [&](int o, R r1, R r2, R rest) {
    CMLBM_FMA_AS_WRITTEN
    m[o] = HALVE ? half * (r2 - r1) : r2 - r1;
    m[o + 9] = rest;
    m[o + 18] = HALVE ? half * (r2 + r1) : r2 + r1;
  };
  {
    const R r1 = fma_r(half, Fx, rho * ux), r2 = fma_r(ux, fma_r(half, Fx, r1), kxx);
    line(K3(0, 0, 0), r1, r2, rho - r2);
  }
  auto first = [&](int o, R F, R w, R m1, R m2) {        // m0 = F/2, m1 a product
    CMLBM_FMA_AS_WRITTEN
    const R r1 = fma_r(half * F, ux, w * m1), r2 = fma_r(ux, fma_r(w, m1, r1), m2);
    line(o, r1, r2, fma_r(F, half, -r2));
  };
  first(K3(0, 0, 1), Fz, p.wc[5], m[K3(1, 0, 1)], half * m[K3(2, 0, 1)]);
  first(K3(0, 1, 0), Fy, p.wc[4], m[K3(1, 1, 0)], half * m[K3(2, 1, 0)]);
  {
    const R m011 = m[K3(0, 1, 1)], m111 = m[K3(1, 1, 1)];
    const R r1 = fma_r(ux, p.wc[6] * m011, p.wc[16] * m111);
    const R r2 = fma_r(ux, fma_r(p.wc[16], m111, r1), p.wc[20] * m[K3(2, 1, 1)]);
    line(K3(0, 1, 1), r1, r2, fma_r(p.wc[6], m011, -r2));
  }
  auto square = [&](int o, R m0, R K, R f, R S, R m2) {  // m0 = f K, m1 = S/2
    CMLBM_FMA_AS_WRITTEN
    const R r1 = fma_r(half, S, ux * m0), r2 = fma_r(ux, fma_r(half, S, r1), m2);
    line(o, r1, r2, fma_r(K, f, -r2));
  };
  square(K3(0, 0, 2), kzz, Z, third, m[K3(1, 0, 2)], m202);
  square(K3(0, 2, 0), kyy, Y, sixth, m[K3(1, 2, 0)], m220);
  auto odd = [&](int o, R w1, R m1, R w2, R m2) {        // m0 = S/2, m1 and m2 products
    CMLBM_FMA_AS_WRITTEN
    const R S = m[o], r1 = fma_r(w1, m1, ux * (half * S)), r2 = fma_r(w2, m2, ux * fma_r(w1, m1, r1));
    line(o, r1, r2, fma_r(S, half, -r2));
  };
  odd(K3(0, 2, 1), p.wc[21], m[K3(1, 2, 1)], p.wc[25], m[K3(2, 2, 1)]);
  odd(K3(0, 1, 2), p.wc[22], m[K3(1, 1, 2)], p.wc[24], m[K3(2, 1, 2)]);
  {
    const R m122 = m[K3(1, 2, 2)];
    const R r1 = fma_r(p.wc[23], m122, ux * (third * T)), r2 = fma_r(ux, fma_r(p.wc[23], m122, r1), m222);
    line(K3(0, 2, 2), r1, r2, fma_r(T, third, -r2));
  }
}

// Relaxation and the inverse pass along x in one, from central moments to populations
// along x (not halved).
template <typename R>
CMLBM_HD void relax_unshift_x27(R (&m)[27], R rho, R inv_rho, R ux, R Fx, R Fy, R Fz, const Rates<R>& p) {
  CMLBM_FMA_AS_WRITTEN
  constexpr R third = R(1.0 / 3.0), half = R(0.5);
  const Diagonal27<R> k(m[K3(2, 0, 0)], m[K3(0, 2, 0)], m[K3(0, 0, 2)], rho, p);
  relax_pairs27(m, p);
  // fourth order, diagonal: m022 = third T
  const R sm = p.per_mass ? inv_rho : R(1);
  const R kxy = k.kxx * k.kyy, kyz = k.kzz * k.kyy;
  const R axz = sm * (k.kzz * k.kxx), ayz = sm * kyz;
  const R axy_xz = fma_r(sm, kxy, axz);
  const R A = m[K3(2, 2, 0)], B = m[K3(2, 0, 2)], C = m[K3(0, 2, 2)];
  const R q1 = fma_r(p.wc[17], C + (A + B), p.w[17] * fma_r(sm, kyz, axy_xz));
  const R q2 = fma_r(p.wc[18], fma_r(R(-2), C, A + B), p.w[18] * fma_r(R(-2), ayz, axy_xz));
  const R q3 = fma_r(p.wc[19], A - B, p.w[19] * fma_r(sm, kxy, -axz));
  const R ab = fma_r(R(2), q1, q2);
  const R m222 = fma_r(p.wc[26], m[K3(2, 2, 2)], p.w[26] * ((sm * sm) * (k.kzz * kxy)));
  unshift_x27<false>(m, rho, ux, Fx, Fy, Fz, p, k.kxx, k.kyy, k.kzz, k.Y, k.Z, half * fma_r(ab, third, q3),
                     half * fma_r(ab, third, -q3), q1 - q2, m222);
}

// Population e scaled by 2^-(number of nonzero components of e).  (One multiply each, an
// exact one: a 16-bit store may fuse it with its subtraction of the rest weight, which
// saves 23 of 1123 instructions of the step.)
template <typename R>
CMLBM_HD void scale27(R (&m)[27]) {
#pragma unroll
  for (int i = 0; i < 27; ++i) {
    const int k = (i / 9 != 1) + ((i / 3) % 3 != 1) + (i % 3 != 1);
    if (k) m[i] *= R(k == 1 ? 0.5 : k == 2 ? 0.25 : 0.125);
  }
}

// Full collision: cube-ordered pre-collision populations in, post-collision out.
template <typename R>
CMLBM_HD void collide27(R (&m)[27], R Fx, R Fy, R Fz, const Rates<R>& p) {
  CMLBM_FMA_AS_WRITTEN
  raw_pass<2>(m);
  raw_pass<1>(m);
  raw_pass<0>(m);
  const R rho = m[K3(0, 0, 0)];
  const R inv_rho = recip(rho);
  const R ux = fma_r(R(0.5), Fx, m[K3(1, 0, 0)]) * inv_rho;
  const R uy = fma_r(R(0.5), Fy, m[K3(0, 1, 0)]) * inv_rho;
  const R uz = fma_r(R(0.5), Fz, m[K3(0, 0, 1)]) * inv_rho;
  shift_pass<0>(m, ux);
  shift_pass<1>(m, uy);
  shift_pass<2>(m, uz);
  // the three inverse passes without their halvings
  relax_unshift_x27(m, rho, inv_rho, ux, Fx, Fy, Fz, p);
  inv_pass_as_written<1, false>(m, uy);
  inv_pass_as_written<2, false>(m, uz);
  scale27(m);
}

// Adds x g to entry b of a rate-adjoint accumulator, or subtracts it (an array or
// anything whose operator[] yields an R&; accumulators that keep the factors
// overload these).
template <typename W, typename R>
CMLBM_HD void add_product(W& gw, int b, R x, R g) {
  gw[b] = fma_r(x, g, R(gw[b]));
}
template <typename W, typename R>
CMLBM_HD void sub_product(W& gw, int b, R x, R g) {
  add_product(gw, b, -x, g);
}

// The same for the adjoint's replay, with the attractor form compiled in, and the pass
// along y as well: m holds the input of the z inverse pass on exit.
template <int PM, typename R>
CMLBM_HD void relax_unshift_xy27(R (&m)[27], R rho, R inv_rho, R ux, R uy, R Fx, R Fy, R Fz, const Rates<R>& p) {
  CMLBM_FMA_AS_WRITTEN
  constexpr R third = R(1.0 / 3.0), half = R(0.5);
  const Diagonal27<R> k(m[K3(2, 0, 0)], m[K3(0, 2, 0)], m[K3(0, 0, 2)], rho, p);
  relax_pairs27(m, p);
  const R sm = PM ? inv_rho : R(1);
  const Attractors27<PM, R> a(k, sm);
  const R A = m[K3(2, 2, 0)], B = m[K3(2, 0, 2)], C = m[K3(0, 2, 2)];
  const R q1 = fma_r(p.wc[17], A + B + C, p.w[17] * a.a1);
  const R q2 = fma_r(p.wc[18], fma_r(R(-2), C, A + B), p.w[18] * a.a2);
  const R q3 = fma_r(p.wc[19], A - B, p.w[19] * a.a3);
  const R ab = fma_r(R(2), q1, q2);
  const R m222 = fma_r(p.wc[26], m[K3(2, 2, 2)], p.w[26] * (k.kxx * k.kyy * k.kzz * (sm * sm)));
  unshift_x27<false>(m, rho, ux, Fx, Fy, Fz, p, k.kxx, k.kyy, k.kzz, k.Y, k.Z, half * fma_r(ab, third, q3),
                     half * fma_r(ab, third, -q3), q1 - q2, m222);
  // the lines along y; those with e_x = +-1 come doubled
#pragma unroll
  for (int l = 0; l < 9; ++l) {
    const int o = line_base<1>(l);
    const R m0 = m[o], m1 = m[o + 3], m2 = m[o + 6];
    R r1, r2;
    if (l / 3 == 1) {
      r1 = fma_r(uy, m0, m1);
      r2 = fma_r(uy, m1 + r1, m2);
      m[o + 3] = m0 - r2;
    } else {
      r1 = fma_r(half, m1, uy * (half * m0));
      const R s = fma_r(half, m1, r1);
      r2 = l % 3 == 2 ? fma_r(half, m2, uy * s) : fma_r(uy, s, half * m2);
      m[o + 3] = fma_r(half, m0, -r2);
    }
    m[o] = half * (r2 - r1);
    m[o + 6] = half * (r2 + r1);
  }
}

// Two adjoints of relaxed moments before their factors: the sums that use wc4 x110 and
// wc26 x222 fuse them.
template <typename R>
struct Unscaled27 {
  R x110, x222;
};

// Adjoint of the relaxation.  m: pre-relaxation central moments (unchanged).  g: on
// entry the adjoint of the relaxed moments, on exit the adjoint of m.  Adds to
// grho, gF* and, through add_product, gw[b] (adjoint of omega_b, b = 4..26).
template <int PM, typename R, typename W>
CMLBM_HD Unscaled27<R> relax27_adj(const R (&m)[27], R rho, const Rates<R>& p, R (&g)[27], R& grho, R& gFx, R& gFy,
                                   R& gFz, W& gw) {
  CMLBM_FMA_AS_WRITTEN
  // recompute the second-order post values and attractor inputs
  const Diagonal27<R> k(m[K3(2, 0, 0)], m[K3(0, 2, 0)], m[K3(0, 0, 2)], rho, p);
  const R kxx = k.kxx, kyy = k.kyy, kzz = k.kzz;
  // per-mass attractors: A = P sm^(k-1), dA/drho = -(k-1) A sm
  const R sm = PM ? R(1) / rho : R(1);
  const Unscaled27<R> x{g[K3(1, 1, 0)], g[K3(2, 2, 2)]};
  R gkxx, gkyy, gkzz;

  // sixth order
  {
    const R G = x.x222;
    const R s2 = sm * sm, kxy = kxx * kyy, gP = p.w[26] * G, gPs = gP * s2;
    if constexpr (PM) {
      const R kxyz = kxy * kzz;
      add_product(gw, 26, fma_r(kxyz, s2, -m[K3(2, 2, 2)]), G);
      grho = fma_r(R(-2) * sm * (kxyz * s2), gP, grho);
    } else {
      add_product(gw, 26, fma_r(kxy, kzz, -m[K3(2, 2, 2)]), G);
    }
    gkxx = gPs * kyy * kzz;
    gkyy = gPs * kxx * kzz;
    gkzz = gPs * kxx * kyy;
    g[K3(2, 2, 2)] = p.wc[26] * G;
  }
  // fifth order and fourth-order off-diagonal: m~ = (1 - w) m
  auto scale = [&](int i, int b) {
    const R G = g[i];
    sub_product(gw, b, m[i], G);
    g[i] = p.wc[b] * G;
  };
  scale(K3(1, 2, 2), 23);
  scale(K3(2, 1, 2), 24);
  scale(K3(2, 2, 1), 25);
  scale(K3(2, 1, 1), 20);
  scale(K3(1, 2, 1), 21);
  scale(K3(1, 1, 2), 22);
  // fourth order diagonal
  {
    const Attractors27<PM, R> a(k, sm);
    const R A = m[K3(2, 2, 0)], B = m[K3(2, 0, 2)], C = m[K3(0, 2, 2)];
    const R gA = g[K3(2, 2, 0)], gB = g[K3(2, 0, 2)], gC = g[K3(0, 2, 2)];
    const R gAB = gA + gB;                                       // twice the adjoint of A + B
    const R gq3 = R(0.5) * (gA - gB);
    const R gq1 = (gC + gAB) * R(1.0 / 3.0);
    const R gq2 = fma_r(R(0.5), gAB, -gC) * R(1.0 / 3.0);
    add_product(gw, 17, a.a1 - (A + B + C), gq1);
    add_product(gw, 18, a.a2 - fma_r(R(-2), C, A + B), gq2);
    add_product(gw, 19, a.a3 - (A - B), gq3);
    const R ga1 = p.w[17] * gq1, ga2 = p.w[18] * gq2, ga12 = fma_r(p.w[18], gq2, ga1);
    const R gaxy = fma_r(p.w[19], gq3, ga12), gaxz = fma_r(-p.w[19], gq3, ga12), gayz = fma_r(R(-2), ga2, ga1);
    if constexpr (PM) grho = fma_r(-sm, fma_r(a.ayz, gayz, fma_r(a.axy, gaxy, a.axz * gaxz)), grho);
    gkxx = fma_r(sm, fma_r(gaxy, kyy, gaxz * kzz), gkxx);
    gkyy = fma_r(sm, fma_r(gayz, kzz, gaxy * kxx), gkyy);
    gkzz = fma_r(sm, fma_r(gayz, kyy, gaxz * kxx), gkzz);
    const R gQ1 = p.wc[17] * gq1, gQ2 = p.wc[18] * gq2, gQ12 = fma_r(p.wc[18], gq2, gQ1);
    g[K3(2, 2, 0)] = fma_r(p.wc[19], gq3, gQ12);
    g[K3(2, 0, 2)] = fma_r(-p.wc[19], gq3, gQ12);
    g[K3(0, 2, 2)] = fma_r(R(-2), gQ2, gQ1);
  }
  // third order
  scale(K3(1, 1, 1), 16);
  auto pair = [&](int i, int j, int bs, int bd) {
    CMLBM_FMA_AS_WRITTEN
    const R gs = R(0.5) * (g[i] + g[j]);
    const R gd = R(0.5) * (g[i] - g[j]);
    sub_product(gw, bs, m[i] + m[j], gs);
    sub_product(gw, bd, m[i] - m[j], gd);
    const R b = p.wc[bd] * gd;
    g[i] = fma_r(p.wc[bs], gs, b);
    g[j] = fma_r(p.wc[bs], gs, -b);
  };
  pair(K3(1, 2, 0), K3(1, 0, 2), 10, 13);
  pair(K3(2, 1, 0), K3(0, 1, 2), 11, 14);
  pair(K3(2, 0, 1), K3(0, 2, 1), 12, 15);
  // second order diagonal; total adjoint of kxx, kyy, kzz
  {
    const R Gx = g[K3(2, 0, 0)] + gkxx, Gy = g[K3(0, 2, 0)] + gkyy, Gz = g[K3(0, 0, 2)] + gkzz;
    const R Gxy = Gx + Gy, Gz3 = Gz * R(1.0 / 3.0);
    const R gt = fma_r(Gxy, R(1.0 / 3.0), Gz3);
    const R gd2 = fma_r(Gxy, R(1.0 / 6.0), -Gz3);
    const R gd1 = R(0.5) * (Gx - Gy);
    sub_product(gw, 7, k.D1, gd1);
    sub_product(gw, 8, k.D2, gd2);
    add_product(gw, 9, rho - k.T, gt);
    grho = fma_r(p.w[9], gt, grho);
    const R gD2 = p.wc[8] * gd2, gT = p.wc[9] * gt;
    g[K3(2, 0, 0)] = fma_r(p.wc[9], gt, fma_r(p.wc[7], gd1, gD2));
    g[K3(0, 2, 0)] = fma_r(p.wc[9], gt, fma_r(-p.wc[7], gd1, gD2));
    g[K3(0, 0, 2)] = fma_r(R(-2), gD2, gT);
  }
  scale(K3(1, 1, 0), 4);
  scale(K3(1, 0, 1), 5);
  scale(K3(0, 1, 1), 6);
  // conserved rows were overwritten by rho and F/2
  grho += g[K3(0, 0, 0)];
  gFx = fma_r(R(0.5), g[K3(1, 0, 0)], gFx);
  gFy = fma_r(R(0.5), g[K3(0, 1, 0)], gFy);
  gFz = fma_r(R(0.5), g[K3(0, 0, 1)], gFz);
  g[K3(0, 0, 0)] = g[K3(1, 0, 0)] = g[K3(0, 1, 0)] = g[K3(0, 0, 1)] = R(0);
  return x;
}

// Adjoint of collide27.  f: cube-ordered pre-collision populations on entry;
// on exit it holds scratch.  g: on entry the adjoint of the post-collision
// populations, on exit the adjoint of f.  s: scratch.  Adds the force and rate
// adjoints.  The forward transform is replayed as collide27 computes it (raw
// sums, u, shifts) and only the central moments c are kept.  The inverse
// passes are differentiated with their inputs recovered from the relaxed
// moments; the shifts in reverse order from their outputs (each shift's
// output is the next one's input, recovered by undoing the later shift); the
// raw sums are linear and need no inputs; rho and u enter through the raw
// moments 000, 100, 010, 001.
template <int PM = -1, typename R, typename W>
CMLBM_HD void collide27_adj(R (&f)[27], R Fx, R Fy, R Fz, const Rates<R>& p, R (&g)[27], R (&s)[27],
                                              R& gFx, R& gFy, R& gFz, W& gw) {
  CMLBM_FMA_AS_WRITTEN
  if constexpr (PM < 0) {                    // the attractor form as p says
    if (p.per_mass)
      collide27_adj<1>(f, Fx, Fy, Fz, p, g, s, gFx, gFy, gFz, gw);
    else
      collide27_adj<0>(f, Fx, Fy, Fz, p, g, s, gFx, gFy, gFz, gw);
    return;
  }
  R(&cm)[27] = f;
  raw_pass<2>(cm);
  raw_pass<1>(cm);
  raw_pass<0>(cm);
  const R rho = cm[K3(0, 0, 0)];
  const R inv_rho = recip(rho);
  const R ux = fma_r(R(0.5), Fx, cm[K3(1, 0, 0)]) * inv_rho;
  const R uy = fma_r(R(0.5), Fy, cm[K3(0, 1, 0)]) * inv_rho;
  const R uz = fma_r(R(0.5), Fz, cm[K3(0, 0, 1)]) * inv_rho;
  shift_pass<0>(cm, ux);
  shift_pass<1>(cm, uy);
  shift_pass<2>(cm, uz);
  R gux = R(0), guy = R(0), guz = R(0), grho = R(0);

  // relax, then replay the inverse passes to get each pass's input
#pragma unroll
  for (int k = 0; k < 27; ++k) s[k] = cm[k];
  relax_unshift_xy27<PM>(s, rho, inv_rho, ux, uy, Fx, Fy, Fz, p);   // s = input of the z inverse pass
  inv_pass_adj<2>(s, uz, g, guz);
  fwd_pass<1>(s, uy);                        // undo the y pass: s = input of the y inverse pass
  inv_pass_adj<1>(s, uy, g, guy);
  fwd_pass<0>(s, ux);                        // s = relaxed central moments
  inv_pass_adj<0>(s, ux, g, gux);

  const Unscaled27<R> x = relax27_adj<PM>(cm, rho, p, g, grho, gFx, gFy, gFz, gw);

  // the shifts z, y, x in reverse; cm holds the output of the shift being
  // differentiated
  {
    const R t = fma_r(-uz, g[K3(1, 1, 2)], g[K3(1, 1, 1)]), g110 = fma_r(p.wc[4], x.x110, -(uz * t));
    shift_pass_adj<2>(cm, uz, g, guz);
    g[K3(1, 1, 0)] = g110;
  }
  unshift_pass<2>(cm, uz);
  shift_pass_adj<1>(cm, uy, g, guy);
  unshift_pass<1>(cm, uy);
  shift_pass_adj<0>(cm, ux, g, gux);

  // u = (j + F/2) / rho with j and rho the raw moments 100, 010, 001 and 000
  g[K3(0, 0, 0)] += fma_r(-fma_r(uz, guz, fma_r(uy, guy, ux * gux)), inv_rho, grho);
  g[K3(1, 0, 0)] = fma_r(gux, inv_rho, g[K3(1, 0, 0)]);
  g[K3(0, 1, 0)] = fma_r(guy, inv_rho, g[K3(0, 1, 0)]);
  g[K3(0, 0, 1)] = fma_r(guz, inv_rho, g[K3(0, 0, 1)]);
  gFx = fma_r(R(0.5), gux * inv_rho, gFx);
  gFy = fma_r(R(0.5), guy * inv_rho, gFy);
  gFz = fma_r(R(0.5), guz * inv_rho, gFz);
  {
    const R t = fma_r(p.wc[26], x.x222, g[K3(0, 2, 2)]), g122 = g[K3(1, 2, 2)];
    raw_pass_adj<0>(g);
    g[K3(0, 2, 2)] = t - g122;
    g[K3(2, 2, 2)] = t + g122;
  }
  raw_pass_adj<1>(g);
  raw_pass_adj<2>(g);
}


// Initial transformed populations fbar = f^eq(rho, u) - S/2 (paper order): the
// central moments about u are the Maxwellian's (Sec. 3: rho c_s^(2k) on the
// even monomials, zero on the odd ones) with -F/2 on the first-order ones (the
// source changes only those, Eq. discretecentralsources); the inverse passes
// return them to populations.
template <typename R>
CMLBM_HD void initial27(R rho, R ux, R uy, R uz, R Fx, R Fy, R Fz, R (&f)[27]) {
  R m[27];
#pragma unroll
  for (int i = 0; i < 27; ++i) m[i] = R(0);
  const R c2 = rho * R(1.0 / 3.0);
  m[K3(0, 0, 0)] = rho;
  m[K3(1, 0, 0)] = R(-0.5) * Fx;
  m[K3(0, 1, 0)] = R(-0.5) * Fy;
  m[K3(0, 0, 1)] = R(-0.5) * Fz;
  m[K3(2, 0, 0)] = m[K3(0, 2, 0)] = m[K3(0, 0, 2)] = c2;
  m[K3(2, 2, 0)] = m[K3(2, 0, 2)] = m[K3(0, 2, 2)] = c2 * R(1.0 / 3.0);
  m[K3(2, 2, 2)] = c2 * R(1.0 / 9.0);
  inv_pass<0>(m, ux);
  inv_pass<1>(m, uy);
  inv_pass<2>(m, uz);
#pragma unroll
  for (int a = 0; a < 27; ++a) f[a] = m[cube27(a)];
}

// Adjoint of initial27 with respect to the force (u fixed): the populations
// are the inverse-pass image of the moments above, linear in F through the
// first-order entries -F/2.  lam: adjoint of f (paper order); adds to gF*.
template <typename R>
CMLBM_HD void initial27_adj_force(R ux, R uy, R uz, const R (&lam)[27], R& gFx, R& gFy, R& gFz) {
  R gm[27], zero[27];
#pragma unroll
  for (int a = 0; a < 27; ++a) {
    gm[cube27(a)] = lam[a];
    zero[a] = R(0);
  }
  R gu = R(0);   // the inputs of the passes only enter the velocity adjoint, unused here
  inv_pass_adj<2>(zero, uz, gm, gu);
  inv_pass_adj<1>(zero, uy, gm, gu);
  inv_pass_adj<0>(zero, ux, gm, gu);
  gFx += R(-0.5) * gm[K3(1, 0, 0)];
  gFy += R(-0.5) * gm[K3(0, 1, 0)];
  gFz += R(-0.5) * gm[K3(0, 0, 1)];
}

}  // namespace cmlbm
