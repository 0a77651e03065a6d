// D3Q15 central-moment collision with forcing (Premnath & Banerjee,
// arXiv:1202.6081, Appendix G).
//
// Steps, per node:
//  1. rho, u from the transformed populations, u including F/2.
//  2. Source S = K D^-1 m^s with the projections m^s printed in Appendix G and
//     the D3Q15 basis K_0..K_14 of Appendix G (inversion as in Eq.
//     sourceformulation1).
//  3. Raw moments of h = fbar + S for the fifteen monomials the D3Q15 kernels
//     use (1, x, y, z, xy, xz, yz, xx, yy, zz, xyy, xxy, xxz, xyz, xxyy); on this
//     lattice they are signed sums over the rest, axis and corner links (the
//     corners by a Walsh-Hadamard transform).
//  4. Binomial shift to central moments, one axis at a time, relaxation of xy, xz, yz (g4..g6),
//     xx-yy, xx+yy-2zz, xx+yy+zz (g7..g9), xyy, xxy, xxz, xyz (g10..g13) toward
//     zero (rho for g9) and xxyy (g14) toward kxx~ kyy~; rho and the first central
//     moments (F/2) are conserved.
//  5. Inverse shift to raw moments and exact inversion of the fifteen raw
//     moments to populations (the K g + S rows of Appendix G), the corners by the
//     inverse transform.
#pragma once

#include "collide_d3q27.hpp"   // Rates<R>, unroll
#include "lattice.hpp"

namespace cmlbm {

// Basis vector K_b of Appendix G evaluated at direction e.
CMLBM_HDC int k15_basis(int b, Vel e) {
  const int x = e.x, y = e.y, z = e.z;
  const int s2 = x * x + y * y + z * z;
  switch (b) {
    case 0: return 1;
    case 1: return x;
    case 2: return y;
    case 3: return z;
    case 4: return x * y;
    case 5: return x * z;
    case 6: return y * z;
    case 7: return x * x - y * y;
    case 8: return s2 - 3 * z * z;
    case 9: return s2 - 2;
    case 10: return 5 * x * s2 - 13 * x;
    case 11: return 5 * y * s2 - 13 * y;
    case 12: return 5 * z * s2 - 13 * z;
    case 13: return x * y * z;
    default: return 30 * (x * x * y * y + x * x * z * z + y * y * z * z) - 40 * s2 + 32;
  }
}

CMLBM_HDC int k15_norm(int b) {
  int d = 0;
  for (int a = 0; a < 15; ++a) d += k15_basis(b, kE15[a]) * k15_basis(b, kE15[a]);
  return d;
}

// Compile-time tables: kB15.v[b][a] = K_b(e_a), kM15.v[m][a] = the monomial m
// (order below) at e_a, kD15[b] = D_b.  Loops over them run through
// unroll so that every entry is a literal constant in the generated code.
struct Tab15 {
  int v[15][15];
};

CMLBM_HDC Vel mono15(int m) {
  constexpr Vel t[15] = {{0, 0, 0}, {1, 0, 0}, {0, 1, 0}, {0, 0, 1}, {1, 1, 0}, {1, 0, 1}, {0, 1, 1}, {2, 0, 0},
                         {0, 2, 0}, {0, 0, 2}, {1, 2, 0}, {2, 1, 0}, {2, 0, 1}, {1, 1, 1}, {2, 2, 0}};
  return t[m];
}

CMLBM_HDC int ipow(int v, int n) { return n == 0 ? 1 : (n == 1 ? v : v * v); }

CMLBM_HDC Tab15 make_basis15() {
  Tab15 t{};
  for (int b = 0; b < 15; ++b)
    for (int a = 0; a < 15; ++a) t.v[b][a] = k15_basis(b, kE15[a]);
  return t;
}

CMLBM_HDC Tab15 make_mono15() {
  Tab15 t{};
  for (int m = 0; m < 15; ++m)
    for (int a = 0; a < 15; ++a)
      t.v[m][a] = ipow(kE15[a].x, mono15(m).x) * ipow(kE15[a].y, mono15(m).y) * ipow(kE15[a].z, mono15(m).z);
  return t;
}

constexpr Tab15 kB15 = make_basis15();
constexpr Tab15 kM15 = make_mono15();

// Source S_a = sum_b K_b(e_a) m^s_b / D_b with the printed m^s (Appendix G).
template <typename R>
CMLBM_HD void source15(R Fx, R Fy, R Fz, R ux, R uy, R uz, R (&S)[15]) {
  const R ux2 = ux * ux, uy2 = uy * uy, uz2 = uz * uz;
  R ms[15];
  ms[0] = R(0);
  ms[1] = Fx;
  ms[2] = Fy;
  ms[3] = Fz;
  ms[4] = Fx * uy + Fy * ux;
  ms[5] = Fx * uz + Fz * ux;
  ms[6] = Fy * uz + Fz * uy;
  ms[7] = R(2) * (Fx * ux - Fy * uy);
  ms[8] = R(2) * (Fx * ux + Fy * uy - R(2) * Fz * uz);
  ms[9] = R(2) * (Fx * ux + Fy * uy + Fz * uz);
  ms[10] = R(5) * (Fx * (R(3) * ux2 + uy2 + uz2) + R(2) * ux * (Fy * uy + Fz * uz)) - R(13) * Fx;
  ms[11] = R(5) * (Fy * (ux2 + R(3) * uy2 + uz2) + R(2) * uy * (Fx * ux + Fz * uz)) - R(13) * Fy;
  ms[12] = R(5) * (Fz * (ux2 + uy2 + R(3) * uz2) + R(2) * uz * (Fx * ux + Fy * uy)) - R(13) * Fz;
  ms[13] = Fx * uy * uz + Fy * ux * uz + Fz * ux * uy;
  ms[14] = R(20) * (Fx * ux * (R(3) * (uy2 + uz2) - R(4)) + Fy * uy * (R(3) * (ux2 + uz2) - R(4)) +
                    Fz * uz * (R(3) * (ux2 + uy2) - R(4)));
  unroll<15>([&](auto b) {
    constexpr int d = k15_norm(decltype(b)::value);
    ms[b] *= R(1.0 / d);
  });
  unroll<15>([&](auto a) {
    R acc = R(0);
    unroll<14>([&](auto b1) {
      constexpr int k = kB15.v[decltype(b1)::value + 1][decltype(a)::value];
      if constexpr (k != 0) acc += R(k) * ms[decltype(b1)::value + 1];
    });
    S[a] = acc;
  });
}

// The fifteen moments the D3Q15 kernels use, in this order.
enum : int { M0 = 0, MX, MY, MZ, MXY, MXZ, MYZ, MXX, MYY, MZZ, MXYY, MXXY, MXXZ, MXYZ, MXXYY };

// The binomial shift between raw and central moments factors into one shift
// per axis, because this set is closed under lowering any one exponent: along
// an axis the moments form triples (exponent 0, 1, 2), pairs (0, 1) and
// singles, and a triple (m0, m1, m2) shifts by u as
// (m0, m1 - u m0, m2 - 2 u m1 + u^2 m0) (raw to central) or
// (m0, m1 + u m0, m2 + 2 u m1 + u^2 m0) (central to raw).
struct Groups15 {
  int t[4][3];   // triples
  int nt;
  int p[4][2];   // pairs
  int np;
};

template <int AX>
CMLBM_HDC Groups15 groups15() {
  if constexpr (AX == 0)
    return {{{0, 1, 7}, {2, 4, 11}, {3, 5, 12}, {8, 10, 14}}, 4, {{6, 13}, {0, 0}, {0, 0}, {0, 0}}, 1};
  else if constexpr (AX == 1)
    return {{{0, 2, 8}, {1, 4, 10}, {7, 11, 14}, {0, 0, 0}}, 3, {{3, 6}, {5, 13}, {0, 0}, {0, 0}}, 2};
  else
    return {{{0, 3, 9}, {0, 0, 0}, {0, 0, 0}, {0, 0, 0}}, 1, {{1, 5}, {2, 6}, {4, 13}, {7, 12}}, 4};
}

// Shift of moments m by u along axis AX (sg = -1: raw to central, +1: back).
template <int AX, typename R>
CMLBM_HD void shift15(R (&m)[15], R u, R sg) {
  constexpr Groups15 G = groups15<AX>();
  const R v = sg * u;
  unroll<G.nt>([&](auto i) {
    constexpr int a = G.t[decltype(i)::value][0], b = G.t[decltype(i)::value][1], c = G.t[decltype(i)::value][2];
    const R nb = m[b] + v * m[a];           // m2 + 2 v m1 + v^2 m0 = m2 + v (m1 + nb)
    m[c] = m[c] + v * (m[b] + nb);
    m[b] = nb;
  });
  unroll<G.np>([&](auto i) {
    constexpr int a = G.p[decltype(i)::value][0], b = G.p[decltype(i)::value][1];
    m[b] += v * m[a];
  });
}

// Raw moments r of populations f (paper order).  The eight corner links' sign
// patterns are the moments 1, x, y, z, xy, xz, yz, xyz, so the corner sums come
// from a three-stage Walsh-Hadamard transform (24 additions); on the corners
// xyy = x, xxy = y, xxz = z and xx = yy = zz = xxyy = 1, and the axis links
// carry only 1, x, y, z, xx, yy, zz.  Corner 7 + i has e_x = -1 when bit 0 of i
// is set, e_y = -1 for bit 1, e_z = -1 for bit 2.
template <typename R>
CMLBM_HD void raw_moments15(const R (&f)[15], R (&r)[15]) {
  const R s0 = f[7] + f[8], d0 = f[7] - f[8];       // (y, z) = (+, +): sum and x-weighted sum
  const R s1 = f[9] + f[10], d1 = f[9] - f[10];     // (-, +)
  const R s2 = f[11] + f[12], d2 = f[11] - f[12];   // (+, -)
  const R s3 = f[13] + f[14], d3 = f[13] - f[14];   // (-, -)
  const R a_p = s0 + s1, y_p = s0 - s1, x_p = d0 + d1, xy_p = d0 - d1;   // z = +1
  const R a_m = s2 + s3, y_m = s2 - s3, x_m = d2 + d3, xy_m = d2 - d3;   // z = -1
  const R c1 = a_p + a_m, cz = a_p - a_m, cy = y_p + y_m, cyz = y_p - y_m;
  const R cx = x_p + x_m, cxz = x_p - x_m, cxy = xy_p + xy_m, cxyz = xy_p - xy_m;
  const R lxx = f[1] + f[2], lyy = f[3] + f[4], lzz = f[5] + f[6];
  r[M0] = ((f[0] + c1) + (lxx + lyy)) + lzz;
  r[MX] = (f[1] - f[2]) + cx;
  r[MY] = (f[3] - f[4]) + cy;
  r[MZ] = (f[5] - f[6]) + cz;
  r[MXY] = cxy;
  r[MXZ] = cxz;
  r[MYZ] = cyz;
  r[MXX] = lxx + c1;
  r[MYY] = lyy + c1;
  r[MZZ] = lzz + c1;
  r[MXYY] = cx;
  r[MXXY] = cy;
  r[MXXZ] = cz;
  r[MXYZ] = cxyz;
  r[MXXYY] = c1;
}

// Populations with raw moments r: the inverse of raw_moments15.  The corner
// moments (1, x, y, z, xy, xz, yz, xyz) = (xxyy, xyy, xxy, xxz, xy, xz, yz, xyz)
// give the eight corners by the inverse transform (the same three stages and
// a factor 1/8); the axis links follow from the xx, x (etc.) moments less the
// corners' parts, the rest population from the density.
template <typename R>
CMLBM_HD void populations_from_raw15(const R (&r)[15], R (&f)[15]) {
  const R c1 = r[MXXYY];
  const R a1p = r[MXXYY] + r[MXXZ], a1m = r[MXXYY] - r[MXXZ];   // 1 + z, 1 - z
  const R axp = r[MXYY] + r[MXZ], axm = r[MXYY] - r[MXZ];       // x + xz, x - xz
  const R ayp = r[MXXY] + r[MYZ], aym = r[MXXY] - r[MYZ];       // y + yz, y - yz
  const R bxyp = r[MXY] + r[MXYZ], bxym = r[MXY] - r[MXYZ];     // xy + xyz, xy - xyz
  // (y, z) corner pairs: the x-even part b and the x-odd part c
  const R b_pp = a1p + ayp, b_mp = a1p - ayp, b_pm = a1m + aym, b_mm = a1m - aym;
  const R c_pp = axp + bxyp, c_mp = axp - bxyp, c_pm = axm + bxym, c_mm = axm - bxym;
  const R h = R(0.125);
  f[7] = h * (b_pp + c_pp);
  f[8] = h * (b_pp - c_pp);
  f[9] = h * (b_mp + c_mp);
  f[10] = h * (b_mp - c_mp);
  f[11] = h * (b_pm + c_pm);
  f[12] = h * (b_pm - c_pm);
  f[13] = h * (b_mm + c_mm);
  f[14] = h * (b_mm - c_mm);
  const R lxx = r[MXX] - c1, lyy = r[MYY] - c1, lzz = r[MZZ] - c1;
  const R lx = r[MX] - r[MXYY], ly = r[MY] - r[MXXY], lz = r[MZ] - r[MXXZ];
  f[1] = R(0.5) * (lxx + lx);
  f[2] = R(0.5) * (lxx - lx);
  f[3] = R(0.5) * (lyy + ly);
  f[4] = R(0.5) * (lyy - ly);
  f[5] = R(0.5) * (lzz + lz);
  f[6] = R(0.5) * (lzz - lz);
  f[0] = ((r[M0] - c1) - lxx) - (lyy + lzz);
}

// Populations with central moments m about u (m is overwritten by the raw
// moments): shift back along z, y, x, then invert.
template <typename R>
CMLBM_HD void populations_from_central15(R (&m)[15], R ux, R uy, R uz, R (&f)[15]) {
  shift15<2>(m, uz, R(1));
  shift15<1>(m, uy, R(1));
  shift15<0>(m, ux, R(1));
  populations_from_raw15(m, f);
}

// Density and velocity (Eqs. densitycalculation, velocitycalculation).
template <typename R>
CMLBM_HD void moments0_15(const R (&f)[15], R Fx, R Fy, R Fz, R& rho, R& ux, R& uy, R& uz, R& inv_rho) {
  CMLBM_FMA_AS_WRITTEN
  rho = R(0);
#pragma unroll
  for (int a = 0; a < 15; ++a) rho += f[a];
  R cx = R(0), cy = R(0), cz = R(0);
#pragma unroll
  for (int a = 7; a < 15; ++a) {
    cx += R(kE15[a].x) * f[a];
    cy += R(kE15[a].y) * f[a];
    cz += R(kE15[a].z) * f[a];
  }
  const R inv = recip(rho);
  inv_rho = inv;
  ux = fma_r(R(0.5), Fx, f[1] - f[2] + cx) * inv;
  uy = fma_r(R(0.5), Fy, f[3] - f[4] + cy) * inv;
  uz = fma_r(R(0.5), Fz, f[5] - f[6] + cz) * inv;
}

// Raw moments of the source S = K D^-1 m^s (Appendix G), in the moment order
// 1, x, y, z, xy, xz, yz, xx, yy, zz, xyy, xxy, xxz, xyz, xxyy.  With K^T K = D
// they follow from the printed projections m^s alone: e.g. the xx moment is
// m^s_7/2 + m^s_8/6 + m^s_9/3 = 2 F_x u_x and the xyy moment is
// (4/5) m^s_1 + m^s_10/10.  Here the sums of products that they and their adjoint share;
// which of two products is fused is free where neither is needed elsewhere, and kept as
// it is so that the gradients keep their bits.
template <typename R>
struct Source15 {
  R ux2, uy2, uz2, Fu, Fv, Fw, Fxy, Fxz, Fyz, Fvw, Fuw, Fuv, cx, cy, cz, xy2, xz2, yz2;
  CMLBM_HD Source15(R Fx, R Fy, R Fz, R ux, R uy, R uz) {
    CMLBM_FMA_AS_WRITTEN
    ux2 = ux * ux;
    uy2 = uy * uy;
    uz2 = uz * uz;
    Fu = Fx * ux;
    Fv = Fy * uy;
    Fw = Fz * uz;
    Fxy = fma_r(Fy, ux, Fx * uy);
    Fxz = fma_r(Fx, uz, Fz * ux);
    Fyz = fma_r(Fz, uy, Fy * uz);
    Fvw = fma_r(Fz, uz, Fv);
    Fuw = fma_r(Fz, uz, Fu);
    Fuv = fma_r(Fy, uy, Fu);
    xy2 = fma_r(uy, uy, ux2);
    xz2 = fma_r(uz, uz, ux2);
    yz2 = fma_r(uz, uz, uy2);
    cx = fma_r(uz, uz, fma_r(R(3), ux2, uy2)) - R(1);
    cy = fma_r(uz, uz, fma_r(R(3), uy2, ux2)) - R(1);
    cz = fma_r(R(3), uz2, xy2) - R(1);
  }
};

// Adds the raw moments of the source to m.
template <typename R>
CMLBM_HD void add_source_raw15(const Source15<R>& q, R Fx, R Fy, R Fz, R ux, R uy, R uz, R (&m)[15]) {
  CMLBM_FMA_AS_WRITTEN
  m[MX] += Fx;
  m[MY] += Fy;
  m[MZ] += Fz;
  m[MXY] += q.Fxy;
  m[MXZ] += q.Fxz;
  m[MYZ] += q.Fyz;
  m[MXX] = fma_r(R(2), q.Fu, m[MXX]);
  m[MYY] = fma_r(R(2), q.Fv, m[MYY]);
  m[MZZ] = fma_r(R(2), q.Fw, m[MZZ]);
  m[MXYY] = fma_r(R(0.5), fma_r(Fx, q.cx, (ux + ux) * q.Fvw), m[MXYY]);
  m[MXXY] = fma_r(R(0.5), fma_r(Fy, q.cy, (uy + uy) * q.Fuw), m[MXXY]);
  m[MXXZ] = fma_r(R(0.5), fma_r(Fz, q.cz, (uz + uz) * q.Fuv), m[MXXZ]);
  m[MXYZ] += fma_r(Fz * ux, uy, fma_r(Fx * uy, uz, Fy * ux * uz));
  m[MXXYY] = fma_r(R(2.0 / 3.0), fma_r(q.Fw, q.xy2, fma_r(q.Fu, q.yz2, q.Fv * q.xz2)), m[MXXYY]);
}

// Its adjoint with respect to F and u (gr: adjoint of m).
template <typename R>
CMLBM_HD void source_raw15_adj(const Source15<R>& q, R Fx, R Fy, R Fz, R ux, R uy, R uz, const R (&gr)[15], R& gFx,
                               R& gFy, R& gFz, R& gux, R& guy, R& guz) {
  CMLBM_FMA_AS_WRITTEN
  const R x2 = R(2) * ux, y2 = R(2) * uy, z2 = R(2) * uz;
  gFx += fma_r(x2, gr[7], fma_r(uz, gr[5], fma_r(uy, gr[4], gr[1])));
  gFy += fma_r(y2, gr[8], fma_r(uz, gr[6], fma_r(ux, gr[4], gr[2])));
  gFz += fma_r(z2, gr[9], fma_r(uy, gr[6], fma_r(ux, gr[5], gr[3])));
  gux += fma_r(R(2) * Fx, gr[7], fma_r(Fz, gr[5], Fy * gr[4]));
  guy += fma_r(R(2) * Fy, gr[8], fma_r(Fz, gr[6], Fx * gr[4]));
  guz += fma_r(R(2) * Fz, gr[9], fma_r(Fy, gr[6], Fx * gr[5]));
  // third order
  const R hx = R(0.5) * q.cx, hy = R(0.5) * q.cy, hz = R(0.5) * q.cz;
  const R uxy = ux * uy, uxz = ux * uz, uyz = uy * uz;
  gFx += fma_r(uxz, gr[12], fma_r(hx, gr[10], uxy * gr[11]));
  gFy += fma_r(uyz, gr[12], fma_r(uxy, gr[10], hy * gr[11]));
  gFz += fma_r(hz, gr[12], fma_r(uxz, gr[10], uyz * gr[11]));
  gux += fma_r(q.Fxz, gr[12], fma_r(fma_r(Fz, uz, fma_r(R(3), q.Fu, q.Fv)), gr[10], q.Fxy * gr[11]));
  guy += fma_r(q.Fyz, gr[12], fma_r(q.Fxy, gr[10], fma_r(Fz, uz, fma_r(R(3), q.Fv, q.Fu)) * gr[11]));
  guz += fma_r(fma_r(Fy, uy, fma_r(R(3), q.Fw, q.Fu)), gr[12], fma_r(q.Fxz, gr[10], q.Fyz * gr[11]));
  gFx = fma_r(uyz, gr[13], gFx);
  gFy = fma_r(uxz, gr[13], gFy);
  gFz = fma_r(uxy, gr[13], gFz);
  gux = fma_r(q.Fyz, gr[13], gux);
  guy = fma_r(q.Fxz, gr[13], guy);
  guz = fma_r(q.Fxy, gr[13], guz);
  // fourth order
  const R c = R(2.0 / 3.0) * gr[14];
  gFx = fma_r(c * ux, q.yz2, gFx);
  gFy = fma_r(c * uy, q.xz2, gFy);
  gFz = fma_r(c * uz, q.xy2, gFz);
  gux = fma_r(c, fma_r(Fx, q.yz2, x2 * q.Fvw), gux);
  guy = fma_r(c, fma_r(Fy, q.xz2, y2 * q.Fuw), guy);
  guz = fma_r(c, fma_r(Fz, q.xy2, z2 * q.Fuv), guz);
}

// shift15 with its multiply-adds as written.  GIVEN: the first triple's first moment,
// shifted, is first.
template <int AX, bool GIVEN = false, typename R>
CMLBM_HD void shift15_as_written(R (&m)[15], R v, R first = R(0)) {
  constexpr Groups15 G = groups15<AX>();
  unroll<G.nt>([&](auto i) {
    CMLBM_FMA_AS_WRITTEN
    constexpr int a = G.t[decltype(i)::value][0], b = G.t[decltype(i)::value][1], c = G.t[decltype(i)::value][2];
    const R nb = GIVEN && a == 0 ? first : fma_r(v, m[a], m[b]);
    m[c] = fma_r(v, m[b] + nb, m[c]);
    m[b] = nb;
  });
  unroll<G.np>([&](auto i) {
    CMLBM_FMA_AS_WRITTEN
    constexpr int a = G.p[decltype(i)::value][0], b = G.p[decltype(i)::value][1];
    m[b] = fma_r(v, m[a], m[b]);
  });
}

// The multiply-adds of the collision are those written and no others, as in D3Q27's.
template <typename R>
CMLBM_HD void collide15(R (&f)[15], R Fx, R Fy, R Fz, const Rates<R>& p) {
  CMLBM_FMA_AS_WRITTEN
  R m[15];
  raw_moments15(f, m);
  const R rho = m[M0];
  const R inv_rho = recip(rho);
  const R ux = fma_r(R(0.5), Fx, m[MX]) * inv_rho;
  const R uy = fma_r(R(0.5), Fy, m[MY]) * inv_rho;
  const R uz = fma_r(R(0.5), Fz, m[MZ]) * inv_rho;
  // raw moments of h = f + S (the source's as in add_source_raw15), then central moments
  // about u
  {
    const R ux2 = ux * ux, uy2 = uy * uy, uz2 = uz * uz;
    const R Fu = Fx * ux, Fv = Fy * uy, Fw = Fz * uz;
    const R xy2 = fma_r(uy, uy, ux2), xz2 = fma_r(ux, ux, uz2), yz2 = fma_r(uy, uy, uz2);
    m[MX] += Fx;
    m[MY] += Fy;
    m[MZ] += Fz;
    m[MXY] += fma_r(Fx, uy, Fy * ux);
    m[MXZ] += fma_r(Fx, uz, Fz * ux);
    m[MYZ] += fma_r(Fz, uy, Fy * uz);
    m[MXX] = fma_r(R(2), Fu, m[MXX]);
    m[MYY] = fma_r(R(2), Fv, m[MYY]);
    m[MZZ] = fma_r(R(2), Fw, m[MZZ]);
    const R cx = fma_r(uz, uz, fma_r(R(3), ux2, uy2)) - R(1), cy = fma_r(uz, uz, fma_r(R(3), uy2, ux2)) - R(1);
    const R cz = fma_r(R(3), uz2, xy2) - R(1);
    m[MXYY] = fma_r(R(0.5), fma_r(ux + ux, fma_r(Fy, uy, Fw), Fx * cx), m[MXYY]);
    m[MXXY] = fma_r(R(0.5), fma_r(uy + uy, fma_r(Fx, ux, Fw), Fy * cy), m[MXXY]);
    m[MXXZ] = fma_r(R(0.5), fma_r(uz + uz, fma_r(Fy, uy, Fu), Fz * cz), m[MXXZ]);
    m[MXYZ] += fma_r(uy, Fz * ux, fma_r(uz, Fx * uy, uz * (Fy * ux)));
    m[MXXYY] = fma_r(R(2.0 / 3.0), fma_r(Fw, xy2, fma_r(Fu, yz2, Fv * xz2)), m[MXXYY]);
  }
  shift15_as_written<0>(m, -ux);
  shift15_as_written<1>(m, -uy);
  shift15_as_written<2>(m, -uz);
  // relaxation; density and the first central moments (F/2) are conserved
  const R d1 = p.wc[7] * (m[MXX] - m[MYY]);
  const R xy2 = m[MXX] + m[MYY], D2 = fma_r(R(-2), m[MZZ], xy2);
  const R t9 = fma_r(p.w[9], rho, p.wc[9] * (xy2 + m[MZZ]));
  const R td = fma_r(p.wc[8], D2, t9 + t9);
  const R txx = fma_r(d1, R(3), td) * R(1.0 / 6.0);
  const R tyy = fma_r(d1, R(-3), td) * R(1.0 / 6.0);
  const R tzz = fma_r(-p.wc[8], D2, t9) * R(1.0 / 3.0);
  const R sm = p.per_mass ? inv_rho : R(1);
  const R xxyy = fma_r(p.wc[14], m[MXXYY], p.w[14] * (txx * tyy * sm));
  // ... and back to raw moments along z and y (shift15), with the relaxed
  // moments that are products fused into the sums that use them
  const R half = R(0.5), hx = half * Fx, hy = half * Fy, hz = half * Fz;
  const R mxy = p.wc[4] * m[MXY];
  const R z1 = fma_r(half, Fz, rho * uz), z2 = fma_r(uz, hz + z1, tzz);
  const R xz = fma_r(hx, uz, p.wc[5] * m[MXZ]), yz = fma_r(hy, uz, p.wc[6] * m[MYZ]);
  const R xyz = fma_r(uz, mxy, p.wc[13] * m[MXYZ]), xxz = fma_r(p.wc[12], m[MXXZ], uz * txx);
  const R y1 = fma_r(half, Fy, rho * uy), y2 = fma_r(uy, hy + y1, tyy);
  const R xy = fma_r(hx, uy, mxy), xyy = fma_r(uy, fma_r(p.wc[4], m[MXY], xy), p.wc[10] * m[MXYY]);
  const R xxy = fma_r(p.wc[11], m[MXXY], uy * txx);
  m[MXXYY] = fma_r(uy, fma_r(p.wc[11], m[MXXY], xxy), xxyy);
  m[M0] = rho;
  m[MX] = hx;
  m[MY] = y1;
  m[MZ] = z1;
  m[MXX] = txx;
  m[MYY] = y2;
  m[MZZ] = z2;
  m[MXY] = xy;
  m[MXZ] = xz;
  m[MYZ] = fma_r(uy, z1, yz);
  m[MXYY] = xyy;
  m[MXXY] = xxy;
  m[MXXZ] = xxz;
  m[MXYZ] = fma_r(uy, xz, xyz);
  shift15_as_written<0>(m, ux);
  populations_from_raw15(m, f);
}

// Initial transformed populations fbar = f^eq(rho, u) - S/2: f^eq has the
// Maxwellian central moments rho, c_s^2 rho (xx, yy, zz), c_s^4 rho (xxyy).
template <typename R>
CMLBM_HD void initial15(R rho, R ux, R uy, R uz, R Fx, R Fy, R Fz, R (&f)[15]) {
  const R c2 = rho * R(1.0 / 3.0);
  R m[15];
#pragma unroll
  for (int k = 0; k < 15; ++k) m[k] = R(0);
  m[M0] = rho;
  m[MXX] = m[MYY] = m[MZZ] = c2;
  m[MXXYY] = rho * R(1.0 / 9.0);
  populations_from_central15(m, ux, uy, uz, f);
  R S[15];
  source15(Fx, Fy, Fz, ux, uy, uz, S);
#pragma unroll
  for (int a = 0; a < 15; ++a) f[a] -= R(0.5) * S[a];
}

// ---------------------------------------------------------------------------
// Adjoint of collide15 (moments in the order of the enum above; the per-axis
// shifts as in the forward collision).
// ---------------------------------------------------------------------------
// Adjoint of shift15: m = its input, g = adjoint of its output (in place ->
// adjoint of its input); adds d/du to gu.  GU, GA: bit i for the second of the two products
// of triple i's sum for gu, and of that for its first moment, being the fused one (free,
// as above).  GIVEN, first: as in shift15_as_written.
template <int AX, unsigned GU, unsigned GA, bool GIVEN = false, typename R>
CMLBM_HD void shift15_adj(const R (&m)[15], R u, R sg, R (&g)[15], R& gu, R first = R(0)) {
  CMLBM_FMA_AS_WRITTEN
  constexpr Groups15 G = groups15<AX>();
  const R v = sg * u, vv = v * v;
  R gv = R(0);
  unroll<G.nt>([&](auto i) {
    CMLBM_FMA_AS_WRITTEN
    constexpr int I = decltype(i)::value, a = G.t[I][0], b = G.t[I][1], c = G.t[I][2];
    const R g1 = g[b], g2 = g[c], nb = GIVEN && a == 0 ? first : fma_r(v, m[a], m[b]), gg = R(2) * g2;
    if constexpr (GU >> I & 1)
      gv += fma_r(gg, nb, g1 * m[a]);
    else
      gv += fma_r(g1, m[a], gg * nb);
    if constexpr (GA >> I & 1)
      g[a] += fma_r(vv, g2, v * g1);
    else
      g[a] += fma_r(v, g1, vv * g2);
    g[b] = fma_r(R(2) * v, g2, g1);
  });
  unroll<G.np>([&](auto i) {
    CMLBM_FMA_AS_WRITTEN
    constexpr int a = G.p[decltype(i)::value][0], b = G.p[decltype(i)::value][1];
    gv = fma_r(g[b], m[a], gv);
    g[a] = fma_r(v, g[b], g[a]);
  });
  gu = fma_r(sg, gv, gu);
}

// Raw moments of h, and the transpose (adjoint) of that linear map.
template <typename R>
CMLBM_HD void raw15(const R (&h)[15], R (&r)[15]) {
  unroll<15>([&](auto m) {
    R acc = R(0);
    unroll<15>([&](auto a) {
      constexpr int k = kM15.v[decltype(m)::value][decltype(a)::value];
      if constexpr (k == 1) acc += h[a];
      if constexpr (k == -1) acc -= h[a];
    });
    r[m] = acc;
  });
}

// gr[12 .. 14] = w[m] x[m - 12], fused into the sums.
template <typename R>
CMLBM_HD void raw15_adj(const R (&gr)[15], const R (&w)[27], const R (&x)[3], R (&gh)[15]) {
  unroll<15>([&](auto a) {
    CMLBM_FMA_AS_WRITTEN
    R acc = R(0);
    unroll<15>([&](auto m) {
      CMLBM_FMA_AS_WRITTEN
      constexpr int M = decltype(m)::value, k = kM15.v[M][decltype(a)::value];
      if constexpr (M >= 12 && k != 0)
        acc = fma_r(k == 1 ? w[M] : -w[M], x[M - 12], acc);
      else if constexpr (k == 1)
        acc += gr[M];
      else if constexpr (k == -1)
        acc -= gr[M];
    });
    gh[a] = acc;
  });
}

// Transpose of the raw-moment inversion at the end of populations15:
// gs = (d f / d s)^T g.
template <typename R>
CMLBM_HD void inverse15_adj(const R (&g)[15], R (&gs)[15]) {
  CMLBM_FMA_AS_WRITTEN
  R c = R(0), cx = R(0), cy = R(0), cz = R(0), cxy = R(0), cxz = R(0), cyz = R(0), cxyz = R(0);
#pragma unroll
  for (int a = 7; a < 15; ++a) {
    const int x = kE15[a].x, y = kE15[a].y, z = kE15[a].z;
    c += g[a];
    cx += R(x) * g[a];
    cy += R(y) * g[a];
    cz += R(z) * g[a];
    cxy += R(x * y) * g[a];
    cxz += R(x * z) * g[a];
    cyz += R(y * z) * g[a];
    cxyz += R(x * y * z) * g[a];
  }
  const R p1 = R(0.5) * (g[1] + g[2]), m1 = R(0.5) * (g[1] - g[2]);
  const R p2 = R(0.5) * (g[3] + g[4]), m2 = R(0.5) * (g[3] - g[4]);
  const R p3 = R(0.5) * (g[5] + g[6]), m3 = R(0.5) * (g[5] - g[6]);
  gs[0] = g[0];
  gs[1] = m1;
  gs[2] = m2;
  gs[3] = m3;
  gs[4] = R(0.125) * cxy;
  gs[5] = R(0.125) * cxz;
  gs[6] = R(0.125) * cyz;
  gs[7] = p1 - g[0];
  gs[8] = p2 - g[0];
  gs[9] = p3 - g[0];
  gs[10] = fma_r(R(0.125), cx, -m1);
  gs[11] = fma_r(R(0.125), cy, -m2);
  gs[12] = fma_r(R(0.125), cz, -m3);
  gs[13] = R(0.125) * cxyz;
  gs[14] = fma_r(R(2), g[0], fma_r(R(0.125), c, -(p1 + p2 + p3)));
}

// Adjoint of source15 with respect to F and u: gS = adjoint of S.
template <typename R>
CMLBM_HD void source15_adj(R Fx, R Fy, R Fz, R ux, R uy, R uz, const R (&gS)[15], R& gFx, R& gFy, R& gFz,
                           R& gux, R& guy, R& guz) {
  R G[15];
  unroll<14>([&](auto b1) {
    constexpr int b = decltype(b1)::value + 1;
    R acc = R(0);
    unroll<15>([&](auto a) {
      constexpr int k = kB15.v[b][decltype(a)::value];
      if constexpr (k != 0) acc += R(k) * gS[a];
    });
    constexpr int d = k15_norm(b);
    G[b] = acc * R(1.0 / d);
  });
  const R ux2 = ux * ux, uy2 = uy * uy, uz2 = uz * uz;
  gFx += G[1];
  gFy += G[2];
  gFz += G[3];
  // ms4..ms6
  gFx += uy * G[4] + uz * G[5];
  gFy += ux * G[4] + uz * G[6];
  gFz += ux * G[5] + uy * G[6];
  gux += Fy * G[4] + Fz * G[5];
  guy += Fx * G[4] + Fz * G[6];
  guz += Fx * G[5] + Fy * G[6];
  // ms7..ms9
  gFx += R(2) * ux * (G[7] + G[8] + G[9]);
  gFy += R(2) * uy * (-G[7] + G[8] + G[9]);
  gFz += R(2) * uz * (G[9] - R(2) * G[8]);
  gux += R(2) * Fx * (G[7] + G[8] + G[9]);
  guy += R(2) * Fy * (-G[7] + G[8] + G[9]);
  guz += R(2) * Fz * (G[9] - R(2) * G[8]);
  // ms10..ms12
  gFx += (R(5) * (R(3) * ux2 + uy2 + uz2) - R(13)) * G[10] + R(10) * ux * (uy * G[11] + uz * G[12]);
  gFy += (R(5) * (ux2 + R(3) * uy2 + uz2) - R(13)) * G[11] + R(10) * uy * (ux * G[10] + uz * G[12]);
  gFz += (R(5) * (ux2 + uy2 + R(3) * uz2) - R(13)) * G[12] + R(10) * uz * (ux * G[10] + uy * G[11]);
  gux += (R(30) * Fx * ux + R(10) * (Fy * uy + Fz * uz)) * G[10] + R(10) * (Fy * ux + Fx * uy) * G[11] +
         R(10) * (Fz * ux + Fx * uz) * G[12];
  guy += R(10) * (Fx * uy + Fy * ux) * G[10] + (R(30) * Fy * uy + R(10) * (Fx * ux + Fz * uz)) * G[11] +
         R(10) * (Fz * uy + Fy * uz) * G[12];
  guz += R(10) * (Fx * uz + Fz * ux) * G[10] + R(10) * (Fy * uz + Fz * uy) * G[11] +
         (R(30) * Fz * uz + R(10) * (Fx * ux + Fy * uy)) * G[12];
  // ms13
  gFx += uy * uz * G[13];
  gFy += ux * uz * G[13];
  gFz += ux * uy * G[13];
  gux += (Fy * uz + Fz * uy) * G[13];
  guy += (Fx * uz + Fz * ux) * G[13];
  guz += (Fx * uy + Fy * ux) * G[13];
  // ms14
  const R ax = R(3) * (uy2 + uz2) - R(4), ay = R(3) * (ux2 + uz2) - R(4), az = R(3) * (ux2 + uy2) - R(4);
  gFx += R(20) * ux * ax * G[14];
  gFy += R(20) * uy * ay * G[14];
  gFz += R(20) * uz * az * G[14];
  gux += R(20) * (Fx * ax + R(6) * ux * (Fy * uy + Fz * uz)) * G[14];
  guy += R(20) * (Fy * ay + R(6) * uy * (Fx * ux + Fz * uz)) * G[14];
  guz += R(20) * (Fz * az + R(6) * uz * (Fx * ux + Fy * uy)) * G[14];
}

// Adjoint of collide15.  f: pre-collision populations.  g: on entry the
// adjoint of the post-collision populations, on exit the adjoint of f.  Adds
// the force adjoint and gw[b] (adjoint of omega_b, b = 4..14).  PM: attractor form,
// 0 literal, 1 per unit mass, -1 as p.per_mass says (run time).  STORED16: populations
// are stored in 16 bits; the shifted z moment is F_z/2 + rho u_z with F_z/2 fused instead of
// rho u_z (free, as above).
template <int PM = -1, bool STORED16 = false, typename R, typename W>
CMLBM_HD void collide15_adj(const R (&f)[15], R Fx, R Fy, R Fz, const Rates<R>& p, R (&g)[15], R& gFx, R& gFy,
                            R& gFz, W& gw) {
  CMLBM_FMA_AS_WRITTEN
  if constexpr (PM < 0) {
    if (p.per_mass)
      collide15_adj<1, STORED16>(f, Fx, Fy, Fz, p, g, gFx, gFy, gFz, gw);
    else
      collide15_adj<0, STORED16>(f, Fx, Fy, Fz, p, g, gFx, gFy, gFz, gw);
    return;
  }
  R rho, ux, uy, uz, inv_rho;
  moments0_15(f, Fx, Fy, Fz, rho, ux, uy, uz, inv_rho);
  R gux = R(0), guy = R(0), guz = R(0), grho = R(0);
  const R sm = PM > 0 ? inv_rho : R(1);

  // forward: central moments c of h = f + S (raw moments of f plus those of S)
  R c[15];
  raw15(f, c);
  const Source15<R> q(Fx, Fy, Fz, ux, uy, uz);
  add_source_raw15(q, Fx, Fy, Fz, ux, uy, uz, c);
  shift15_as_written<0>(c, -ux);
  shift15_as_written<1>(c, -uy);
  shift15_as_written<2>(c, -uz);
  // relaxed central moments t (conserved rows: rho and F/2)
  const R D1 = c[7] - c[8], xy2 = c[7] + c[8], D2 = fma_r(R(-2), c[9], xy2), T = xy2 + c[9];
  const R d1 = p.wc[7] * D1;
  const R t9 = fma_r(p.w[9], rho, p.wc[9] * T);
  const R td = fma_r(p.wc[8], D2, t9 + t9);
  const R txx = fma_r(R(3), d1, td) * R(1.0 / 6.0);
  const R tyy = fma_r(R(-3), d1, td) * R(1.0 / 6.0);
  const R tzz = fma_r(-p.wc[8], D2, t9) * R(1.0 / 3.0);
  R t[15];
  t[0] = rho;
  t[1] = R(0.5) * Fx;
  t[2] = R(0.5) * Fy;
  t[3] = R(0.5) * Fz;
#pragma unroll
  for (int m = 4; m < 7; ++m) t[m] = p.wc[m] * c[m];
  t[7] = txx;
  t[8] = tyy;
  t[9] = tzz;
#pragma unroll
  for (int m = 10; m < 14; ++m) t[m] = p.wc[m] * c[m];
  t[14] = fma_r(p.wc[14], c[14], p.w[14] * (txx * tyy * sm));

  // back through the inversion and the shifts central -> raw (z, y, x order
  // reversed: the forward applies z, then y, then x)
  R gt[15];
  inverse15_adj(g, gt);
  {
    R v[15];   // input of the x shift = t shifted along z and y
#pragma unroll
    for (int m = 0; m < 15; ++m) v[m] = t[m];
    const R z = STORED16 ? fma_r(R(0.5), Fz, uz * rho) : fma_r(uz, rho, t[3]);
    shift15_as_written<2, true>(v, uz, z);
    // along y (shift15), with the relaxed moments that are products fused into the sums
    // that use them
    {
      const R n2 = fma_r(uy, v[0], v[2]), n4 = fma_r(uy, v[1], v[4]), n11 = fma_r(p.wc[11], c[11], uy * v[7]);
      v[8] = fma_r(uy, v[2] + n2, v[8]);
      v[10] = fma_r(uy, fma_r(p.wc[4], c[4], n4), v[10]);
      v[14] = fma_r(uy, fma_r(p.wc[11], c[11], n11), v[14]);
      v[2] = n2;
      v[4] = n4;
      v[11] = n11;
      v[6] = fma_r(uy, v[3], v[6]);
      v[13] = fma_r(uy, v[5], v[13]);
    }
    const R g6 = gt[6] + ux * gt[13];            // (both rounded)
    shift15_adj<0, 0, 0>(v, ux, R(1), gt, gux);
    gt[6] = g6;
    shift15_as_written<1>(v, -uy);               // undo: v = input of the y shift
    shift15_adj<1, 0, 0>(v, uy, R(1), gt, guy);
    shift15_adj<2, 1, 1, true>(t, uz, R(1), gt, guz, z);
  }
  // relaxation
  grho += gt[0];
  gFx = fma_r(R(0.5), gt[1], gFx);
  gFy = fma_r(R(0.5), gt[2], gFy);
  gFz = fma_r(R(0.5), gt[3], gFz);
  R gc[15];
  gc[0] = gc[1] = gc[2] = gc[3] = R(0);
#pragma unroll
  for (int m = 4; m < 7; ++m) {
    gc[m] = p.wc[m] * gt[m];
    sub_product(gw, m, c[m], gt[m]);
  }
#pragma unroll
  for (int m = 10; m < 14; ++m) {
    gc[m] = p.wc[m] * gt[m];
    sub_product(gw, m, c[m], gt[m]);
  }
  R gtxx = gt[7], gtyy = gt[8];
  const R gtzz = gt[9];
  {
    const R G = gt[14], gA = p.w[14] * G;
    gc[14] = p.wc[14] * G;
    if constexpr (PM > 0) {
      const R txy = txx * tyy;
      add_product(gw, 14, fma_r(txy, sm, -c[14]), G);
      grho = fma_r(-sm * (txy * sm), gA, grho);
      gtxx = fma_r(gA * tyy, sm, gtxx);
      gtyy = fma_r(gA * txx, sm, gtyy);
    } else {
      add_product(gw, 14, fma_r(txx, tyy, -c[14]), G);
      gtxx = fma_r(gA, tyy, gtxx);
      gtyy = fma_r(gA, txx, gtyy);
    }
  }
  {
    const R gxy = gtxx + gtyy, gzz3 = gtzz * R(1.0 / 3.0);
    const R gt9 = fma_r(gxy, R(1.0 / 3.0), gzz3);
    const R gd2 = fma_r(gxy, R(1.0 / 6.0), -gzz3);
    const R gd1 = R(0.5) * (gtxx - gtyy);
    sub_product(gw, 7, D1, gd1);
    sub_product(gw, 8, D2, gd2);
    add_product(gw, 9, rho - T, gt9);
    grho = fma_r(p.w[9], gt9, grho);
    const R gD2 = p.wc[8] * gd2, gT = p.wc[9] * gt9;
    gc[7] = fma_r(p.wc[9], gt9, fma_r(p.wc[7], gd1, gD2));
    gc[8] = fma_r(p.wc[9], gt9, fma_r(-p.wc[7], gd1, gD2));
    gc[9] = fma_r(R(-2), gD2, gT);
  }
  // back through the shifts raw -> central (forward order x, y, z)
  {
    R v[15];   // input of the z shift: c unshifted along z
#pragma unroll
    for (int m = 0; m < 15; ++m) v[m] = c[m];
    shift15_as_written<2>(v, uz);
    const R g4 = fma_r(p.wc[4], gt[4], -(uz * gc[13]));   // (gc4 = wc4 gt4 fused into its own update)
    shift15_adj<2, 0, 0>(v, uz, R(-1), gc, guz);
    gc[4] = g4;
    shift15_as_written<1>(v, uy);   // input of the y shift
    shift15_adj<1, 6, 7>(v, uy, R(-1), gc, guy);
    shift15_as_written<0>(v, ux);   // raw moments of h
    shift15_adj<0, 14, 15>(v, ux, R(-1), gc, gux);
  }
  // raw moments (of f and of the source), density and velocity
  R gh[15];
  const R unscaled[3] = {gt[12], gt[13], gt[14]};
  raw15_adj(gc, p.wc, unscaled, gh);
  source_raw15_adj(q, Fx, Fy, Fz, ux, uy, uz, gc, gFx, gFy, gFz, gux, guy, guz);
  const R inv = inv_rho;
  const R gjx = gux * inv, gjy = guy * inv, gjz = guz * inv;
  grho = fma_r(-fma_r(uz, guz, fma_r(uy, guy, ux * gux)), inv, grho);
  gFx = fma_r(R(0.5), gjx, gFx);
  gFy = fma_r(R(0.5), gjy, gFy);
  gFz = fma_r(R(0.5), gjz, gFz);
  // (e = 0 adds 0 gj: a NaN or infinite gj reaches every population)
  auto along = [&](int e, R gu, R gj, R acc) {
    CMLBM_FMA_AS_WRITTEN
    return e == 0 ? fma_r(R(0), gj, acc) : fma_r(e > 0 ? gu : -gu, inv, acc);
  };
#pragma unroll
  for (int a = 0; a < 15; ++a)
    g[a] = along(kE15[a].z, guz, gjz, along(kE15[a].y, guy, gjy, along(kE15[a].x, gux, gjx, gh[a] + grho)));
}

// Adjoint of the force dependence of initial15 (u0 fixed): fbar = f^eq - S/2.
template <typename R>
CMLBM_HD void initial15_adj_force(R ux, R uy, R uz, const R (&lam)[15], R& gFx, R& gFy, R& gFz) {
  R gS[15];
#pragma unroll
  for (int a = 0; a < 15; ++a) gS[a] = R(-0.5) * lam[a];
  R gux = R(0), guy = R(0), guz = R(0);
  source15_adj(R(0), R(0), R(0), ux, uy, uz, gS, gFx, gFy, gFz, gux, guy, guz);
}

}  // namespace cmlbm
