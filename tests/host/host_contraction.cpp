// Host build of the collision and its adjoint with the types of both arithmetics, for
// the test that a compiler's freedom to fuse multiplies and adds changes none of their bits.
#include "host_collide.cpp"

namespace {

template <typename R>
struct RateSum {
  R* p;
  R& operator[](int b) const { return p[b]; }
};

// out: the adjoint of f (Q), of the force (3) and of the rates (23, the first Q - 4 used)
template <int Q, int PM, bool STORED16 = false, typename R>
void adjoint(const R* f, const R* F, const double* omega, const R* g_in, R* out) {
  const cmlbm::Rates<R> p = rates<R>(Q, omega, PM);
  R gF[3] = {}, gw[27] = {}, m[Q], g[Q];
  RateSum<R> acc{gw};
  for (int a = 0; a < Q; ++a) {
    const int k = Q == 27 ? cmlbm::cube27(a) : a;
    m[k] = f[a];
    g[k] = g_in[a];
  }
  if constexpr (Q == 27) {
    R s[27];
    cmlbm::collide27_adj<PM>(m, F[0], F[1], F[2], p, g, s, gF[0], gF[1], gF[2], acc);
  } else {
    cmlbm::collide15_adj<PM, STORED16>(m, F[0], F[1], F[2], p, g, gF[0], gF[1], gF[2], acc);
  }
  for (int a = 0; a < Q; ++a) out[a] = g[Q == 27 ? cmlbm::cube27(a) : a];
  for (int i = 0; i < 3; ++i) out[Q + i] = gF[i];
  for (int b = 4; b < 27; ++b) out[Q + 3 + b - 4] = gw[b];
}

template <typename R>
void adjoint(int q, const R* f, const R* F, const double* omega, int per_mass, const R* g_in, R* out) {
  if (q == 27)
    per_mass ? adjoint<27, 1>(f, F, omega, g_in, out) : adjoint<27, 0>(f, F, omega, g_in, out);
  else
    per_mass ? adjoint<15, 1>(f, F, omega, g_in, out) : adjoint<15, 0>(f, F, omega, g_in, out);
}

}  // namespace

extern "C" {

void hc_adjoint_bits_f64(int q, const double* f, const double* F, const double* omega, int per_mass, const double* g,
                         double* out) {
  adjoint<double>(q, f, F, omega, per_mass, g, out);
}

void hc_adjoint_bits_f32(int q, const float* f, const float* F, const double* omega, int per_mass, const float* g,
                         float* out) {
  adjoint<float>(q, f, F, omega, per_mass, g, out);
}

// (the arithmetic over 16-bit storage: D3Q15's differs in which product of a sum is fused)
void hc_adjoint_bits_16(int q, const float* f, const float* F, const double* omega, int per_mass, const float* g,
                        float* out) {
  if (q == 27)
    adjoint<float>(q, f, F, omega, per_mass, g, out);
  else
    per_mass ? adjoint<15, 1, true>(f, F, omega, g, out) : adjoint<15, 0, true>(f, F, omega, g, out);
}

}  // extern "C"
