// Harmonic terms of the Cartesian expansions.  Included by fmm_impl.h.
#pragma once

// D[g] = -d^g (1/r) obeys Laplace's equation away from the
// source, D[x, y, z + 2] = -D[x + 2, y, z] - D[x, y + 2, z], so an expansion
// is fixed by its terms with z exponent 0 or 1: (m + 1)^2 up to degree m.
// Reduced index: by degree m, then z = 0 (x ascending), then z = 1.
// ---------------------------------------------------------------------------
constexpr __host__ __device__ int hterms(int m) { return m < 0 ? 0 : (m + 1) * (m + 1); }
constexpr __host__ __device__ int h_degree(int i) {
  int m = 0;
  while ((m + 1) * (m + 1) <= i) ++m;
  return m;
}
// exponents x | y << 8 | z << 16 of reduced term i
constexpr __host__ __device__ int h_exp(int i) {
  const int m = h_degree(i), r = i - m * m;
  return r <= m ? (r | (m - r) << 8) : ((r - m - 1) | (m - 1 - (r - m - 1)) << 8 | 1 << 16);
}
constexpr __host__ __device__ int h_index(int x, int y, int z) {
  const int m = x + y + z;
  return m * m + (z ? m + 1 + x : x);
}
constexpr __host__ __device__ int binom(int n, int k) {
  int b = 1;
  for (int i = 1; i <= k; ++i) b = b * (n - k + i) / i;
  return b;
}
// Moments (or evaluation coefficients) f of the full expansion carried over to
// reduced term (x, y, e): sum over the full terms that the recurrence sends
// there, (x - 2l, y - 2m, 2(l + m) + e) with weight (-1)^(l+m) C(l+m, l).
template <typename F>
__device__ __forceinline__ double h_reduce(int i, F&& f) {
  const int ex = h_exp(i), x = mi_a(ex), y = mi_b(ex), e = mi_c(ex);
  double s = 0.0;
  for (int l = 0; 2 * l <= x; ++l)
    for (int m = 0; 2 * m <= y; ++m) {
      const double w = (double)(((l + m) & 1) ? -binom(l + m, l) : binom(l + m, l));
      s += w * f(mi_index(x - 2 * l, y - 2 * m, 2 * (l + m) + e));
    }
  return s;
}
constexpr __host__ __device__ int h_parity(int i) {
  const int ex = h_exp(i);
  return ((ex & 1) << 2) | (((ex >> 8) & 1) << 1) | ((ex >> 16) & 1);
}
// The same from the terms of one degree, in graded order, everything but the
// values known at compile time.
template <int I, int N>
__device__ __forceinline__ double h_reduce_deg(const double (&d)[N]) {
  constexpr int ex = h_exp(I), x = ex & 255, y = (ex >> 8) & 255, e = ex >> 16, m = x + y + e;
  static_assert(N == ndeg(m), "the terms of one degree");
  double s = 0.0;
  static_for<x / 2 + 1>([&](auto lc) {
    constexpr int l = decltype(lc)::value;
    static_for<y / 2 + 1>([&](auto kc) {
      constexpr int k = decltype(kc)::value;
      constexpr double w = ((l + k) & 1) ? -binom(l + k, l) : binom(l + k, l);
      s = fma(w, d[mi_index(x - 2 * l, y - 2 * k, 2 * (l + k) + e) - nterms(m - 1)], s);
    });
  });
  return s;
}
