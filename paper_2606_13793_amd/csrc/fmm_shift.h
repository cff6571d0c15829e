// Shifts between levels in harmonic terms, on the matrix cores.  Included by
// fmm_impl.h.
#pragma once

// M2M, L2L and their transposes are one matrix.  With t = b + g over the full
// terms and the harmonic ones D_a spanning them (D_t = sum_a w(a, t) D_a),
//   C(a, b) = sum_g 2^-|b| 4^-|g| / g! w(a, b + g),  |g| = |a| - |b|,
//   M2M      M(P, a) = sum_q sum_b chi_{a+b}(q) C(a, b) M(2P + q, b)
//   L2L      L(2P + q, b) = own(q, b) + sum_a chi_{a+b}(q) C(a, b) / 2 L(P, a)
// (chi: parities of the terms over the child's sign; w is h_reduce's, and keeps
// degree and parity).  Sorting a into its 8 parity classes e makes the sign
// chi_e(q) chi_b(q): a gather (M2M, transposed L2L) is a mirror folding of the
// children about their parent, fold8, and 8 products over b; a scatter (L2L,
// transposed M2M) is 8 products over the class's terms and an inverse Walsh sum,
// which a lane holds whole.
// Multipoles are planes [term][(n + 6)^3], so there a lane's column of a product
// is the parent (stores run along z); locals are rows [cell][hrow], so there it
// is the term.
template <int P>
struct ShiftShape {
  static constexpr int HT = hterms(P), NS = (HT + 3) / 4, NPS = blk_psteps(P), NTC = (NPS + 3) / 4, NTB = (HT + 15) / 16;
  static constexpr int SPW = (NS + 3) / 4;  // gather: K steps of each of the 4 waves
  static constexpr int GATHER = NS * 8 * NTC * 64, SCATTER = 8 * NPS * NTB * 64, PLAIN = HT * HT;
  static constexpr int TABLE = GATHER + SCATTER + PLAIN;
};

__device__ inline double shift_coef(int a, int b) {
  const int ea = h_exp(a), eb = h_exp(b), x = mi_a(ea), y = mi_b(ea), e = mi_c(ea);
  double s = 0.0;
  for (int l = 0; 2 * l <= x; ++l)
    for (int m = 0; 2 * m <= y; ++m) {
      const int g[3] = {x - 2 * l - mi_a(eb), y - 2 * m - mi_b(eb), 2 * (l + m) + e - mi_c(eb)};
      if (g[0] < 0 || g[1] < 0 || g[2] < 0) continue;
      double f = 1.0;
      for (int i = 0; i < 3; ++i)
        for (int k = 2; k <= g[i]; ++k) f *= k;
      const double w = (double)(((l + m) & 1) ? -binom(l + m, l) : binom(l + m, l));
      s += w * ldexp(1.0 / f, -h_degree(b) - 2 * (g[0] + g[1] + g[2]));
    }
  return s;
}
// Fragments of the gather [step][class][tile][64] (k-group kq: b = 4 s + kq;
// lane: term 16 tile + i of the class), then of the scatter [class][step][tile]
// [64] (k-group: term 4 s + kq of the class; lane: b = 16 tile + i), then C[b][a].
template <int P>
__global__ void k_shift_table(double* __restrict__ W) {
  using S = ShiftShape<P>;
  const int id = blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= S::TABLE) return;
  const int i = id & 15, kq = (id >> 4) & 3;
  int a, b;
  if (id < S::GATHER) {
    const int f = id >> 6, j = 16 * (f % S::NTC) + i;
    a = j < 4 * S::NPS ? c_ft<P>.pt[(f / S::NTC) & 7][j] : -1;
    b = 4 * (f / (8 * S::NTC)) + kq;
  } else if (id < S::GATHER + S::SCATTER) {
    const int f = (id - S::GATHER) >> 6;
    a = c_ft<P>.pt[f / (S::NTB * S::NPS)][4 * (f / S::NTB % S::NPS) + kq];
    b = 16 * (f % S::NTB) + i;
  } else {
    a = (id - S::GATHER - S::SCATTER) % S::HT;
    b = (id - S::GATHER - S::SCATTER) / S::HT;
  }
  W[id] = a >= 0 && b < S::HT ? shift_coef(a, b) : 0.0;
}

// Gather.  Segments: n = parents per axis, a = the children's values, b = the
// parents' (ROWS: or null), u = M2M: copy of b in FP32, or null; ROWS: the
// cotangents of the M2L's rows, planes [column][(n + 6)^3] over the parents in H,
// the class sums over 8.  hm: terms written (the others are zero).
// Block: 16 parents, 4 waves, each a quarter of the K steps: the loads of a wave
// are all issued before its first product, and the quarters are added in LDS.
// What bounds it: reading the children's values (M2M of 256^3, p = 6, 4 levels:
// 68 us; 164 with a thread per term and its coefficient list).
template <int P, bool ROWS, typename H>
__global__ __launch_bounds__(256, 2) void k_gather(const Seg* __restrict__ segs, int nseg, const Seg one,
                                                   const double* __restrict__ W, int hm) {
  using S = ShiftShape<P>;
  constexpr int HT = S::HT, HR = hrow(P), NTC = S::NTC, SPW = S::SPW, RS = 17;
  __shared__ double red[4 * 8 * NTC * 16 * RS];
  const Seg& sg = nseg ? find_seg(segs, nseg, blockIdx.x) : one;
  const int np = sg.n, npp = np + 6, nc = 2 * np + (ROWS ? 0 : 6);
  const long long nps = (long long)np * np * np, ncpp = (long long)npp * npp * npp, ncc = (long long)nc * nc * nc;
  const long long P0 = (long long)((int)blockIdx.x - sg.first_block) * 16;
  const int lane = threadIdx.x & 63, i = lane & 15, kq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const long long pc = min(P0 + i, nps - 1);
  const int p2 = (int)(pc % np), p1 = (int)((pc / np) % np), p0 = (int)(pc / ((long long)np * np));
  const auto src = gmem(sg.a);
  // v[u][m]: the child whose place in the parent has bits m (M2M: upper; ROWS:
  // lower), the pair along z in one load
  typedef double dz2 __attribute__((ext_vector_type(2), aligned(8)));
  double v[SPW][8];
#pragma unroll
  for (int u = 0; u < SPW; ++u) {
    const int b = min(4 * (w * SPW + u) + kq, HT - 1);  // (past the last: the table is zero)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int x = q >> 1, y = q & 1;
      if constexpr (ROWS) {
        const long long c = ((long long)(2 * p0 + 1 - x) * nc + 2 * p1 + 1 - y) * nc + 2 * p2;
        v[u][2 * q] = src[(c + 1) * HR + b];
        v[u][2 * q + 1] = src[c * HR + b];
      } else {
        const dz2 t = *(const __attribute__((address_space(1))) dz2*)(src + b * ncc +
                                                                     ((long long)(2 * p0 + x + 3) * nc + 2 * p1 + y + 3) * nc + 2 * p2 + 3);
        v[u][2 * q] = t[0];
        v[u][2 * q + 1] = t[1];
      }
    }
  }
  d4 acc[8][NTC];
#pragma unroll
  for (int e = 0; e < 8; ++e)
#pragma unroll
    for (int t = 0; t < NTC; ++t) acc[e][t] = d4{0, 0, 0, 0};
  const auto wt = gmem(W);
#pragma unroll
  for (int u = 0; u < SPW; ++u) {
    const int s = w * SPW + u;
    if (s >= S::NS) break;  // (uniform)
    const int b = min(4 * s + kq, HT - 1), par = c_ft<P>.par[b];
    double tb[8][NTC], a[8];
    if (!ROWS || sg.b)
#pragma unroll
      for (int e = 0; e < 8; ++e)
#pragma unroll
        for (int t = 0; t < NTC; ++t) tb[e][t] = (wt + ((s * 8 + e) * NTC + t) * 64)[(unsigned)lane];
    fold8<8>(v[u], par & 4 ? -1.0 : 1.0, par & 2 ? -1.0 : 1.0, par & 1 ? -1.0 : 1.0, a);
    if constexpr (ROWS) {
      if (4 * s + kq < HT && P0 + i < nps) {
        const int m = c_ft<P>.deg[b];
        H* const to = static_cast<H*>(sg.u) + (7 * m * m + b) * ncpp + ((long long)(p0 + 3) * npp + p1 + 3) * npp + p2 + 3;
#pragma unroll
        for (int e = 0; e < 8; ++e) to[e * (2 * m + 1) * ncpp] = static_cast<H>(0.125 * a[e]);
      }
      if (!sg.b) continue;
    }
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int t = 0; t < NTC; ++t)
        acc[e][t] = ROWS ? __builtin_amdgcn_mfma_f64_16x16x4f64(a[e], tb[e][t], acc[e][t], 0, 0, 0)
                         : __builtin_amdgcn_mfma_f64_16x16x4f64(tb[e][t], a[e], acc[e][t], 0, 0, 0);
  }
  if (ROWS && !sg.b) return;
#pragma unroll
  for (int e = 0; e < 8; ++e)
#pragma unroll
    for (int t = 0; t < NTC; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        red[(((w * 8 + e) * NTC + t) * 16 + Mf<double>::row(r, kq)) * RS + i] = acc[e][t][r];
  __syncthreads();
  for (int q = threadIdx.x; q < 16 * HT; q += 256) {
    // (rows: the terms of a parent; planes: the parents of a term)
    const int a = ROWS ? q % HT : q >> 4, pl = ROWS ? q / HT : q & 15;
    const long long p = P0 + pl;
    if (p >= nps) continue;
    const int e = c_ft<P>.par[a], j = c_ft<P>.idx[a];
    const int at = ((e * NTC + (j >> 4)) * 16 + (ROWS ? pl : j & 15)) * RS + (ROWS ? j & 15 : pl);
    double x = 0.0;
#pragma unroll
    for (int k = 0; k < 4; ++k) x += red[k * 8 * NTC * 16 * RS + at];
    if constexpr (ROWS) {
      sg.b[p * HR + a] = 0.5 * x;
    } else {
      const int q2 = (int)(p % np), q1 = (int)((p / np) % np), q0 = (int)(p / ((long long)np * np));
      const long long to = a * ncpp + ((long long)(q0 + 3) * npp + q1 + 3) * npp + q2 + 3;
      if (a >= hm) x = 0.0;
      sg.b[to] = x;
      if (sg.u) static_cast<float*>(sg.u)[to] = (float)x;
    }
  }
}

// Scatter.  Segments: n = parents per axis, a = the parents' values, b = the children's (planes: added to), ROWS: c = the
// M2L's rows [parent][frow], sums over the children's signs times 8.
// Block: 16 parents, one wave for each 16 terms b: it holds the 8 classes of a
// (parent, term) in one lane, so the inverse Walsh sum needs no exchange.
// What bounds it: the children's values (transposed M2M of 128^3, p = 6, a level:
// 37 us with a thread per term, 15 with what the results add to read after the
// products, 9 with it read first; L2L of 256^3, 3 levels: 104 -> 87 us).
template <int P, bool ROWS>
__global__ __launch_bounds__(64 * ShiftShape<P>::NTB) void k_scatter(const Seg* __restrict__ segs, int nseg, const Seg one,
                                                                    const double* __restrict__ W) {
  using S = ShiftShape<P>;
  constexpr int HT = S::HT, HR = hrow(P), FR = frow(P), NPS = S::NPS, NTB = S::NTB;
  const Seg& sg = nseg ? find_seg(segs, nseg, blockIdx.x) : one;
  const int np = sg.n, npp = np + 6, nc = 2 * np + (ROWS ? 0 : 6);
  const long long nps = (long long)np * np * np, ncpp = (long long)npp * npp * npp, ncc = (long long)nc * nc * nc;
  const long long P0 = (long long)((int)blockIdx.x - sg.first_block) * 16;
  const int lane = threadIdx.x & 63, i = lane & 15, kq = lane >> 4;
  const int t = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // the lane's 4 results (parent, term), clamped into the grid; what they add to
  // is read before anything else
  typedef double dz2 __attribute__((ext_vector_type(2), aligned(8)));
  const int tb0 = 16 * t;
  double own[4][8];
  long long at[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = Mf<double>::row(r, kq), b = min(tb0 + (ROWS ? i : row), HT - 1);
    const long long p = min(P0 + (ROWS ? row : i), nps - 1);
    const int p2 = (int)(p % np), p1 = (int)((p / np) % np), p0 = (int)(p / ((long long)np * np));
    if constexpr (ROWS) {
      at[r] = (((long long)(2 * p0) * nc + 2 * p1) * nc + 2 * p2) * HR + b;
      const auto from = gmem(sg.c + p * FR + fold_at(0, b));
#pragma unroll
      for (int e = 0; e < 8; ++e) own[r][e] = from[2 * e];
    } else {
      at[r] = b * ncc + ((long long)(2 * p0 + 3) * nc + 2 * p1 + 3) * nc + 2 * p2 + 3;
      const auto from = gmem(sg.b + at[r]);
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const dz2 z = *(const __attribute__((address_space(1))) dz2*)(from + ((long long)(q >> 1) * nc + (q & 1)) * nc);
        own[r][2 * q] = z[0];
        own[r][2 * q + 1] = z[1];
      }
    }
  }
  d4 acc[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) acc[e] = d4{0, 0, 0, 0};
  {
    const long long pc = min(P0 + i, nps - 1);
    const int p2 = (int)(pc % np), p1 = (int)((pc / np) % np), p0 = (int)(pc / ((long long)np * np));
    const auto src = gmem(sg.a + (ROWS ? pc * HR : ((long long)(p0 + 3) * npp + p1 + 3) * npp + p2 + 3));
    const auto wt = gmem(W + S::GATHER + t * 64);
    double v[8][NPS], tb[8][NPS];
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int s = 0; s < NPS; ++s) {
        // (a class's places past its last term: the table is zero)
        v[e][s] = src[max((int)c_ft<P>.pt[e][4 * s + kq], 0) * (ROWS ? 1LL : ncpp)];
        tb[e][s] = (wt + (e * NPS + s) * NTB * 64)[(unsigned)lane];
      }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int e = 0; e < 8; ++e)
#pragma unroll
      for (int s = 0; s < NPS; ++s)
        acc[e] = ROWS ? __builtin_amdgcn_mfma_f64_16x16x4f64(v[e][s], tb[e][s], acc[e], 0, 0, 0)
                      : __builtin_amdgcn_mfma_f64_16x16x4f64(tb[e][s], v[e][s], acc[e], 0, 0, 0);
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = Mf<double>::row(r, kq), b = tb0 + (ROWS ? i : row);
    if (b >= HT || P0 + (ROWS ? row : i) >= nps) continue;
    const int pb = c_ft<P>.par[b];
    double y[8];
    if constexpr (ROWS) {
#pragma unroll
      for (int e = 0; e < 8; ++e) y[e] = fma(0.125, own[r][e], 0.5 * acc[e][r]);
      walsh8(y);
      double* const to = sg.b + at[r];
#pragma unroll
      for (int m = 0; m < 8; ++m)  // minus bits
        to[((long long)((m & 4 ? 0 : 1) * nc + (m & 2 ? 0 : 1)) * nc + (m & 1 ? 0 : 1)) * HR] = chi(pb, m) * y[m];
    } else {
#pragma unroll
      for (int e = 0; e < 8; ++e) y[e] = acc[e][r];
      walsh8(y);
      double* const to = sg.b + at[r];
#pragma unroll
      for (int q = 0; q < 4; ++q)  // upper bits
        *reinterpret_cast<dz2*>(to + ((long long)(q >> 1) * nc + (q & 1)) * nc) =
            dz2{own[r][2 * q] + chi(pb, 2 * q) * y[2 * q], own[r][2 * q + 1] + chi(pb, 2 * q + 1) * y[2 * q + 1]};
    }
  }
}

// Harmonic multipoles of the cells of 4^3 unigrid cells, one thread each.
// Segments: n = unigrid cells per axis, field, b = planes, u = copy in FP32 or
// null.  hm: terms written (the others are zero).
// What bounds it: reading the densities and writing the planes (whole lines, as
// the lanes of a wave run along z).
template <int P, typename TI>
__global__ __launch_bounds__(256) void k_p2mh(const Seg* __restrict__ segs, int nseg, IoArg io, int hm) {
  const Seg& sg = find_seg(segs, nseg, blockIdx.x);
  const int n = sg.n, nk = n >> 2, gp = nk + 6;
  const TI* __restrict__ rho = io_rho<TI>(io, sg.field);
  const long long T = (long long)((int)blockIdx.x - sg.first_block) * 256 + threadIdx.x;
  if (T >= (long long)nk * nk * nk) return;
  const int t2 = (int)(T % nk), t1 = (int)((T / nk) % nk), t0 = (int)(T / ((long long)nk * nk));
  double v[64];
  p2m2_slots(rho + (((long long)4 * t0) * n + 4 * t1) * n + 4 * t2, n, v);
  const long long ncp = (long long)gp * gp * gp, cp = ((long long)(t0 + 3) * gp + t1 + 3) * gp + t2 + 3;
  static_for<P + 1>([&](auto dc) {
    constexpr int m = decltype(dc)::value;
    double d[ndeg(m)];
    static_for<ndeg(m)>([&](auto ec) { d[decltype(ec)::value] = p2m2_term<nterms(m - 1) + decltype(ec)::value>(v); });
    static_for<2 * m + 1>([&](auto rc) {
      constexpr int i = m * m + decltype(rc)::value;
      const double x = i < hm ? h_reduce_deg<i>(d) : 0.0;
      sg.b[i * ncp + cp] = x;
      if (sg.u) static_cast<float*>(sg.u)[i * ncp + cp] = (float)x;
    });
    // (one degree at a time: the scheduler would otherwise form every term
    // before the first store and hold them all in registers)
    __builtin_amdgcn_sched_barrier(0);
  });
}

// Upward pass of a folded field from its unigrid: harmonic multipoles of the
// cells of 4^3 unigrid cells (level k) and of the two levels above.
// Segments: n = unigrid cells per axis, field, split = levels (1 to 3),
// a, c, d = planes of levels k, k - 1, k - 2 (FP64, written), b, t, u = their
// copies in FP32, or null.
// Block: 16^3 unigrid cells, 64 cells of level k, 8 and 1 above.  The lane's cell
// is P2M's (one wave would do; the 4 waves share the terms by degree), its values
// stay in LDS, and the shifts are plain sums of the matrix C over the 8 children's
// sums of a parity: 8 parents would leave half of a matrix product empty.
// What bounds it: on small grids the latency of one pass from the densities to
// the planes, of which separate launches had one each.
constexpr int up_owner(int P, int m) {  // the wave that forms degree m
  int load[4] = {}, own = 0;
  for (int d = P; d >= m; --d) {
    own = 0;
    for (int w = 1; w < 4; ++w)
      if (load[w] < load[own]) own = w;
    load[own] += ndeg(d);
  }
  return own;
}
template <int P, typename TI>
__global__ __launch_bounds__(256) void k_up(const Seg* __restrict__ segs, int nseg, IoArg io,
                                            const double* __restrict__ C, int hm) {
  constexpr int HT = hterms(P), CS = 65;
  __shared__ double cell[HT * CS];         // [term][cell]
  __shared__ double sums[8 * HT * 8];      // [class][term][parent]
  __shared__ double mid[HT * 9];           // [term][level k - 1]
  const Seg& sg = find_seg(segs, nseg, blockIdx.x);
  const int n = sg.n, nk = n >> 2, lb = (int)blockIdx.x - sg.first_block, nr = n >> 4;
  const int b0 = lb / (nr * nr), b1 = (lb / nr) % nr, b2 = lb % nr;
  const TI* __restrict__ rho = io_rho<TI>(io, sg.field);
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  auto put = [&](const double* planes, void* copy, int g, int x, int y, int z, int term, double v) {
    const int gp = g + 6;
    const long long at = term * ((long long)gp * gp * gp) + ((long long)(x + 3) * gp + y + 3) * gp + z + 3;
    const_cast<double*>(planes)[at] = v;
    if (copy) static_cast<float*>(copy)[at] = (float)v;
  };
  {
    const int t0 = 4 * b0 + (lane >> 4), t1 = 4 * b1 + ((lane >> 2) & 3), t2 = 4 * b2 + (lane & 3);
    double v[64];
    p2m2_slots(rho + (((long long)4 * t0) * n + 4 * t1) * n + 4 * t2, n, v);
    static_for<P + 1>([&](auto dc) {
      constexpr int m = decltype(dc)::value;
      if (w != up_owner(P, m)) return;
      double d[ndeg(m)];
      static_for<ndeg(m)>([&](auto ec) { d[decltype(ec)::value] = p2m2_term<nterms(m - 1) + decltype(ec)::value>(v); });
      static_for<2 * m + 1>([&](auto rc) {
        constexpr int i = m * m + decltype(rc)::value;
        const double x = i < hm ? h_reduce_deg<i>(d) : 0.0;
        cell[i * CS + lane] = x;
        put(sg.a, sg.b, nk, t0, t1, t2, i, x);
      });
      // (one degree at a time: the scheduler would otherwise form every term
      // before the first store and hold them all in registers)
      __builtin_amdgcn_sched_barrier(0);
    });
  }
  // sums over the children's signs: chi_{e + parity(b)}; bits of a child: upper
  auto fold = [&](const double* from, int stride, int np, auto child) {
    for (int q = threadIdx.x; q < np * HT; q += 256) {
      const int p = q % np, b = q / np, par = c_ft<P>.par[b];
      double r[8], a[8];
#pragma unroll
      for (int m = 0; m < 8; ++m) r[m] = from[b * stride + child(p, m)];
      fold8<8>(r, par & 4 ? -1.0 : 1.0, par & 2 ? -1.0 : 1.0, par & 1 ? -1.0 : 1.0, a);
#pragma unroll
      for (int e = 0; e < 8; ++e) sums[(e * HT + b) * np + p] = a[e];
    }
  };
  if (sg.split < 2) return;
  __syncthreads();
  fold(cell, CS, 8, [](int p, int m) {
    return 16 * (2 * (p >> 2) + (m >> 2)) + 4 * (2 * ((p >> 1) & 1) + ((m >> 1) & 1)) + 2 * (p & 1) + (m & 1);
  });
  __syncthreads();
  for (int q = threadIdx.x; q < 8 * HT; q += 256) {
    const int p = q & 7, a = q >> 3, nb = hterms(c_ft<P>.deg[a]);
    const double* x = sums + c_ft<P>.par[a] * (HT * 8) + p;
    double v = 0.0;
#pragma unroll 4
    for (int b = 0; b < nb; ++b) v = fma(C[b * HT + a], x[b * 8], v);
    if (a >= hm) v = 0.0;
    mid[a * 9 + p] = v;
    put(sg.c, sg.t, nk >> 1, 2 * b0 + (p >> 2), 2 * b1 + ((p >> 1) & 1), 2 * b2 + (p & 1), a, v);
  }
  if (sg.split < 3) return;
  __syncthreads();
  fold(mid, 9, 1, [](int, int m) { return m; });
  __syncthreads();
  // (4 lanes share a sum)
  for (int q = threadIdx.x; q < 4 * HT; q += 256) {
    const int a = q >> 2, nb = hterms(c_ft<P>.deg[a]);
    const double* x = sums + c_ft<P>.par[a] * HT;
    double v = 0.0;
#pragma unroll 4
    for (int b = q & 3; b < nb; b += 4) v = fma(C[b * HT + a], x[b], v);
    v += __shfl_xor(v, 1);
    v += __shfl_xor(v, 2);
    if (a >= hm) v = 0.0;
    if ((q & 3) == 0) put(sg.d, sg.u, nk >> 2, b0, b1, b2, a, v);
  }
}
