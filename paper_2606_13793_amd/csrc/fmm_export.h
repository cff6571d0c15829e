// Expansions of folded fields in full Cartesian terms, for fmm_debug_expansions.
// Included by fmm_impl.h.
#pragma once

// Multipoles of cells first .. first + gridDim.x - 1 (C order) of a level, [cell][nt
// terms].  The kernels keep harmonic terms only (planes; null for FMM-1's finest
// level, which they do not form): those are theirs, and what harmonic terms leave
// open comes from the copy of the density that the last solve left.  So the full
// sums f_a = sum_s rho_s w_s^a / a!, w = (the cell's centre - s) / its size, are
// formed first, and each harmonic term's difference from the plane is added to the
// full term of the same exponents, which enters that harmonic term alone and with
// weight 1.
// Thread = term; nothing here is on a solve's path.
template <int P, typename TI>
__global__ void k_export_m(const TI* __restrict__ rho, const double* __restrict__ planes, int n, int level, int hm, int nt,
                           long long first, double* __restrict__ out) {
  constexpr int NT = nterms(P), HT = hterms(P);
  __shared__ double pw[(P + 1) * 256];  // (1024 >> 2 places along an axis)
  __shared__ double f[NT];
  const int m = n >> level, nk = 1 << level;
  const long long c = first + blockIdx.x;
  const int c2 = (int)(c % nk), c1 = (int)((c / nk) % nk), c0 = (int)(c / ((long long)nk * nk));
  for (int i = threadIdx.x; i < m; i += blockDim.x) {
    double w = 1.0;
    for (int k = 0; k <= P; ++k, w *= (m - 1 - 2 * i) / (2.0 * m * k)) pw[k * 256 + i] = w;
  }
  __syncthreads();
  const int t = threadIdx.x;
  if (t < NT) {
    const int ex = c_mi_exp[t];
    const double *px = pw + 256 * mi_a(ex), *py = pw + 256 * mi_b(ex), *pz = pw + 256 * mi_c(ex);
    const TI* cell = rho + (((long long)m * c0) * n + m * c1) * n + m * c2;
    double s = 0.0;
    for (int x = 0; x < m; ++x) {
      double sx = 0.0;
      for (int y = 0; y < m; ++y) {
        const TI* row = cell + ((long long)x * n + y) * n;
        double sy = 0.0;
        for (int z = 0; z < m; ++z) sy = fma(pz[z], (double)row[z], sy);
        sx = fma(py[y], sy, sx);
      }
      s = fma(px[x], sx, s);
    }
    f[t] = s;
  }
  __syncthreads();
  double d = 0.0;
  if (planes && t < hm) {
    const int np = nk + 6;
    d = planes[t * ((long long)np * np * np) + ((long long)(c0 + 3) * np + c1 + 3) * np + c2 + 3] -
        h_reduce(t, [&](int a) { return f[a]; });
  }
  __syncthreads();
  if (planes && t < HT) f[c_ft<P>.full[t]] += d;
  __syncthreads();
  if (t < nt) out[blockIdx.x * (long long)nt + t] = f[t];
}
template <int P>
hipError_t export_multipoles(const fmm_plan* pl, int level, long long first, long long cnt, double* dev, hipStream_t s) {
  const double* planes = level <= block_level(pl, pl->F) ? (const double*)pl->lev[level].M : nullptr;
  const dim3 g((unsigned)cnt), th((nterms(P) + 63) / 64 * 64);
  const int hm = hterms(pl->nmax);
  if (pl->precision == 0)
    hipLaunchKernelGGL((k_export_m<P, double>), g, th, 0, s, (const double*)pl->fld[0].rho_copy, planes, pl->n, level, hm,
                       pl->NMX, first, dev);
  else
    hipLaunchKernelGGL((k_export_m<P, float>), g, th, 0, s, (const float*)pl->fld[0].rho_copy, planes, pl->n, level, hm,
                       pl->NMX, first, dev);
  return hipGetLastError();
}

// Complete locals of such cells, [cell][term], full terms from the harmonic ones by
// Laplace's equation.  Lc: the level's complete locals, or null for FMM-1's finest
// level, which keeps its M2L part only, Walsh-folded over each parent's children
// (Lw): that is unfolded, and the shift of the parent's complete local (Lp; null
// where nothing comes from above) added.
template <int P, typename H>
__global__ void k_export_l(const double* __restrict__ Lc, const H* __restrict__ Lw, const double* __restrict__ Lp, int level,
                           long long first, double* __restrict__ out) {
  constexpr int NT = nterms(P), HT = hterms(P), HR = hrow(P), FR = frow(P);
  __shared__ double own[HT];
  __shared__ double par[NT];
  const int nk = 1 << level, t = threadIdx.x;
  const long long c = first + blockIdx.x;
  const int c2 = (int)(c % nk), c1 = (int)((c / nk) % nk), c0 = (int)(c / ((long long)nk * nk));
  const long long pc = ((long long)(c0 >> 1) * (nk / 2) + (c1 >> 1)) * (nk / 2) + (c2 >> 1);
  const int minus = 7 - (((c0 & 1) << 2) | ((c1 & 1) << 1) | (c2 & 1));
  if (t < HT) {
    double v = 0.0;
    if (Lc)
      v = Lc[c * HR + t];
    else
      for (int k = 0; k < 8; ++k) v += 0.125 * chi(k ^ c_ft<P>.par[t], minus) * (double)Lw[pc * FR + fold_at(k, t)];
    own[t] = v;
  }
  const int ex = t < NT ? c_mi_exp[t] : 0, x = mi_a(ex), y = mi_b(ex), z = mi_c(ex);
  auto full = [&](const double* h) {
    const int k = z >> 1;
    double v = 0.0;
    for (int l = 0; l <= k; ++l) v += binom(k, l) * h[h_index(x + 2 * l, y + 2 * (k - l), z & 1)];
    return k & 1 ? -v : v;
  };
  if (t < NT) par[t] = Lp ? full(Lp + pc * HR) : 0.0;
  __syncthreads();
  if (t >= NT) return;
  double v = full(own);
  for (int s = t; s < NT && Lp; ++s) {
    const int es = c_mi_exp[s], gx = mi_a(es) - x, gy = mi_b(es) - y, gz = mi_c(es) - z;
    if (gx < 0 || gy < 0 || gz < 0) continue;
    const double w = chi((gx & 1) << 2 | (gy & 1) << 1 | (gz & 1), minus) * c_mi_invfact[mi_index(gx, gy, gz)];
    v = fma(ldexp(w, -(x + y + z + 1) - 2 * (gx + gy + gz)), par[s], v);
  }
  out[blockIdx.x * (long long)NT + t] = v;
}
template <int P>
hipError_t export_locals(const fmm_plan* pl, int level, long long first, long long cnt, double* dev, hipStream_t s) {
  const Level& lv = pl->lev[level];
  const dim3 g((unsigned)cnt), th((nterms(P) + 63) / 64 * 64);
  if (level <= block_level(pl, pl->F))
    hipLaunchKernelGGL((k_export_l<P, double>), g, th, 0, s, lv.Lc, nullptr, nullptr, level, first, dev);
  else {
    const double* up = level > 3 ? pl->lev[level - 1].Lc : nullptr;
    if (bottom_low(pl, pl->F))
      hipLaunchKernelGGL((k_export_l<P, float>), g, th, 0, s, nullptr, (const float*)lv.Lw, up, level, first, dev);
    else
      hipLaunchKernelGGL((k_export_l<P, double>), g, th, 0, s, nullptr, (const double*)lv.Lw, up, level, first, dev);
  }
  return hipGetLastError();
}
