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
