// Transposes of the folded kernels (fmm_fold.h).  Included by fmm_impl.h.
//
// The solve on the folded kernels is, with all maps linear,
//   Mh_{F-1} = harmonic P2M rho, Mh_{k-1} = M2M Mh_k,
//   Lw_k = M2L Mh_{k-1} (Walsh-folded over children), Lc_k = unfold Lw_k + L2L Lc_{k-1},
//   (phi, g) = unfold(block stencil fold(rho) + L2P Lw_F + L2P' Lc_{F-1}).
// The backward pass runs the transposes in reverse:
//   k_blk_adj_l    cotangents -> Lw_bar_F, Lc_bar_{F-1}          (L2P^T; FMM-2:
//                  Lc_bar_F, and the folded cotangents for M2P^T, k_m2lf OP 3)
//   k_l2lf_adj     Lc_bar_k -> Lw_bar_k, Lc_bar_{k-1}, k = F-1..3
//   k_m2lf (OP 1)  Lw_bar_k -> Mh_bar_{k-1}, every level           (M2L^T)
//   k_m2mf_adj     Mh_bar_{k-1} -> Mh_bar_k (+=), k = 3..F-1
//   k_block_adj    cotangents, Mh_bar_{F-1} -> rho_bar           (stencil^T, P2M^T)
// The interaction relation is symmetric and mirror-symmetric, so each
// transpose gathers over the same 6^3 cells (12^3 unigrid cells) around an oct
// and folds the same way.  L2P^T, the stencil and the chains are FP64 in every
// plan, M2L^T runs in the compute type of the forward M2L of its level.
#pragma once

// The stencil transpose has 8 columns, the sources of the positive octant:
// products of 16 x 4 x 4, fragments of 4 columns and 4 k-groups.
// [4 outputs][54 steps][8 patterns][4 kq][4][2]; then P2M^T,
// [8][blk_psteps][4 kq][4][2]
constexpr __host__ __device__ int blka_off_p() { return 4 * BLK_STEPS * 8 * 32; }
constexpr __host__ __device__ int blka_off_l(int P) { return blka_off_p() + 8 * blk_psteps(P) * 32; }
// L2P^T: own locals [8 steps][tiles][64], level F-1 [8 patterns][8 steps][64]
constexpr __host__ __device__ int blka_ltiles(int P) { return (hterms(P) + 15) / 16; }
constexpr __host__ __device__ int blka_off_lp(int P) { return blka_off_l(P) + 8 * blka_ltiles(P) * 64; }
constexpr __host__ __device__ int blka_table(int P) { return blka_off_lp(P) + 64 * 64; }

template <int P>
__global__ void k_blk_adj_table(const double* __restrict__ G, double* __restrict__ W, int nmax, int dl) {
  constexpr int OFF_P = blka_off_p(), OFF_L = blka_off_l(P), OFF_LP = blka_off_lp(P), END = blka_table(P), np = blk_psteps(P),
                LT = blka_ltiles(P);
  const int id = blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= END) return;
  const bool quads = id < OFF_L;
  const int lane = id & 63, j = quads ? ((id >> 1) & 3) + 4 * (id & 1) : lane & 15, kq = quads ? (id >> 3) & 3 : lane >> 4;
  double x = 0.0;
  if (id < OFF_P) {
    // source sp of the positive octant, targets at y = the 8 images of u
    const int e = (id >> 5) & 7, st = (id >> 8) % BLK_STEPS, o = (id >> 8) / BLK_STEPS, pair = 4 * (st / 6) + kq;
    const int jj[3] = {pair / 6, pair % 6, st % 6};
    for (int minus = 0; minus < 8; ++minus) {
      int t = 0, v = 0, neg = 0;  // the target's place in its own block, the source seen from there, tau
      for (int a = 0; a < 3; ++a) {
        const int u2 = (minus >> (2 - a)) & 1 ? -(2 * jj[a] + 1) : 2 * jj[a] + 1;  // 2 y
        const int B = (u2 + 4 + 16) / 8 - 2, r2 = u2 - 8 * B;                      // block offset, 2 (y - 4 B)
        const int sp2 = 2 * ((j >> (2 - a)) & 1) + 1;
        const int v2 = r2 < 0 ? 8 * B - sp2 : sp2 - 8 * B;
        neg = neg << 1 | (r2 < 0);
        t = t << 1 | (r2 > 2 || r2 < -2);
        v = v * 12 + (v2 + 11) / 2;
      }
      const int eo = o ? 8 >> o : 0;  // the axis of output o
      x += chi(e, minus) * chi(eo, minus) * chi(eo, neg) * G[((size_t)t * 1728 + v) * 4 + o];
    }
  } else if (id < OFF_L) {
    const int s = (id - OFF_P) >> 5, e = s / np;
    const int b = c_ft<P>.pt[e][4 * (s % np) + kq];
    if (b >= 0 && h_degree(b) <= nmax) {
      // P2M weights w^a / a!, w = -(1/8 or 3/8)
      const double w[3] = {(j & 4) ? -0.375 : -0.125, (j & 2) ? -0.375 : -0.125, (j & 1) ? -0.375 : -0.125};
      x = 8.0 * h_reduce(b, [&](int bt) {
            const int ex = c_mi_exp[bt];
            double m = c_mi_invfact[bt];
            for (int i = 0; i < mi_a(ex); ++i) m *= w[0];
            for (int i = 0; i < mi_b(ex); ++i) m *= w[1];
            for (int i = 0; i < mi_c(ex); ++i) m *= w[2];
            return m;
          });
    }
  } else if (id < OFF_LP) {
    const int f = (id - OFF_L) >> 6, s = f / LT, b = 16 * (f % LT) + j;
    if (b < hterms(P)) x = 0.125 * h_reduce(b, [&](int bt) { return l2p_coef(bt, s, kq); });
  } else {
    const int f = (id - OFF_LP) >> 6, e = f >> 3, s = f & 7;
    const int b = j < 4 * np ? c_ft<P>.pt[e][j] : -1;
    if (b >= 0) x = h_reduce(b, [&](int bt) { return blk_l2p(bt, s, kq, dl); });
  }
  W[id] = x;
}

// L2P^T.  A block takes 16 consecutive 4^3 blocks (C order), folds their
// scaled cotangents into Y(e; t, o), and wave e multiplies pattern e by the
// transposed tables: Lw_bar_F columns (e, b) to padded planes
// [column][(nb + 6)^3] in the compute type of the transposed M2L, and the
// terms of parity e of Lc_bar_{F-1}, [block][hrow].  Bound by its traffic
// (reads 4 values a cell, writes 8 (p + 1)^2 a block); the blocks are the columns
// of the products, so that a wave's store to a plane is a run of 16 along z
// straight from its registers (128^3, p = 6: 63 us, through LDS 78).
// FMM-2: no own part; lb takes Y itself, planes [32 e + 4 t + o][(nb + 6)^3].
template <int P, typename TI, typename H, int DL>
__global__ __launch_bounds__(512) void k_blk_adj_l(const TI* __restrict__ dphi, const TI* __restrict__ dg, int n,
                                                   const double* __restrict__ W, H* __restrict__ lb,
                                                   double* __restrict__ lc) {
  constexpr int HR = hrow(P), NT = blka_ltiles(P), HT = hterms(P), NPT = 4 * blk_psteps(P);
  constexpr int OFF_L = blka_off_l(P), OFF_P = blka_off_lp(P);
  constexpr int YS = 33;  // LDS row stride
  __shared__ double lds[8 * 16 * YS];
  const int nb = n >> 2, nbp = nb + 6;
  const long long nblk = (long long)nb * nb * nb, N = (long long)n * n * n, ncp = (long long)nbp * nbp * nbp;
  const long long B0 = (long long)blockIdx.x * 16;
  const double dx = 1.0 / n, sphi = (DL == 1 ? 0.5 : 0.25) * dx * dx, sgr = (DL == 1 ? -0.25 : -0.0625) * dx;
  {
    // thread (o, t, block): blocks fastest
    const int bl = threadIdx.x & 15, t = (threadIdx.x >> 4) & 7, o = threadIdx.x >> 7;
    const long long B = B0 + bl;
    double y[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) y[m] = 0.0;
    if (B < nblk && (o == 0 || dg)) {
      const int b2 = (int)(B % nb), b1 = (int)((B / nb) % nb), b0 = (int)(B / ((long long)nb * nb));
      const TI* src = o == 0 ? dphi : dg + (o - 1) * N;
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const int x = m & 4 ? 1 - ((t >> 2) & 1) : 2 + ((t >> 2) & 1), yy = m & 2 ? 1 - ((t >> 1) & 1) : 2 + ((t >> 1) & 1),
                  z = m & 1 ? 1 - (t & 1) : 2 + (t & 1);
        y[m] = (double)src[((long long)(4 * b0 + x) * n + 4 * b1 + yy) * n + 4 * b2 + z];
      }
    }
    walsh8(y);
    const double sc = o == 0 ? sphi : sgr;
    const int eo = o ? 8 >> o : 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      // (a constant register index: the exchange e ^ eo is done by the LDS address)
      lds[((e ^ eo) * 16 + bl) * YS + 4 * t + o] = sc * y[e];
    }
  }
  __syncthreads();
  if constexpr (DL == 2) {
    const int bl = threadIdx.x & 15;
    const long long B = B0 + bl;
    if (B < nblk) {
      const int b2 = (int)(B % nb), b1 = (int)((B / nb) % nb), b0 = (int)(B / ((long long)nb * nb));
      const long long cp = ((long long)(b0 + 3) * nbp + b1 + 3) * nbp + b2 + 3;
      for (int c = threadIdx.x >> 4; c < 256; c += 32)
        lb[c * ncp + cp] = static_cast<H>(lds[((c >> 5) * 16 + bl) * YS + (c & 31)]);
    }
    if (!lc) return;
  }
  const int lane = threadIdx.x & 63, i = lane & 15, kq = lane >> 4;
  const int e = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  d4 acc[NT], ap = d4{0, 0, 0, 0};
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = d4{0, 0, 0, 0};
#pragma unroll
  for (int s = 0; s < 8; ++s) {
    const double a = lds[(e * 16 + i) * YS + 4 * s + kq];
#pragma unroll
    for (int t = 0; t < NT && DL == 1; ++t)
      acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(W[OFF_L + (s * NT + t) * 64 + lane], a, acc[t], 0, 0, 0);
    if (lc) ap = __builtin_amdgcn_mfma_f64_16x16x4f64(W[OFF_P + (e * 8 + s) * 64 + lane], a, ap, 0, 0, 0);
  }
  // rows of the results: columns b of pattern e, places in class e
  const long long B = B0 + i;
  if (B >= nblk) return;
  if constexpr (DL == 1) {
    const int b2 = (int)(B % nb), b1 = (int)((B / nb) % nb), b0 = (int)(B / ((long long)nb * nb));
    H* const to = lb + ((long long)(b0 + 3) * nbp + b1 + 3) * nbp + b2 + 3;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int b = 16 * t + 4 * v + kq;
        if (b >= HT) continue;
        const int m = c_ft<P>.deg[b];
        to[(7 * m * m + b + e * (2 * m + 1)) * ncp] = static_cast<H>(acc[t][v]);
      }
  }
  if (lc)
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int j = 4 * v + kq, b = j < NPT ? c_ft<P>.pt[e][j] : -1;
      if (b >= 0) lc[B * HR + b] = ap[v];
    }
}

// Transpose of the block stencil (P2P^T, M2P^T and the finest P2M^T), plus the
// P2M^T of level F - 1: rho_bar of a 4^3 block from the cotangents of the 12^3
// cells around, one output (phi, gx, gy, gz) in the LDS tile at a time, and
// the adjoint harmonic multipoles of its own level F-1 cell (planes; or null).
// Tiles and folding as in k_block.  Products of 16 x 4 x 4 (17 cycles; lane =
// column + 4 (row / 4) + 16 (row % 4) of the result), as one of 16 x 16 x 4 (64
// cycles) would have 8 dead columns.  Then table loads bound a wave, so a
// fragment of 8 columns is one load and serves the NX row tiles (128^3, p = 6: 210
// us with 16 columns, 237 with narrow products for one row tile, 133 now; one row
// tile per block, which small grids take to fill the device, 163).
template <int P, typename TI, typename TO, int NX, int DL>
__global__ __launch_bounds__(BLK_THREADS, 2) void k_block_adj(const TI* __restrict__ dphi, const TI* __restrict__ dg,
                                                              const double* __restrict__ W,
                                                              const double* __restrict__ Mb, TO* __restrict__ drho,
                                                              int n, int tpa) {
  typedef double d2v __attribute__((ext_vector_type(2)));
  constexpr int NE = 4, KS = 2, NR = NX, NPS = blk_psteps(P), CS = 9;
  constexpr int EP = KS * 8 * NX * 16 * CS, TILE = blk_tile(NX), SZ = EP > TILE ? EP : TILE;
  __shared__ __attribute__((aligned(16))) double lds[SZ];
  const int nb = n >> 2, lb = blockIdx.x;
  const int bx0 = (lb / (tpa * tpa)) * NX, by0 = ((lb / tpa) % tpa) * 4, bz0 = (lb % tpa) * 4;
  const long long N = (long long)n * n * n;
  const double dx = 1.0 / n;
  const int lane = threadIdx.x & 63, i = lane & 15, kq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), ks = w & 1, e0 = (w >> 1) * NE;
  const double sx0 = e0 ? -1.0 : 1.0;
  constexpr int OFF_P = blka_off_p();
  double acc[NR][NE][2] = {};
  const unsigned quad = (lane >> 4) * 4 + (lane & 3);
  const double* ctr = lds + 6 * BLK_PLANE + blk_row(4 * (i >> 2) + 6) + 4 * (i & 3);
#pragma unroll 1
  for (int o = 0; o < (dg ? 4 : 1); ++o) {
    __syncthreads();
    // the accumulators' scale, with the Walsh sum's 1/8
    const double sc = 0.125 * (o == 0 ? (DL == 1 ? 0.5 : 0.25) * dx * dx : (DL == 1 ? -0.25 : -0.0625) * dx);
    stage_cells<NX>(lds, o == 0 ? dphi : dg + (o - 1) * N, (TI*)nullptr, n, 4 * bx0 - 4, 4 * by0 - 4, 4 * bz0 - 4,
                    [sc](TI v) { return sc * (double)v; });
    __syncthreads();
    // the sign of a minus image along the output's own axis
    const double sx = o == 1 ? -sx0 : sx0, sy = o == 2 ? -1.0 : 1.0, sz = o == 3 ? -1.0 : 1.0;
    const auto wb = gmem(W + o * (BLK_STEPS * 256) + e0 * 32);
    auto bread = [&](int s, d2v (&b)[NE]) {
#pragma unroll
      for (int e = 0; e < NE; ++e) b[e] = *(const __attribute__((address_space(1))) d2v*)(wb + s * 256 + e * 32 + 2 * quad);
    };
    // as in k_block
    double r[NR][8], a[NR][NE];
    d2v b[2][NE];
    const double* p[4];
    auto aread = [&](auto jc) {
#pragma unroll
      for (int m = 0; m < NR; ++m)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          r[m][2 * q] = p[q][m * 4 * BLK_PLANE + 6 + decltype(jc)::value];
          r[m][2 * q + 1] = p[q][m * 4 * BLK_PLANE + 5 - decltype(jc)::value];
        }
    };
    blk_images(ctr, c_blk_place[4 * ks + kq], p);
    bread(6 * ks, b[0]);
    aread(std::integral_constant<int, 0>{});
#pragma unroll 1
    for (int grp = ks; grp < BLK_GROUPS; grp += KS) {
      const int gn = grp + KS < BLK_GROUPS ? grp + KS : ks;  // (past the last: read, not used)
      const int pn = c_blk_place[4 * gn + kq];
      static_for<6>([&](auto jc) {
        constexpr int jz = decltype(jc)::value, u = jz & 1;
#pragma unroll
        for (int m = 0; m < NR; ++m) fold8<NE>(r[m], sx, sy, sz, a[m]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (jz < 5) {
          bread(6 * grp + jz + 1, b[u ^ 1]);
        } else {
          bread(6 * gn, b[u ^ 1]);
          blk_images(ctr, pn, p);
        }
        aread(std::integral_constant<int, (jz + 1) % 6>{});
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int m = 0; m < NR; ++m)
#pragma unroll
          for (int e = 0; e < NE; ++e)
#pragma unroll
            for (int g = 0; g < 2; ++g)
              acc[m][e][g] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[m][e], b[u][e][g], acc[m][e][g], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      });
    }
  }
  // (the shorter K slice takes the multipoles)
  if (Mb && ks == 1) {
    const int cy = min(by0 + (i >> 2), nb - 1), cz = min(bz0 + (i & 3), nb - 1), nbp = nb + 6;
    const long long ncp = (long long)nbp * nbp * nbp;
    const double* wp = W + OFF_P + e0 * (NPS * 32) + 2 * quad;
#pragma unroll
    for (int m = 0; m < NR; ++m) {
      const long long cell = ((long long)(min(bx0 + m, nb - 1) + 3) * nbp + cy + 3) * nbp + cz + 3;
#pragma unroll
      for (int e = 0; e < NE; ++e)
#pragma unroll
        for (int s = 0; s < NPS; ++s) {
          const int bt = c_ft<P>.pt[e0 + e][4 * s + kq];
          // (the stencil's accumulators carry the Walsh sum's 1/8)
          const double v = Mb[(bt >= 0 ? bt : 0) * ncp + cell];
          const d2v b = *reinterpret_cast<const d2v*>(wp + (e * NPS + s) * 32);
#pragma unroll
          for (int g = 0; g < 2; ++g)
            acc[m][e][g] = __builtin_amdgcn_mfma_f64_4x4x4f64(bt >= 0 ? 0.125 * v : 0.0, b[g], acc[m][e][g], 0, 0, 0);
        }
    }
  }
  __syncthreads();
  constexpr int ROWS = NX * 16, ES = ROWS * CS;
#pragma unroll
  for (int m = 0; m < NR; ++m)
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
      for (int g = 0; g < 2; ++g)
        lds[(ks * 8 + e0 + e) * ES + (16 * m + kq + 4 * ((lane >> 2) & 3)) * CS + 4 * g + (lane & 3)] = acc[m][e][g];
  __syncthreads();
  for (int q = threadIdx.x; q < ROWS * 8; q += BLK_THREADS) {
    double* x = lds + (q >> 3) * CS + (q & 7);
    double y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      y[e] = x[e * ES];
#pragma unroll
      for (int k = 1; k < KS; ++k) y[e] += x[(k * 8 + e) * ES];
    }
    walsh8(y);
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e * ES] = y[e];
  }
  __syncthreads();
  const int z = threadIdx.x & 15, y = threadIdx.x >> 4, qy = y & 3, qz = z & 3;
  const int uy = 4 * by0 + y, uz = 4 * bz0 + z;
  const double* const res = lds + ((qy < 2) << 1 | (qz < 2)) * ES + (4 * (y >> 2) + (z >> 2)) * CS +
                            ((qy == 0 || qy == 3) << 1 | (qz == 0 || qz == 3));
  if (uy < n && uz < n)
    static_for<4 * NX>([&](auto xc) {
      constexpr int x = decltype(xc)::value, qx = x & 3;
      constexpr int at = (qx < 2 ? 4 * ES : 0) + (qx == 0 || qx == 3 ? 4 : 0) + 16 * (x >> 2) * CS;
      const int ux = 4 * bx0 + x;
      if (ux < n) drho[((long long)ux * n + uy) * n + uz] = (TO)res[at];
    });
}
