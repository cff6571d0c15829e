// Mirror-folded kernels of the finest level.  Included by fmm_impl.h (needs
// its constant tables and helpers).
//
// An oct (the 8 children of one cell, Sec. 2.2) is its own mirror image about
// its centre along each axis, and so are the 6^3 cells that hold the sources
// of its targets.  With t a target and s a source in the positive octant of
// the oct's centre, and tau, sigma in {+1,-1}^3 their mirror signs,
//   out(tau t, b) = sum_{s, sigma} K(tau t - sigma s) in(sigma s, a)
// and, as a derivative of 1/r of order g picks up the sign of an axis where
// g is odd, K[g](tau t - sigma s) = tau^g K[g](t - tau sigma s).  The sum over
// sigma is a convolution over the group {+1,-1}^3: Walsh sums over the 8
// mirror images turn it into 8 independent products, one per parity pattern e,
//   IN(e; s, a)  = sum_sigma chi_e(sigma) sigma^a in(sigma s, a)
//   OUT(e; t, b) = sum_{s, a} K^(e; t, b; s, a) IN(e; s, a)
//   tau^b out(tau t, b) = 1/8 sum_e chi_e(tau) OUT(e; t, b)
// with 1/8 of the multiply-adds of the unfolded sum (chi_e(sigma) = -1 for
// each axis with e = 1 and sigma = -1).  Pairs that the interaction list
// excludes have zero K; the exclusion is mirror-symmetric too.
#pragma once

// chi_e(sigma) with sigma given by its minus bits
__host__ __device__ __forceinline__ double chi(int e, int minus) {
  int b = e & minus;
  b ^= b >> 2;
  return ((b ^ (b >> 1)) & 1) ? -1.0 : 1.0;
}

// ---------------------------------------------------------------------------
// Finest block kernel.  A block is 4^3 unigrid cells: an oct of level F for
// FMM-1, a level-F cell for FMM-2.  FMM-1: its sources are the 12^3 unigrid cells of the 6^3 level-F cells
// around: M2P of a level-F source is a linear map of its 8 densities (P2M,
// then M2P: 8 numbers fix all its multipoles), so P2M, M2P (Sec. 4) and the
// near field, eq. (direct), are one matrix of 12^3 sources by 64 targets x
// (phi, g), tabulated once per plan for the order and truncation.  Folded, it
// is 8 products of K = 216 by 32 columns.  L2P adds K rows to them:
//  - the own locals (M2L part of the 8 level-F cells), Walsh-folded over the
//    children, K = (p + 1)^2 harmonic terms, the same table for every e;
//  - the complete local of the block's own cell (level F-1 for FMM-1: L2L then
//    L2P as one exact evaluation): only terms of parity e enter pattern e.
// FMM-2: the 12^3 cells around are the near field, eq. (direct), the own local
// is the level-F one, and M2P (k_m2lf, FO_M2P) comes from a buffer in the
// epilogue.
// ---------------------------------------------------------------------------
constexpr int BLK_K = 216, BLK_STEPS = BLK_K / 4;
constexpr int BLK_THREADS = 512;
// LDS tile of densities: (4 NX + 8) x 24 x 24 cells, z rows of 28 (16 lanes
// 4 octs apart in y and z, 4 consecutive z each, then hit distinct banks)
constexpr int BLK_ROW = 28, BLK_PLANE = 24 * BLK_ROW;
constexpr __host__ __device__ int blk_tile(int nx) { return (4 * nx + 8) * BLK_PLANE; }

// row stride of the folded locals per (parent, pattern), in terms
constexpr __host__ __device__ int hrow(int P) { return (hterms(P) + 3) / 4 * 4; }
// K steps of the own-local part: whole groups of 16 terms (a lane takes 4
// consecutive terms, one vector load), then steps of 4
constexpr __host__ __device__ int blk_lsteps(int P) { return (hterms(P) + 3) / 4; }
// reduced term of K index (step s, k group kq) of the own-local part
constexpr __host__ __device__ int blk_lterm(int P, int s, int kq) {
  const int full = hterms(P) / 16 * 4;  // steps in whole groups
  return s < full ? (s / 4) * 16 + 4 * kq + s % 4 : 4 * s + kq;
}
// K steps of the level F-1 part: the most terms of one parity pattern
constexpr __host__ __device__ int blk_psteps(int P) {
  int most = 0;
  for (int e = 0; e < 8; ++e) {
    int c = 0;
    for (int i = 0; i < hterms(P); ++i) c += h_parity(i) == e;
    most = c > most ? c : most;
  }
  return (most + 3) / 4;
}
// the k-th reduced term of parity e, or -1
constexpr __host__ __device__ int blk_pterm(int P, int e, int k) {
  for (int i = 0; i < hterms(P); ++i)
    if (h_parity(i) == e && k-- == 0) return i;
  return -1;
}
// table layout (elements): the folded stencil [54][8][2][64], the own locals
// [steps][2][64], the level F-1 locals [8][steps][2][64]
constexpr __host__ __device__ int blk_off_l() { return BLK_STEPS * 8 * 2 * 64; }
constexpr __host__ __device__ int blk_off_p(int P) { return blk_off_l() + blk_lsteps(P) * 2 * 64; }
constexpr __host__ __device__ int blk_table(int P) { return blk_off_p(P) + 8 * blk_psteps(P) * 2 * 64; }

// The unfolded stencil G[t][v][o], t in the positive octant (bits: 1/2 or 3/2
// from the centre), v = (12 v0 + v1) 12 + v2 the source, in the units of the
// bottom accumulators (phi = dx^2/2 acc, g = -dx/4 acc).
__global__ void k_blk_green(const double* __restrict__ Dtab, double* __restrict__ G, int NMX, int ND, int dl) {
  const int id = blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= 8 * 1728 * 4) return;
  const int o = id & 3, v = (id >> 2) % 1728, t = (id >> 2) / 1728;
  const int vv[3] = {v / 144, (v / 12) % 12, v % 12};
  const int tb[3] = {(t >> 2) & 1, (t >> 1) & 1, t & 1};
  int d[3];
  bool near = true;
  for (int a = 0; a < 3; ++a) {
    d[a] = 3 - (vv[a] >> 1);
    near = near && d[a] >= -1 && d[a] <= 1;
  }
  double x = 0.0;
  if (dl == 2) {
    x = p2p2_delta_coef(6 + tb[0] - vv[0], 6 + tb[1] - vv[1], 6 + tb[2] - vv[2], o);
  } else if (near) {
    const int dt = (9 + tb[0] - vv[0]) * 49 + (9 + tb[1] - vv[1]) * 7 + (9 + tb[2] - vv[2]);
    x = o == 0 ? 2.0 * c_p2p_phi[dt] : -4.0 * c_p2p_g[(o - 1) * 343 + dt];
  } else {
    const int dd = (d[0] + 3) * 49 + (d[1] + 3) * 7 + d[2] + 3;
    const double* D = Dtab + ((size_t)dd * 8 + t) * ND;
    for (int al = 0; al < NMX; ++al) {
      const int ex = c_mi_exp[al];
      const int ax = mi_a(ex), ay = mi_b(ex), az = mi_c(ex);
      double c = ldexp(c_mi_invfact[al], -2 * (ax + ay + az));
      if (((vv[0] & ax) + (vv[1] & ay) + (vv[2] & az)) & 1) c = -c;
      x = fma(c, D[mi_index(ax + (o == 1), ay + (o == 2), az + (o == 3))], x);
    }
  }
  G[id] = x;
}

// L2P from the complete local of the block's cell to target t of the positive
// octant, in the units of the accumulators.
__device__ __forceinline__ double blk_l2p(int bt, int t, int o, int dl) {
  if (dl == 1) return l2p_parent_coef(bt, 7, t, o);
  const double w[3] = {(t & 4) ? 0.375 : 0.125, (t & 2) ? 0.375 : 0.125, (t & 1) ? 0.375 : 0.125};
  return l2p_w_coef(bt, w, 1.0, 1.0, o);
}

// The block kernel's B table in the compute type (layout above); lane = j +
// 16 kq, column 16 tile + j = (t, o).  The 1/8 of the inverse Walsh sum is
// left to the epilogue.
template <typename H>
__global__ void k_blk_table(const double* __restrict__ G, H* __restrict__ W, int P, int dl) {
  const int id = blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= blk_table(P)) return;
  const int lane = id & 63, tile = (id >> 6) & 1, j = lane & 15, kq = lane >> 4, col = 16 * tile + j;
  const int t = col >> 2, o = col & 3;
  double x = 0.0;
  if (id < blk_off_l()) {
    const int e = (id >> 7) & 7, k = 4 * (id >> 10) + kq;
    const int jj[3] = {k / 36, (k / 6) % 6, k % 6};
    for (int minus = 0; minus < 8; ++minus) {
      int v = 0;
      for (int a = 0; a < 3; ++a) v = v * 12 + (((minus >> (2 - a)) & 1) ? 5 - jj[a] : 6 + jj[a]);
      x += chi(e, minus) * G[((size_t)t * 1728 + v) * 4 + o];
    }
  } else if (id < blk_off_p(P)) {
    const int b = blk_lterm(P, (id - blk_off_l()) >> 7, kq);
    if (b < hterms(P)) x = h_reduce(b, [&](int bt) { return l2p_coef(bt, t, o); });
  } else {
    const int s = (id - blk_off_p(P)) >> 7, np = blk_psteps(P), e = s / np;
    const int b = blk_pterm(P, e, 4 * (s % np) + kq);
    if (b >= 0) x = 8.0 * h_reduce(b, [&](int bt) { return blk_l2p(bt, t, o, dl); });
  }
  W[id] = static_cast<H>(x);
}

// (pattern, term) of folded-local column col (columns sorted by the degree of
// the term, the pattern slow inside a degree), packed pattern << 8 | term; -1
// past the last
constexpr __host__ __device__ int m2lf_col(int P, int col) {
  if (col >= 8 * hterms(P)) return -1;
  const int m = h_degree(col / 8), in = col - 8 * m * m;
  return (in / (2 * m + 1)) << 8 | (m * m + in % (2 * m + 1));
}
// Index tables of the folded kernels of one order.
template <int P>
struct FoldTab {
  short col[8 * hterms(P)];             // m2lf_col
  unsigned char full[hterms(P)];        // full-term index of a reduced term
  unsigned char par[hterms(P)];         // its parity pattern
  signed char pt[8][4 * blk_psteps(P)];  // blk_pterm
  constexpr FoldTab() : col(), full(), par(), pt() {
    for (int i = 0; i < 8 * hterms(P); ++i) col[i] = (short)m2lf_col(P, i);
    int cnt[8] = {};
    for (auto& row : pt)
      for (auto& v : row) v = -1;
    for (int i = 0; i < hterms(P); ++i) {
      const int ex = h_exp(i), e = h_parity(i);
      full[i] = (unsigned char)mi_index(ex & 255, (ex >> 8) & 255, ex >> 16);
      par[i] = (unsigned char)e;
      pt[e][cnt[e]++] = (signed char)i;
    }
  }
};
template <int P>
__constant__ const FoldTab<P> c_ft = FoldTab<P>();

// in-place Walsh transform of 8 values
template <typename H>
__device__ __forceinline__ void walsh8(H (&y)[8]) {
#pragma unroll
  for (int bit = 1; bit < 8; bit <<= 1)
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (!(e & bit)) {
        const H u = y[e], v = y[e | bit];
        y[e] = u + v;
        y[e | bit] = u - v;
      }
}

// Walsh sums of the 8 mirror images r[minus bits] for the NE patterns
// NE eg .. NE eg + NE - 1: s = the weight of the minus images along each axis,
// chi of the axis where eg fixes it (x for NE <= 4; y for NE <= 2; z for NE = 1) times the
// images' own sign.
template <int NE, typename H>
__device__ __forceinline__ void fold8(const H (&r)[8], H sx, H sy, H sz, H (&a)[NE]) {
  H x[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) x[q] = fma(sx, r[4 + q], r[q]);
  if constexpr (NE == 8) {
    H y[4];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int q = 0; q < 4; ++q) y[q] = h ? fma(-sx, r[4 + q], r[q]) : x[q];
      const H p0 = fma(sy, y[2], y[0]), p1 = fma(sy, y[3], y[1]), m0 = fma(-sy, y[2], y[0]), m1 = fma(-sy, y[3], y[1]);
      a[4 * h] = fma(sz, p1, p0);
      a[4 * h + 1] = fma(-sz, p1, p0);
      a[4 * h + 2] = fma(sz, m1, m0);
      a[4 * h + 3] = fma(-sz, m1, m0);
    }
  } else if constexpr (NE == 4) {
    const H p0 = fma(sy, x[2], x[0]), p1 = fma(sy, x[3], x[1]), m0 = fma(-sy, x[2], x[0]), m1 = fma(-sy, x[3], x[1]);
    a[0] = fma(sz, p1, p0);
    a[1] = fma(-sz, p1, p0);
    a[2] = fma(sz, m1, m0);
    a[3] = fma(-sz, m1, m0);
  } else {
    const H y0 = fma(sy, x[2], x[0]), y1 = fma(sy, x[3], x[1]);
    if constexpr (NE == 2) {
      a[0] = fma(sz, y1, y0);
      a[1] = fma(-sz, y1, y0);
    } else {
      a[0] = fma(sz, y1, y0);
    }
  }
}

// Segments: n = unigrid cells per axis, tpa = tiles along y and z, tz = tiles
// along x, field, t = copy of the density to leave in the plan (or null),
// u = own locals [block][8][hrow] in the compute type (or null: F = 2),
// d = complete locals of the blocks' cells [block][hrow] (or null), c = FMM-2:
// M2P, [block][4][4^3] in the compute type.
// Tile: NX x 4 x 4 blocks; wave w takes row tile X = w % NX (the 4 x 4 blocks
// of plane X) and the NX patterns from NX (w / NX).
// What bounds it: the matrix cores (54 + 13 + 3 K steps of 16 products per row
// tile at p = 6).  A lane reads the 8 mirror images of its operand from the LDS
// tile and folds them itself (12 adds for 8 products); B is read through the
// caches, each fragment once per wave, the NX waves of a plane sharing it.
template <int P, typename CT, typename TI, typename TO, int NX, int DL>
__global__ __launch_bounds__(BLK_THREADS, (blk_tile(NX) * sizeof(typename Mf<CT>::H) > 80000 ? 2 : 4)) void k_block(const Seg* __restrict__ segs, int nseg, IoArg io,
                                                          const typename Mf<CT>::H* __restrict__ W,
                                                          unsigned int* __restrict__ stamp_cnt,
                                                          unsigned long long* __restrict__ stamp_done) {
  using M = Mf<CT>;
  using H = typename M::H;
  using Acc = typename M::Acc;
  constexpr int NE = NX, HR = hrow(P), NLS = blk_lsteps(P), NPS = blk_psteps(P);
  constexpr int OFF_L = blk_off_l(), OFF_P = blk_off_p(P);
  // epilogue image of the block's results, [8][NX * 16][33]
  constexpr int EP = 8 * NX * 16 * 33, TILE = blk_tile(NX), SZ = EP > TILE ? EP : TILE;
  __shared__ __attribute__((aligned(16))) H lds[SZ];
  __shared__ int spt[8 * NPS * 4];
  const Seg& sg = find_seg(segs, nseg, blockIdx.x);
  const int n = sg.n, nb = n >> 2;
  const TI* __restrict__ rho = io_rho<TI>(io, sg.field);
  TO* __restrict__ phi = io_phi<TO>(io, sg.field);
  TO* __restrict__ g = io_g<TO>(io, sg.field);
  TI* __restrict__ keep = static_cast<TI*>(sg.t);
  const int lb = blockIdx.x - sg.first_block;
  const int bx0 = (lb / (sg.tpa * sg.tpa)) * NX, by0 = ((lb / sg.tpa) % sg.tpa) * 4, bz0 = (lb % sg.tpa) * 4;
  for (int t = threadIdx.x; t < 8 * NPS * 4; t += BLK_THREADS) spt[t] = c_ft<P>.pt[t / (NPS * 4)][t % (NPS * 4)];
  // the densities of the tile and 4 cells around, zero outside the grid
  {
    constexpr int CNT = (4 * NX + 8) * 24 * 24, FB = 9;
    const int x0 = 4 * bx0 - 4, y0 = 4 * by0 - 4, z0 = 4 * bz0 - 4;
    const auto grho = gmem(rho);
#pragma unroll 1
    for (int e0 = threadIdx.x; e0 < CNT; e0 += FB * BLK_THREADS) {
      TI v[FB];
#pragma unroll
      for (int u = 0; u < FB; ++u) {
        const int e = e0 + u * BLK_THREADS, z = z0 + e % 24, y = y0 + (e / 24) % 24, x = x0 + e / 576;
        const bool in = e < CNT && x >= 0 && y >= 0 && z >= 0 && x < n && y < n && z < n;
        v[u] = in ? grho[((long long)x * n + y) * n + z] : TI(0);
      }
#pragma unroll
      for (int u = 0; u < FB; ++u) {
        const int e = e0 + u * BLK_THREADS, tz = e % 24, ty = (e / 24) % 24, tx = e / 576;
        if (e < CNT) {
          lds[tx * BLK_PLANE + ty * BLK_ROW + tz] = static_cast<H>(v[u]);
          if (keep && tx >= 4 && tx < 4 * NX + 4 && ty >= 4 && ty < 20 && tz >= 4 && tz < 20 && x0 + tx < n &&
              y0 + ty < n && z0 + tz < n)
            keep[((long long)(x0 + tx) * n + y0 + ty) * n + z0 + tz] = v[u];
        }
      }
    }
  }
  const int lane = threadIdx.x & 63, i = lane & 15, kq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), X = w % NX, eg = w / NX, e0 = eg * NE;
  const H sx = (e0 & 4) ? H(-1) : H(1), sy = (e0 & 2) ? H(-1) : H(1), sz = (e0 & 1) ? H(-1) : H(1);
  Acc acc[NE][2];
#pragma unroll
  for (int e = 0; e < NE; ++e) acc[e][0] = acc[e][1] = Acc{0, 0, 0, 0};
  __syncthreads();
  // ---- the 12^3 densities: K index k = (36 jx + 6 jy + jz), image "plus" at
  // centre + j, "minus" at centre - 1 - j along each axis
  {
    const H* ctr = lds + (4 * X + 6) * BLK_PLANE + (4 * (i >> 2) + 6) * BLK_ROW + 4 * (i & 3) + 6;
    int jx = 0, jy = 0, jz = kq;
    auto aread = [&](H (&r)[8]) {
      const int px = jx * BLK_PLANE, mx = -BLK_PLANE - px, py = jy * BLK_ROW, my = -BLK_ROW - py;
      const H *pp = ctr + px + py, *pm = ctr + px + my, *mp = ctr + mx + py, *mm = ctr + mx + my;
      r[0] = pp[jz];
      r[1] = pp[-1 - jz];
      r[2] = pm[jz];
      r[3] = pm[-1 - jz];
      r[4] = mp[jz];
      r[5] = mp[-1 - jz];
      r[6] = mm[jz];
      r[7] = mm[-1 - jz];
      jz += 4;
      if (jz >= 6) {
        jz -= 6;
        if (++jy == 6) {
          jy = 0;
          jx = jx < 5 ? jx + 1 : 5;  // (past the last step: a read that is not used)
        }
      }
    };
    const auto wb = gmem(W + e0 * 128 + lane);
    auto bread = [&](int s, H (&b)[NE][2]) {
#pragma unroll
      for (int e = 0; e < NE; ++e)
#pragma unroll
        for (int t = 0; t < 2; ++t) b[e][t] = wb[s * 1024 + e * 128 + t * 64];
    };
    H r[2][8], b[2][NE][2], a[NE];
    aread(r[0]);
    bread(0, b[0]);
#pragma unroll 1
    for (int s = 0; s < BLK_STEPS; s += 2) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int sn = s + u + 1 < BLK_STEPS ? s + u + 1 : BLK_STEPS - 1;
        bread(sn, b[u ^ 1]);
        aread(r[u ^ 1]);
        fold8<NE>(r[u], sx, NE <= 2 ? sy : H(1), NE == 1 ? sz : H(1), a);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int e = 0; e < NE; ++e) {
          acc[e][0] = M::op(a[e], b[u][e][0], acc[e][0]);
          acc[e][1] = M::op(a[e], b[u][e][1], acc[e][1]);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  // ---- L2P; the lane's block, clamped into the grid
  const int cx = min(bx0 + X, nb - 1), cy = min(by0 + (i >> 2), nb - 1), cz = min(bz0 + (i & 3), nb - 1);
  const long long cell = ((long long)cx * nb + cy) * nb + cz;
  if (sg.u) {
    typedef H h4 __attribute__((ext_vector_type(4)));
    const auto own = gmem(static_cast<const H*>(sg.u) + (cell * 8 + e0) * HR);
    const H* wl = W + OFF_L + lane;
    constexpr int FULL = hterms(P) / 16;
#pragma unroll 1
    for (int c = 0; c < FULL; ++c) {
      h4 a[NE];
#pragma unroll
      for (int e = 0; e < NE; ++e)
        a[e] = *(const __attribute__((address_space(1))) h4*)(own + e * HR + 16 * c + 4 * kq);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const H b0 = wl[(4 * c + v) * 128], b1 = wl[(4 * c + v) * 128 + 64];
#pragma unroll
        for (int e = 0; e < NE; ++e) {
          acc[e][0] = M::op(a[e][v], b0, acc[e][0]);
          acc[e][1] = M::op(a[e][v], b1, acc[e][1]);
        }
      }
    }
#pragma unroll
    for (int s = 4 * FULL; s < NLS; ++s) {
      const H b0 = wl[s * 128], b1 = wl[s * 128 + 64];
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        const H a = own[e * HR + 4 * s + kq];
        acc[e][0] = M::op(a, b0, acc[e][0]);
        acc[e][1] = M::op(a, b1, acc[e][1]);
      }
    }
  }
  if (sg.d) {
    const auto par = gmem(sg.d + cell * HR);
    const H* wp = W + OFF_P + e0 * (NPS * 128) + lane;
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
      for (int s = 0; s < NPS; ++s) {
        const int bt = spt[(e0 + e) * (NPS * 4) + 4 * s + kq];
        const double v = par[bt >= 0 ? bt : 0];
        const H a = bt >= 0 ? static_cast<H>(v) : H(0);
        acc[e][0] = M::op(a, wp[(e * NPS + s) * 128], acc[e][0]);
        acc[e][1] = M::op(a, wp[(e * NPS + s) * 128 + 64], acc[e][1]);
      }
  }
  // ---- inverse Walsh sums over the patterns: results to LDS as [pattern]
  // [block][33], each thread transforms whole octets in place, then the block
  // writes z runs of 16 unigrid cells
  __syncthreads();
  constexpr int NR = NX * 16, ES = NR * 33;
#pragma unroll
  for (int e = 0; e < NE; ++e)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int v = 0; v < 4; ++v) lds[(e0 + e) * ES + (16 * X + M::row(v, kq)) * 33 + 16 * t + i] = acc[e][t][v];
  __syncthreads();
#pragma unroll 1
  for (int q = threadIdx.x; q < NR * 32; q += BLK_THREADS) {
    H* x = lds + (q >> 5) * 33 + (q & 31);
    H y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = x[e * ES];
    walsh8(y);
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e * ES] = y[e];
  }
  __syncthreads();
  // phi = sphi acc, g_d = sgr tau_d acc, with the Walsh sum's 1/8 in acc
  const H* const m2p = reinterpret_cast<const H*>(sg.c);
  const double dx = 1.0 / n, sphi = (DL == 1 ? 0.5 : 0.25) * dx * dx, sgr = (DL == 1 ? -0.25 : -0.0625) * dx;
  const long long N = (long long)n * n * n;
  const int ncomp = g ? 4 : 1;
#pragma unroll 1
  for (int q = threadIdx.x; q < 4 * NX * 256 * ncomp; q += BLK_THREADS) {
    const int z = q & 15, y = (q >> 4) & 15, x = (q >> 8) % (4 * NX), o = (q >> 8) / (4 * NX);
    const int ux = 4 * bx0 + x, uy = 4 * by0 + y, uz = 4 * bz0 + z;
    if (ux >= n || uy >= n || uz >= n) continue;
    // position in the block 0..3: the minus images are 0, 1 (3/2, 1/2 out)
    const int qx = x & 3, qy = y & 3, qz = z & 3;
    const int minus = ((qx < 2) << 2) | ((qy < 2) << 1) | (qz < 2);
    const int t = ((qx == 0 || qx == 3) << 2) | ((qy == 0 || qy == 3) << 1) | (qz == 0 || qz == 3);
    const int row = 16 * (x >> 2) + 4 * (y >> 2) + (z >> 2);
    double val = 0.125 * (double)lds[minus * ES + row * 33 + 4 * t + o];
    if (o && (minus >> (3 - o)) & 1) val = -val;
    if constexpr (DL == 2)
      val += (double)m2p[((((long long)(ux >> 2) * nb + (uy >> 2)) * nb + (uz >> 2)) * 4 + o) * 64 + (qx * 4 + qy) * 4 + qz];
    const long long u = ((long long)ux * n + uy) * n + uz;
    if (o == 0)
      phi[u] = (TO)(sphi * val);
    else
      g[(o - 1) * N + u] = (TO)(sgr * val);
  }
  if (stamp_cnt) {
    // the field's last block records when the field is complete
    __syncthreads();
    if (threadIdx.x == 0) {
      __threadfence();
      if (atomicAdd(stamp_cnt + sg.field, 1u) == (unsigned int)(sg.tpa * sg.tpa * sg.tz) - 1)
        stamp_done[sg.field] = wall_clock64();
    }
  }
}

// ---------------------------------------------------------------------------
// M2L, eq. (M2L), folded.  Rows are the octs O of the source grid (level
// k - 1); the sources are the 6^3 cells around (27 in the positive octant),
// the targets the 64 level-k children of the oct's 8 cells P.  Both sides keep
// harmonic terms only, and |a| + |b| <= p.
// Columns (kappa, b): the targets of the positive octant are the 8 children of
// its cell P; their Walsh pattern kappa over those children takes the place of
// the child, so that a row of the result is already folded the way k_block
// reads it:
//   Lw[P][kappa][b] = sum_children chi_kappa(sigma) sigma^b L(child, b)
//                   = chi_kappa(tau) sum_e chi_e(tau) OUT(e; kappa, b) / 8,
// P the cell tau of the oct.  Columns are sorted by |b| (kappa slow inside a
// degree), K by |a| (K index 27 a + source), so a tile of 16 columns needs a
// prefix of K: ceil(27 (p - |b| + 1)^2 / 4) steps.
// ---------------------------------------------------------------------------
constexpr __host__ __device__ int fold_ntiles(int op, int P) {
  return op == FO_M2L ? (8 * hterms(P) + 15) / 16 : op == FO_M2P ? 16 : (hterms(P) + 15) / 16;
}
constexpr __host__ __device__ int fold_steps(int op, int P, int nmax, int t) {
  if (op == FO_M2P) return (27 * hterms(nmax) + 3) / 4;
  const int m = h_degree(op == FO_M2L ? 16 * t / 8 : 16 * t);
  if (op == FO_M2L) return (27 * hterms(P - m < nmax ? P - m : nmax) + 3) / 4;
  return m > nmax ? 0 : op == FO_M2LT ? 54 * hterms(P - m) : 27 * 64;
}

// B fragments in the compute type, [fragment (tile, step)][8 patterns][64];
// tiles[t] = (steps, first fragment).
template <typename H>
__global__ void k_m2lf_table(const double* __restrict__ Dtab, const int2* __restrict__ tiles, H* __restrict__ W, int P,
                             int nmax, int ND, long long cnt) {
  const long long id = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (id >= cnt) return;
  const int lane = (int)(id & 63), e = (int)(id >> 6) & 7, f = (int)(id >> 9);
  int t = 0;
  while (tiles[t].y + tiles[t].x <= f) ++t;
  const int k = 4 * (f - tiles[t].y) + (lane >> 4), cb = m2lf_col(P, 16 * t + (lane & 15));
  const int a = k / 27, s = k % 27, kap = cb >> 8, b = cb & 255;
  double x = 0.0;
  if (cb >= 0 && a < hterms(nmax) && h_degree(a) + h_degree(b) <= P) {
    const int ea = h_exp(a), eb = h_exp(b), pa = h_parity(a), pb = h_parity(b);
    const int g = mi_index(mi_a(ea) + mi_a(eb), mi_b(ea) + mi_b(eb), mi_c(ea) + mi_c(eb));
    const int j[3] = {s / 9, (s / 3) % 3, s % 3};
    for (int minus = 0; minus < 8; ++minus) {
      int dd = 0;
      bool near = true;
      for (int ax = 0; ax < 3; ++ax) {
        const int d = (minus >> (2 - ax)) & 1 ? j[ax] + 1 : -j[ax];
        near = near && d >= -1 && d <= 1;
        dd = dd * 7 + d + 3;
      }
      if (near) continue;
      double y = 0.0;
      for (int q = 0; q < 8; ++q) y += chi(kap ^ pb, 7 - q) * Dtab[((size_t)dd * 8 + q) * ND + g];
      x += chi(e ^ pa, minus) * y;
    }
    x = ldexp(x, -(h_degree(b) + 1) - 3);
  }
  W[id] = static_cast<H>(x);
}

// OP 1 is the transpose: rows are the octs of source cells J, the operands the
// cotangents of the Lw rows of the 27 x 8 cells P around (K index 27 column +
// P, columns sorted by |b|; an image's sign is chi_kappa), columns the terms a
// of one J, the results M_bar(J = sigma, a) = sigma^a sum_e chi_e(sigma) OUT(e; a).
// OP 2 is FMM-2's M2P (Sec. 4): rows are the octs of level F, K as in M2L with
// every term, columns (o, t) the outputs at the 4^3 unigrid cells t of the
// positive octant's cell.  OP 3 is its transpose: K index 27 (32 kappa + 4 t + o)
// + P over the cotangents of the cells P, folded about each P's own centre.
//
// Segments: n = source grid cells per axis, tpa = tiles along y and z, tz =
// tiles along x; OP 0: a = harmonic multipoles of the source grid in the compute
// type, [term][(n + 6)^3] (terms padded to a multiple of 4), u = result in the
// compute type or b = result in FP64, [n^3][8][hrow]; OP 2: the same, u =
// [n^3][4][4^3]; OP 1, 3: a = cotangent planes [K term][(n + 6)^3] in the compute
// type, b = result, planes [term][(n + 6)^3].
// Tile: MT x 4 x 4 octs.  8 waves: 8 / NE groups of NE patterns, KS slices of
// the K steps, MT / NR groups of NR row tiles (a row tile: the 4 x 4 octs of a
// plane).  A block sums NT column tiles over all 8 patterns, so the inverse
// Walsh sums happen in its epilogue.  Blocks: column groups x T tiles, the
// heaviest group (lowest degrees) first; a group whose K loop is long against
// the launch shares it among several blocks (grid.parts), each summing a run
// of chunks: they leave their sums in `part`, which k_m2lf_sum adds in order.
// What bounds it: the matrix cores.  LDS holds 4 terms of the tile's cells and
// 2 around; a lane reads the 8 mirror images of an operand and folds them (8
// adds for two patterns), which NT products amortise; each B fragment is read
// from L2 once per wave for NR row tiles.
//
// what column col stands for, -1 past the last
template <int P, int OP>
__device__ __forceinline__ int fold_colmap(int col) {
  if constexpr (OP == 0) return col < 8 * hterms(P) ? c_ft<P>.col[col] : -1;
  return col < (OP == 2 ? 256 : hterms(P)) ? col : -1;
}
// result q of a group of row tiles: consecutive threads take the columns of a
// row, or for planes the rows
template <int OP, int NT>
__device__ __forceinline__ int m2lf_qcol(int q) { return OP & 1 ? (q >> 4) % (16 * NT) : q % (16 * NT); }
template <int OP, int NT>
__device__ __forceinline__ int m2lf_qrow(int q) { return OP & 1 ? q & 15 : (q / (16 * NT)) & 15; }
// inverse Walsh sum over the patterns, to the 8 cells of the oct of `row`
template <int P, typename H, int OP>
__device__ __forceinline__ void m2lf_put(const Seg& sg, int cb, int ox, int oy0, int oz0, int row, double (&y)[8]) {
  constexpr int HR = hrow(P);
  const int ns = sg.n, nsp = ns + 6, no = ns >> 1, oy = oy0 + (row >> 2), oz = oz0 + (row & 3);
  if (cb < 0 || ox >= no || oy >= no || oz >= no) return;
  walsh8(y);
  if constexpr (OP == 2) {
    H* const ut = static_cast<H*>(sg.u);
    const int o = cb >> 6, eo = o ? 8 >> o : 0, t0 = (cb >> 4) & 3, t1 = (cb >> 2) & 3, t2 = cb & 3;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const long long p = ((long long)(2 * ox + 1 - ((m >> 2) & 1)) * ns + (2 * oy + 1 - ((m >> 1) & 1))) * ns +
                          (2 * oz + 1 - (m & 1));
      const int pos = ((m & 4 ? 3 - t0 : t0) * 4 + (m & 2 ? 3 - t1 : t1)) * 4 + (m & 1 ? 3 - t2 : t2);
      ut[(p * 4 + o) * 64 + pos] = static_cast<H>(m & eo ? -y[m] : y[m]);
    }
  } else if constexpr (OP & 1) {
    const int pa = c_ft<P>.par[cb];
    const long long ncellp = (long long)nsp * nsp * nsp;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const long long c = ((long long)(2 * ox + 4 - ((m >> 2) & 1)) * nsp + (2 * oy + 4 - ((m >> 1) & 1))) * nsp +
                          (2 * oz + 4 - (m & 1));
      sg.b[cb * ncellp + c] = chi(pa, m) * y[m];
    }
  } else {
    const int kap = cb >> 8, b = cb & 255;
    H* const ut = static_cast<H*>(sg.u);
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      // cell tau of the oct: minus bits m
      const long long p = ((long long)(2 * ox + 1 - ((m >> 2) & 1)) * ns + (2 * oy + 1 - ((m >> 1) & 1))) * ns +
                          (2 * oz + 1 - (m & 1));
      const double v = chi(kap, m) * y[m];
      if (ut)
        ut[(p * 8 + kap) * HR + b] = static_cast<H>(v);
      else
        sg.b[(p * 8 + kap) * HR + b] = v;
    }
  }
}
template <int P, typename CT, int OP, int MT, int NT, int NE, int KS>
__global__ __launch_bounds__(512, 2) void k_m2lf(const Seg* __restrict__ segs, int nseg, int T,
                                                 const int2* __restrict__ tiles,
                                                 const typename Mf<CT>::H* __restrict__ W, const M2lGrid grid,
                                                 double* __restrict__ part) {
  using M = Mf<CT>;
  using H = typename M::H;
  using Acc = typename M::Acc;
  constexpr int NR = MT * KS / NE, NG = 8 / NE, NX = MT / NR;
  static_assert(NG * KS * NX == 8, "8 waves");
  constexpr int CELLS = (2 * MT + 4) * 144, CS = 16 * NT + 1;
  constexpr int EP = KS * NX * 8 * 16 * CS, SZ = EP > 4 * CELLS ? EP : 4 * CELLS;
  __shared__ __attribute__((aligned(16))) H lds[SZ];
  __shared__ int4 ktab[108];  // per K index of a chunk: plus image, and the distances to the minus ones
  constexpr int NTERM = OP == 3 ? 256 : OP == 1 ? 8 * hterms(P) : hrow(P);
  __shared__ float4 tsg[NTERM];  // per K term: the sign of a minus image along each axis
  __shared__ int scol[16 * NT];
  int grp = 0;
  while (grp + 1 < grid.ng && (int)blockIdx.x >= grid.first[grp + 1]) ++grp;
  const int T0 = grp * NT, np = grid.parts[grp], rb = (int)blockIdx.x - grid.first[grp], lbk = rb / np, ip = rb % np;
  const Seg& sg = find_seg(segs, nseg, lbk);
  const int nsp = sg.n + 6, tb = lbk - sg.first_block;
  const int ox0 = (tb / (sg.tpa * sg.tpa)) * MT, oy0 = ((tb / sg.tpa) % sg.tpa) * 4, oz0 = (tb % sg.tpa) * 4;
  const long long ncellp = (long long)nsp * nsp * nsp;
  const auto src = gmem(reinterpret_cast<const H*>(sg.a));
  int vt[NT], off[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int2 e = tiles[T0 + t];
    vt[t] = e.x;
    off[t] = e.y;
  }
  for (int k = threadIdx.x; k < 108; k += 512) {
    const int s = k % 27, jx = s / 9, jy = (s / 3) % 3, jz = s % 3;
    ktab[k] = int4{(k / 27) * CELLS + jx * 144 + jy * 12 + jz, (2 * jx + 1) * 144, (2 * jy + 1) * 12, 2 * jz + 1};
  }
  for (int c = threadIdx.x; c < 16 * NT; c += 512) {
    const int col = 16 * T0 + c;
    scol[c] = fold_colmap<P, OP>(col);
  }
  for (int t = threadIdx.x; t < NTERM; t += 512) {
    const int e = OP == 3 ? t >> 5 : OP == 1 ? c_ft<P>.col[t] >> 8 : t < hterms(P) ? c_ft<P>.par[t] : 0;
    tsg[t] = float4{e & 4 ? -1.f : 1.f, e & 2 ? -1.f : 1.f, e & 1 ? -1.f : 1.f, 0.f};
  }
  const int lane = threadIdx.x & 63, i = lane & 15, kq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int e0 = (w % NG) * NE, ks = (w / NG) % KS, xg = w / (NG * KS);
  const H sx = (e0 & 4) ? H(-1) : H(1), sy = (e0 & 2) ? H(-1) : H(1), sz = (e0 & 1) ? H(-1) : H(1);
  // the lane's oct: image "plus 0" of the wave's first row tile
  const H* ctr = lds + (2 * xg * NR + 3) * 144 + (2 * (i >> 2) + 3) * 12 + 2 * (i & 3) + 3;
  Acc acc[NR][NE][NT];
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[r][e][t] = Acc{0, 0, 0, 0};
  const H* we = W + e0 * 64 + lane;
  // K steps [sa, sb) of chunk c (steps 27 c ..), column tiles 0 .. NA - 1
  auto run = [&](auto nac, int c, int sa, int sb) {
    constexpr int NA = decltype(nac)::value;
    int s = sa + (ks - sa % KS + KS) % KS;
    if (s >= sb) return;
    auto aread = [&](int st, H (&r)[NR][8], float (&g)[3]) {
      const int k = 4 * (st - 27 * c) + kq;  // < 108
      const int4 q = ktab[k];
      const float4 sg4 = tsg[4 * c + ((k * 38) >> 10)];  // k / 27
      g[0] = sg4.x;
      g[1] = sg4.y;
      g[2] = sg4.z;
      const H *p0 = ctr + q.x, *p1 = p0 - q.z, *p2 = p0 - q.y, *p3 = p1 - q.y;
#pragma unroll
      for (int m = 0; m < NR; ++m) {
        r[m][0] = p0[m * 288];
        r[m][1] = p0[m * 288 - q.w];
        r[m][2] = p1[m * 288];
        r[m][3] = p1[m * 288 - q.w];
        r[m][4] = p2[m * 288];
        r[m][5] = p2[m * 288 - q.w];
        r[m][6] = p3[m * 288];
        r[m][7] = p3[m * 288 - q.w];
      }
    };
    auto bread = [&](int st, H (&b)[NE][NA]) {
#pragma unroll
      for (int t = 0; t < NA; ++t) {
        const auto p = gmem(we + (size_t)(off[t] + st) * 512);
#pragma unroll
        for (int e = 0; e < NE; ++e) b[e][t] = p[e * 64];
      }
    };
    H r[2][NR][8], b[2][NE][NA], a[NE];
    float g[2][3];
    aread(s, r[0], g[0]);
    bread(s, b[0]);
#pragma unroll 1
    for (; s < sb; s += 2 * KS) {
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int st = s + u * KS, sn = st + KS < sb ? st + KS : s;
        if (u == 0 || st < sb) {
          bread(sn, b[u ^ 1]);
          aread(sn, r[u ^ 1], g[u ^ 1]);
          __builtin_amdgcn_sched_barrier(0);
          const H gx = NE <= 4 ? sx * (H)g[u][0] : (H)g[u][0], gy = NE <= 2 ? sy * (H)g[u][1] : (H)g[u][1], gz = NE == 1 ? sz * (H)g[u][2] : (H)g[u][2];
#pragma unroll
          for (int m = 0; m < NR; ++m) {
            fold8<NE>(r[u][m], gx, gy, gz, a);
#pragma unroll
            for (int e = 0; e < NE; ++e)
#pragma unroll
              for (int t = 0; t < NA; ++t) acc[m][e][t] = M::op(a[e], b[u][e][t], acc[m][e][t]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  };
  // terms 4 c .. 4 c + 3 per chunk: 27 K steps
  const int nch = (vt[0] + 26) / 27, c1 = (ip + 1) * nch / np;
  for (int c = ip * nch / np; c < c1; ++c) {
    __syncthreads();
    constexpr int CNT = 4 * CELLS, FB = 7;
#pragma unroll 1
    for (int q0 = threadIdx.x; q0 < CNT; q0 += FB * 512) {
      H v[FB];
#pragma unroll
      for (int u = 0; u < FB; ++u) {
        const int q = q0 + u * 512, cell = q % CELLS, z = 2 * oz0 + 1 + cell % 12, y = 2 * oy0 + 1 + (cell / 12) % 12,
                  x = 2 * ox0 + 1 + cell / 144;
        v[u] = q < CNT && x < nsp && y < nsp && z < nsp
                   ? src[(4 * c + q / CELLS) * ncellp + ((long long)x * nsp + y) * nsp + z]
                   : H(0);
      }
#pragma unroll
      for (int u = 0; u < FB; ++u)
        if (q0 + u * 512 < CNT) lds[q0 + u * 512] = v[u];
    }
    __syncthreads();
    const int end = min(27 * c + 27, vt[0]);
    int cur = 27 * c;
    count_down<NT>([&](auto nac) {
      constexpr int NA = decltype(nac)::value;
      const int to = min(end, vt[NA - 1]);
      if (to > cur) {
        run(nac, c, cur, to);
        cur = to;
      }
    });
  }
  // the 8 patterns' sums of result q of row tile r, through LDS (one row tile
  // of each row group at a time), then from all parts of the K loop
  constexpr int NQ = NX * 16 * 16 * NT;
  double* const slot = part + (size_t)blockIdx.x * (NR * NQ * 8);
  auto stage = [&](int r) {
    __syncthreads();
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          lds[(((ks * NX + xg) * 8 + e0 + e) * 16 + M::row(v, kq)) * CS + 16 * t + i] = acc[r][e][t][v];
    __syncthreads();
  };
  auto load = [&](int q, double (&y)[8]) {
    const int col = m2lf_qcol<OP, NT>(q), row = m2lf_qrow<OP, NT>(q), xr = q / (256 * NT);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      double x = 0.0;
#pragma unroll
      for (int k = 0; k < KS; ++k) x += (double)lds[(((k * NX + xr) * 8 + e) * 16 + row) * CS + col];
      y[e] = x;
    }
  };
  if (np > 1) {
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      stage(r);
#pragma unroll 1
      for (int q = threadIdx.x; q < NQ; q += 512) {
        double y[8];
        load(q, y);
#pragma unroll
        for (int e = 0; e < 8; ++e) slot[(size_t)(r * 8 + e) * NQ + q] = y[e];
      }
    }
    return;
  }
#pragma unroll
  for (int r = 0; r < NR; ++r) {
    stage(r);
#pragma unroll 1
    for (int q = threadIdx.x; q < NQ; q += 512) {
      const int cb = scol[m2lf_qcol<OP, NT>(q)];
      double y[8];
      load(q, y);
      m2lf_put<P, H, OP>(sg, cb, ox0 + (q / (256 * NT)) * NR + r, oy0, oz0, m2lf_qrow<OP, NT>(q), y);
    }
  }
}

// Adds the parts of the shared groups of a k_m2lf launch, in order.  Blocks:
// (group, tile), the groups with several parts only (sum_first: first block).
template <int P, typename H, int OP, int MT, int NT, int NR>
__global__ __launch_bounds__(256) void k_m2lf_sum(const Seg* __restrict__ segs, int nseg, int T, const M2lGrid grid,
                                                  const double* __restrict__ part) {
  constexpr int NQ = MT / NR * 256 * NT;
  int g = 0, left = (int)blockIdx.x / T;  // (a tile per T blocks of each shared group)
  while (grid.parts[g] == 1 || left-- > 0) ++g;
  const int lbk = (int)blockIdx.x % T, np = grid.parts[g];
  const Seg& sg = find_seg(segs, nseg, lbk);
  const int tb = lbk - sg.first_block;
  const int ox0 = (tb / (sg.tpa * sg.tpa)) * MT, oy0 = ((tb / sg.tpa) % sg.tpa) * 4, oz0 = (tb % sg.tpa) * 4;
  const double* slot = part + ((size_t)grid.first[g] + (size_t)lbk * np) * (NR * NQ * 8);
  for (int x = blockIdx.y * 256 + threadIdx.x; x < NR * NQ; x += gridDim.y * 256) {
    const int r = x / NQ, q = x % NQ, col = 16 * NT * g + m2lf_qcol<OP, NT>(q);
    const int cb = fold_colmap<P, OP>(col);
    if (cb < 0) continue;
    double y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = slot[(size_t)(r * 8 + e) * NQ + q];
    for (int k = 1; k < np; ++k)
#pragma unroll
      for (int e = 0; e < 8; ++e) y[e] += slot[(size_t)k * (NR * NQ * 8) + (size_t)(r * 8 + e) * NQ + q];
    m2lf_put<P, H, OP>(sg, cb, ox0 + (q / (256 * NT)) * NR + r, oy0, oz0, m2lf_qrow<OP, NT>(q), y);
  }
}

// The other operators' B fragments, as k_m2lf_table.
template <typename H>
__global__ void k_m2lf_adj_table(const double* __restrict__ Dtab, const int2* __restrict__ tiles, H* __restrict__ W,
                                 int P, int nmax, int ND, long long cnt) {
  const long long id = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (id >= cnt) return;
  const int lane = (int)(id & 63), e = (int)(id >> 6) & 7, f = (int)(id >> 9);
  int t = 0;
  while (tiles[t].y + tiles[t].x <= f) ++t;
  const int k = 4 * (f - tiles[t].y) + (lane >> 4), s = k % 27, cb = m2lf_col(P, k / 27), a = 16 * t + (lane & 15);
  const int kap = cb >> 8, b = cb & 255;
  double x = 0.0;
  if (cb >= 0 && a < hterms(nmax) && h_degree(a) + h_degree(b) <= P) {
    const int ea = h_exp(a), eb = h_exp(b), pb = h_parity(b);
    const int g = mi_index(mi_a(ea) + mi_a(eb), mi_b(ea) + mi_b(eb), mi_c(ea) + mi_c(eb));
    const int j[3] = {s / 9, (s / 3) % 3, s % 3};
    for (int minus = 0; minus < 8; ++minus) {
      int dd = 0;
      bool near = true;
      for (int ax = 0; ax < 3; ++ax) {
        const int d = (minus >> (2 - ax)) & 1 ? -j[ax] - 1 : j[ax];  // P - J
        near = near && d >= -1 && d <= 1;
        dd = dd * 7 + d + 3;
      }
      if (near) continue;
      double y = 0.0;
      for (int q = 0; q < 8; ++q) y += chi(kap ^ pb, 7 - q) * Dtab[((size_t)dd * 8 + q) * ND + g];
      x += chi(e ^ kap, minus) * y;
    }
    x = ldexp(x, -(h_degree(b) + 1) - 3);
  }
  W[id] = static_cast<H>(x);
}

// FMM-2: M2P, and its transpose, from the derivatives at the 64 unigrid
// positions of a level-F cell.
template <typename H>
__global__ void k_m2pf_table(const double* __restrict__ Dtab2, const int2* __restrict__ tiles, H* __restrict__ W, int P,
                             int nmax, int ND, long long cnt, int adj) {
  const long long id = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (id >= cnt) return;
  const int lane = (int)(id & 63), e = (int)(id >> 6) & 7, f = (int)(id >> 9);
  int t = 0;
  while (tiles[t].y + tiles[t].x <= f) ++t;
  const int k = 4 * (f - tiles[t].y) + (lane >> 4), s = k % 27, kt = k / 27, col = 16 * t + (lane & 15);
  const int a = adj ? col : kt;
  double x = 0.0;
  if (a < hterms(nmax)) {
    const int ea = h_exp(a), pa = h_parity(a), j[3] = {s / 9, (s / 3) % 3, s % 3};
    const int o = adj ? kt & 3 : col >> 6, eo = o ? 8 >> o : 0, kap = kt >> 5;
    const int g = mi_index(mi_a(ea) + (o == 1), mi_b(ea) + (o == 2), mi_c(ea) + (o == 3));
    for (int minus = 0; minus < 8; ++minus) {
      int dd = 0;
      bool near = true;
      for (int ax = 0; ax < 3; ++ax) {
        const int m = (minus >> (2 - ax)) & 1;
        const int d = adj ? (m ? -j[ax] - 1 : j[ax]) : (m ? j[ax] + 1 : -j[ax]);  // P - J
        near = near && d >= -1 && d <= 1;
        dd = dd * 7 + d + 3;
      }
      if (near) continue;
      const double* D = Dtab2 + (size_t)dd * 64 * ND + g;
      if (!adj) {
        x += chi(e ^ pa, minus) * D[(size_t)(col & 63) * ND];
      } else {
        // the target's images about its own cell's centre: 1/2, 3/2 out on either side
        double y = 0.0;
        for (int im = 0; im < 8; ++im) {
          int sub = 0;
          for (int ax = 0; ax < 3; ++ax) {
            const int b = (kt >> (4 - ax)) & 1;
            sub = sub * 4 + ((im >> (2 - ax)) & 1 ? 1 - b : 2 + b);
          }
          y += chi(kap ^ eo, im) * D[(size_t)sub * ND];
        }
        x += chi(e ^ kap, minus) * y;
      }
    }
    x *= adj ? 1.0 / 64 : 1.0 / 8;
  }
  W[id] = static_cast<H>(x);
}

// L2L, eq. (L2L), in harmonic terms: the complete locals of the cells of one
// level, [cell][hrow], from the M2L's rows (Walsh-folded over the children) and
// the complete locals of the level above (null: the coarsest level).  With
// S[b][pat] the shift's partial sum over the g of parity pattern pat
// (coefficient lists of plan time, over the full terms b + g, which a block
// expands once from the harmonic ones),
//   L(child, b) = chi_b(sigma) sum_kappa chi_kappa(sigma) (Lw[kappa][b] / 8 + S[b][kappa ^ parity(b)]).
// Thread (parent of 16, slot of 32): terms slot, slot + 32, ...
// Segments: n = cells per axis of level k - 1, a = its complete locals (or
// null), c = M2L rows of level k, b = the result.
constexpr int L2LF_ROWS = 16, L2LF_THREADS = 512;
template <int P>
__global__ __launch_bounds__(L2LF_THREADS) void k_l2lf(const Seg* __restrict__ segs, int nseg,
                                                       const int* __restrict__ cs, const int* __restrict__ cidx,
                                                       const double* __restrict__ ccoef) {
  constexpr int NL = nterms(P), HT = hterms(P), HR = hrow(P), E = l2l_entries(P), SS = NL + 1;
  __shared__ int s_cs[8 * NL + 1];
  __shared__ int s_idx[E];
  __shared__ double s_coef[E];
  __shared__ double s_src[L2LF_ROWS * SS];
  __shared__ double s_h[L2LF_ROWS * HR];
  const Seg& sg = find_seg(segs, nseg, blockIdx.x);
  const int ns = sg.n;
  const long long nps = (long long)ns * ns * ns, P0 = (long long)(blockIdx.x - sg.first_block) * L2LF_ROWS;
  const bool up = sg.a != nullptr;
  if (up) {
    for (int t = threadIdx.x; t <= 8 * NL; t += L2LF_THREADS) s_cs[t] = cs[t];
    for (int t = threadIdx.x; t < E; t += L2LF_THREADS) {
      s_idx[t] = cidx[t];
      s_coef[t] = ccoef[t];
    }
    for (int t = threadIdx.x; t < L2LF_ROWS * HR; t += L2LF_THREADS)
      s_h[t] = P0 + t / HR < nps ? sg.a[P0 * HR + t] : 0.0;
    __syncthreads();
    // full terms: (x, y, 2k + e) = (-1)^k sum_l C(k, l) (x + 2l, y + 2(k - l), e)
    for (int t = threadIdx.x; t < L2LF_ROWS * NL; t += L2LF_THREADS) {
      const int r = t / NL, f = t - r * NL, ex = c_mi_exp[f], z = mi_c(ex), k = z >> 1;
      double v = 0.0;
      for (int l = 0; l <= k; ++l)
        v += (double)binom(k, l) * s_h[r * HR + h_index(mi_a(ex) + 2 * l, mi_b(ex) + 2 * (k - l), z & 1)];
      s_src[r * SS + f] = (k & 1) ? -v : v;
    }
    __syncthreads();
  }
  const int slot = threadIdx.x & 31, r = threadIdx.x >> 5;
  const long long Pc = P0 + r;
  if (Pc >= nps) return;
  const int p2 = (int)(Pc % ns), p1 = (int)((Pc / ns) % ns), p0 = (int)(Pc / ((long long)ns * ns));
  const double* __restrict__ row = sg.c + Pc * 8 * HR;
  const double* src = s_src + r * SS;
  double* __restrict__ out = sg.b;
  for (int b = slot; b < HT; b += 32) {
    const int bt = c_ft<P>.full[b], pb = c_ft<P>.par[b];
    double y[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) y[k] = row[k * HR + b];
    double S[8];
#pragma unroll
    for (int pat = 0; pat < 8; ++pat) {
      double x = 0.0;
      if (up)
#pragma unroll 2
        for (int j = s_cs[8 * bt + pat]; j < s_cs[8 * bt + pat + 1]; ++j) x = fma(s_coef[j], src[s_idx[j]], x);
      S[pat] = x;
    }
    // S over the patterns of the full shift; its Walsh index is kappa = pat ^ pb,
    // so transform both sums apart and give S its sign chi_b
#pragma unroll
    for (int bit = 1; bit < 8; bit <<= 1)
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (!(e & bit)) {
          const double u = y[e], v = y[e | bit], a = S[e], c = S[e | bit];
          y[e] = u + v;
          y[e | bit] = u - v;
          S[e] = a + c;
          S[e | bit] = a - c;
        }
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const long long c = ((long long)(2 * p0 + 1 - ((m >> 2) & 1)) * (2 * ns) + (2 * p1 + 1 - ((m >> 1) & 1))) * (2 * ns) +
                          (2 * p2 + 1 - (m & 1));
      out[c * HR + b] = fma(0.125 * chi(pb, m), y[m], S[m]);
    }
  }
}
