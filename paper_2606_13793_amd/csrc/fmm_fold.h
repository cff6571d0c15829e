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
constexpr int BLK_THREADS = 256;
// LDS tile of densities: (4 NX + 8) x 24 x 24 cells, one element of padding
// after every 4 rows: the 16 lanes of an operand read are 4 cells apart in z and
// 4 rows in y, 97 elements, so in FP64 they hit 16 distinct pairs of the 32 banks
// (with rows of 28 and no other padding, all 4 y hit the same ones).
constexpr int BLK_PLANE = 24 * 24 + 6;
constexpr __host__ __device__ int blk_row(int y) { return 24 * y + (y >> 2); }
constexpr __host__ __device__ int blk_tile(int nx) { return (4 * nx + 8) * BLK_PLANE; }

// K order of the stencil: step 6 g + jz, k-group kq: source (jx, jy, jz) with
// 6 jx + jy = 4 g + kq.  A lane's (jx, jy) stays for 6 steps, and jz is the same
// for all lanes, so the addresses of the mirror images cost nothing per step.
constexpr int BLK_GROUPS = BLK_STEPS / 6;
// place of a lane's (jx, jy): the plus image (from 6 cells before the block's
// centre along z; bits 0-11), the distance of the minus image along y (9 bits
// from 12) and jx (from 21)
constexpr __host__ __device__ int blk_place(int pair) {
  if (pair >= 36) pair = 35;
  const int jx = pair / 6, jy = pair % 6;
  return (jx * BLK_PLANE + blk_row(6 + jy) - blk_row(6)) | (blk_row(6 + jy) - blk_row(5 - jy)) << 12 | jx << 21;
}
static_assert(5 * BLK_PLANE + blk_row(11) - blk_row(6) < 4096 && blk_row(11) < 512, "bits of a place");

// row stride of complete locals per cell, in terms
constexpr __host__ __device__ int hrow(int P) { return (hterms(P) + 3) / 4 * 4; }
// Folded locals of a parent: pairs of terms (2q, 2q + 1), 8 patterns, 2 terms.
// A pair is a column tile of the M2L, so that its stores are whole aligned lines
// and its K loop is as long as its lower degree needs; the block kernel reads 4
// patterns of a pair as one run.
constexpr __host__ __device__ int frow(int P) { return (hterms(P) + 1) / 2 * 16; }
constexpr __host__ __device__ int fold_at(int kappa, int b) { return 16 * (b >> 1) + 2 * kappa + (b & 1); }
// the own-local part runs two K steps at a time: k-group kq of step 2 s + v has
// term 8 s + 2 kq + v
constexpr __host__ __device__ int blk_lpairs(int P) { return (hterms(P) + 7) / 8; }
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
// table layout (elements): the folded stencil [54][8][64][2 column tiles], the
// own locals [steps][64][2], the level F-1 locals [8][steps][64][2]
constexpr __host__ __device__ int blk_off_l() { return BLK_STEPS * 8 * 2 * 64; }
constexpr __host__ __device__ int blk_off_p(int P) { return blk_off_l() + 2 * blk_lpairs(P) * 2 * 64; }
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

// (pattern, term) of column col of the transpose's K order (sorted by the degree
// of the term, the pattern slow inside a degree), packed pattern << 8 | term; -1
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
  unsigned char deg[hterms(P)];         // its degree
  unsigned char idx[hterms(P)];         // its place among the terms of that pattern
  signed char pt[8][4 * blk_psteps(P)];  // the terms of each pattern, -1 past the last
  constexpr FoldTab() : col(), full(), par(), deg(), idx(), pt() {
    for (int i = 0; i < 8 * hterms(P); ++i) col[i] = (short)m2lf_col(P, i);
    int cnt[8] = {};
    for (auto& row : pt)
      for (auto& v : row) v = -1;
    for (int i = 0; i < hterms(P); ++i) {
      const int ex = h_exp(i), e = h_parity(i);
      full[i] = (unsigned char)mi_index(ex & 255, (ex >> 8) & 255, ex >> 16);
      par[i] = (unsigned char)e;
      deg[i] = (unsigned char)h_degree(i);
      idx[i] = (unsigned char)cnt[e];
      pt[e][cnt[e]++] = (signed char)i;
    }
  }
};
template <int P>
__constant__ const FoldTab<P> c_ft = FoldTab<P>();
struct BlkPlaces {
  int v[36];
  constexpr BlkPlaces() : v() {
    for (int i = 0; i < 36; ++i) v[i] = blk_place(i);
  }
  __device__ int operator[](int i) const { return v[i]; }
};
__constant__ const BlkPlaces c_blk_place = BlkPlaces();

// The block kernel's B table in the compute type (layout above); lane = j +
// 16 kq, column 16 tile + j = (t, o).  The 1/8 of the inverse Walsh sum is
// left to the epilogue.
// (The order is a template parameter so that the offsets and class tables are
// constants: 137 us of plan creation at p = 6 before.)
template <int P, typename H>
__global__ void k_blk_table(const double* __restrict__ G, H* __restrict__ W, int dl) {
  constexpr int OFF_L = blk_off_l(), OFF_P = blk_off_p(P), END = blk_table(P), np = blk_psteps(P);
  const int id = blockIdx.x * blockDim.x + threadIdx.x;
  if (id >= END) return;
  const int lane = (id >> 1) & 63, tile = id & 1, j = lane & 15, kq = lane >> 4, col = 16 * tile + j;
  const int t = col >> 2, o = col & 3;
  double x = 0.0;
  if (id < OFF_L) {
    const int e = (id >> 7) & 7, st = id >> 10, pair = 4 * (st / 6) + kq;
    const int jj[3] = {pair / 6, pair % 6, st % 6};
    for (int minus = 0; minus < 8; ++minus) {
      int v = 0;
      for (int a = 0; a < 3; ++a) v = v * 12 + (((minus >> (2 - a)) & 1) ? 5 - jj[a] : 6 + jj[a]);
      x += chi(e, minus) * G[((size_t)t * 1728 + v) * 4 + o];
    }
  } else if (id < OFF_P) {
    const int st = (id - OFF_L) >> 7, b = 8 * (st >> 1) + 2 * kq + (st & 1);
    if (b < hterms(P)) x = h_reduce(b, [&](int bt) { return l2p_coef(bt, t, o); });
  } else {
    const int s = (id - OFF_P) >> 7, e = s / np;
    const int b = c_ft<P>.pt[e][4 * (s % np) + kq];
    if (b >= 0) x = 8.0 * h_reduce(b, [&](int bt) { return blk_l2p(bt, t, o, dl); });
  }
  W[id] = static_cast<H>(x);
}

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
// chi of the axis where eg fixes it (x for NE <= 4; y for NE = 2) times the images'
// own sign.
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
    static_assert(NE == 2, "2, 4 or 8 patterns");
    const H y0 = fma(sy, x[2], x[0]), y1 = fma(sy, x[3], x[1]);
    a[0] = fma(sz, y1, y0);
    a[1] = fma(-sz, y1, y0);
  }
}

// Stages the (4 NX + 8) x 24 x 24 cells from (x0, y0, z0) of an n^3 grid into the
// LDS tile, times sc, zero outside the grid; keep (or null) gets a copy of the
// block's own cells.  252 threads take 21 rows of 12 pairs at a time; the pairs
// are aligned to their element only.
template <int NX, typename TI, typename H, typename Val>
__device__ __forceinline__ void stage_cells(H* __restrict__ lds, const TI* __restrict__ src, TI* __restrict__ keep, int n,
                                            int x0, int y0, int z0, Val&& val) {
  typedef TI ti2 __attribute__((ext_vector_type(2), aligned(sizeof(TI))));
  constexpr int ROWS = (4 * NX + 8) * 24, FB = 7;
  const long long at = ((long long)x0 * n + y0) * n + z0;
  const auto g = gmem(src + at);  // (only dereferenced inside the grid)
  const int zc = threadIdx.x % 12, r0 = threadIdx.x / 12, z = z0 + 2 * zc;
  const bool zok = z >= 0 && z < n && threadIdx.x < 252;
  if (threadIdx.x >= 252) return;
#pragma unroll 1
  for (int r = r0; r < ROWS; r += 21 * FB) {
    ti2 v[FB];
#pragma unroll
    for (int u = 0; u < FB; ++u) {
      const int row = r + 21 * u, tx = row / 24, ty = row - 24 * tx;
      const bool in = zok && row < ROWS && (unsigned)(x0 + tx) < (unsigned)n && (unsigned)(y0 + ty) < (unsigned)n;
      v[u] = in ? *(const __attribute__((address_space(1))) ti2*)(g + (unsigned)((tx * n + ty) * n + 2 * zc)) : ti2{0, 0};
    }
#pragma unroll
    for (int u = 0; u < FB; ++u) {
      const int row = r + 21 * u, tx = row / 24, ty = row - 24 * tx;
      if (row >= ROWS) continue;
      H* const to = lds + tx * BLK_PLANE + blk_row(ty) + 2 * zc;
      to[0] = val(v[u][0]);
      to[1] = val(v[u][1]);
      if (keep && tx >= 4 && tx < 4 * NX + 4 && ty >= 4 && ty < 20 && zc >= 2 && zc < 10 && x0 + tx < n && y0 + ty < n &&
          z < n)
        *(ti2*)(keep + at + (unsigned)((tx * n + ty) * n + 2 * zc)) = v[u];
    }
  }
}

// The lane's pointers to the images of source (jx, jy) with x plus or minus, y
// plus or minus, at 6 cells before the block's centre along z.
template <typename H>
__device__ __forceinline__ void blk_images(const H* ctr, int q, const H* (&p)[4]) {
  const int dx = 2 * BLK_PLANE * (q >> 21) + BLK_PLANE, dy = (q >> 12) & 511;
  p[0] = ctr + (q & 4095);
  p[1] = p[0] - dy;
  p[2] = p[0] - dx;
  p[3] = p[1] - dx;
}

// Segments: n = unigrid cells per axis, tpa = tiles along y and z, tz = tiles
// along x, field, t = copy of the density to leave in the plan (or null),
// u = own locals [block][frow] in the compute type (or null: F = 2),
// d = complete locals of the blocks' cells [block][hrow] (or null), c = FMM-2:
// M2P, [block][4][4^3] in the compute type.
// Tile: NX x 4 x 4 blocks, NT of the 2 column tiles (one: t = 0 the inner, 1 the
// outer cells along x; blockIdx.y).  4 waves, each with one half of the patterns
// and NR row tiles (the 4 x 4 blocks of a plane) of one of KS slices of the K steps.
// What bounds it: the matrix cores (54 + 14 + 3 K steps of 16 products per row
// tile at p = 6), and, as vector operations do not run beside FP64 products,
// everything else a wave executes.  So a lane folds the 8 mirror images of its
// operand from the LDS tile itself (12 adds for 8 products) at addresses formed
// once for 6 steps, B comes through the caches at a uniform base, both column
// tiles in one load, and the epilogue forms addresses once per thread.  FP32
// products take half as long, and there B's loads bound a wave: each fragment
// serves two row tiles (256^3, p = 6, FP32: 666 us -> 515; FP64, where that is no
// gain, 875 against 862; 1146 before the addresses were formed per group and the
// own locals read as runs).  FP64 at 256^3: 370 us of products for the stencil and
// 115 for L2P at 2.4 GHz, and 949 MB of locals, 200 us of copy rate.  Blocks are
// small so that a CU holds two (FP32: three or four): one's staging and stores
// run beside the other's products.
// PHI: calls for the potential alone, FP64: the 8 columns (t, phi) as products of
// 16 x 4 x 4 (17 cycles; FP32 has none of that rate) over the same table, each
// fragment for two row tiles, as loads bound a wave then (128^3, p = 6: 109 us with
// the 24 columns of g, 68 without).
// blocks (of 4 waves) per compute unit
template <typename CT, int NX>
constexpr int blk_occ = Mf<CT>::IDX == 0 ? 2 : NX == 2 ? 3 : 4;
template <int P, typename CT, typename TI, typename TO, int NX, int NT, int DL, bool PHI>
__global__ __launch_bounds__(BLK_THREADS, (blk_occ<CT, NX>)) void k_block(
    const Seg* __restrict__ segs, int nseg, IoArg io, const typename Mf<CT>::H* __restrict__ W,
    unsigned int* __restrict__ stamp_cnt, unsigned long long* __restrict__ stamp_done) {
  using M = Mf<CT>;
  using H = typename M::H;
  static_assert(!PHI || (Mf<CT>::IDX == 0 && NT == 2), "FP64, all positions");
  using Acc = std::conditional_t<PHI, H, typename M::Acc>;
  typedef H h2 __attribute__((ext_vector_type(2)));
  constexpr int NE = 4, KS = Mf<CT>::IDX == 0 && !PHI ? 2 / NX : 2, NR = NX * KS / 2, HR = hrow(P), FR = frow(P);
  constexpr int NLP = blk_lpairs(P), NPS = blk_psteps(P), OFF_L = blk_off_l(), OFF_P = blk_off_p(P);
  // own-local pairs of steps of the last K slice, which has one group less
  constexpr int LSPLIT = KS == 1 ? NLP : NLP < (8 + NPS + 2 * NLP) / 4 ? NLP : (8 + NPS + 2 * NLP) / 4;
  // epilogue image of the results of NXR row tiles, [slice][half][4][NXR * 16][CS]
  constexpr int NXR = NX / NR, CS = PHI ? 9 : 16 * NT + 1, ES = NXR * 16 * CS;
  constexpr int EP = KS * 8 * ES, TILE = blk_tile(NX), SZ = EP > TILE ? EP : TILE;
  __shared__ __attribute__((aligned(16))) H lds[SZ];
  __shared__ int spt[8 * NPS * 4];
  const Seg& sg = find_seg(segs, nseg, blockIdx.x);
  const int n = sg.n, nb = n >> 2;
  TO* __restrict__ phi = io_phi<TO>(io, sg.field);
  TO* __restrict__ g = io_g<TO>(io, sg.field);
  const int lb = blockIdx.x - sg.first_block;
  const int bx0 = (lb / (sg.tpa * sg.tpa)) * NX, by0 = ((lb / sg.tpa) % sg.tpa) * 4, bz0 = (lb % sg.tpa) * 4;
  for (int t = threadIdx.x; t < 8 * NPS * 4; t += BLK_THREADS) spt[t] = c_ft<P>.pt[t / (NPS * 4)][t % (NPS * 4)];
  const int t0 = NT == 1 ? blockIdx.y : 0;  // column tile
  stage_cells<NX>(lds, io_rho<TI>(io, sg.field), t0 ? nullptr : static_cast<TI*>(sg.t), n, 4 * bx0 - 4, 4 * by0 - 4, 4 * bz0 - 4,
                  [](TI v) { return static_cast<H>(v); });
  const int lane = threadIdx.x & 63, i = lane & 15, kq = lane >> 4;
  // the wave's first row tile, K slice and half of the patterns
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), X = KS == 1 ? w & 1 : 0, ks = KS == 1 ? 0 : w & 1,
            half = w >> 1, e0 = half * NE;
  const H sx = half ? H(-1) : H(1);
  Acc acc[NR][NE][NT];
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[r][e][t] = Acc{};
  // the lane's B elements (PHI: column lane % 4 of each tile's phi)
  const unsigned bl = PHI ? 8u * (lane & 3) + 32u * kq : 2u * lane;
  auto mul = [](H a, H b, Acc c) {
    if constexpr (PHI) return __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, 0, 0, 0);
    else return M::op(a, b, c);
  };
  auto products = [&](const H (&a)[NR][NE], const H (&b)[NE][NT]) {
#pragma unroll
    for (int r = 0; r < NR; ++r)
#pragma unroll
      for (int e = 0; e < NE; ++e)
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[r][e][t] = mul(a[r][e], b[e][t], acc[r][e][t]);
  };
  __syncthreads();
  // ---- the 12^3 densities
  {
    const H* ctr = lds + (4 * X + 6) * BLK_PLANE + blk_row(4 * (i >> 2) + 6) + 4 * (i & 3);
    const auto wb = gmem(W + e0 * 128 + t0);  // (uniform base, the lane as a 32-bit offset)
    auto bread = [&](int s, H (&b)[NE][NT]) {
#pragma unroll
      for (int e = 0; e < NE; ++e)
        if constexpr (NT == 2) {
          const h2 v = *(const __attribute__((address_space(1))) h2*)(wb + s * 1024 + e * 128 + bl);
          b[e][0] = v[0], b[e][1] = v[1];
        } else {
          b[e][0] = (wb + s * 1024 + e * 128)[2u * lane];
        }
    };
    const H* p[4];
    H r[NR][8], b[2][NE][NT], a[NR][NE];
    auto aread = [&](auto jc) {
#pragma unroll
      for (int m = 0; m < NR; ++m)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          r[m][2 * q] = p[q][m * 4 * BLK_PLANE + 6 + decltype(jc)::value];
          r[m][2 * q + 1] = p[q][m * 4 * BLK_PLANE + 5 - decltype(jc)::value];
        }
    };
    // operands are read one step ahead: images as soon as the last are folded
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
        for (int m = 0; m < NR; ++m) fold8<NE>(r[m], sx, H(1), H(1), a[m]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (jz < 5) {
          bread(6 * grp + jz + 1, b[u ^ 1]);
        } else {
          bread(6 * gn, b[u ^ 1]);
          blk_images(ctr, pn, p);
        }
        aread(std::integral_constant<int, (jz + 1) % 6>{});
        __builtin_amdgcn_sched_barrier(0);
        products(a, b[u]);
        __builtin_amdgcn_sched_barrier(0);
      });
    }
  }
  // ---- L2P; the lane's blocks, clamped into the grid
  long long cell[NR];
#pragma unroll
  for (int r = 0; r < NR; ++r)
    cell[r] = ((long long)min(bx0 + X + r, nb - 1) * nb + min(by0 + (i >> 2), nb - 1)) * nb + min(bz0 + (i & 3), nb - 1);
  if (DL == 1 && sg.u) {
    typedef H h8 __attribute__((ext_vector_type(8), aligned(16)));
    const auto wl = gmem(W + OFF_L + t0);
    const auto own = gmem(static_cast<const H*>(sg.u) + 2 * e0);
    h8 x[2][NR];
    H y[2][2][NT];
    // pair of steps s: 4 patterns of 2 terms are one run
    auto read = [&](int s, h8 (&x)[NR], H (&y)[2][NT]) {
      const int q = min(4 * s + kq, FR / 16 - 1);  // (past the last: the table is zero)
#pragma unroll
      for (int r = 0; r < NR; ++r) x[r] = *(const __attribute__((address_space(1))) h8*)(own + cell[r] * FR + 16 * q);
#pragma unroll
      for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int t = 0; t < NT; ++t) y[v][t] = (wl + s * 256 + v * 128 + t)[bl];
    };
    const int s0 = KS == 1 || ks ? 0 : LSPLIT, s1 = KS == 1 || !ks ? NLP : LSPLIT;
    auto step = [&](const h8 (&x)[NR], const H (&y)[2][NT]) {
#pragma unroll
      for (int v = 0; v < 2; ++v)
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
          for (int e = 0; e < NE; ++e)
#pragma unroll
            for (int t = 0; t < NT; ++t) acc[r][e][t] = mul(x[r][2 * e + v], y[v][t], acc[r][e][t]);
    };
    if (s0 < s1) {
      read(s0, x[0], y[0]);
#pragma unroll 1
      for (int s = s0; s < s1; s += 2) {
        read(min(s + 1, s1 - 1), x[1], y[1]);
        __builtin_amdgcn_sched_barrier(0);
        step(x[0], y[0]);
        __builtin_amdgcn_sched_barrier(0);
        read(min(s + 2, s1 - 1), x[0], y[0]);
        __builtin_amdgcn_sched_barrier(0);
        if (s + 1 < s1) step(x[1], y[1]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
  if (sg.d && ks == 0) {
    const auto wp = gmem(W + OFF_P + e0 * (NPS * 128) + t0);
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const auto par = gmem(sg.d + cell[r] * HR);
      double v[NE][NPS];
#pragma unroll
      for (int e = 0; e < NE; ++e)
#pragma unroll
        for (int s = 0; s < NPS; ++s) {
          const int bt = spt[(e0 + e) * (NPS * 4) + 4 * s + kq];
          const double x = par[bt >= 0 ? bt : 0];
          v[e][s] = bt >= 0 ? x : 0.0;
        }
#pragma unroll
      for (int e = 0; e < NE; ++e)
#pragma unroll
        for (int s = 0; s < NPS; ++s) {
          const H a = static_cast<H>(v[e][s]);
#pragma unroll
          for (int t = 0; t < NT; ++t)
            acc[r][e][t] = mul(a, (wp + (e * NPS + s) * 128 + t)[bl], acc[r][e][t]);
        }
    }
  }
  // phi = sphi acc, g_d = sgr tau_d acc, with the Walsh sum's 1/8.  Thread (y, z)
  // of the tile's 16 x 16 columns along x; position in the block 0..3: the minus
  // images are 0, 1 (3/2, 1/2 out)
  const H* const m2p = reinterpret_cast<const H*>(sg.c);
  const double dx = 1.0 / n, sphi = (DL == 1 ? 0.5 : 0.25) * dx * dx, sgr = (DL == 1 ? -0.25 : -0.0625) * dx;
  const long long N = (long long)n * n * n;
  const int z = threadIdx.x & 15, y = threadIdx.x >> 4, qy = y & 3, qz = z & 3;
  const int uy = 4 * by0 + y, uz = 4 * bz0 + z, myz = (qy < 2) << 1 | (qz < 2);
  const int tyz = (qy == 0 || qy == 3) << 1 | (qz == 0 || qz == 3);
  const H* const res = lds + myz * ES + (4 * (y >> 2) + (z >> 2)) * CS + (PHI ? 1 : 4) * tyz;
  const double sc[4] = {0.125 * sphi, 0.125 * sgr, (qy < 2 ? -0.125 : 0.125) * sgr, (qz < 2 ? -0.125 : 0.125) * sgr};
  const long long blk0 = ((long long)bx0 * nb + (uy >> 2)) * nb + (uz >> 2), pyz = qy * 4 + qz;
  const unsigned at = (unsigned)(y * n + z);
  static_for<NR>([&](auto rc) {
    constexpr int R = decltype(rc)::value;
    // inverse Walsh sums: over y and z in the wave, over x (the two halves of the
    // patterns) when the results are read back as z runs
    __syncthreads();
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int v = 0; v < (PHI ? 1 : 4); ++v) {
        H x[NE];
#pragma unroll
        for (int e = 0; e < NE; ++e)
          if constexpr (PHI) x[e] = acc[R][e][t];
          else x[e] = acc[R][e][t][v];
        const H p0 = x[0] + x[1], m0 = x[0] - x[1], p1 = x[2] + x[3], m1 = x[2] - x[3];
        const int row = PHI ? kq + 4 * ((lane >> 2) & 3) : M::row(v, kq), col = PHI ? 4 * t + (lane & 3) : 16 * t + i;
        H* const to = lds + (ks * 2 + half) * 4 * ES + (16 * X + row) * CS + col;
        to[0] = p0 + p1;
        to[ES] = m0 + m1;
        to[2 * ES] = p0 - p1;
        to[3 * ES] = m0 - m1;
      }
    __syncthreads();
    if (uy < n && uz < n)
      static_for<4 * NXR>([&](auto xc) {
        constexpr int x = decltype(xc)::value, qx = x & 3, XT = x >> 2, XB = R + XT;
        // (column tile 1: the outer two cells along x)
        constexpr int outer = qx == 0 || qx == 3, ro = (PHI ? 4 : NT == 2 ? 16 : 0) * outer + 16 * XT * CS;
        if (NT == 1 && outer != t0) return;
        const int ux = 4 * (bx0 + XB) + qx;
        if (ux >= n) return;
        const long long row = ((long long)ux * n + 4 * by0) * n + 4 * bz0;  // (uniform)
#pragma unroll
        for (int o = 0; o < 4; ++o) {
          if (o && (PHI || !g)) break;
          H a = res[ro + o], c = res[4 * ES + ro + o];
          if constexpr (KS == 2) {
            a += res[8 * ES + ro + o];
            c += res[12 * ES + ro + o];
          }
          double val = (double)(qx < 2 ? a - c : a + c) * (o == 1 && qx < 2 ? -sc[1] : sc[o]);
          if constexpr (DL == 2)
            val = fma((double)m2p[((blk0 + (long long)XB * nb * nb) * 4 + o) * 64 + qx * 16 + pyz], o ? sgr : sphi, val);
          if (o == 0)
            (phi + row)[at] = (TO)val;
          else
            (g + (o - 1) * N + row)[at] = (TO)val;
        }
      });
  });
  if (stamp_cnt) {
    // the field's last block records when the field is complete
    __syncthreads();
    if (threadIdx.x == 0) {
      __threadfence();
      if (atomicAdd(stamp_cnt + sg.field, 1u) == (unsigned int)(sg.tpa * sg.tpa * sg.tz * (NT == 1 ? 2 : 1)) - 1)
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
//   Lw[P][(kappa, b)] = sum_children chi_kappa(sigma) sigma^b L(child, b)
//                   = chi_kappa(tau) sum_e chi_e(tau) OUT(e; kappa, b) / 8,
// P the cell tau of the oct.  Columns are sorted by |b| (kappa slow inside a
// degree), K by |a| (K index 27 a + source), so a tile of 16 columns needs a
// prefix of K: ceil(27 (p - |b| + 1)^2 / 4) steps.
// ---------------------------------------------------------------------------
constexpr __host__ __device__ int fold_ntiles(int op, int P) {
  return op == FO_M2L ? (8 * hterms(P) + 15) / 16 : op == FO_M2P ? 16 : (hterms(P) + 15) / 16;
}
// steps of the forward operators before the chunks, for term 0
constexpr int FOLD_HEAD = 7;
constexpr __host__ __device__ int fold_steps(int op, int P, int nmax, int t) {
  const int m = h_degree(op == FO_M2L ? 2 * t : 16 * t);
  if (op == FO_M2L || op == FO_M2P) {
    const int q = op == FO_M2P || nmax < P - m ? nmax : P - m;
    return FOLD_HEAD + 27 * ((hterms(q) - 1 + 3) / 4);
  }
  return m > nmax ? 0 : op == FO_M2LT ? 54 * hterms(P - m) : 27 * 64;
}
// (term, source) of k-group kq of a step; the term past the last for padding
__host__ __device__ inline void fold_k(int op, int st, int kq, int* term, int* src) {
  const bool head = op == FO_M2L || op == FO_M2P;
  if (head && st < FOLD_HEAD) {
    *term = 4 * st + kq < 27 ? 0 : 0xffff;
    *src = (4 * st + kq) % 27;
    return;
  }
  const int c = st - (head ? FOLD_HEAD : 0);
  *term = (head ? 1 : 0) + 4 * (c / 27) + kq;
  *src = c % 27;
}

// B fragments in the compute type, [fragment (tile, step)][4 pairs of
// patterns][64][2];
// tiles[t] = (steps, first fragment).
template <typename H>
__global__ void k_m2lf_table(const double* __restrict__ Dtab, const int2* __restrict__ tiles, H* __restrict__ W, int P,
                             int nmax, int ND, long long cnt) {
  const long long id = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (id >= cnt) return;
  const int lane = (int)(id >> 1) & 63, e = ((int)(id >> 7) & 3) * 2 + (int)(id & 1), f = (int)(id >> 9);
  int t = 0;
  while (tiles[t].y + tiles[t].x <= f) ++t;
  const int kap = (lane >> 1) & 7, b = 2 * t + (lane & 1);  // fold_at
  int a, s;
  fold_k(FO_M2L, f - tiles[t].y, lane >> 4, &a, &s);
  double x = 0.0;
  if (b < hterms(P) && a < hterms(nmax) && h_degree(a) + h_degree(b) <= P) {
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
// cotangents of the Lw rows of the 27 x 8 cells P around (K terms: the columns,
// sorted by |b|; an image's sign is chi_kappa), columns the terms a
// of one J, the results M_bar(J = sigma, a) = sigma^a sum_e chi_e(sigma) OUT(e; a).
// OP 2 is FMM-2's M2P (Sec. 4): rows are the octs of level F, K as in M2L with
// every term, columns (o, t) the outputs at the 4^3 unigrid cells t of the
// positive octant's cell.  OP 3 is its transpose: K term 32 kappa + 4 t + o of
// the cotangents of the cells P, folded about each P's own centre.
//
// Segments: n = source grid cells per axis, tpa = tiles along y and z, tz =
// tiles along x; OP 0: a = harmonic multipoles of the source grid in the compute
// type, [term][(n + 6)^3] (terms padded to a multiple of 4), u = result in the
// compute type or b = result in FP64, [n^3][frow], or t = complete locals of the
// children, [(2 n)^3][hrow] (the coarsest level); OP 2: the same, u =
// [n^3][4][4^3]; OP 1, 3: a = cotangent planes [K term][(n + 6)^3] in the compute
// type, b = result, planes [term][(n + 6)^3].
// Tile: MT x 4 x 4 octs.  NW waves: 8 / NE groups of NE patterns, MT / NR
// groups of NR row tiles (a row tile: the 4 x 4 octs of a plane).  A block sums
// NT column tiles over all 8 patterns, so the inverse Walsh sums happen in its
// epilogue.  Blocks: column groups x T tiles, the heaviest group (lowest
// degrees) first; a group whose K loop is long against the launch shares it
// among several blocks (grid.parts), each summing a run of chunks: they leave
// their sums in `part`, which k_m2lf_sum adds in order.
// What bounds it: the matrix cores, and in FP64 every vector operation beside
// them, as those do not overlap (an FP64 product of 16 x 16 x 4 takes 64 cycles
// of a SIMD, a fused multiply-add 4.5).  So a lane folds the 8 mirror images of
// its operand once for NE x NT products (12 adds for 4 patterns), its addresses
// change every third step, B comes at a uniform base, the next step's operands
// and the next chunk's planes are read beside the products.  Two blocks run per
// compute unit, so that one's staging and stores lie beside the other's
// products.  At 64^3 source cells, p = 6 (the finest level of a 256^3 grid):
// FP64 1785 us -> 1436 us (835 us of products at 2.4 GHz), FP32 1216 -> 885 us,
// of which the 839 (420) MB of results are 180 (90) us of copy rate.
//
// LDS tile of k_m2lf: rows of 12 cells along z, the even cells first (the 16
// octs of an operand read are 2 cells apart in z and in y), with a stride of 14:
// two rows are 28 elements, so in FP64 the 16 lanes of a read hit 16 distinct
// pairs of the 32 banks
constexpr int FOLD_ROW = 14, FOLD_PLANE = 12 * FOLD_ROW;
constexpr __host__ __device__ int fold_z(int z) { return (z & 1) * 6 + (z >> 1); }
// what column col stands for: OP 0 the column and its pattern from bit 16; -1
// past the last
template <int P, int OP>
__device__ __forceinline__ int fold_colmap(int col) {
  if constexpr (OP == 0) return 2 * (col >> 4) + (col & 1) < hterms(P) ? col | ((col >> 1) & 7) << 16 : -1;
  return col < (OP == 2 ? 256 : hterms(P)) ? col : -1;
}
// result q of a group of row tiles: consecutive threads take the columns of a
// row, or for planes the rows
template <int OP, int NT>
__device__ __forceinline__ int m2lf_qcol(int q) { return OP & 1 ? (q >> 4) % (16 * NT) : q % (16 * NT); }
template <int OP, int NT>
__device__ __forceinline__ int m2lf_qrow(int q) { return OP & 1 ? q & 15 : (q / (16 * NT)) & 15; }
// inverse Walsh sum over the patterns, to the 8 cells of the oct (dx, row) of the
// tile at octs (ox0, oy0, oz0) (uniform; the lane's part of an address is a
// 32-bit offset)
template <int P, typename H, int OP>
__device__ __forceinline__ void m2lf_put(const Seg& sg, int cb, int ox0, int oy0, int oz0, int dx, int row,
                                         double (&y)[8]) {
  constexpr int FR = frow(P);
  const int ns = sg.n, nsp = ns + 6, no = ns >> 1, dy = row >> 2, dz = row & 3;
  if (cb < 0 || ox0 + dx >= no || oy0 + dy >= no || oz0 + dz >= no) return;
  walsh8(y);
  if constexpr (OP == 2) {
    H* const ut = static_cast<H*>(sg.u);
    const int o = cb >> 6, eo = o ? 8 >> o : 0, t0 = (cb >> 4) & 3, t1 = (cb >> 2) & 3, t2 = cb & 3;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const long long p = ((long long)(2 * (ox0 + dx) + 1 - ((m >> 2) & 1)) * ns + (2 * (oy0 + dy) + 1 - ((m >> 1) & 1))) * ns +
                          (2 * (oz0 + dz) + 1 - (m & 1));
      const int pos = ((m & 4 ? 3 - t0 : t0) * 4 + (m & 2 ? 3 - t1 : t1)) * 4 + (m & 1 ? 3 - t2 : t2);
      ut[(p * 4 + o) * 64 + pos] = static_cast<H>(m & eo ? -y[m] : y[m]);
    }
  } else if constexpr (OP & 1) {
    const int pa = c_ft<P>.par[cb];
    double* const b0 = sg.b + ((long long)(2 * ox0 + 4) * nsp + 2 * oy0 + 4) * nsp + 2 * oz0 + 4;
    double* const bl = b0 + cb * ((long long)nsp * nsp * nsp) + (2 * (dx * nsp + dy) * nsp + 2 * dz);
#pragma unroll
    for (int m = 0; m < 8; ++m)
      bl[-(((m >> 2) & 1) * nsp + ((m >> 1) & 1)) * nsp - (m & 1)] = chi(pa, m) * y[m];
  } else {
    const int kap = cb >> 16;
    const unsigned off = (unsigned)((2 * (dx * ns + dy) * ns + 2 * dz) * FR + (cb & 0xffff));
    if (sg.t) {
      // coarsest level: nothing comes from above, so the locals of the children
      // c are complete, L(2P + c, b) = chi_b(c) / 8 sum_kappa chi_kappa(c) Lw; the 8
      // patterns of a term are 8 lanes two apart
      const int b = 2 * ((cb & 0xffff) >> 4) + (cb & 1), nc = 2 * ns;
      const double sc = 0.125 * chi(c_ft<P>.par[b], kap);
      double* const out = static_cast<double*>(sg.t);
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        double v = chi(kap, m) * y[m];
#pragma unroll
        for (int bit = 1; bit < 8; bit <<= 1) {
          const double o = __shfl_xor(v, 2 * bit);
          v = kap & bit ? o - v : v + o;
        }
        const int x0 = 2 * (2 * (ox0 + dx) + (m & 4 ? 0 : 1)) + (kap & 4 ? 0 : 1),
                  x1 = 2 * (2 * (oy0 + dy) + (m & 2 ? 0 : 1)) + (kap & 2 ? 0 : 1),
                  x2 = 2 * (2 * (oz0 + dz) + (m & 1 ? 0 : 1)) + (kap & 1 ? 0 : 1);
        out[(((long long)x0 * nc + x1) * nc + x2) * hrow(P) + b] = sc * v;
      }
      return;
    }
    const long long p0 = ((long long)2 * ox0 * ns + 2 * oy0) * ns + 2 * oz0;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      // cell tau of the oct: minus bits m
      const long long p = (p0 + ((m & 4 ? 0 : 1) * ns + (m & 2 ? 0 : 1)) * ns + (m & 1 ? 0 : 1)) * FR;
      const double v = chi(kap, m) * y[m];
      if (sg.u)
        (static_cast<H*>(sg.u) + p)[off] = static_cast<H>(v);
      else
        (sg.b + p)[off] = v;
    }
  }
}
// column tiles per pass of the epilogue
template <int NT>
constexpr int m2lf_nte = NT % 2 ? NT : NT / 2;
// Tile shapes of the folded M2L by variant (rows of octs, column tiles per
// group, patterns per wave, waves): forward, and transposes, whose few
// column tiles are dominated by the first.
// X: FP32 products, which take half the time, so that folding an operand has to
// serve more of them.
template <int OP, int V, int X>
struct M2lShape {  // V = -1: none
  static constexpr int MT = 1, NT = 1, NE = 2, NW = 0;
};
template <int X> struct M2lShape<0, 0, X> { static constexpr int MT = 1, NT = 2, NE = 2, NW = 4; };
template <> struct M2lShape<0, 1, 0> { static constexpr int MT = 2, NT = 2, NE = 4, NW = 4; };
template <> struct M2lShape<0, 1, 1> { static constexpr int MT = 2, NT = 4, NE = 2, NW = 4; };
template <int X> struct M2lShape<1, 0, X> { static constexpr int MT = 1, NT = 1, NE = 2, NW = 4; };
template <int X> struct M2lShape<1, 1, X> { static constexpr int MT = 4, NT = 1, NE = 8, NW = 4; };
template <int V, int X> struct M2lShape<2, V, X> : M2lShape<0, V, X> {};
template <int V, int X> struct M2lShape<3, V, X> : M2lShape<1, V, X> {};

template <typename CT, int OP, typename S>
struct M2lLds {
  using H = typename Mf<CT>::H;
  static constexpr int NR = S::NW ? 8 * S::MT / (S::NE * S::NW) : 1, NX = S::MT / NR, CS = 16 * m2lf_nte<S::NT> + 1;
  static constexpr int CELLS = (2 * S::MT + 4) * FOLD_PLANE, NPL = OP == FO_M2L || OP == FO_M2P ? 5 : 4;
  static constexpr int EP = NX * 8 * 16 * CS, SZ = EP > NPL * CELLS ? EP : NPL * CELLS;
  static constexpr int BYTES = S::NW ? (int)(SZ * sizeof(H)) + 64 * S::NT : 0;
};
template <int P, typename CT, int OP, typename S>
__device__ __forceinline__ void m2lf_run(const M2lArgs& args, int block, char* smem) {
  using M = Mf<CT>;
  using H = typename M::H;
  using Acc = typename M::Acc;
  using L = M2lLds<CT, OP, S>;
  constexpr int MT = S::MT, NT = S::NT, NE = S::NE, NW = S::NW;
  constexpr int NR = L::NR, NG = 8 / NE, NX = L::NX, THR = 64 * NW;
  static_assert(NG * NX == NW && NX * NR == MT && NE % 2 == 0, "the waves' shares");
  constexpr bool HEAD = OP == FO_M2L || OP == FO_M2P;
  constexpr int NTERM = OP == 3 ? 256 : OP == 1 ? 8 * hterms(P) : hterms(P);
  constexpr int ROW = FOLD_ROW, PLANE = FOLD_PLANE;
  constexpr int NTE = m2lf_nte<NT>, CELLS = L::CELLS, CS = L::CS;
  typedef H hp __attribute__((ext_vector_type(2)));  // two patterns of a fragment
  typedef H h2 __attribute__((ext_vector_type(2), aligned(sizeof(H))));
  constexpr int RPP = (2 * MT + 4) * 12, RPT = THR / 6, FB = (4 * RPP + RPT - 1) / RPT;
  H* const lds = reinterpret_cast<H*>(smem);
  int* const scol = reinterpret_cast<int*>(smem + L::SZ * sizeof(H));
  const M2lGrid& grid = args.grid;
  const int2* __restrict__ tiles = args.tiles;
  const H* __restrict__ W = static_cast<const H*>(args.W);
  int grp = 0;
  while (grp + 1 < grid.ng && block >= grid.first[grp + 1]) ++grp;
  const int T0 = grp * NT, np = grid.parts[grp], rb = block - grid.first[grp], lbk = rb / np, ip = rb % np;
  const Seg& sg = find_seg(args.segs, args.nseg, lbk);
  const int nsp = sg.n + 6, tb = lbk - sg.first_block;
  const int ox0 = (tb / (sg.tpa * sg.tpa)) * MT, oy0 = ((tb / sg.tpa) % sg.tpa) * 4, oz0 = (tb % sg.tpa) * 4;
  const long long ncellp = (long long)nsp * nsp * nsp;
  // chunks and first fragment of each column tile
  int nc[NT], off[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int2 e = tiles[T0 + t];
    nc[t] = e.x ? (e.x - (HEAD ? FOLD_HEAD : 0)) / 27 : 0;
    off[t] = e.y;
  }
  for (int c = threadIdx.x; c < 16 * NT; c += THR) scol[c] = fold_colmap<P, OP>(16 * T0 + c);
  const int lane = threadIdx.x & 63, i = lane & 15, kq = lane >> 4;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int e0 = (w % NG) * NE, xg = w / NG;
  // the lane's oct: its first cell but two, in the wave's first row tile
  const H* const oct = lds + 2 * xg * NR * PLANE + 2 * (i >> 2) * ROW + (i & 3);
  Acc acc[NR][NE][NT];
#pragma unroll
  for (int r = 0; r < NR; ++r)
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[r][e][t] = Acc{0, 0, 0, 0};
  // Planes of the tile's cells and two around from term t0 on (zero past the
  // terms and the grid), to registers and then to slots at, at + 1, ...: CNT
  // planes of RPP rows of 6 pairs along z.  The pairs are aligned to their
  // element only; one that reaches past the grid is halo.
  const int pz = threadIdx.x % 6, r0 = threadIdx.x / 6;
  const auto src =
      gmem(reinterpret_cast<const H*>(sg.a) + ((long long)(2 * ox0 + 1) * nsp + 2 * oy0 + 1) * nsp + 2 * oz0 + 1);
  auto fetch = [&](auto cnt, int t0, h2* v) {
    constexpr int ROWS = decltype(cnt)::value * RPP, N = (ROWS + RPT - 1) / RPT;
    const bool zok = 2 * oz0 + 2 * pz + 2 < nsp && r0 < RPT;
    const auto p = src + t0 * ncellp;
    unsigned in = 0;
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int row = r0 + u * RPT, pn = row / RPP, q = row - pn * RPP, x = q / 12, y = q - 12 * x;
      const bool ok = zok && row < ROWS && t0 + pn < NTERM && 2 * ox0 + 1 + x < nsp && 2 * oy0 + 1 + y < nsp;
      v[u] = *(const __attribute__((address_space(1))) h2*)(p + (ok ? pn * ncellp + (unsigned)((x * nsp + y) * nsp + 2 * pz) : 0));
      in |= (unsigned)ok << u;
    }
    return in;
  };
  auto place = [&](auto cnt, const h2* v, unsigned in, int at) {
    constexpr int ROWS = decltype(cnt)::value * RPP, N = (ROWS + RPT - 1) / RPT;
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int row = r0 + u * RPT, pn = row / RPP, q = row - pn * RPP;
      if (row >= ROWS || r0 >= RPT) continue;
      H* const to = lds + (at + pn) * CELLS + q * ROW + pz;
      const bool ok = in >> u & 1;
      to[0] = ok ? v[u][0] : H(0);
      to[6] = ok ? v[u][1] : H(0);
    }
  };
  constexpr std::integral_constant<int, 1> one{};
  constexpr std::integral_constant<int, 4> four{};
  constexpr bool AHEAD = FB <= 10;  // the next chunk is read beside a chunk's products
  h2 nv[FB];
  unsigned nin = 0;
  auto bread = [&](auto nac, int st, H (&b)[NE][decltype(nac)::value]) {
#pragma unroll
    for (int t = 0; t < decltype(nac)::value; ++t) {
      // (uniform base, the lane as a 32-bit offset)
      const auto p = gmem(W + ((size_t)(off[t] + st) * 8 + e0) * 64);
#pragma unroll
      for (int e = 0; e < NE; e += 2) {
        const hp v = *(const __attribute__((address_space(1))) hp*)(p + e * 64 + 2u * lane);
        b[e][t] = v[0], b[e + 1][t] = v[1];
      }
    }
  };
  auto products = [&](auto nac, const H (&a)[NR][NE], H (&b)[NE][decltype(nac)::value]) {
#pragma unroll
    for (int m = 0; m < NR; ++m)
#pragma unroll
      for (int e = 0; e < NE; ++e)
#pragma unroll
        for (int t = 0; t < decltype(nac)::value; ++t) acc[m][e][t] = M::op(a[m][e], b[e][t], acc[m][e][t]);
  };
  // chi of the axes the wave's patterns share
  const H cx = NE <= 4 && (e0 & 4) ? H(-1) : H(1), cy = NE <= 2 && (e0 & 2) ? H(-1) : H(1);
  // the 27 sources of chunk c
  auto run = [&](auto nac, int c, bool more) {
    constexpr int NA = decltype(nac)::value;
    const int t = (HEAD ? 1 : 0) + 4 * c + kq;  // the lane's term, and the signs of its minus images
    const int par = t >= NTERM ? 0 : OP == 3 ? t >> 5 : OP == 1 ? c_ft<P>.col[t] >> 8 : c_ft<P>.par[t];
    const H gx = par & 4 ? -cx : cx, gy = par & 2 ? -cy : cy, gz = par & 1 ? H(-1) : H(1);
    const int base = (HEAD ? FOLD_HEAD : 0) + 27 * c;
    const H* const pl = oct + kq * CELLS;
    const H* p[4];
    auto images = [&](int q) {
      const int jx = q / 3, jy = q - 3 * jx;
      p[0] = pl + (3 + jx) * PLANE + (3 + jy) * ROW;
      p[1] = pl + (3 + jx) * PLANE + (2 - jy) * ROW;
      p[2] = pl + (2 - jx) * PLANE + (3 + jy) * ROW;
      p[3] = pl + (2 - jx) * PLANE + (2 - jy) * ROW;
    };
    auto aread = [&](auto jc, H (&r)[NR][8]) {
      constexpr int jz = decltype(jc)::value;
#pragma unroll
      for (int m = 0; m < NR; ++m)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          r[m][2 * q] = p[q][m * 2 * PLANE + fold_z(3 + jz)];
          r[m][2 * q + 1] = p[q][m * 2 * PLANE + fold_z(2 - jz)];
        }
    };
    // operands are read one step ahead: images as soon as the last are folded
    H r[NR][8], b[3][NE][NA];
    images(0);
    bread(nac, base, b[0]);
    aread(std::integral_constant<int, 0>{}, r);
    if (AHEAD && more) {
      nin = fetch(four, (HEAD ? 1 : 0) + 4 * (c + 1), nv);
      asm volatile("" ::: "memory");  // (the loads stay up here)
    }
#pragma unroll 1
    for (int q = 0; q < 9; ++q)
      static_for<3>([&](auto jc) {
        constexpr int jz = decltype(jc)::value, nx = (jz + 1) % 3;
        H a[NR][NE];
#pragma unroll
        for (int m = 0; m < NR; ++m) fold8<NE>(r[m], gx, gy, gz, a[m]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (jz == 2) {
          const int qn = q < 8 ? q + 1 : 0;  // (past the last: read, not used)
          images(qn);
          bread(nac, base + 3 * qn, b[nx]);
        } else {
          bread(nac, base + 3 * q + jz + 1, b[nx]);
        }
        aread(std::integral_constant<int, nx>{}, r);
        __builtin_amdgcn_sched_barrier(0);
        products(nac, a, b[jz]);
        __builtin_amdgcn_sched_barrier(0);
      });
  };
  const int c0 = ip * nc[0] / np, c1 = (ip + 1) * nc[0] / np;
  const bool head = HEAD && ip == 0;
  if (c0 < c1) nin = fetch(four, (HEAD ? 1 : 0) + 4 * c0, nv);
  if (head) {
    h2 hv[(RPP + RPT - 1) / RPT];
    const unsigned hin = fetch(one, 0, hv);
    place(one, hv, hin, 4);
  }
  if (c0 < c1) place(four, nv, nin, 0);
  __syncthreads();
  if (head) {
    // term 0: 4 sources a step, at the lane's own places
    const H* const pl = oct + 4 * CELLS;
    H b[2][NE][NT];
    bread(std::integral_constant<int, NT>{}, 0, b[0]);
    static_for<FOLD_HEAD>([&](auto uc) {
      constexpr int u = decltype(uc)::value;
      H r[NR][8];
      const int s = min(4 * u + kq, 26), jx = s / 9, jy = (s / 3) % 3, jz = s % 3;
      const int xo[2] = {(3 + jx) * PLANE, (2 - jx) * PLANE}, yo[2] = {(3 + jy) * ROW, (2 - jy) * ROW},
                zo[2] = {((1 + jz) & 1) * 6 + ((3 + jz) >> 1), (jz & 1) * 6 + ((2 - jz) >> 1)};
#pragma unroll
      for (int m = 0; m < NR; ++m)
#pragma unroll
        for (int q = 0; q < 8; ++q) r[m][q] = pl[xo[q >> 2] + yo[(q >> 1) & 1] + zo[q & 1] + m * 2 * PLANE];
      if constexpr (u + 1 < FOLD_HEAD) bread(std::integral_constant<int, NT>{}, u + 1, b[(u + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
      H a[NR][NE];
#pragma unroll
      for (int m = 0; m < NR; ++m) fold8<NE>(r[m], cx, cy, H(1), a[m]);
      products(std::integral_constant<int, NT>{}, a, b[u & 1]);
      __builtin_amdgcn_sched_barrier(0);
    });
  }
  for (int c = c0; c < c1; ++c) {
    // the tiles that have chunk c are a prefix of the group
    int na = NT;
    while (na > 1 && nc[na - 1] <= c) --na;
    count_down<NT>([&](auto nac) {
      if (na == decltype(nac)::value) run(nac, c, c + 1 < c1);
    });
    if (c + 1 < c1) {
      __syncthreads();
      if (!AHEAD) nin = fetch(four, (HEAD ? 1 : 0) + 4 * (c + 1), nv);
      place(four, nv, nin, 0);
      __syncthreads();
    }
  }
  // the 8 patterns' sums of result q of row tile r, through LDS (one row tile
  // of each row group and NTE column tiles at a time), then from all parts of
  // the K loop
  constexpr int NQ = NX * 16 * 16 * NTE;
  double* const slot = args.part + (size_t)block * (MT * 16 * 16 * NT * 8);
  static_for<NR * (NT / NTE)>([&](auto rpc) {
    constexpr int rp = decltype(rpc)::value, r = rp / (NT / NTE), t0 = rp % (NT / NTE) * NTE;
    if (scol[16 * t0] < 0) return;  // (uniform: no columns there)
    __syncthreads();
#pragma unroll
    for (int e = 0; e < NE; ++e)
#pragma unroll
      for (int t = 0; t < NTE; ++t)
#pragma unroll
        for (int v = 0; v < 4; ++v)
          lds[((xg * 8 + e0 + e) * 16 + M::row(v, kq)) * CS + 16 * t + i] = acc[r][e][t0 + t][v];
    __syncthreads();
#pragma unroll 1
    for (int q = threadIdx.x; q < NQ; q += THR) {
      const int col = m2lf_qcol<OP, NTE>(q), row = m2lf_qrow<OP, NTE>(q), xr = q / (256 * NTE);
      double y[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) y[e] = (double)lds[((xr * 8 + e) * 16 + row) * CS + col];
      if (np > 1) {
#pragma unroll
        for (int e = 0; e < 8; ++e) slot[(size_t)(rp * 8 + e) * NQ + q] = y[e];
      } else {
        m2lf_put<P, H, OP>(sg, scol[16 * t0 + col], ox0, oy0, oz0, xr * NR + r, row, y);
      }
    }
  });
}

// a: the FP64 share of a launch (its blocks first), b: the FP32 share
template <int P, int OP, typename SA, typename SB>
__global__ __launch_bounds__(256, 2) void k_m2lf(const M2lArgs a, const M2lArgs b) {
  constexpr int LA = M2lLds<double, OP, SA>::BYTES, LB = M2lLds<float, OP, SB>::BYTES;
  static_assert(SA::NW % 4 == 0 && SB::NW % 4 == 0 && SA::NW <= 4 && SB::NW <= 4, "4 waves");
  __shared__ __attribute__((aligned(16))) char smem[LA > LB ? LA : LB];
  if constexpr (!SB::NW) {
    m2lf_run<P, double, OP, SA>(a, blockIdx.x, smem);
  } else if constexpr (!SA::NW) {
    m2lf_run<P, float, OP, SB>(b, blockIdx.x, smem);
  } else {
    const int first = (int)a.grid.blocks;
    if ((int)blockIdx.x < first)
      m2lf_run<P, double, OP, SA>(a, blockIdx.x, smem);
    else
      m2lf_run<P, float, OP, SB>(b, (int)blockIdx.x - first, smem);
  }
}

// Adds the parts of the shared groups of a k_m2lf launch, in order: MT x NT
// blocks for each tile of each such group (the FP64 share's na first).
template <int P, typename H, int OP, typename S>
__device__ __forceinline__ void m2lf_add(const M2lArgs& args, int block) {
  constexpr int MT = S::MT, NT = S::NT, NR = 8 * MT / (S::NE * S::NW), SUB = MT * NT;
  constexpr int NTE = m2lf_nte<NT>, NP = NT / NTE, NQ = MT / NR * 256 * NTE;
  const M2lGrid& grid = args.grid;
  const int sub = block % SUB, tile = block / SUB, T = args.T;
  int g = 0, left = tile / T;  // (a tile per T blocks of each shared group)
  while (grid.parts[g] == 1 || left-- > 0) ++g;
  const int lbk = tile % T, np = grid.parts[g];
  const Seg& sg = find_seg(args.segs, args.nseg, lbk);
  const int tb = lbk - sg.first_block;
  const int ox0 = (tb / (sg.tpa * sg.tpa)) * MT, oy0 = ((tb / sg.tpa) % sg.tpa) * 4, oz0 = (tb % sg.tpa) * 4;
  const double* slot = args.part + ((size_t)grid.first[g] + (size_t)lbk * np) * (NR * NP * NQ * 8);
  for (int x = sub * 256 + threadIdx.x; x < NR * NP * NQ; x += SUB * 256) {
    const int rp = x / NQ, q = x % NQ, col = 16 * (NT * g + rp % NP * NTE) + m2lf_qcol<OP, NTE>(q);
    const int cb = fold_colmap<P, OP>(col);
    if (cb < 0) continue;
    double y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = slot[(size_t)(rp * 8 + e) * NQ + q];
    // (several parts' loads in flight; the sum keeps its order)
#pragma unroll 4
    for (int k = 1; k < np; ++k)
#pragma unroll
      for (int e = 0; e < 8; ++e) y[e] += slot[(size_t)k * (NR * NP * NQ * 8) + (size_t)(rp * 8 + e) * NQ + q];
    m2lf_put<P, H, OP>(sg, cb, ox0, oy0, oz0, (q / (256 * NTE)) * NR + rp / NP, m2lf_qrow<OP, NTE>(q), y);
  }
}
template <int P, int OP, typename SA, typename SB>
__global__ __launch_bounds__(256) void k_m2lf_sum(const M2lArgs a, const M2lArgs b, int na) {
  if constexpr (SA::NW > 0)
    if ((int)blockIdx.x < na) m2lf_add<P, double, OP, SA>(a, blockIdx.x);
  if constexpr (SB::NW > 0)
    if ((int)blockIdx.x >= na) m2lf_add<P, float, OP, SB>(b, (int)blockIdx.x - na);
}

// The other operators' B fragments, as k_m2lf_table.
template <typename H>
__global__ void k_m2lf_adj_table(const double* __restrict__ Dtab, const int2* __restrict__ tiles, H* __restrict__ W,
                                 int P, int nmax, int ND, long long cnt) {
  const long long id = blockIdx.x * (long long)blockDim.x + threadIdx.x;
  if (id >= cnt) return;
  const int lane = (int)(id >> 1) & 63, e = ((int)(id >> 7) & 3) * 2 + (int)(id & 1), f = (int)(id >> 9);
  int t = 0;
  while (tiles[t].y + tiles[t].x <= f) ++t;
  int kt, s;
  fold_k(FO_M2LT, f - tiles[t].y, lane >> 4, &kt, &s);
  const int cb = m2lf_col(P, kt), a = 16 * t + (lane & 15);
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
  const int lane = (int)(id >> 1) & 63, e = ((int)(id >> 7) & 3) * 2 + (int)(id & 1), f = (int)(id >> 9);
  int t = 0;
  while (tiles[t].y + tiles[t].x <= f) ++t;
  const int col = 16 * t + (lane & 15);
  int kt, s;
  fold_k(adj ? FO_M2PT : FO_M2P, f - tiles[t].y, lane >> 4, &kt, &s);
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
