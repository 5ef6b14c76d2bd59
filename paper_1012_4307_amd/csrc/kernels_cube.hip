// kernels_cube.hip -- fused 3D kernels of the V(1,1) red-black cycle (Sec. 4.2
// of bin Zubair, Reps, Vanroose: one red-black SOR sweep before and after the
// coarse-grid correction, full weighting, trilinear interpolation).  Each
// level is visited by two kernels, as in 2D:
//
//   down: t = S_rb(0; b), rc = FW(b - M t)           reads b, k^2, writes rc
//   up:   t again, v = t + P ec, u = S_rb(v; b)      reads ec, b, k^2, writes u
//
// A block owns a column of the grid, an x-y tile times a chunk of z planes,
// and marches through its planes: a thread owns one pair of x-adjacent columns
// of the tile (one red and one black node in every plane), keeps the last four
// planes of its two columns in registers, so that z neighbours never leave the
// thread, and exchanges x and y neighbours through LDS.  The phases of the
// sweep run skewed by one plane each: in one step the red relaxation works on
// plane z, the black one on z - 1 (it needs red on z - 2 .. z), the residual
// (down) or the red post-relaxation (up) on z - 2, the full weighting or the
// black post-relaxation on z - 3.  What a phase reads from LDS was written in
// the step before into the other half of a double buffer, so a step has one
// barrier, and the loads of plane z + 1 are in flight while plane z is worked
// on.  Halos (three nodes) are recomputed, no grid-wide synchronisation.
//
// What bounds it: the issue and latency of a step (one barrier, an LDS round
// trip, 160-220 vector instructions of a thread at 2-3 waves per SIMD: 0.8-1.3
// us), not HBM.  Finest level of a 129^3 cycle, FP64: down 20 us (56 MB, 2.8
// TB/s), up 34 us (94 MB, 2.8 TB/s); FP32 17 and 26 us.  The separate kernels
// of the general cycle make seven passes over a level, and their residual +
// full weighting forms every fine residual 3.4 times (27 per coarse node): the
// whole cycle took 390 us FP64, 300 us FP32, now 112 and 96 us (148 and 119 before
// its coarse end was a dense map).
#include "ecs_cube.h"

namespace ecs {

namespace {

// Tile: 36 pairs = 72 staged columns (66 of them owned: levels of 2^k + 1
// nodes split into 65 / 66 without a nearly empty last tile), rows by threads.
constexpr int PX = 36;
constexpr int kOwn = 2 * PX - 6;  // owned fine columns
constexpr int CXD = PX - 3;       // owned coarse columns of the down kernel

template <typename R>
__device__ __forceinline__ cplx<R> zc() {
  return mk<R>(0, 0);
}
template <typename R>
__device__ __forceinline__ cplx<R> pick(bool c, cplx<R> a, cplx<R> b) {
  return mk<R>(c ? a.re : b.re, c ? a.im : b.im);
}
template <typename R>
__device__ __forceinline__ cplx<R> keep(bool c, cplx<R> a) {
  return mk<R>(c ? a.re : R(0), c ? a.im : R(0));
}
// acc + w u by four fused multiply-adds
template <typename R>
__device__ __forceinline__ cplx<R> fma_c(cplx<R> w, cplx<R> u, cplx<R> acc) {
  return mk<R>(fma(-w.im, u.im, fma(w.re, u.re, acc.re)), fma(w.im, u.re, fma(w.re, u.im, acc.im)));
}
// GS: omega = 1 known at compile time; a relaxed node then forgets its old
// value and has no residual, so a down step writes and weights the red residuals
// alone (five reads in even planes, four in odd ones, of nine) and an up step
// corrects the black nodes alone.  129^3 FP64 down 24.0 -> 22.1 us, up 34.3 ->
// 32.1; 97^3 FP32, still with an FP32 diagonal (diag3), 14.3 -> 13.8 and 18.9 ->
// 17.8.
template <bool GS, typename R>
__device__ __forceinline__ cplx<R> relaxed(R omega, cplx<R> v) {
  if constexpr (GS) return v;
  else return omega * v;
}
// 1 / d in FP64: the hardware estimate of 1 / |d|^2 and Newton steps y <- y +
// y (1 - a y) in fused arithmetic, each of which doubles the correct bits: one is
// enough for an FP32 result; after two the reciprocal is the correctly rounded
// one (no difference from the division over 2^27 random arguments), at a third of
// its instructions.
template <typename R>
__device__ __forceinline__ cplx<double> inv_d(cplx<double> d) {
  const double a = abs2(d);
  double s = __builtin_amdgcn_rcp(a);
  s = fma(s, fma(-a, s, 1.0), s);
  if constexpr (sizeof(R) == 8) s = fma(s, fma(-a, s, 1.0), s);
  return mk<double>(d.re * s, -d.im * s);
}

// What rounding 1 / D to FP32 leaves off, which the post-relaxation adds back: that
// error is the same at all nodes where D is (see diag3).  Nothing in FP64.
template <typename R>
struct Rest {
  cplx<R> v;
  __device__ __forceinline__ void set(cplx<double> inv) {
    if constexpr (sizeof(R) == 4) v = cvt<R>(inv - cvt<double>(cvt<R>(inv)));
  }
};
// acc + t / D
template <typename R>
__device__ __forceinline__ cplx<R> add_over(cplx<R> t, cplx<R> inv, const Rest<R> &rest, cplx<R> acc) {
  if constexpr (sizeof(R) == 4) acc = fma_c(rest.v, t, acc);
  return fma_c(t, inv, acc);
}
template <typename R>
__device__ __forceinline__ cplx<R> over(cplx<R> t, cplx<R> inv, const Rest<R> &rest) {
  if constexpr (sizeof(R) == 4) return fma_c(t, inv, rest.v * t);
  else return t * inv;
}

// one x-y plane of a level as a buffer resource (empty outside [0, n2))
template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const T *base, int k, bool in, int64_t plane) {
  return __builtin_amdgcn_make_buffer_rsrc((void *)(base + (in ? k : 0) * plane), 0,
                                           in ? (int)(plane * (int64_t)sizeof(T)) : 0, kRsrcWord3);
}

// What a thread holds of its two columns.  Column 0 is the red one in even
// steps (planes gz0, gz0 + 2, ...), column 1 in odd ones; the neighbours of a
// column-0 node in x and y are column-1 nodes of other threads and vice versa.
template <typename R>
struct Cols {
  int i[2];                // x index
  int j;                   // y index
  bool in[2];              // interior in x and y
  bool a0;                 // column 0 is the left one (a) of the pair
  int side[2];             // thread offset (+-1) of the column's x neighbour in the next pair
  cplx<R> wo[2], wn[2];    // x weights of the neighbour in the own pair / in the next pair
  cplx<R> ym[2], yp[2];    // y weights
  cplx<double> xy[2];      // the diagonal's x and y weights
  uint32_t ob[2], ok[2];   // byte offsets within a plane (outside: kOutside)
};

template <typename R>
__device__ __forceinline__ Cols<R> cols_of(const Grid<R> &g, int gx0, int gy0, int gz0, int l, int y, bool live) {
  Cols<R> q;
  const int ia = gx0 + 2 * l;
  q.j = gy0 + y;
  const bool yin = live && q.j >= 1 && q.j <= g.n1 - 2;
  q.a0 = ((ia + q.j + gz0) & 1) == 0;
  const cplx<R> ym = yin ? g.cm1[q.j] : zc<R>(), yp = yin ? g.cp1[q.j] : zc<R>();
#pragma unroll
  for (int c = 0; c < 2; c++) {
    const bool left = (c == 0) == q.a0;
    q.i[c] = left ? ia : ia + 1;
    q.in[c] = yin && q.i[c] >= 1 && q.i[c] <= g.n0 - 2;
    q.side[c] = left ? -1 : 1;
    const cplx<R> xm = q.in[c] ? g.cm0[q.i[c]] : zc<R>(), xp = q.in[c] ? g.cp0[q.i[c]] : zc<R>();
    q.wo[c] = pick(left, xp, xm);
    q.wn[c] = pick(left, xm, xp);
    // off the interior every weight and b are 0, so the iterate and the
    // residual stay 0 there without masks (in z the end planes' weights are 0
    // too); the diagonal only has to be invertible
    q.ym[c] = keep(q.in[c], ym);
    q.yp[c] = keep(q.in[c], yp);
    q.xy[c] = q.in[c] ? cvt<double>(xm) + cvt<double>(xp) + cvt<double>(ym) + cvt<double>(yp)
                     : mk<double>(1, 0);
    const uint32_t p = (uint32_t)(q.j * g.n0 + q.i[c]);
    q.ob[c] = q.in[c] ? p * (uint32_t)sizeof(cplx<R>) : kOutside;
    q.ok[c] = q.in[c] ? p * (uint32_t)sizeof(R) : kOutside;
  }
  return q;
}

// thread index of a neighbour, kept inside the block (the clamped reads are of
// halo nodes whose results nobody uses)
template <int NT>
__device__ __forceinline__ int in_block(int t) {
  return t < 0 ? 0 : t >= NT ? NT - 1 : t;
}

// The z weights of a plane (0 on the end planes; planes beyond the grid take
// the end planes').
template <typename R>
__device__ __forceinline__ cplx<R> zweight(const cplx<R> *w, int k, int n2) {
  return w[k < 0 ? 0 : k >= n2 ? n2 - 1 : k];
}

// The diagonal of a node, in FP64 for both types.  Where k^2 and the mesh are
// uniform it has the same rounding error at all nodes, which acts like an error of
// k^2 and is not averaged away, so FP32 neither forms it nor its inverse in FP32:
// error of a 97^3 cycle (k = 9) against 64 bits 2.6e-7 with both in FP32, 8.4e-8 so
// (the general kernels' correction form, u + (b - M u) / D: 1.9e-7), the cycle 69.9
// -> 71.4 us (finest up 17.8 -> 18.9); over 20 cycles of 17^3 to 161^3 0.22 to 0.94
// of the general kernels' error.
template <typename R>
__device__ __forceinline__ cplx<double> diag3(cplx<double> xy, cplx<R> zm, cplx<R> zp, R k2, const Grid<R> &g) {
  const cplx<double> z = cvt<double>(zm) + cvt<double>(zp) + cvt<double>(g.c);
  return xy + z + (double)k2 * cvt<double>(g.beta);
}

// off-diagonal sum plus `acc` at a column-r node: own / on = x neighbours in
// the own and the next pair, n + ym / yp = y neighbours, zm / zp in z.  FP32 sums
// axis by axis, half the roundings of a chain on the growing sum (8.4e-8 against
// 9.5e-8); FP64 is faster with the chain (129^3 112 us, 114 by axis) and its error
// is that of its weights (against 80-bit arithmetic 1.9e-16 to 4.0e-16 at 17^3 and
// 33^3, by axis 1.6e-16 to 6.2e-16, the general kernels 1.7e-16 to 4.5e-16).
template <typename R>
__device__ __forceinline__ cplx<R> offd3(const Cols<R> &q, int r, cplx<R> acc, cplx<R> own, const cplx<R> *n, int nx,
                                         int nym, int nyp, cplx<R> wzm, cplx<R> zm, cplx<R> wzp, cplx<R> zp) {
  if constexpr (sizeof(R) == 4) {
    const cplx<R> x = fma_c(q.wn[r], n[nx], q.wo[r] * own);
    const cplx<R> y = fma_c(q.yp[r], n[nyp], q.ym[r] * n[nym]);
    const cplx<R> z = fma_c(wzp, zp, wzm * zm);
    return acc + ((x + y) + z);
  }
  acc = fma_c(q.wo[r], own, acc);
  acc = fma_c(wzm, zm, acc);
  acc = fma_c(wzp, zp, acc);
  acc = fma_c(q.wn[r], n[nx], acc);
  acc = fma_c(q.ym[r], n[nym], acc);
  return fma_c(q.yp[r], n[nyp], acc);
}

// ----------------------------------------------------------------- down
// CY coarse rows (2 CY + 5 staged rows) x CXD coarse columns x cz coarse
// planes; staged planes 2 K0 - 3 + [0, 2 cz + 5).
template <int CY>
struct DownTile {
  static constexpr int ROWS = 2 * CY + 5;
  static constexpr int NT = (PX * ROWS + 63) / 64 * 64;
};

template <typename R, int CY, bool GS>
__global__ __launch_bounds__(DownTile<CY>::NT) void k_down3(Grid<R> f, Grid<R> c, const cplx<R> *__restrict__ b,
                                                            cplx<R> *__restrict__ rc, R omega, int tx, int ty, int cz,
                                                            int tiles) {
  constexpr int ROWS = DownTile<CY>::ROWS, NT = DownTile<CY>::NT;
  // [half][thread]; the residuals by position, a in [0, NT), b in [NT, 2 NT)
  // (GS: only the red ones, at their thread)
  __shared__ cplx<R> sRed[2][NT], sBlk[2][NT], sRes[2][GS ? NT : 2 * NT];
  const int tid = threadIdx.x;
  const int tile = xcd_tile(tiles);
  if (tile < 0) return;
  const int I0 = (tile % tx) * CXD, J0 = ((tile / tx) % ty) * CY, K0 = (tile / (tx * ty)) * cz;
  const int gx0 = 2 * I0 - 3, gy0 = 2 * J0 - 3, gz0 = 2 * K0 - 3;
  const int y = tid / PX, l = tid - y * PX;
  const Cols<R> q = cols_of(f, gx0, gy0, gz0, l, y, y < ROWS);
  const R om1 = R(1) - omega;
  const int64_t plane = (int64_t)f.n0 * f.n1;
  const int nb[2] = {in_block<NT>(tid + q.side[0]), in_block<NT>(tid + q.side[1])};
  const int ym = in_block<NT>(tid - PX), yp = in_block<NT>(tid + PX);
  const int pos[2] = {q.a0 ? tid : tid + NT, q.a0 ? tid + NT : tid};
  // full weighting: thread -> coarse column, its centre in pair fl + 1, column b, row 2 fj + 3
  const int fj = tid / CXD, fl = tid - fj * CXD;
  const bool fw = tid < CXD * CY && I0 + fl < c.n0 && J0 + fj < c.n1;
  const bool fin = fw && I0 + fl >= 1 && I0 + fl <= c.n0 - 2 && J0 + fj >= 1 && J0 + fj <= c.n1 - 2;
  const int ft = fw ? (2 * fj + 3) * PX + fl + 1 : PX + 1;
  cplx<R> acc = zc<R>();

  // slot = step & 3 of a plane; plane z + 1 is loaded into the slot that plane
  // z - 3 no longer needs
  cplx<R> B[2][4], D[2][4], T[2][4], resB = zc<R>();
  cplx<R> zm[4], zp[4];  // z weights of the planes (uniform)
  R K2[2];
#pragma unroll
  for (int m = 0; m < 4; m++) {
    zm[m] = zp[m] = zc<R>();
#pragma unroll
    for (int e = 0; e < 2; e++) B[e][m] = D[e][m] = T[e][m] = zc<R>();
  }
  auto load = [&](int k, int m) {
    zm[m] = zweight(f.cm2, k, f.n2);
    zp[m] = zweight(f.cp2, k, f.n2);
    const bool zin = k >= 1 && k <= f.n2 - 2;
    const __amdgpu_buffer_rsrc_t rb = plane_rsrc(b, k, zin, plane), rk = plane_rsrc(f.k2, k, zin, plane);
#pragma unroll
    for (int e = 0; e < 2; e++) {
      B[e][m] = ld_c(rb, q.ob[e], cplx<R>());
      K2[e] = ld_r(rk, q.ok[e], R());
    }
  };
  load(gz0, 0);
  const int steps = 2 * cz + 6;
  auto step = [&](int s, auto M) {
    constexpr int m0 = decltype(M)::value, m1 = (m0 + 3) & 3, m2 = (m0 + 2) & 3, m3 = (m0 + 1) & 3;
    constexpr int r = m0 & 1, h = m0 & 1, ho = 1 - h;
    const int z = gz0 + s;
    // plane z has arrived; its diagonals, and red from zero: omega b / D
    {
#pragma unroll
      for (int e = 0; e < 2; e++) D[e][m0] = cvt<R>(inv_d<R>(diag3(q.xy[e], zm[m0], zp[m0], K2[e], f)));
    }
    load(z + 1, m3);
    T[r][m0] = relaxed<GS>(omega, B[r][m0]) * D[r][m0];
    sRed[h][tid] = T[r][m0];
    // black on z - 1, and its residual (1 - w)(b + o)
    const cplx<R> tb = offd3(q, r, B[r][m1], T[1 - r][m1], sRed[ho], nb[r], ym, yp, zm[m1], T[r][m2], zp[m1],
                             T[r][m0]);
    T[r][m1] = relaxed<GS>(omega, tb) * D[r][m1];
    sBlk[h][tid] = T[r][m1];
    // residual of plane z - 2: red (1 - w) b + o, black from the step before
    if constexpr (GS) {
      sRes[h][tid] = offd3(q, r, zc<R>(), T[1 - r][m2], sBlk[ho], nb[r], ym, yp, zm[m2], T[r][m3], zp[m2], T[r][m1]);
    } else {
      sRes[h][pos[r]] = offd3(q, r, om1 * B[r][m2], T[1 - r][m2], sBlk[ho], nb[r], ym, yp, zm[m2], T[r][m3], zp[m2],
                              T[r][m1]);
      sRes[h][pos[1 - r]] = resB;
      resB = om1 * tb;
    }
    // full weighting of plane z - 3: its x-y average, then 1/4, 1/2, 1/4 in z
    if (fw) {
      const cplx<R> *ra = sRes[ho], *rb = ra + NT;
      cplx<R> S;
      if constexpr (GS && (m0 & 1) == 0)  // red: the centre (b) and the corners (a)
        S = R(0.25) * ra[ft] + R(0.0625) * (ra[ft - PX] + ra[ft - PX + 1] + ra[ft + PX] + ra[ft + PX + 1]);
      else if constexpr (GS)  // red: the neighbours in x (a) and y (b)
        S = R(0.125) * (ra[ft] + ra[ft + 1] + ra[ft - PX] + ra[ft + PX]);
      else
        S = R(0.25) * rb[ft] + R(0.125) * (ra[ft] + ra[ft + 1] + rb[ft - PX] + rb[ft + PX]) +
            R(0.0625) * (ra[ft - PX] + ra[ft - PX + 1] + ra[ft + PX] + ra[ft + PX + 1]);
      if constexpr ((m0 & 1) == 0) {
        acc = acc + R(0.5) * S;  // s - 3 odd: the centre plane
      } else {
        const int K = K0 + (s - 7) / 2;
        if (s >= 7 && K < c.n2)
          rc[((int64_t)K * c.n1 + J0 + fj) * c.n0 + I0 + fl] =
              keep(fin && K >= 1 && K <= c.n2 - 2, acc + R(0.25) * S);
        acc = R(0.25) * S;
      }
    }
    __syncthreads();
  };
  for (int s = 0; s < steps; s += 4) {
    step(s, std::integral_constant<int, 0>());
    if (s + 1 < steps) step(s + 1, std::integral_constant<int, 1>());
    if (s + 2 < steps) step(s + 2, std::integral_constant<int, 2>());
    if (s + 3 < steps) step(s + 3, std::integral_constant<int, 3>());
  }
}

// ------------------------------------------------------------------- up
// ROWS staged rows (ROWS - 6 owned) x kOwn owned columns x cz owned planes
// (cz even); staged planes Z0 - 3 + [0, cz + 6).  The pre-smoothed iterate is
// recomputed from b, as in 2D.  The coarse correction is interpolated in x and
// y per coarse plane and pair (column a is odd: the mean of two coarse columns;
// four cached reads a pair), and between two coarse planes in registers.
template <typename R, int ROWS, int NT, bool GS>
__global__ __launch_bounds__(NT) void k_up3(Grid<R> f, Grid<R> c, const cplx<R> *__restrict__ b,
                                            const cplx<R> *__restrict__ ec, cplx<R> *__restrict__ u, R omega, int tx,
                                            int ty, int cz, int tiles) {
  static_assert(PX * ROWS <= NT, "every staged pair has a thread");
  __shared__ cplx<R> sRed[2][NT], sBlk[2][NT], sRel[2][NT];
  const int tid = threadIdx.x;
  const int tile = xcd_tile(tiles);
  if (tile < 0) return;
  const int gx0 = (tile % tx) * kOwn - 3, gy0 = ((tile / tx) % ty) * (ROWS - 6) - 3;
  const int Z0 = (tile / (tx * ty)) * cz, gz0 = Z0 - 3;
  const int y = tid / PX, l = tid - y * PX;
  const Cols<R> q = cols_of(f, gx0, gy0, gz0, l, y, y < ROWS);
  const R om1 = R(1) - omega;
  const int64_t plane = (int64_t)f.n0 * f.n1, cplane = (int64_t)c.n0 * c.n1;
  const int nb[2] = {in_block<NT>(tid + q.side[0]), in_block<NT>(tid + q.side[1])};
  const int ym = in_block<NT>(tid - PX), yp = in_block<NT>(tid + PX);
  const bool yown = y >= 3 && y < ROWS - 3 && q.j < f.n1;
  uint32_t os[2], oe[4];  // byte offsets of the stores and of the pair's four coarse nodes
#pragma unroll
  for (int e = 0; e < 2; e++) {
    const int x = q.i[e] - gx0;
    const bool own = yown && x >= 3 && x < 3 + kOwn && q.i[e] < f.n0;
    os[e] = own ? (uint32_t)(q.j * f.n0 + q.i[e]) * (uint32_t)sizeof(cplx<R>) : kOutside;
  }
  {
    // coarse columns of the pair: that of b and the one before it
    const int Ib = (gx0 + 2 * l + 1) >> 1, Ja = q.j >> 1, Jb = Ja + (q.j & 1);
    const bool yin = y < ROWS && q.j >= 1 && q.j <= f.n1 - 2;
#pragma unroll
    for (int w = 0; w < 4; w++) {
      const int I = (w & 1) ? Ib : Ib - 1, J = (w >> 1) ? Jb : Ja;
      oe[w] = yin && I >= 0 && I < c.n0 ? (uint32_t)(J * c.n0 + I) * (uint32_t)sizeof(cplx<R>) : kOutside;
    }
  }

  // per plane (slot = step & 3): b and 1 / D of both columns; of the red node
  // t, v = t + P e (not GS: its new value does not use it) and the post-relaxed
  // u; of the black node v
  cplx<R> B[2][4], D[2][4], T[4], vR[4], vB[4], uR[4], nB[2], Ec[2], En[2];
  Rest<R> X[2][4];
  cplx<R> zm[4], zp[4], nzm, nzp;  // z weights of the planes (uniform)
  R K2[2];
#pragma unroll
  for (int m = 0; m < 4; m++) {
    zm[m] = zp[m] = zc<R>();
    T[m] = vR[m] = vB[m] = uR[m] = zc<R>();
#pragma unroll
    for (int e = 0; e < 2; e++) {
      B[e][m] = D[e][m] = zc<R>();
      X[e][m].set(zc<double>());
    }
  }
  Ec[0] = Ec[1] = En[0] = En[1] = zc<R>();
  auto load = [&](int k) {
    nzm = zweight(f.cm2, k, f.n2);
    nzp = zweight(f.cp2, k, f.n2);
    const bool zin = k >= 1 && k <= f.n2 - 2;
    const __amdgpu_buffer_rsrc_t rb = plane_rsrc(b, k, zin, plane), rk = plane_rsrc(f.k2, k, zin, plane);
#pragma unroll
    for (int e = 0; e < 2; e++) {
      nB[e] = ld_c(rb, q.ob[e], cplx<R>());
      K2[e] = ld_r(rk, q.ok[e], R());
    }
  };
  load(gz0);
  const int steps = cz + 6;
  auto step = [&](int s, auto M) {
    constexpr int m0 = decltype(M)::value, m1 = (m0 + 3) & 3, m2 = (m0 + 2) & 3, m3 = (m0 + 1) & 3;
    constexpr int r = m0 & 1, h = m0 & 1, ho = 1 - h;
    const int z = gz0 + s;
    {
      zm[m0] = nzm;
      zp[m0] = nzp;
#pragma unroll
      for (int e = 0; e < 2; e++) {
        B[e][m0] = nB[e];
        const cplx<double> inv = inv_d<R>(diag3(q.xy[e], nzm, nzp, K2[e], f));
        D[e][m0] = cvt<R>(inv);
        X[e][m0].set(inv);
      }
    }
    load(z + 1);
    // even steps work on the fine plane z - 1 = 2 K and fetch coarse plane
    // K + 1; odd ones on 2 K + 1, the mean of the two
    cplx<R> raw[4];
    if constexpr ((m0 & 1) == 0) {
      const int K = (z - 1) / 2 + 1;  // z - 1 is even, so the division is exact
      const __amdgpu_buffer_rsrc_t re = plane_rsrc(ec, K, K >= 0 && K < c.n2, cplane);
#pragma unroll
      for (int w = 0; w < 4; w++) raw[w] = ld_c(re, oe[w], cplx<R>());
    }
    T[m0] = relaxed<GS>(omega, B[r][m0]) * D[r][m0];
    sRed[h][tid] = T[m0];
    // black t on z - 1, then v = t + P e on both nodes of the pair
    {
      const cplx<R> tb = offd3(q, r, B[r][m1], T[m1], sRed[ho], nb[r], ym, yp, zm[m1], T[m2],
                               zp[m1], T[m0]);
      cplx<R> pb = Ec[r], pr = Ec[1 - r];
      if constexpr ((m0 & 1) != 0) {
        pb = R(0.5) * (pb + En[r]);
        pr = R(0.5) * (pr + En[1 - r]);
      }
      vB[m1] = fma_c(relaxed<GS>(omega, tb), D[r][m1], pb);
      if constexpr (!GS) vR[m1] = T[m1] + pr;
      sBlk[h][tid] = vB[m1];
    }
    // red post-relaxation on z - 2
    {
      const cplx<R> o = offd3(q, r, B[r][m2], vB[m2], sBlk[ho], nb[r], ym, yp, zm[m2], vB[m3],
                              zp[m2], vB[m1]);
      if constexpr (GS) uR[m2] = over(o, D[r][m2], X[r][m2]);
      else uR[m2] = add_over(omega * o, D[r][m2], X[r][m2], om1 * vR[m2]);
      sRel[h][tid] = uR[m2];
    }
    // black post-relaxation on z - 3; both nodes are final
    if (s >= 6) {
      const cplx<R> o = offd3(q, r, B[r][m3], uR[m3], sRel[ho], nb[r], ym, yp, zm[m3], uR[m0],
                              zp[m3], uR[m2]);
      cplx<R> uB;
      if constexpr (GS) uB = over(o, D[r][m3], X[r][m3]);
      else uB = add_over(omega * o, D[r][m3], X[r][m3], om1 * vB[m3]);
      const bool zin = z - 3 >= 1 && z - 3 <= f.n2 - 2;
      const __amdgpu_buffer_rsrc_t ro = plane_rsrc(u, z - 3, z - 3 < f.n2, plane);
      st_c(ro, os[r], keep(q.in[r] && zin, uB));
      st_c(ro, os[1 - r], keep(q.in[1 - r] && zin, uR[m3]));
    }
    if constexpr ((m0 & 1) == 0) {
      const cplx<R> ea = R(0.25) * ((raw[0] + raw[1]) + (raw[2] + raw[3])), eb = R(0.5) * (raw[1] + raw[3]);
#pragma unroll
      for (int e = 0; e < 2; e++) En[e] = keep(q.in[e], pick((e == 0) == q.a0, ea, eb));
    } else {
      Ec[0] = En[0];
      Ec[1] = En[1];
    }
    __syncthreads();
  };
  for (int s = 0; s < steps; s += 4) {
    step(s, std::integral_constant<int, 0>());
    if (s + 1 < steps) step(s + 1, std::integral_constant<int, 1>());
    if (s + 2 < steps) step(s + 2, std::integral_constant<int, 2>());
    if (s + 3 < steps) step(s + 3, std::integral_constant<int, 3>());
  }
}

// A launch shape: z planes per block and the time it is expected to take.
struct Shape {
  int cz;
  int64_t cost;
};

// Planes per block, a multiple of `unit`: every block runs extra + per_plane cz
// steps, 256 blocks (one per CU) at a time, so the chunk with the fewest steps
// over all rounds is taken: a longer chunk repeats fewer halo planes, a shorter
// one fills the chip, and a last round of a few blocks costs as much as a full
// one (129^3 FP64: 376 down blocks in two rounds 46 us, 248 in one 23 us).
Shape chunk(int64_t xy_tiles, int planes, int unit, int per_plane, int64_t step_cost) {
  Shape best{unit, INT64_MAX};
  for (int cz = unit; cz <= 32 * unit; cz += unit) {
    const int64_t tiles = xy_tiles * ((planes + cz - 1) / cz);
    const int64_t cost = (tiles + 255) / 256 * (per_plane * cz + 6) * step_cost;
    if (cost < best.cost) best = {cz, cost};
    if (cz >= planes) break;
  }
  return best;
}

template <int CY>
Shape down_shape(int n0, int n1, int n2, int64_t step_cost) {
  return chunk((int64_t)((n0 + CXD - 1) / CXD) * ((n1 + CY - 1) / CY), n2, 1, 2, step_cost);
}
template <int ROWS>
Shape up_shape(int n0, int n1, int n2, int64_t step_cost) {
  return chunk((int64_t)((n0 + kOwn - 1) / kOwn) * ((n1 + ROWS - 7) / (ROWS - 6)), n2, 2, 1, step_cost);
}

template <typename R, int CY>
void launch_down3_t(const Grid<R> &f, const Grid<R> &c, const cplx<R> *b, cplx<R> *rc, R omega, int cz,
                    hipStream_t s) {
  const int tx = (c.n0 + CXD - 1) / CXD, ty = (c.n1 + CY - 1) / CY;
  const int tiles = tx * ty * ((c.n2 + cz - 1) / cz);
  const dim3 grid(xcd_padded(tiles)), block(DownTile<CY>::NT);
  if (omega == R(1)) launch_k((k_down3<R, CY, true>), grid, block, 0, s, f, c, b, rc, omega, tx, ty, cz, tiles);
  else launch_k((k_down3<R, CY, false>), grid, block, 0, s, f, c, b, rc, omega, tx, ty, cz, tiles);
}

template <typename R, int ROWS>
void launch_up3_t(const Grid<R> &f, const Grid<R> &c, const cplx<R> *b, const cplx<R> *ec, cplx<R> *u, R omega,
                  int cz, hipStream_t s) {
  constexpr int NT = (PX * ROWS + 63) / 64 * 64;
  const int tx = (f.n0 + kOwn - 1) / kOwn, ty = (f.n1 + ROWS - 7) / (ROWS - 6);
  const int tiles = tx * ty * ((f.n2 + cz - 1) / cz);
  const dim3 grid(xcd_padded(tiles)), block(NT);
  if (omega == R(1)) launch_k((k_up3<R, ROWS, NT, true>), grid, block, 0, s, f, c, b, ec, u, omega, tx, ty, cz, tiles);
  else launch_k((k_up3<R, ROWS, NT, false>), grid, block, 0, s, f, c, b, ec, u, omega, tx, ty, cz, tiles);
}

}  // namespace

// Tile heights: tall tiles repeat fewer halo rows, low ones have fewer waves to
// run through a step (a step of the low tile costs 9 where the tall one's costs
// 10, measured), so the low tile wins where the level fits one round anyway.
// 33^3 FP64: down 9.2 us with 4 coarse rows, 10.8 with 6; 129^3: 25.4 and 22.7;
// up 10.7 us with 10 rows, 11.1 with 14; 129^3: 59 and 36.5.  The tall up tile
// of FP64 is 14 rows, 8 waves of 242 VGPRs (17 rows spill: 142 us); FP32 holds
// 17 rows (26.1 us at 129^3 against 29.3 with 14).
template <typename R>
void launch_down3_rb(const Grid<R> &f, const Grid<R> &c, const cplx<R> *b, cplx<R> *rc, R omega, hipStream_t s) {
  const Shape tall = down_shape<6>(c.n0, c.n1, c.n2, 10), low = down_shape<4>(c.n0, c.n1, c.n2, 9);
  if (low.cost < tall.cost) launch_down3_t<R, 4>(f, c, b, rc, omega, low.cz, s);
  else launch_down3_t<R, 6>(f, c, b, rc, omega, tall.cz, s);
}

template <typename R>
void launch_up3_rb(const Grid<R> &f, const Grid<R> &c, const cplx<R> *b, const cplx<R> *ec, cplx<R> *u, R omega,
                   hipStream_t s) {
  constexpr int TALL = sizeof(R) == 8 ? 14 : 17;
  const Shape tall = up_shape<TALL>(f.n0, f.n1, f.n2, 10), low = up_shape<10>(f.n0, f.n1, f.n2, 9);
  if (low.cost < tall.cost) launch_up3_t<R, 10>(f, c, b, ec, u, omega, low.cz, s);
  else launch_up3_t<R, TALL>(f, c, b, ec, u, omega, tall.cz, s);
}

#define ECS_INST_CUBE(R)                                                                                        \
  template void launch_down3_rb<R>(const Grid<R> &, const Grid<R> &, const cplx<R> *, cplx<R> *, R,             \
                                   hipStream_t);                                                                \
  template void launch_up3_rb<R>(const Grid<R> &, const Grid<R> &, const cplx<R> *, const cplx<R> *, cplx<R> *, \
                                 R, hipStream_t);
ECS_INST_CUBE(double)
ECS_INST_CUBE(float)

}  // namespace ecs
