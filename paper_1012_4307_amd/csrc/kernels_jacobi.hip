// kernels_jacobi.hip -- fused 2D kernels of general omega-Jacobi cycles with one
// sweep before and after the coarse-grid correction (the F cycles of Sec. 5 of
// bin Zubair, Reps, Vanroose).  Algorithm 1 visits a level in groups, the gamma
// visits its parent makes in a row, with the level's right-hand side unchanged;
// one kernel covers everything the level does between two visits of the next
// one:
//
//   first visit:   x = J(0),                 rc = FW(b - M x)
//   later visits:  x = J(J(x + P e)),        rc = FW(b - M x)
//                  (the post-sweep of one visit, the pre-sweep of the next)
//   after the last: x = J(x + P e)
//
// gamma + 1 launches for gamma visits, where a launch per step takes 3 gamma.
// On the levels in question (a few hundred nodes per axis and less) a launch
// costs more than its bytes.  A block owns a tile, stages it with a halo (two
// nodes, two more per further sweep) and recomputes the halo, phases exchanging
// neighbours through LDS; x is written to the other of two buffers, since the
// neighbouring blocks read the old one.
//
// What bounds them: launch latency and the phases of a block on all levels but
// the finest of a large grid.  641^2 FP64: first visit 7.5 us (4.9 TB/s of its 37
// MB with the stores), after the last 7.0 us; 321^2 4.7, later visits 6.8, after
// the last 4.3; 81^2 4.0, 5.3, 4.8.  The three launches of a visit took 3.5 + 4.8
// + 4.7 us on average over the levels, 9.4 us for the last on 641^2.  An F_1^3 cycle on 641^2
// is 33 launches instead of 55: 268 -> 198 us; F_1^4 on 385^2 280 -> 185 us.
#include "ecs_jacobi.h"

namespace ecs {

namespace {

template <typename R>
__device__ __forceinline__ cplx<R> zj() {
  return mk<R>(0, 0);
}

// The diagonal of a node.  It, its inverse and their products are FP64 for both
// types: where k^2 and the mesh are uniform an FP32 rounding of the diagonal is the
// same at all nodes, acts like an error of k^2 and is not averaged away.  FP32
// cycles of 129^2 to 641^2 against the 64-bit one: 1.1 to 1.2 times the error of the
// general kernels (which correct by the quotient of the residual) with an FP32
// diagonal, 0.4 to 0.9 times so.  A kernel takes up to 0.2 us more, an FP32 cycle 2
// to 4% (F_1^3 on 641^2 137.5 -> 143.2 us).
template <typename R>
__device__ __forceinline__ cplx<double> diag_j(cplx<R> xm, cplx<R> xp, cplx<R> ym, cplx<R> yp, R k2, cplx<R> beta,
                                               cplx<R> c) {
  return cvt<double>(xm) + cvt<double>(xp) + cvt<double>(ym) + cvt<double>(yp) +
         ((double)k2 * cvt<double>(beta) + cvt<double>(c));
}

// 1 / a; for an FP32 result the hardware estimate and one Newton step, 46 bits
template <typename R>
__device__ __forceinline__ double recip(double a) {
  if constexpr (sizeof(R) == 8) return 1.0 / a;
  const double s = __builtin_amdgcn_rcp(a);
  return fma(s, fma(-a, s, 1.0), s);
}

// MODE 0: first visit, 2: later ones.  Tile: CX x CY coarse nodes from (I0, J0);
// residuals are needed on fine columns 2 I0 + [-1, 2 CX), x on [-2, 2 CX + 1),
// and one node further out for each sweep that reads neighbours.
// Lanes are columns, the 4 waves take every fourth row, a thread keeps b, D,
// 1 / D and the iterate of its nodes in registers.
template <typename R, int CY, int MODE>
__global__ __launch_bounds__(256) void k_jac_down(Grid<R> f, Grid<R> c, const cplx<R> *__restrict__ b,
                                                  const cplx<R> *__restrict__ x, const cplx<R> *__restrict__ e,
                                                  cplx<R> *__restrict__ out, cplx<R> *__restrict__ rc, R omega,
                                                  int tiles_x, int tiles) {
  constexpr int H = 2 + MODE, CX = (64 - (2 * H - 1)) / 2;
  constexpr int WX = 2 * CX + 2 * H - 1, WY = 2 * CY + 2 * H - 1, RPW = (WY + 3) / 4;
  __shared__ cplx<R> s0[WY][64], s1[WY][64];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tile = xcd_tile(tiles);
  if (tile < 0) return;
  const int I0 = (tile % tiles_x) * CX, J0 = (tile / tiles_x) * CY;
  const int gx0 = 2 * I0 - H, gy0 = 2 * J0 - H, n0 = f.n0, n1 = f.n1;
  const double om1 = 1.0 - (double)omega;
  const int i = gx0 + lane;
  const bool xin = lane < WX && i >= 1 && i <= n0 - 2;
  const cplx<R> xm = xin ? f.cm0[i] : zj<R>(), xp = xin ? f.cp0[i] : zj<R>();
  const int lm = lane > 0 ? lane - 1 : 0, lp = lane < 63 ? lane + 1 : 63;  // clamped: halo results nobody uses
  // interior rows of the window through buffer resources: 0 elsewhere
  const int jl = min(max(gy0, 1), n1 - 1), jh = min(max(gy0 + WY, 1), n1 - 1);
  const __amdgpu_buffer_rsrc_t rb = rows_rsrc(b, jl, jh, n0), rk = rows_rsrc(f.k2, jl, jh, n0);
  const __amdgpu_buffer_rsrc_t rx = rows_rsrc(MODE ? x : b, jl, jh, n0);
  const uint32_t oc = col_off<cplx<R>>(xin, i), ok = col_off<R>(xin, i);
  // the correction's rows; its column i / 2 and the next (the same when i is even)
  const int Jl = min(max(gy0 >> 1, 0), c.n1), Jh = min((gy0 + WY) / 2 + 2, c.n1);
  const __amdgpu_buffer_rsrc_t re = rows_rsrc(MODE ? e : b, Jl, Jh, c.n0);
  const uint32_t oa = col_off<cplx<R>>(xin, i >> 1), ob = col_off<cplx<R>>(xin, (i >> 1) + (i & 1));
  cplx<R> B[RPW], X[RPW], ym[RPW], yp[RPW], ea[RPW], eb[RPW], ec[RPW], ed[RPW];
  cplx<double> D[RPW], V[RPW];
  R K[RPW];
#pragma unroll
  for (int r = 0; r < RPW; r++) {
    const int ly = wv + 4 * r, j = gy0 + ly;
    const bool yin = ly < WY && j >= 1 && j <= n1 - 2;
    const int jc = yin ? j : 1;
    ym[r] = yin ? f.cm1[jc] : zj<R>();
    yp[r] = yin ? f.cp1[jc] : zj<R>();
    const uint32_t q = row_off<cplx<R>>(j - jl, n0);
    B[r] = ld_c(rb, oc + q, cplx<R>());
    K[r] = ld_r(rk, ok + row_off<R>(j - jl, n0), R());
    if constexpr (MODE != 0) {
      X[r] = ld_c(rx, oc + q, cplx<R>());
      const uint32_t q0 = row_off<cplx<R>>((j >> 1) - Jl, c.n0), q1 = row_off<cplx<R>>((j >> 1) + (j & 1) - Jl, c.n0);
      ea[r] = ld_c(re, oa + q0, cplx<R>());
      eb[r] = ld_c(re, ob + q0, cplx<R>());
      ec[r] = ld_c(re, oa + q1, cplx<R>());
      ed[r] = ld_c(re, ob + q1, cplx<R>());
    }
  }
  // diagonals; x = J(0) or v = x + P e (0 off the interior)
#pragma unroll
  for (int r = 0; r < RPW; r++) {
    const int ly = wv + 4 * r, j = gy0 + ly;
    if (ly < WY) {
      const bool in = xin && j >= 1 && j <= n1 - 2;
      D[r] = in ? diag_j(xm, xp, ym[r], yp[r], K[r], f.beta, f.c) : mk<double>(1, 0);
      const double s = recip<R>(abs2(D[r]));
      V[r] = mk<double>(D[r].re * s, -D[r].im * s);
      if constexpr (MODE == 0) X[r] = cvt<R>((double)omega * (cvt<double>(B[r]) * V[r]));
      else X[r] = in ? X[r] + R(0.25) * ((ea[r] + eb[r]) + (ec[r] + ed[r])) : zj<R>();
      s0[ly][lane] = X[r];
    }
  }
  __syncthreads();
  auto offd = [&](const cplx<R>(*s)[64], int ly, int r) {
    return xm * s[ly][lm] + xp * s[ly][lp] + ym[r] * s[ly - 1][lane] + yp[r] * s[ly + 1][lane];
  };
  if constexpr (MODE != 0) {
    // two sweeps, each a ring further in (from s0 to s1 and back)
#pragma unroll
    for (int sw = 0; sw < 2; sw++) {
      cplx<R>(*from)[64] = sw == 0 ? s0 : s1;
      cplx<R>(*to)[64] = sw == 0 ? s1 : s0;
#pragma unroll
      for (int r = 0; r < RPW; r++) {
        const int ly = wv + 4 * r, j = gy0 + ly;
        if (ly >= 1 + sw && ly <= WY - 2 - sw) {
          const cplx<R> o = offd(from, ly, r);
          X[r] = (xin && j >= 1 && j <= n1 - 2)
                     ? cvt<R>(om1 * cvt<double>(X[r]) + (double)omega * (cvt<double>(B[r] + o) * V[r]))
                     : zj<R>();
          to[ly][lane] = X[r];
        }
      }
      __syncthreads();
    }
  }
  // x of the owned nodes; residual b - M x, 0 off the interior
  const __amdgpu_buffer_rsrc_t ro = rows_rsrc(out, 2 * J0, min(2 * J0 + 2 * CY, n1), n0);
  const uint32_t oo = col_off<cplx<R>>(lane >= H && lane < H + 2 * CX && i < n0, i);
#pragma unroll
  for (int r = 0; r < RPW; r++) {
    const int ly = wv + 4 * r, j = gy0 + ly;
    if (ly >= H && ly < H + 2 * CY && j < n1) st_c(ro, oo + row_off<cplx<R>>(j - 2 * J0, n0), X[r]);
    if (ly >= H - 1 && ly <= H + 2 * CY - 1) {
      const cplx<R> o = offd(s0, ly, r);
      s1[ly][lane] =
          (xin && j >= 1 && j <= n1 - 2) ? cvt<R>(cvt<double>(B[r] + o) - D[r] * cvt<double>(X[r])) : zj<R>();
    }
  }
  __syncthreads();
  // full weighting: lane = coarse column, its fine node in column H + 2 lane
  if (lane < CX) {
    const int I = I0 + lane, p = H + 2 * lane;
    for (int cy = wv; cy < CY; cy += 4) {
      const int J = J0 + cy, y = H + 2 * cy;
      if (I >= c.n0 || J >= c.n1) continue;
      cplx<R> acc = zj<R>();
      if (I >= 1 && I <= c.n0 - 2 && J >= 1 && J <= c.n1 - 2)
        acc = R(0.25) * s1[y][p] + R(0.125) * (s1[y][p - 1] + s1[y][p + 1] + s1[y - 1][p] + s1[y + 1][p]) +
              R(0.0625) * (s1[y - 1][p - 1] + s1[y - 1][p + 1] + s1[y + 1][p - 1] + s1[y + 1][p + 1]);
      rc[(int64_t)J * c.n0 + I] = acc;
    }
  }
}

// out = J(x + P e): the correction and the first post-sweep.  62 x TY owned nodes,
// staged with a ring of one.  AP: also A.y = A out (UpApply, no dot product), which
// needs out on a ring of one and the staging on a ring of two: 60 x TY owned nodes.
// 65^2 FP64, where a step of GMRES is a chain of small launches: 3.8 us here and
// 4.5 of the matvec -> 4.4 in one, a solve of 66 steps 2.93 -> 2.55 ms.
template <typename R, int TY, bool AP>
__global__ __launch_bounds__(256) void k_jac_up(Grid<R> f, Grid<R> c, const cplx<R> *__restrict__ b,
                                                const cplx<R> *__restrict__ x, const cplx<R> *__restrict__ e,
                                                cplx<R> *__restrict__ out, R omega, int tiles_x, int tiles,
                                                UpApply<R> A) {
  constexpr int H = AP ? 2 : 1, TX = 64 - 2 * H, WY = TY + 2 * H, RPW = (WY + 3) / 4;
  __shared__ cplx<R> s0[WY][64], s1[AP ? WY : 1][64];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int tile = xcd_tile(tiles);
  if (tile < 0) return;
  const int x0 = (tile % tiles_x) * TX, y0 = (tile / tiles_x) * TY;
  const int n0 = f.n0, n1 = f.n1, i = x0 - H + lane, gy0 = y0 - H;
  const double om1 = 1.0 - (double)omega;
  const bool xin = i >= 1 && i <= n0 - 2;
  const cplx<R> xm = xin ? f.cm0[i] : zj<R>(), xp = xin ? f.cp0[i] : zj<R>();
  const int lm = lane > 0 ? lane - 1 : 0, lp = lane < 63 ? lane + 1 : 63;
  const int jl = min(max(gy0, 1), n1 - 1), jh = min(max(gy0 + WY, 1), n1 - 1);
  const __amdgpu_buffer_rsrc_t rb = rows_rsrc(b, jl, jh, n0), rk = rows_rsrc(f.k2, jl, jh, n0),
                               rx = rows_rsrc(x, jl, jh, n0);
  const uint32_t oc = col_off<cplx<R>>(xin, i), ok = col_off<R>(xin, i);
  const int Jl = min(max(gy0 >> 1, 0), c.n1), Jh = min((gy0 + WY) / 2 + 2, c.n1);
  const __amdgpu_buffer_rsrc_t re = rows_rsrc(e, Jl, Jh, c.n0);
  const uint32_t oa = col_off<cplx<R>>(xin, i >> 1), ob = col_off<cplx<R>>(xin, (i >> 1) + (i & 1));
  cplx<R> B[RPW], X[RPW], ym[RPW], yp[RPW], ea[RPW], eb[RPW], ec[RPW], ed[RPW];
  R K[RPW];
#pragma unroll
  for (int r = 0; r < RPW; r++) {
    const int ly = wv + 4 * r, j = gy0 + ly;
    const bool yin = ly < WY && j >= 1 && j <= n1 - 2;
    const int jc = yin ? j : 1;
    ym[r] = yin ? f.cm1[jc] : zj<R>();
    yp[r] = yin ? f.cp1[jc] : zj<R>();
    const uint32_t q = row_off<cplx<R>>(j - jl, n0);
    B[r] = ld_c(rb, oc + q, cplx<R>());
    K[r] = ld_r(rk, ok + row_off<R>(j - jl, n0), R());
    X[r] = ld_c(rx, oc + q, cplx<R>());
    const uint32_t q0 = row_off<cplx<R>>((j >> 1) - Jl, c.n0), q1 = row_off<cplx<R>>((j >> 1) + (j & 1) - Jl, c.n0);
    ea[r] = ld_c(re, oa + q0, cplx<R>());
    eb[r] = ld_c(re, ob + q0, cplx<R>());
    ec[r] = ld_c(re, oa + q1, cplx<R>());
    ed[r] = ld_c(re, ob + q1, cplx<R>());
  }
#pragma unroll
  for (int r = 0; r < RPW; r++) {
    const int ly = wv + 4 * r, j = gy0 + ly;
    if (ly < WY) {
      X[r] = (xin && j >= 1 && j <= n1 - 2) ? X[r] + R(0.25) * ((ea[r] + eb[r]) + (ec[r] + ed[r])) : zj<R>();
      s0[ly][lane] = X[r];
    }
  }
  __syncthreads();
  const __amdgpu_buffer_rsrc_t ro = rows_rsrc(out, y0, min(y0 + TY, n1), n0);
  const uint32_t oo = col_off<cplx<R>>(lane >= H && lane < TX + H && i < n0, i);
  // A's weights, in flight during the sweep
  const cplx<R> am = AP && xin ? A.cm0[i] : zj<R>(), ap = AP && xin ? A.cp0[i] : zj<R>();
#pragma unroll
  for (int r = 0; r < RPW; r++) {
    const int ly = wv + 4 * r, j = gy0 + ly;
    if (ly >= 1 && ly <= WY - 2 && j < n1) {
      cplx<R> v = zj<R>();
      if (xin && j >= 1 && j <= n1 - 2) {
        const cplx<double> d = diag_j(xm, xp, ym[r], yp[r], K[r], f.beta, f.c);
        const cplx<R> o =
            xm * s0[ly][lm] + xp * s0[ly][lp] + ym[r] * s0[ly - 1][lane] + yp[r] * s0[ly + 1][lane];
        v = cvt<R>(om1 * cvt<double>(X[r]) +
                   (double)omega * (recip<R>(abs2(d)) * (cvt<double>(B[r] + o) * conjg(d))));
      }
      if constexpr (AP) {
        X[r] = v;
        s1[ly][lane] = v;
      }
      if (ly >= H && ly < TY + H) st_c(ro, oo + row_off<cplx<R>>(j - y0, n0), v);
    }
  }
  if constexpr (AP) {
    __syncthreads();
    const __amdgpu_buffer_rsrc_t ry = rows_rsrc(A.y, y0, min(y0 + TY, n1), n0);
#pragma unroll
    for (int r = 0; r < RPW; r++) {
      const int ly = wv + 4 * r, j = gy0 + ly;
      if (ly >= H && ly < TY + H && j < n1) {
        cplx<R> v = zj<R>();
        if (xin && j >= 1 && j <= n1 - 2) {
          const cplx<R> aym = A.cm1[j], ayp = A.cp1[j];
          const cplx<R> d = am + ap + aym + ayp + (K[r] * A.beta + A.c);
          cplx<R> o = am * s1[ly][lm] + ap * s1[ly][lp];
          o = o + aym * s1[ly - 1][lane] + ayp * s1[ly + 1][lane];
          v = d * X[r] - o;
        }
        st_c(ry, oo + row_off<cplx<R>>(j - y0, n0), v);
      }
    }
  }
}

template <typename R, int CY, int MODE>
void launch_jac(const Grid<R> &f, const Grid<R> &c, const cplx<R> *b, const cplx<R> *x, const cplx<R> *e, cplx<R> *out,
                cplx<R> *rc, R omega, hipStream_t s) {
  constexpr int CX = (64 - (2 * (2 + MODE) - 1)) / 2;
  const int tx = (c.n0 + CX - 1) / CX, tiles = tx * ((c.n1 + CY - 1) / CY);
  launch_k((k_jac_down<R, CY, MODE>), dim3(xcd_padded(tiles)), dim3(256), 0, s, f, c, b, x, e, out, rc, omega, tx,
           tiles);
}

}  // namespace

template <typename R>
void launch_jacobi_down(const Grid<R> &f, const Grid<R> &c, const cplx<R> *b, const cplx<R> *x, const cplx<R> *e,
                        cplx<R> *out, cplx<R> *rc, R omega, hipStream_t s) {
  // two coarse rows a block fill the chip up to 257 coarse rows (a level of 321^2
  // has 488 blocks of them); four repeat fewer halo rows above
  const bool low = c.n1 <= 257;
  if (x == nullptr) {
    if (low) launch_jac<R, 2, 0>(f, c, b, x, e, out, rc, omega, s);
    else launch_jac<R, 4, 0>(f, c, b, x, e, out, rc, omega, s);
  } else {
    if (low) launch_jac<R, 2, 2>(f, c, b, x, e, out, rc, omega, s);
    else launch_jac<R, 4, 2>(f, c, b, x, e, out, rc, omega, s);
  }
}

template <typename R>
void launch_jacobi_up(const Grid<R> &f, const Grid<R> &c, const cplx<R> *b, const cplx<R> *x, const cplx<R> *e,
                      cplx<R> *out, R omega, hipStream_t s, const UpApply<R> *ap) {
  const auto go = [&](auto rows, auto with) {
    constexpr int TY = decltype(rows)::value;
    constexpr bool AP = decltype(with)::value;
    constexpr int TX = AP ? 60 : 62;
    const int tx = (f.n0 + TX - 1) / TX, tiles = tx * ((f.n1 + TY - 1) / TY);
    launch_k((k_jac_up<R, TY, AP>), dim3(xcd_padded(tiles)), dim3(256), 0, s, f, c, b, x, e, out, omega, tx, tiles,
             AP ? *ap : UpApply<R>{});
  };
  // six rows a block while the level then is a few blocks per CU, 14 above (with
  // A two fewer: two and four row slots of a wave as well)
  const bool low = f.n1 <= 513;
  if constexpr (sizeof(R) == 8) {  // an Arnoldi step's vectors are FP64
    if (ap && low) return go(std::integral_constant<int, 4>(), std::true_type());
    if (ap) return go(std::integral_constant<int, 12>(), std::true_type());
  }
  if (low) go(std::integral_constant<int, 6>(), std::false_type());
  else go(std::integral_constant<int, 14>(), std::false_type());
}

template void launch_jacobi_up<double>(const Grid<double> &, const Grid<double> &, const cplx<double> *,
                                       const cplx<double> *, const cplx<double> *, cplx<double> *, double, hipStream_t,
                                       const UpApply<double> *);
template void launch_jacobi_up<float>(const Grid<float> &, const Grid<float> &, const cplx<float> *,
                                      const cplx<float> *, const cplx<float> *, cplx<float> *, float, hipStream_t,
                                      const UpApply<float> *);
template void launch_jacobi_down<double>(const Grid<double> &, const Grid<double> &, const cplx<double> *,
                                         const cplx<double> *, const cplx<double> *, cplx<double> *, cplx<double> *,
                                         double, hipStream_t);
template void launch_jacobi_down<float>(const Grid<float> &, const Grid<float> &, const cplx<float> *,
                                        const cplx<float> *, const cplx<float> *, cplx<float> *, cplx<float> *, float,
                                        hipStream_t);

}  // namespace ecs
