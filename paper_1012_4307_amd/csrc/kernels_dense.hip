// kernels_dense.hip -- the coarse end of a multigrid cycle as one dense map
// (Sec. 4.2, Algorithm 1).  What Algorithm 1 does from a small level down, for
// the right-hand side the level above restricts to it and a zero first iterate,
// is linear in that right-hand side: a fixed N x N matrix, N the level's
// interior nodes, for any cycle indices, sweeps and smoother, and also for the
// repeated visits of an F or W cycle taken together.  The matrices are built
// once per set-up, from the coarsest inverse up, in FP64; a cycle applies the
// finest of them with one multiplication.
//
// What bounds it: launch latency and one round trip to L2.  The alternative, a
// single workgroup walking the levels in LDS with a barrier after every colour
// or transfer, is a chain of latencies: 33^2 .. 9^2 took 15.5 us FP64, 12.4
// FP32 per cycle, the 25^2 .. 4^2 end of an F_1^4 cycle 16.4 us per visit, at
// 13 visits per cycle on 385^2 (10 maps now).  The map of a 33^2 level reads
// 14.8 MB (FP64) over all CUs instead: 3.8 us, in FP32 3.5; 41^2 8 and 5.2 us.
//
// FP32 products and sums are FP64: the entries are rounded once already, and sums
// of up to 25 products a lane in FP32 left a grid that is one map (41^2
// omega-Jacobi) 9.0e-8 from the 64-bit cycle, where the level by level one was
// 6.0e-8; now 3.7e-8, at the same 3.5 us on 33^2 and 4.7 -> 5.2 us on 41^2.
#include "ecs_dense.h"
#include "ecs_reduce.h"

namespace ecs {

namespace {

// node of unknown c of a level with ni x nj interior nodes per plane (float
// reciprocals: exact, c < 4096)
struct Interior {
  int n0, n1, n2, ni, nij;
  float ri, rij;
  __device__ Interior(int a0, int a1, int a2) : n0(a0), n1(a1), n2(a2), ni(a0 - 2), nij((a0 - 2) * (a1 - 2)) {
    ri = 1.0f / (float)ni;
    rij = 1.0f / (float)nij;
  }
  __device__ __forceinline__ int node(int c) const {
    int k = 0;
    if (n2 > 1) {
      k = (int)(((float)c + 0.5f) * rij);
      c -= k * nij;
      k++;
    }
    const int j = (int)(((float)c + 0.5f) * ri);
    return (k * n1 + j + 1) * n0 + (c - j * ni) + 1;
  }
};

// two FP32 entries per 16-byte load, one FP64 entry
template <typename R>
struct alignas(16) Quad {
  static constexpr int V = 16 / (int)sizeof(cplx<R>);
  cplx<R> v[V];
};

constexpr int kChunk = 1024;  // entries of b staged at a time

// One wave per row: every load of the row (up to a chunk) is issued before b is
// staged, the lanes' partial sums meet in one wave sum.  b is staged in LDS once
// per block of four rows.  Rows keep their block, so each XCD reads the same
// eighth of the map every time and finds it in its L2.  A batched launch
// applies a row, held in registers, to every right-hand side in turn (per
// right-hand side the single launch's arithmetic).
template <typename R, bool MR>
__global__ __launch_bounds__(256) void k_dense(const cplx<R> *__restrict__ G, int N, int n0, int n1, int n2,
                                               const cplx<R> *__restrict__ b, cplx<R> *__restrict__ u, RhsSet rs) {
  constexpr int V = Quad<R>::V, Q = kChunk / (64 * V);
  __shared__ __align__(16) cplx<R> sb[kChunk];
  const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row = blockIdx.x * 4 + wv, ld = dense_ld(N);
  const Interior in(n0, n1, n2);
  const int nn = n0 * n1 * n2;
  const __amdgpu_buffer_rsrc_t rg = __builtin_amdgcn_make_buffer_rsrc(
      (void *)(G + (int64_t)(row < N ? row : 0) * ld), 0, row < N ? ld * (int)sizeof(cplx<R>) : 0, kRsrcWord3);
  Quad<R> g[Q];
  auto load = [&](int c0) {
#pragma unroll
    for (int q = 0; q < Q; q++)
      g[q] = __builtin_bit_cast(Quad<R>, __builtin_amdgcn_raw_buffer_load_b128(
                                             rg, (uint32_t)((c0 + V * (lane + 64 * q)) * (int)sizeof(cplx<R>)), 0, 0));
  };
  load(0);
  const int p = blockIdx.x * 256 + threadIdx.x;  // the grid has at least nn threads
  const int i = p % n0, j = (p / n0) % n1, k = p / (n0 * n1);
  const bool edge = p < nn && (i == 0 || i == n0 - 1 || j == 0 || j == n1 - 1 || (n2 > 1 && (k == 0 || k == n2 - 1)));
  const int count = MR ? rs.count : 1;
  for (int y = 0; y < count; y++) {
    const int64_t off = MR ? rs.slot[y] * rhs_stride(nn) : 0;
    cplx<double> acc = mk<double>(0, 0);
    for (int c0 = 0; c0 < N; c0 += kChunk) {
      cplx<R> v[4];
#pragma unroll
      for (int e = 0; e < 4; e++) {
        const int c = c0 + (int)threadIdx.x + 256 * e;
        v[e] = c < N ? b[off + in.node(c)] : mk<R>(0, 0);
      }
      if (N > kChunk && (c0 > 0 || y > 0)) load(c0);
      if (c0 > 0 || y > 0) __syncthreads();  // the chunk before has been read
#pragma unroll
      for (int e = 0; e < 4; e++) sb[threadIdx.x + 256 * e] = v[e];
      __syncthreads();
#pragma unroll
      for (int q = 0; q < Q; q++) {
        const Quad<R> x = *reinterpret_cast<const Quad<R> *>(&sb[V * (lane + 64 * q)]);
#pragma unroll
        for (int h = 0; h < V; h++) acc = acc + cvt<double>(g[q].v[h]) * cvt<double>(x.v[h]);
      }
    }
    const double re = wave_sum(acc.re), im = wave_sum(acc.im);
    if (lane == 0 && row < N) u[off + in.node(row)] = mk<R>((R)re, (R)im);
    if (edge) u[off + p] = mk<R>(0, 0);
  }
}

// One block per column of the map: the level operations on the unit vector of
// that unknown, vectors in LDS.  A thread keeps the places, inverse diagonals
// and weights' indices of its unknowns (one in NT) over all phases; the next
// level's map is applied eight rows per wave at a time, enough loads in flight
// for its L2 latency (one row at a time took 118 of a visit's 155 us on 41^2).
template <int NODES, int COARSE, int UNK, int NT>
__global__ __launch_bounds__(NT) void k_dense_gen(DenseGen a) {
  constexpr int E = (UNK + NT - 1) / NT, RW = 8;
  __shared__ cplx<double> su[NODES], sw[NODES], scb[COARSE], sce[COARSE];
  __shared__ int first, last;  // the non-zero range of the restricted residual
  const Grid<double> &f = a.f;
  const int tid = threadIdx.x, n0 = f.n0, n1 = f.n1, n2 = f.n2, nn = n0 * n1 * n2, nc = a.c0 * a.c1 * a.c2;
  const int s1 = n0, s2 = n0 * n1;
  const bool three = n2 > 1;
  const Interior in(n0, n1, n2), cin(a.c0, a.c1, a.c2);
  const int N = three ? in.nij * (n2 - 2) : in.nij, Nc = three ? cin.nij * (a.c2 - 2) : cin.nij;
  const int unit = in.node(blockIdx.x);
  const double om = a.omega;
  cplx<double> *u = su, *w = sw;
  int P[E], I[E], J[E], K[E];
  cplx<double> d[E];
#pragma unroll
  for (int e = 0; e < E; e++) {
    const int c = tid + e * NT;
    P[e] = c < N ? in.node(c) : -1;
    const int p = c < N ? P[e] : in.node(0);
    I[e] = p % n0;
    J[e] = (p / n0) % n1;
    K[e] = p / s2;
    d[e] = f.cm0[I[e]] + f.cp0[I[e]] + f.cm1[J[e]] + f.cp1[J[e]];
    if (three) d[e] = d[e] + f.cm2[K[e]] + f.cp2[K[e]];
    d[e] = d[e] + (f.k2[p] * f.beta + f.c);
  }
  for (int p = tid; p < nn; p += NT) su[p] = sw[p] = mk<double>(0, 0);
  for (int q = tid; q < nc; q += NT) sce[q] = mk<double>(0, 0);
  __syncthreads();
  // b - M x at unknown e
  auto resid = [&](int e, const cplx<double> *x) {
    const int p = P[e];
    cplx<double> r = f.cm0[I[e]] * x[p - 1] + f.cp0[I[e]] * x[p + 1] + f.cm1[J[e]] * x[p - s1] + f.cp1[J[e]] * x[p + s1];
    if (three) r = r + f.cm2[K[e]] * x[p - s2] + f.cp2[K[e]] * x[p + s2];
    return r + mk<double>(p == unit ? 1.0 : 0.0, 0.0) - d[e] * x[p];
  };
  auto sweeps = [&](int nu) {
    for (int q = 0; q < nu; q++) {
      for (int colour = 0; colour < (a.red_black ? 2 : 1); colour++) {
        cplx<double> *to = a.red_black ? u : w;
#pragma unroll
        for (int e = 0; e < E; e++)
          if (P[e] >= 0 && (!a.red_black || ((I[e] + J[e] + K[e]) & 1) == colour))
            to[P[e]] = u[P[e]] + om * cdiv(resid(e, u), d[e]);
        __syncthreads();
      }
      if (!a.red_black) {
        cplx<double> *t = u;
        u = w;
        w = t;
      }
    }
  };
  for (int rep = 0; rep < a.reps; rep++) {
    sweeps(a.nu1);
#pragma unroll
    for (int e = 0; e < E; e++)
      if (P[e] >= 0) w[P[e]] = resid(e, u);  // w's boundary stays 0
    if (tid == 0) {
      first = Nc;
      last = -1;
    }
    __syncthreads();
    for (int c = tid; c < Nc; c += NT) {
      const int q = cin.node(c), Ic = q % a.c0, Jc = (q / a.c0) % a.c1, Kc = q / (a.c0 * a.c1);
      const int p = (2 * Kc * n1 + 2 * Jc) * n0 + 2 * Ic;
      cplx<double> acc = mk<double>(0, 0);
      for (int dz = three ? -1 : 0; dz <= (three ? 1 : 0); dz++) {
        const cplx<double> *r0 = w + p + dz * s2;
        const cplx<double> s = 0.25 * r0[0] + 0.125 * (r0[-1] + r0[1] + r0[-s1] + r0[s1]) +
                               0.0625 * (r0[-s1 - 1] + r0[-s1 + 1] + r0[s1 - 1] + r0[s1 + 1]);
        acc = acc + (!three ? 1.0 : dz == 0 ? 0.5 : 0.25) * s;
      }
      scb[c] = acc;
      // on the first visit the unit vector has reached a few nodes only
      if (acc.re != 0 || acc.im != 0) {
        atomicMin(&first, c);
        atomicMax(&last, c);
      }
    }
    __syncthreads();
    {
      const cplx<double> *X = rep == 0 ? a.X1 : a.X2;
      const int lane = tid & 63, ld = dense_ld(Nc);
      for (int r0 = (tid >> 6) * RW; r0 < Nc; r0 += NT / 64 * RW) {
        cplx<double> acc[RW];
#pragma unroll
        for (int h = 0; h < RW; h++) acc[h] = mk<double>(0, 0);
#pragma unroll 2
        for (int c = (first & ~63) + lane; c <= last; c += 64) {
          const cplx<double> x = scb[c];
#pragma unroll
          for (int h = 0; h < RW; h++) acc[h] = acc[h] + X[(int64_t)(r0 + h < Nc ? r0 + h : r0) * ld + c] * x;
        }
#pragma unroll
        for (int h = 0; h < RW; h++) {
          const double re = wave_sum(acc[h].re), im = wave_sum(acc[h].im);
          if (lane == 0 && r0 + h < Nc) sce[cin.node(r0 + h)] = mk<double>(re, im);
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < E; e++) {
      if (P[e] < 0) continue;
      const int I1 = I[e] & 1, J1 = (J[e] & 1) * a.c0, K1 = three ? (K[e] & 1) * a.c0 * a.c1 : 0;
      const cplx<double> *c = sce + ((K[e] >> 1) * a.c1 + (J[e] >> 1)) * a.c0 + (I[e] >> 1);
      const cplx<double> lo = 0.25 * ((c[0] + c[I1]) + (c[J1] + c[J1 + I1]));
      const cplx<double> hi = 0.25 * ((c[K1] + c[K1 + I1]) + (c[K1 + J1] + c[K1 + J1 + I1]));
      u[P[e]] = u[P[e]] + 0.5 * (lo + hi);
    }
    __syncthreads();
    sweeps(a.nu2);
  }
  const int ld = dense_ld(N);
#pragma unroll
  for (int e = 0; e < E; e++) {
    if (P[e] < 0) continue;
    cplx<double> *row = a.G + (int64_t)(tid + e * NT) * ld;
    row[blockIdx.x] = u[P[e]];
    if (blockIdx.x == 0 && ld > N) row[N] = mk<double>(0, 0);
  }
}

}  // namespace

template <typename R>
void launch_dense(const cplx<R> *G, int N, int n0, int n1, int n2, const cplx<R> *b, cplx<R> *u, hipStream_t s,
                  const RhsSet &rs) {
  const dim3 grid((N + 3) / 4), block(256);
  if (multi_rhs(rs)) launch_k((k_dense<R, true>), grid, block, 0, s, G, N, n0, n1, n2, b, u, rs);
  else launch_k((k_dense<R, false>), grid, block, 0, s, G, N, n0, n1, n2, b, u, rs);
}

void launch_dense_gen(const DenseGen &a, hipStream_t s) {
  const int n2 = a.f.n2, nodes = a.f.n0 * a.f.n1 * n2, coarse = a.c0 * a.c1 * a.c2;
  const int N = (a.f.n0 - 2) * (a.f.n1 - 2) * (n2 > 1 ? n2 - 2 : 1);
  // small levels: three blocks per CU
  if (nodes <= 1152 && coarse <= 320 && N <= 1024)
    launch_k((k_dense_gen<1152, 320, 1024, 512>), dim3(N), dim3(512), 0, s, a);
  else
    launch_k((k_dense_gen<kDenseNodes, kDenseCoarse, kDenseMax, 1024>), dim3(N), dim3(1024), 0, s, a);
}

template void launch_dense<double>(const cplx<double> *, int, int, int, int, const cplx<double> *, cplx<double> *,
                                   hipStream_t, const RhsSet &);
template void launch_dense<float>(const cplx<float> *, int, int, int, int, const cplx<float> *, cplx<float> *,
                                  hipStream_t, const RhsSet &);

}  // namespace ecs
