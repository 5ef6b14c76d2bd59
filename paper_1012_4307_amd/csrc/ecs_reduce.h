// ecs_reduce.h -- block reductions and the device-side Bi-CGSTAB scalar
// recurrence shared by the kernels that fuse a dot product into their pass.
#pragma once

#include "ecs_krylov.h"

namespace ecs {

constexpr int kRedThreads = 256;  // 4 waves of 64

// The wave's sum in every lane: the butterfly v += v[lane ^ o], o = 32, 16,
// ..., 1, with each exchange done in registers rather than through the LDS
// crossbar -- lanes ^ 32 and ^ 16 by the permlane swaps (each returns both
// halves of the swapped pair: a lane takes the half that came from the other
// side), ^ 8 by a row rotation by 8 (exact within a 16-lane row), and ^ 4, 2,
// 1 by rotations by 4, 2, 1: after the ^ 8 step every value repeats with
// period 8 within its row (then 4, then 2), so a lane's rotation partner
// holds the same value as its xor partner.  Every addition has the same
// operands in the same order as the plain butterfly, so the sums are equal
// bit for bit.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), CTRL, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), CTRL, 0xF, 0xF, false);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double lane_xor32(double v) {
  const bool low = (__lane_id() & 32) == 0;
  const auto lo = __builtin_amdgcn_permlane32_swap(__double2loint(v), __double2loint(v), false, false);
  const auto hi = __builtin_amdgcn_permlane32_swap(__double2hiint(v), __double2hiint(v), false, false);
  return __hiloint2double(low ? hi[1] : hi[0], low ? lo[1] : lo[0]);
}
__device__ __forceinline__ double lane_xor16(double v) {
  const bool even = (__lane_id() & 16) == 0;
  const auto lo = __builtin_amdgcn_permlane16_swap(__double2loint(v), __double2loint(v), false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(__double2hiint(v), __double2hiint(v), false, false);
  return __hiloint2double(even ? hi[1] : hi[0], even ? lo[1] : lo[0]);
}
__device__ __forceinline__ double wave_sum(double v) {
  v += lane_xor32(v);
  v += lane_xor16(v);
  v += dpp_move<0x128>(v);  // row_ror:8
  v += dpp_move<0x124>(v);  // row_ror:4
  v += dpp_move<0x122>(v);  // row_ror:2
  v += dpp_move<0x121>(v);  // row_ror:1
  return v;
}

// block-wide sum of a complex value over the first NW waves of the block; result
// in thread 0.  lds: one entry for each wave of the block.
template <int NW>
__device__ __forceinline__ cplx<double> block_sum_n(cplx<double> v, cplx<double> *lds) {
  v.re = wave_sum(v.re);
  v.im = wave_sum(v.im);
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) lds[wid] = v;
  __syncthreads();
  cplx<double> s = mk<double>(0, 0);
  if (threadIdx.x == 0)
    for (int q = 0; q < NW; q++) s = s + lds[q];
  return s;
}
__device__ __forceinline__ cplx<double> block_sum(cplx<double> v, cplx<double> *lds /* >= 4 */) {
  return block_sum_n<kRedThreads / 64>(v, lds);
}

// This thread's share of a second-stage reduction: x[t] + x[t + B] + ... over
// the entries below n (t = threadIdx.x, B = kRedThreads), added in that order.
// The loads of a chunk are all issued before the first add: a plain strided
// loop waits for each load before issuing the next, one memory round trip
// per entry.
__device__ __forceinline__ cplx<double> strided_sum(const cplx<double> *x, int n) {
  constexpr int U = 16;
  cplx<double> s = mk<double>(0, 0);
  for (int b0 = threadIdx.x; b0 < n; b0 += U * kRedThreads) {
    cplx<double> v[U];
#pragma unroll
    for (int u = 0; u < U; u++) {
      const int b = b0 + u * kRedThreads;
      v[u] = x[b < n ? b : b0];
    }
#pragma unroll
    for (int u = 0; u < U; u++)
      if (b0 + u * kRedThreads < n) s = s + v[u];
  }
  return s;
}

// The recurrence's products and quotients, with the fused operations written out:
// the compiler fuses a * b - c * d one way or the other depending on the code
// around it, and the recurrence runs in kernels of several kinds.
__device__ __forceinline__ cplx<double> mul_rec(cplx<double> a, cplx<double> b) {
  return mk<double>(fma(a.re, b.re, -(a.im * b.im)), fma(a.re, b.im, a.im * b.re));
}
__device__ __forceinline__ double abs2_rec(cplx<double> a) { return fma(a.re, a.re, a.im * a.im); }
__device__ __forceinline__ cplx<double> div_rec(cplx<double> a, cplx<double> b) {
  const double inv = 1.0 / abs2_rec(b);
  return inv * mul_rec(a, conjg(b));
}

// Bi-CGSTAB scalar recurrence on the reduced dot products d0, d1.
__device__ inline void bicg_update(BicgScalars *S, int mode, cplx<double> d0, cplx<double> d1) {
  const cplx<double> zero = mk<double>(0, 0);
  switch (mode) {
    case kBicgAlpha:  // alpha = rho / (r^, v)
      if (abs2_rec(d0) == 0 || S->bad) { S->bad = 1; S->alpha = zero; break; }
      S->alpha = div_rec(S->rho, d0);
      break;
    case kBicgOmega:  // omega = (t, s) / (t, t)
      if (d1.re == 0 || S->bad) { S->bad = 1; S->omega = zero; break; }
      S->omega = (1.0 / d1.re) * d0;
      break;
    case kBicgInit:  // (re)start: rho = (r^, r) = ||r||^2, p = r on the first step
      S->breakdowns += S->bad;
      S->rnorm2 = d0.re;
      S->est = sqrt(d0.re) / S->bnorm;
      S->rho = mk<double>(d0.re, 0);
      S->alpha = mk<double>(1, 0);
      S->omega = mk<double>(1, 0);
      S->beta = zero;
      S->bad = !(S->est == S->est) || isinf(S->est) || d0.re == 0;
      break;
    case kBicgNormRho: {  // end of a step: ||r||^2 = d0, rho1 = (r^, r) = d1, beta for the next step
      S->rnorm2 = d0.re;
      S->est = sqrt(d0.re) / S->bnorm;
      if (!(S->est == S->est) || isinf(S->est)) S->bad = 1;
      if (abs2_rec(d1) == 0 || abs2_rec(S->rho) == 0 || abs2_rec(S->omega) == 0 || S->bad) {
        S->bad = 1; S->beta = zero; S->alpha = zero; S->omega = zero;
        break;
      }
      S->beta = mul_rec(div_rec(d1, S->rho), div_rec(S->alpha, S->omega));
      S->rho = d1;
      break;
    }
  }
}

// A following kernel's share of a reduction (BicgFold), in two parts so that the
// kernel can issue its own loads in between: each thread's partials, then the
// sums (strided_sum and block_sum over the same entries: the one-block
// reduction's bits) and the update, which every thread reads from LDS.
constexpr int kFoldU = kFoldPartials / kRedThreads;
template <int NP>
struct FoldLoads {
  cplx<double> v[NP][kFoldU];
};
template <int NP>
__device__ __forceinline__ FoldLoads<NP> fold_load(const cplx<double> *partials, int nb) {
  FoldLoads<NP> L;
#pragma unroll
  for (int q = 0; q < NP; q++)
#pragma unroll
    for (int u = 0; u < kFoldU; u++) {
      const int b = (int)threadIdx.x + u * kRedThreads;
      L.v[q][u] = partials[(int64_t)q * nb + (b < nb ? b : 0)];
    }
  return L;
}
template <int NP>
__device__ __forceinline__ void fold_finish(const FoldLoads<NP> &L, const BicgScalars *in, BicgScalars *out, int nb,
                                            int mode, cplx<double> *red, BicgScalars *sh) {
  cplx<double> d[2] = {mk<double>(0, 0), mk<double>(0, 0)};
#pragma unroll
  for (int q = 0; q < NP; q++) {
    cplx<double> s = mk<double>(0, 0);
#pragma unroll
    for (int u = 0; u < kFoldU; u++)
      if ((int)threadIdx.x + u * kRedThreads < nb) s = s + L.v[q][u];
    d[q] = block_sum(s, red);
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *sh = *in;
    bicg_update(sh, mode, d[0], d[1]);
    if (blockIdx.x == 0) *out = *sh;
  }
  __syncthreads();
}

}  // namespace ecs
