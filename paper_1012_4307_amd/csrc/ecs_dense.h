// ecs_dense.h -- the coarse end of a cycle as a dense map (not part of the
// public ABI): argument blocks and launchers of kernels_dense.hip.
#pragma once

#include "ecs_internal.h"

namespace ecs {

// A level takes part in the dense end when its map and the vectors of its
// construction fit: kDenseMax unknowns, kDenseNodes nodes, kDenseCoarse nodes
// on the next level.
constexpr int kDenseMax = 1600;
constexpr int kDenseNodes = 2304;
constexpr int kDenseCoarse = 448;

// rows of a map lie dense_ld(N) elements apart (16-byte aligned in FP32)
__host__ __device__ __forceinline__ int dense_ld(int n) { return (n + 1) & ~1; }

// u = G b on a level's interior nodes (row-major unknowns, x fastest), u = 0 on
// its boundary; b and u hold the level with its boundary.  G: N rows.
template <typename R>
void launch_dense(const cplx<R> *G, int N, int n0, int n1, int n2, const cplx<R> *b, cplx<R> *u, hipStream_t s,
                  const RhsSet &rs = one_rhs());

// Builds the map of `reps` visits of a level in a row, from a zero iterate:
// each is nu1 sweeps, the residual's full weighting, the next level's map (X1
// on the first visit, X2 on the later ones), the correction, nu2 sweeps.
struct DenseGen {
  Grid<double> f;                // the level
  int c0, c1, c2;                // nodes of the next level
  const cplx<double> *X1, *X2;   // maps of the next level
  int reps, nu1, nu2, red_black; // red_black: SOR in two colours, else omega-Jacobi
  double omega;
  cplx<double> *G;
};
void launch_dense_gen(const DenseGen &a, hipStream_t s);

}  // namespace ecs
