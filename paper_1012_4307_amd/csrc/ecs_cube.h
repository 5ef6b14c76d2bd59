// ecs_cube.h -- launchers of the fused 3D V(1,1) red-black cycle (not part of
// the public ABI).
#pragma once

#include <type_traits>

#include "ecs_internal.h"

namespace ecs {

// 3D counterparts of launch_down_rb / launch_up_rb: zero-guess red-black
// sweep, residual and full weighting; the sweep recomputed, trilinear
// correction and red-black post-sweep into u
template <typename R>
void launch_down3_rb(const Grid<R> &fine, const Grid<R> &coarse, const cplx<R> *b, cplx<R> *rc, R omega,
                     hipStream_t s);
template <typename R>
void launch_up3_rb(const Grid<R> &fine, const Grid<R> &coarse, const cplx<R> *b, const cplx<R> *ec, cplx<R> *u,
                   R omega, hipStream_t s);

}  // namespace ecs
