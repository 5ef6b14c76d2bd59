// ecs_jacobi.h -- launchers of the fused omega-Jacobi level kernels (not part
// of the public ABI).
#pragma once

#include <type_traits>

#include "ecs_internal.h"

namespace ecs {

// out = J(0) (x null) or J(J(x + P e)), and rc = FW(b - M out); out of place.
template <typename R>
void launch_jacobi_down(const Grid<R> &fine, const Grid<R> &coarse, const cplx<R> *b, const cplx<R> *x,
                        const cplx<R> *e, cplx<R> *out, cplx<R> *rc, R omega, hipStream_t s);

// out = J(x + P e), out of place; with ap (kUpApplyOnly) y = A out as well.
template <typename R>
void launch_jacobi_up(const Grid<R> &fine, const Grid<R> &coarse, const cplx<R> *b, const cplx<R> *x,
                      const cplx<R> *e, cplx<R> *out, R omega, hipStream_t s, const UpApply<R> *ap = nullptr);

}  // namespace ecs
