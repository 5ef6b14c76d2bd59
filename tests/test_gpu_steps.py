"""GPU parity of every step of the multigrid-preconditioned solve against the
FP64 CPU oracle, element by element, through the C ABI.

Tolerances: the FP64 path differs from the oracle only by rounding order,
so single steps must agree to 1e-13 (relative to the largest entry) and a
whole cycle to 1e-12; the FP32 cycle must agree to 1e-5 per step and 2e-4 per
cycle (a few FP32 ulps amplified by the coarse-level solves)."""
import math

import numpy as np
import pytest

from helpers import gpu_for, oracle_for, ragged_workload, relerr, to_gpu, to_np
from paper_1012_4307_amd import workloads as W

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-13, "f32": 1e-5}
CYCLE_TOL = {"f64": 1e-12, "f32": 2e-4}


def cases():
    c1 = W.small_constant_k()
    c2 = W.coulomb(E=2.0, n=129)
    rg = ragged_workload()
    return {"small_constant_k": c1, "coulomb129": c2, "ragged97": rg}


CASES = cases()


@pytest.fixture(scope="module", params=list(CASES))
def case(request):
    return CASES[request.param]


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_operator_apply(case, dt):
    w = case
    P = oracle_for(w)
    S = gpu_for(w, dt)
    rng = np.random.default_rng(5)
    x = W.random_complex(w.shape, rng)
    for op in ("A", "M", "AT"):
        y = to_np(S.apply(to_gpu(x), op))
        assert relerr(y, P.apply(x, which=op)) < 1e-13, op
        assert np.all(y[0] == 0) and np.all(y[:, -1] == 0)


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_smoother_sweep(case, dt):
    w = case
    P = oracle_for(w)
    S = gpu_for(w, dt)
    cdt = np.complex64 if dt == "f32" else np.complex128
    rng = np.random.default_rng(6)
    for level in (0, 1):
        shape = S.level_shape(level)
        b = W.random_complex(shape, rng)
        u = W.random_complex(shape, rng)
        if dt == "f32":
            b = b.astype(cdt).astype(np.complex128)
            u = u.astype(cdt).astype(np.complex128)
        for ns in (1, 2):
            got = to_np(S.smooth(to_gpu(b.astype(cdt)), to_gpu(u.astype(cdt)), level, ns))
            ref = P.smooth(b, u, level, w.cycle["smoother"], w.cycle["omega"], ns)
            assert relerr(got, ref) < TOL[dt] * (10 if dt == "f32" else 1), (level, ns)


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_residual_restrict_and_prolong(case, dt):
    w = case
    P = oracle_for(w)
    S = gpu_for(w, dt)
    cdt = np.complex64 if dt == "f32" else np.complex128
    rng = np.random.default_rng(7)
    for level in range(S.nlev - 1):
        shape = S.level_shape(level)
        b = W.random_complex(shape, rng).astype(cdt).astype(np.complex128)
        u = W.random_complex(shape, rng).astype(cdt).astype(np.complex128)
        rc = to_np(S.residual_restrict(to_gpu(b.astype(cdt)), to_gpu(u.astype(cdt)), level))
        ref = P.restrict(P.residual(b, u, level), level)
        assert relerr(rc, ref) < TOL[dt] * (10 if dt == "f32" else 1), level
        ec = W.random_complex(S.level_shape(level + 1), rng).astype(cdt).astype(np.complex128)
        up = to_np(S.prolong_correct(to_gpu(ec.astype(cdt)), to_gpu(u.astype(cdt)), level))
        assert relerr(up, P.prolong_add(ec, u, level)) < TOL[dt], level


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_coarse_solve(case, dt):
    w = case
    P = oracle_for(w)
    S = gpu_for(w, dt)
    cdt = np.complex64 if dt == "f32" else np.complex128
    rng = np.random.default_rng(8)
    b = W.random_complex(S.level_shape(S.nlev - 1), rng).astype(cdt).astype(np.complex128)
    x = to_np(S.coarse_solve(to_gpu(b.astype(cdt))))
    assert relerr(x, P.coarse_solve(b)) < (1e-12 if dt == "f64" else 1e-5)


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_vcycle(case, dt):
    w = case
    P = oracle_for(w)
    S = gpu_for(w, dt)
    rng = np.random.default_rng(9)
    for v in (w.rhs[0], W.random_complex(w.shape, rng)):
        z = to_np(S.vcycle(to_gpu(v)))
        assert relerr(z, P.mg_apply(v)) < CYCLE_TOL[dt]


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_vcycle_native_dtype(dt):
    """The cycle on vectors in its own dtype (no conversion passes) equals the
    oracle's cycle of the same right-hand side."""
    import torch
    w = W.coulomb(E=2.0, n=257)
    P = oracle_for(w)
    S = gpu_for(w, dt)
    v = W.random_complex(w.shape, np.random.default_rng(14))
    vd = to_gpu(v).to(torch.complex64 if dt == "f32" else torch.complex128)
    z = S.vcycle_native(vd)
    assert z.dtype == vd.dtype
    ref = P.mg_apply(to_np(vd).astype(np.complex128))
    assert relerr(to_np(z).astype(np.complex128), ref) < CYCLE_TOL[dt]


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_vcycle_tail_schedules(dt):
    """The single-workgroup tail over every admissible range of coarse levels:
    the whole cycle (33^2 grid), the dense solve alone, and coarsest grids of
    9, 4, 225 and 49 unknowns (64, 64, 4 and 16 threads per row of the dense
    solve), against the oracle's cycle.  FP32 cycles also run the wide tail:
    from a 65^2 level, the whole cycle of a 65^2 grid, and from a ragged 49^2
    level."""
    rng = np.random.default_rng(12)
    runs = [(W.coulomb(E=1.0, n=33), (33, 17, 9, 5, 3)),
            (ragged_workload(), (3, 4, 7, 13, 25)),
            (ragged_workload(n=129, coarsest=17), (17, 33)),
            (W.coulomb(E=2.0, n=129, coarsest=9), (9, 17, 33))]
    if dt == "f32":
        runs += [(W.coulomb(E=2.0, n=257, coarsest=9), (65,)), (W.coulomb(E=1.0, n=65, coarsest=9), (65,)),
                 (ragged_workload(n=193, coarsest=7), (49, 65))]
    for w, tails in runs:
        P = oracle_for(w)
        S = gpu_for(w, dt)
        for v in (w.rhs[0], W.random_complex(w.shape, rng)):
            ref = P.mg_apply(v)
            for tn in tails:
                S.set_tuning(tail_nodes=tn)
                assert relerr(to_np(S.vcycle(to_gpu(v))), ref) < CYCLE_TOL[dt], (w.name, w.n, tn)


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_vcycle_two_level_kernels(dt):
    """Levels run two per kernel (down: levels l, l+1 in one block with the
    intermediate right-hand side in LDS; up: levels l+1, l): every pairing
    the schedule allows -- none, only the smallest levels, all levels above
    the tail, an odd count with a single level on top -- against the oracle."""
    rng = np.random.default_rng(13)
    runs = [(W.coulomb(E=2.0, n=257), (0, 33, 65, 129, 257)),
            (ragged_workload(n=193, coarsest=7), (0, 25, 49, 97, 193)),
            (W.coulomb(E=1.0, n=65), (0, 65))]
    for w, pgs in runs:
        P = oracle_for(w)
        S = gpu_for(w, dt)
        v = W.random_complex(w.shape, rng)
        ref = P.mg_apply(v)
        for pg in pgs:
            for tn in (9, 33):
                S.set_tuning(tail_nodes=tn, pair_grid=pg)
                assert relerr(to_np(S.vcycle(to_gpu(v))), ref) < CYCLE_TOL[dt], (w.name, w.n, pg, tn)


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_vcycle_tile_heights(dt):
    """Every tile height of the fused down and up kernels (coarse rows per
    block 2..6, 8, and 16 in FP32; fine rows 4..32), applied on every level
    above the tail of a ragged grid, against the oracle's cycle."""
    w = ragged_workload(n=193, coarsest=7)
    P = oracle_for(w)
    S = gpu_for(w, dt)
    v = W.random_complex(w.shape, np.random.default_rng(16))
    ref = P.mg_apply(v)
    downs = (2, 3, 4, 5, 6, 8) + ((16,) if dt == "f32" else ())
    for d in downs:
        for u in (4, 8, 10, 12, 16, 32):
            S.set_tuning(down_rows=d, up_rows=u, small_grid=3, tail_nodes=33, pair_grid=0)
            assert relerr(to_np(S.vcycle(to_gpu(v))), ref) < CYCLE_TOL[dt], (d, u)


@pytest.mark.parametrize("omega", [1.0, 0.85])
def test_tile_height_kept_over_a_change_of_type(omega):
    """A schedule with 16 coarse rows a block, which FP32 cycles have, stays set when
    the context's cycle becomes an FP64 one: the cycle is the oracle's on every
    node (fine levels of 193 and 97 coarse rows, no multiples of 8 or 16)."""
    import ctypes
    import torch
    import paper_1012_4307_amd as E
    w = ragged_workload(n=385, coarsest=7, omega=omega)
    P = oracle_for(w)
    v = W.random_complex(w.shape, np.random.default_rng(23))
    S = gpu_for(w, "f32")
    S.set_tuning(down_rows=16, small_grid=3, pair_grid=0)
    assert relerr(to_np(S.vcycle(to_gpu(v))), P.mg_apply(v)) < CYCLE_TOL["f32"]
    L, d = E.lib(), S.precond.to_c()
    d.vcycle_dtype = E.F64
    assert L.ecs_set_precond(S._h, ctypes.byref(d)) == 0
    n = ctypes.c_size_t()
    assert L.ecs_workspace_size(S._h, None, ctypes.byref(n)) == 0
    ws = torch.empty(n.value + 256, dtype=torch.uint8, device="cuda")
    assert L.ecs_set_workspace(S._h, ctypes.c_void_p((ws.data_ptr() + 255) & ~255), n.value) == 0
    got = to_np(S.vcycle(to_gpu(v)))
    assert relerr(got, P.mg_apply(v)) < CYCLE_TOL["f64"]
    # no part of the result comes from what the buffers held
    for other in (1.0, -3.0):
        S.vcycle(to_gpu(other * W.random_complex(w.shape, np.random.default_rng(5))))
        assert np.array_equal(to_np(S.vcycle(to_gpu(v))), got)


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("omega", [1.0, 0.85])
@pytest.mark.parametrize("n,coarsest", [(37, 10), (125, 32), (193, 7)])
def test_vcycle_relaxation_factor(dt, omega, n, coarsest):
    """The forms of the fused kernels with omega = 1 known at compile time and
    with any omega, one and two levels per kernel, on grids of less than one tile
    and one column beyond a tile (125 = 120 + 5, 63 = 60 + 3), against the
    oracle's cycle."""
    w = ragged_workload(n=n, coarsest=coarsest, omega=omega)
    P = oracle_for(w)
    S = gpu_for(w, dt)
    v = W.random_complex(w.shape, np.random.default_rng(n))
    ref = P.mg_apply(v)
    for tuning in (dict(pair_grid=0), dict(pair_grid=n), dict(pair_grid=0, small_grid=3, down_rows=4, up_rows=8)):
        S.set_tuning(tail_nodes=9, **tuning)
        got = to_np(S.vcycle(to_gpu(v)))
        assert relerr(got, ref) < CYCLE_TOL[dt], tuning
        assert np.all(got[[0, -1]] == 0) and np.all(got[:, [0, -1]] == 0)


@pytest.mark.parametrize("gf,gc,smoother,omega,nu", [(2, 2, "rbgs", 1.05, 1), (1, 2, "jacobi", 0.8, 1),
                                                      (1, 4, "jacobi", 0.5, 2), (1, 1, "rbgs", 1.0, 2)])
def test_general_cycles(gf, gc, smoother, omega, nu):
    """Algorithm 1 with other cycle indices (W, F, F_1^4) and sweep counts."""
    w = W.coulomb(E=1.0, n=129)
    cyc = dict(smoother=smoother, omega=omega, nu1=nu, nu2=nu, gamma_f=gf, gamma_c=gc, coarsest=5)
    for prec in (dict(kind="qd", lam0=0.0), dict(kind="csl", beta1=-1.0, beta2=-0.5),
                 dict(kind="csg", theta_alpha=math.pi / 13)):
        P = oracle_for(w, prec=prec, cycle=cyc)
        S = gpu_for(w, "f64", prec=prec, cycle=cyc)
        z = to_np(S.vcycle(to_gpu(w.rhs[0])))
        assert relerr(z, P.mg_apply(w.rhs[0])) < 1e-12, (prec["kind"], gf, gc)


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("gf,gc,smoother,omega,nu1,nu2", [(1, 4, "jacobi", 0.8, 1, 1), (1, 3, "jacobi", 0.5, 2, 1),
                                                          (2, 2, "rbgs", 1.05, 0, 2), (1, 2, "rbgs", 1.0, 1, 0),
                                                          (2, 3, "jacobi", 0.8, 1, 2)])
def test_general_cycle_tail(dt, gf, gc, smoother, omega, nu1, nu2):
    """General cycles whose coarse end runs as one single-workgroup schedule:
    every tail start (none, the last levels, the whole hierarchy), unequal
    and zero sweep counts, against the oracle; the captured cycle replays the
    eager one bit for bit."""
    import torch
    rng = np.random.default_rng(15)
    cyc = dict(smoother=smoother, omega=omega, nu1=nu1, nu2=nu2, gamma_f=gf, gamma_c=gc)
    runs = [(ragged_workload(n=97, coarsest=4), 4, (3, 7, 13, 25, 33)),
            (W.paper_mp2(L=6.25, n_int=64, n_layer=16)[0], 6, (3, 11, 21, 33)),
            (W.coulomb(E=1.0, n=33), 5, (9, 33))]
    for w, c, tails in runs:
        cy = dict(cyc, coarsest=c)
        prec = dict(kind="csl", beta1=-1.0, beta2=-0.5)
        P = oracle_for(w, prec=prec, cycle=cy)
        S = gpu_for(w, dt, prec=prec, cycle=cy)
        v = W.random_complex(w.shape, rng)
        ref = P.mg_apply(v)
        for tn in tails:
            S.set_tuning(tail_nodes=tn)
            S.set_graphs(False)
            ze = S.vcycle(to_gpu(v))
            assert relerr(to_np(ze), ref) < (1e-12 if dt == "f64" else CYCLE_TOL[dt]), (w.name, tn)
            S.set_graphs(True)
            for _ in range(3):
                zg = S.vcycle(to_gpu(v))
                torch.cuda.synchronize()
                assert torch.equal(zg, ze), (w.name, tn)


def test_3d_steps_and_cycle():
    w = W.cube_constant_k(n=33, k=6.0)
    P = oracle_for(w)
    S = gpu_for(w, "f64")
    rng = np.random.default_rng(10)
    x = W.random_complex(w.shape, rng)
    for op in ("A", "M", "AT"):
        assert relerr(to_np(S.apply(to_gpu(x), op)), P.apply(x, which=op)) < 1e-13
    b = W.random_complex(w.shape, rng)
    assert relerr(to_np(S.smooth(to_gpu(b), to_gpu(x))), P.smooth(b, x)) < 1e-13
    rc = to_np(S.residual_restrict(to_gpu(b), to_gpu(x)))
    assert relerr(rc, P.restrict(P.residual(b, x))) < 1e-13
    ec = W.random_complex(S.level_shape(1), rng)
    assert relerr(to_np(S.prolong_correct(to_gpu(ec), to_gpu(x))), P.prolong_add(ec, x)) < 1e-13
    assert relerr(to_np(S.vcycle(to_gpu(b))), P.mg_apply(b)) < 1e-12
    S32 = gpu_for(w, "f32")
    assert relerr(to_np(S32.vcycle(to_gpu(b))), P.mg_apply(b)) < 2e-4


@pytest.mark.parametrize("n,coarsest", [(97, 4), (65, 5)])
def test_3d_steps_and_cycle_wide(n, coarsest):
    """3D grids wider than one 64-node x-tile of the 3D kernels (97^3 ragged,
    unsymmetric layers, random k^2; 65^3 one node over the tile): every step
    and one cycle (both dtypes) against the oracle."""
    w = ragged_workload(n=n, coarsest=coarsest, dim=3, seed=33)
    P = oracle_for(w)
    S = gpu_for(w, "f64")
    rng = np.random.default_rng(11)
    x = W.random_complex(w.shape, rng)
    for op in ("A", "M", "AT"):
        y = to_np(S.apply(to_gpu(x), op))
        assert relerr(y, P.apply(x, which=op)) < 1e-13, op
        assert np.all(y[0] == 0) and np.all(y[:, :, -1] == 0)
    b = W.random_complex(w.shape, rng)
    assert relerr(to_np(S.smooth(to_gpu(b), to_gpu(x))), P.smooth(b, x)) < 1e-13
    rc = to_np(S.residual_restrict(to_gpu(b), to_gpu(x)))
    assert relerr(rc, P.restrict(P.residual(b, x))) < 1e-13
    ec = W.random_complex(S.level_shape(1), rng)
    assert relerr(to_np(S.prolong_correct(to_gpu(ec), to_gpu(x))), P.prolong_add(ec, x)) < 1e-13
    ref = P.mg_apply(b)
    assert relerr(to_np(S.vcycle(to_gpu(b))), ref) < 1e-12
    S32 = gpu_for(w, "f32")
    assert relerr(to_np(S32.vcycle(to_gpu(b))), ref) < 2e-4


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("n,coarsest,omega", [(5, 3, 1.0), (9, 5, 1.0), (17, 9, 1.15), (33, 5, 1.0), (53, 14, 0.9),
                                              (73, 10, 1.15)])
def test_3d_fused_cycle(dt, n, coarsest, omega):
    """The fused 3D down / up kernels against the oracle's cycle, with random k^2
    and unsymmetric layers: one coarse plane, levels below one tile, one node
    beyond a tile in x (73 = 66 + 7) and rows, chunks and planes that do not
    divide; the graph replay gives the same bits."""
    w = ragged_workload(n=n, coarsest=coarsest, omega=omega, dim=3)
    P = oracle_for(w)
    S = gpu_for(w, dt)
    cdt = np.complex64 if dt == "f32" else np.complex128
    v = W.random_complex(w.shape, np.random.default_rng(n)).astype(cdt)
    got = to_np(S.vcycle_native(to_gpu(v)))
    assert relerr(got, P.mg_apply(v.astype(np.complex128))) < (2e-4 if dt == "f32" else 1e-12)
    for a in range(3):
        assert np.all(np.take(got, [0, -1], axis=a) == 0)
    S.set_graphs(True)
    assert np.array_equal(to_np(S.vcycle_native(to_gpu(v))), got)


@pytest.mark.parametrize("n,coarsest,k,omega", [(17, 5, 9.0, 1.0), (33, 5, 5.0, 1.0), (97, 4, 9.0, 1.0),
                                                (97, 4, 9.0, 0.9)])
def test_3d_fp32_cycle_accuracy(n, coarsest, k, omega):
    """The FP32 3D cycle at constant k on a mesh that is uniform inside the layers,
    where the diagonal has the same rounding error at every node: within two FP32
    roundings (2 x 2^-24, relative in the 2-norm) of the oracle's 64-bit cycle.  A
    relaxation's sums, its store and the corrections' are a few independent
    roundings of half a unit each at most; an error common to all nodes, of a
    diagonal or an inverse formed in FP32, exceeds that (1.3e-7 to 2.6e-7 here)."""
    w = W.cube_constant_k(n=n, k=k, coarsest=coarsest)
    err = fp32_cycle_error(w, dict(w.cycle, omega=omega))
    assert err < 2.0 ** -23, err


def fp32_cycle_error(w, cycle):
    """Error of the FP32 cycle against the oracle's, relative in the 2-norm."""
    P = oracle_for(w, cycle=cycle)
    S = gpu_for(w, "f32", cycle=cycle)
    v = W.random_complex(w.shape, np.random.default_rng(w.n[0])).astype(np.complex64)
    ref = P.mg_apply(v.astype(np.complex128))
    return np.linalg.norm(to_np(S.vcycle_native(to_gpu(v))) - ref) / np.linalg.norm(ref)


@pytest.mark.parametrize("dim,n,coarsest,smoother", [(2, 33, 5, "rbgs"), (2, 41, 6, "jacobi"), (3, 13, 4, "rbgs"),
                                                     (3, 13, 4, "jacobi")])
def test_fp32_dense_map_accuracy(dim, n, coarsest, smoother):
    """A grid that is one FP32 dense map, of two and more products a lane and of more
    than are staged at a time (41): within one FP32 rounding (2^-24, relative in the
    2-norm) of the oracle's cycle.  The map's entries and the result are rounded by
    half a unit at most, independently; the sums are FP64."""
    w = W.coulomb(E=2.0, n=n, coarsest=coarsest) if dim == 2 else W.cube_constant_k(n=n, k=5.0, coarsest=coarsest)
    err = fp32_cycle_error(w, dict(w.cycle, smoother=smoother, omega=1.0 if smoother == "rbgs" else 0.8))
    assert err < 2.0 ** -24, err


@pytest.mark.parametrize("n,coarsest,gamma,omega", [(129, 5, 3, 0.6), (257, 5, 1, 0.8), (385, 4, 1, 0.8)])
def test_fp32_jacobi_cycle_accuracy(n, coarsest, gamma, omega):
    """FP32 omega-Jacobi cycles on the fused level kernels, where the relaxation uses
    the diagonal's inverse directly: within two FP32 roundings (2 x 2^-24, relative
    in the 2-norm) of the oracle's cycle, as with the 3D cycle's."""
    w = W.coulomb(E=2.0, n=n, coarsest=coarsest)
    err = fp32_cycle_error(w, dict(w.cycle, smoother="jacobi", omega=omega, gamma_c=gamma))
    assert err < 2.0 ** -23, err


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("dim,n,coarsest,gf,gc,smoother,nu1,nu2",
                         [(2, 81, 6, 1, 3, "jacobi", 1, 1), (2, 41, 6, 1, 4, "jacobi", 1, 2),
                          (2, 93, 47, 1, 1, "rbgs", 1, 1), (2, 9, 3, 1, 1, "rbgs", 1, 1), (2, 5, 5, 1, 1, "rbgs", 1, 1),
                          (3, 17, 3, 1, 1, "rbgs", 1, 1), (3, 21, 6, 2, 2, "jacobi", 1, 1),
                          (3, 25, 4, 1, 3, "rbgs", 2, 1), (3, 19, 10, 1, 2, "jacobi", 0, 2)])
def test_dense_coarse_end(dt, dim, n, coarsest, gf, gc, smoother, nu1, nu2):
    """The dense map of the coarse end against the oracle's cycle: one unknown
    on the coarsest level, odd and even numbers of unknowns, 1521 and 2025
    unknowns (more than the 1024 staged at a time), 3D maps, the whole grid as
    one map, one level, repeated visits with exchanged cycle indices, zero
    sweeps."""
    if coarsest < n:
        w = ragged_workload(n=n, coarsest=coarsest, dim=dim)
    else:
        w = W.coulomb(E=1.0, n=n, coarsest=coarsest)
    cy = dict(smoother=smoother, omega=0.9, nu1=nu1, nu2=nu2, gamma_f=gf, gamma_c=gc, coarsest=coarsest)
    P = oracle_for(w, cycle=cy)
    S = gpu_for(w, dt, cycle=cy)
    v = W.random_complex(w.shape, np.random.default_rng(n))
    got = to_np(S.vcycle(to_gpu(v)))
    assert relerr(got, P.mg_apply(v)) < (1e-12 if dt == "f64" else CYCLE_TOL[dt])
    for a in range(dim):
        assert np.all(np.take(got, [0, -1], axis=a) == 0)


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("n,coarsest,gf,gc", [(61, 16, 1, 1), (113, 8, 1, 3), (125, 32, 2, 2), (113, 8, 2, 1),
                                              (545, 18, 1, 2)])
def test_fused_jacobi_cycle(dt, n, coarsest, gf, gc):
    """The fused omega-Jacobi level kernels against the oracle's cycle: one coarse
    column and row beyond a tile (61: 31 = 30 + 1; 113: 57 = 2 x 28 + 1; 125 = 2 x
    62 + 1), groups of one, two and three visits, low and tall tiles (545)."""
    w = ragged_workload(n=n, coarsest=coarsest, kind="csl", smoother="jacobi", omega=0.8)
    cy = dict(w.cycle, gamma_f=gf, gamma_c=gc)
    P = oracle_for(w, cycle=cy)
    S = gpu_for(w, dt, cycle=cy)
    v = W.random_complex(w.shape, np.random.default_rng(n))
    got = to_np(S.vcycle(to_gpu(v)))
    assert relerr(got, P.mg_apply(v)) < (1e-12 if dt == "f64" else CYCLE_TOL[dt])
    assert np.all(got[[0, -1]] == 0) and np.all(got[:, [0, -1]] == 0)


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_exchanged_maps_only_below_level_one(dt):
    """The workspace of an F cycle holds maps for the exchanged cycle indices from
    level 2 on: against a W cycle, which has none, 21^2 and 11^2 maps more and no
    41^2 one."""
    import ctypes
    import paper_1012_4307_amd as E
    w = ragged_workload(n=81, coarsest=6, kind="csl", smoother="jacobi", omega=0.8)

    def size(gf, gc):
        n = ctypes.c_size_t()
        S = gpu_for(w, dt, cycle=dict(w.cycle, gamma_f=gf, gamma_c=gc))
        assert E.lib().ecs_workspace_size(S._h, None, ctypes.byref(n)) == 0
        return n.value

    entry = 16 + (8 if dt == "f32" else 0)
    maps = entry * (19 * 19 * (19 * 19 + 1) + 81 * 82)
    assert abs(size(1, 2) - size(2, 2) - maps) <= 8 * 256


def test_schedule_change_launches_nothing():
    """A schedule set while the context's stream is being captured, by a program that
    then drops the graph: the eager cycles after it use the new schedule's FP32 map
    (the dense end from 17^2 instead of 33^2)."""
    import torch
    w = W.coulomb(E=2.0, n=129)
    P = oracle_for(w)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        S = gpu_for(w, "f32")
        v = W.random_complex(w.shape, np.random.default_rng(8))
        ref = P.mg_apply(v)
        assert relerr(to_np(S.vcycle(to_gpu(v))), ref) < CYCLE_TOL["f32"]
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            S.set_tuning(tail_nodes=17)
        del g
        assert relerr(to_np(S.vcycle(to_gpu(v))), ref) < CYCLE_TOL["f32"]


def skewed(w):
    """The workload with another mesh width, contour and layers on every axis."""
    dim = w.dim
    lo, hi = (-1.0, -1.3, -0.8)[:dim], (1.0, 0.9, 1.5)[:dim]
    ecs = (((-0.55, np.pi / 5), (0.6, np.pi / 7)), (None, (0.3, np.pi / 4)),
           ((-0.5, np.pi / 9), (0.9, np.pi / 6)))[:dim]
    return W.Workload(w.name + "_skewed", dim, w.n, lo, hi, ecs, w.k2, w.rhs, w.precond, w.cycle, w.krylov, w.nlev)


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("dim,n,coarsest,smoother,gamma,omega", [
    (3, 33, 5, "rbgs", 1, 1.0), (3, 53, 14, "rbgs", 1, 0.9), (3, 13, 4, "rbgs", 1, 1.0), (3, 19, 10, "jacobi", 2, 0.8),
    (2, 33, 5, "rbgs", 1, 1.0), (2, 193, 7, "rbgs", 1, 1.0), (2, 385, 7, "rbgs", 1, 0.9), (2, 41, 6, "jacobi", 3, 0.8),
    (2, 113, 8, "jacobi", 1, 0.8), (2, 145, 10, "jacobi", 3, 0.7)])
def test_cycles_with_other_weights_on_every_axis(dt, dim, n, coarsest, smoother, gamma, omega):
    """The fused kernels and the dense maps take each axis's own weights: cycles on
    grids with another mesh width, contour and layers per axis against the oracle."""
    w = skewed(ragged_workload(n=n, coarsest=coarsest, dim=dim, smoother=smoother, omega=omega))
    cy = dict(w.cycle, gamma_c=gamma)
    P = oracle_for(w, cycle=cy)
    S = gpu_for(w, dt, cycle=cy)
    v = W.random_complex(w.shape, np.random.default_rng(n))
    ref = P.mg_apply(v)
    for tuning in (dict(), dict(tail_nodes=9, pair_grid=0, small_grid=3)) if dim == 2 else (dict(),):
        S.set_tuning(**tuning)
        assert relerr(to_np(S.vcycle(to_gpu(v))), ref) < CYCLE_TOL[dt], tuning


@pytest.mark.parametrize("method,smoother,inner,n", [("bicgstab", "rbgs", 0, 193), ("gmres", "rbgs", 0, 193),
                                                     ("fgmres", "rbgs", 4, 193), ("gmres", "jacobi", 0, 57),
                                                     ("bicgstab", "rbgs", 0, 545)])
def test_operator_with_other_weights_on_every_axis(method, smoother, inner, n):
    """The matvec inside the cycle's last kernel takes each axis's own weights: the
    solve reaches its tolerance by the oracle's operator, in at most one step more
    than with the separate matvec (which a timed one is)."""
    import paper_1012_4307_amd as E
    kind, om = ("csl", 0.8) if smoother == "jacobi" else ("qd", 1.0)
    w = skewed(ragged_workload(n=n, coarsest={193: 7, 57: 29, 545: 18}[n], kind=kind, smoother=smoother, omega=om))
    P = oracle_for(w)
    kr = E.Krylov(method=method, restart=30, rtol=1e-8, maxit=3000, inner=inner)
    S = gpu_for(w, "f32" if inner else "f64", krylov=kr)
    b = w.rhs[0].copy()
    b[[0, -1]] = b[:, [0, -1]] = 0
    x, st = S.solve(to_gpu(b))
    assert st["status"] == 0, st
    assert np.linalg.norm((b - P.apply(to_np(x)))[1:-1, 1:-1]) <= 1.05e-8 * np.linalg.norm(b)
    if inner == 0:
        S.timing("apply_A", True)
        _, other = S.solve(to_gpu(b))
        assert abs(st["iterations"] - other["iterations"]) <= max(1, 0.02 * other["iterations"]), (st, other)


def test_full_size_vcycle_sampled():
    """The benchmark grid (2049^2, h = 0.25, 9 levels): one FP64 cycle checked
    against the oracle on the whole grid (one oracle cycle takes seconds)."""
    w = W.large_coulomb(n=2049)
    P = oracle_for(w)
    S = gpu_for(w, "f64")
    z = to_np(S.vcycle(to_gpu(w.rhs[0])))
    assert relerr(z, P.mg_apply(w.rhs[0])) < 1e-12
    S32 = gpu_for(w, "f32")
    z32 = to_np(S32.vcycle(to_gpu(w.rhs[0])))
    assert relerr(z32, P.mg_apply(w.rhs[0])) < 2e-4


def test_vcycle_graph_replay_matches_eager():
    """The captured cycle graph, replayed several times with other eager work
    and synchronisations in between, reproduces the eager cycle bit for bit
    (both dtypes)."""
    import torch
    w = W.coulomb(E=2.0, n=257)
    for dt in ("f64", "f32"):
        S = gpu_for(w, dt)
        v = to_gpu(w.rhs[0])
        S.set_graphs(False)
        ref = S.vcycle(v)
        S.set_graphs(True)
        x = to_gpu(W.random_complex(w.shape, np.random.default_rng(3)))
        for r in range(4):
            z = S.vcycle(v)
            torch.cuda.synchronize()
            y = S.apply(x, "A")
            torch.cuda.synchronize()
            assert torch.equal(z, ref), (dt, r)
        assert torch.isfinite(y.abs()).all()
        # the default mode launches this fused cycle eagerly
        S.set_graphs("auto")
        assert torch.equal(S.vcycle(v), ref), dt


def test_sampled_timing_and_launch_mode_arguments():
    """Kernel timing of one launch in `every` (the 1st, (every+1)-th, ...):
    ten cycles timed one in four give three timed fine-level down launches,
    all with the same algorithmic bytes; launch modes outside
    never/always/auto and negative timing arguments are rejected."""
    import torch
    import paper_1012_4307_amd as E
    w = W.coulomb(E=2.0, n=257)
    S = gpu_for(w, "f32")
    v = to_gpu(w.rhs[0]).to(torch.complex64)
    S.timing("down", True, every=4)
    for _ in range(10):
        S.vcycle_native(v)
    n, ms, by = S.timing_read("down")
    S.timing("down", False)
    assert n == 3 and ms > 0, (n, ms)
    assert by == pytest.approx(3 * 257 * 257 * 4 * 3.5)  # read b, k^2; write the coarse quarter
    S.timing("down", True)
    for _ in range(5):
        S.vcycle_native(v)
    n, _, _ = S.timing_read("down")
    S.timing("down", False)
    assert n == 5
    assert E.lib().ecs_set_graphs(S._h, 3) == -1
    assert E.lib().ecs_timing_enable(S._h, 7, -1) == -1
    with pytest.raises(ValueError):
        S.timing("down", True, every=0)
