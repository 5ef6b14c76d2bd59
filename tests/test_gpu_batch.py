"""Batched solve (Bi-CGSTAB rounds over independent systems, each on its own
stream; a system's right-hand sides solved together, every kernel of an
iteration serving all of them in one launch) and the cycle autotuner."""
import math

import numpy as np
import pytest

from helpers import gpu_for, oracle_for, relerr, to_gpu, to_np
import paper_1012_4307_amd as E
from paper_1012_4307_amd import workloads as W

pytestmark = pytest.mark.gpu


def small_batch():
    descs = W.batch_systems(count=6, sizes=(65, 129))
    return [W.batch_inputs(d) for d in descs]


def test_batch_equals_individual_solves():
    """Every right-hand side of every system: the batched iterate equals the
    one the single-system solve produces (same kernels in the same order), and
    its true residual, recomputed by the oracle, meets the tolerance."""
    import torch
    ws = small_batch()
    kr = E.Krylov(method="bicgstab", rtol=1e-8, maxit=5000)
    streams = [torch.cuda.Stream() for _ in range(3)]
    solvers, rhs = [], []
    for q, w in enumerate(ws):
        with torch.cuda.stream(streams[q % 3]):
            solvers.append(gpu_for(w, "f64" if q % 2 else "f32", krylov=kr))
        rhs.append(torch.stack([to_gpu(b) for b in w.rhs]))
    torch.cuda.synchronize()
    xs, stats = E.batch_solve(solvers, rhs, kr)
    torch.cuda.synchronize()
    for q, w in enumerate(ws):
        assert stats[q]["status"] == 0, stats[q]
        P = oracle_for(w)
        for r, b in enumerate(w.rhs):
            with torch.cuda.stream(streams[q % 3]):
                x1, st = solvers[q].solve(to_gpu(b), krylov=kr)
            torch.cuda.synchronize()
            assert torch.equal(xs[q][r], x1), (q, r)
            xn = to_np(xs[q][r])
            res = np.linalg.norm((b - P.apply(xn))[1:-1, 1:-1]) / np.linalg.norm(b[1:-1, 1:-1])
            assert res <= 1.05e-8, (q, r, res)


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_multi_rhs_groups_equal_single_solves(dt):
    """Ten right-hand sides of one system (a group of 8 solved together, then a
    group of 2), one of them zero, with initial guesses, beside a second system
    with its own tolerance and an omega-Jacobi cycle (taken one right-hand
    side at a time): every solution equals the single solve from the same
    guess bit for bit, and its residual recomputed by the oracle meets the
    system's tolerance."""
    import dataclasses
    import torch
    w = W.coulomb(E=1.5, n=257)
    rng = np.random.default_rng(77)
    rhs = [W.random_complex(w.shape, rng) for _ in range(10)]
    rhs[5] = np.zeros(w.shape, complex)
    guesses = [0.01 * W.random_complex(w.shape, rng) for _ in range(10)]
    wj = W.small_constant_k(n=65, beta2=-0.5)
    rj = [W.random_complex(wj.shape, rng) for _ in range(3)]
    kr = E.Krylov(method="bicgstab", rtol=1e-9, maxit=5000)
    krj = E.Krylov(method="bicgstab", rtol=1e-7, maxit=5000)
    streams = [torch.cuda.Stream() for _ in range(2)]
    with torch.cuda.stream(streams[0]):
        S = gpu_for(w, dt, krylov=kr)
    with torch.cuda.stream(streams[1]):
        Sj = gpu_for(wj, dt, krylov=krj)
    B = torch.stack([to_gpu(b) for b in rhs])
    X0 = torch.stack([to_gpu(g) for g in guesses])
    Bj = torch.stack([to_gpu(b) for b in rj])
    torch.cuda.synchronize()
    xs, stats = E.batch_solve([S, Sj], [B, Bj], [kr, krj], x0=[X0, None])
    torch.cuda.synchronize()
    assert stats[0]["status"] == 0 and stats[1]["status"] == 0, stats
    P, Pj = oracle_for(w), oracle_for(wj)
    for q, (Sv, Pv, bs, xb, krv, tol) in enumerate(((S, P, rhs, xs[0], kr, 1e-9), (Sj, Pj, rj, xs[1], krj, 1e-7))):
        for r, b in enumerate(bs):
            x0 = X0[r] if q == 0 else None
            with torch.cuda.stream(streams[q]):
                x1, st = Sv.solve(to_gpu(b), x0=x0, krylov=krv)
            torch.cuda.synchronize()
            assert torch.equal(xb[r], x1), (q, r)
            if not b.any():
                assert int(torch.count_nonzero(xb[r])) == 0
                continue
            xn = to_np(xb[r])
            res = np.linalg.norm((b - Pv.apply(xn))[1:-1, 1:-1]) / np.linalg.norm(b[1:-1, 1:-1])
            assert res <= 1.05 * tol, (q, r, res)
    # through the ABI: a workspace sized for fewer right-hand sides at once
    # than the group of 8 is refused before any launch
    import ctypes
    S.ws = None
    S._ensure_workspace(dataclasses.replace(kr, nrhs=2))
    d = kr.to_c()
    xo = torch.empty_like(B)
    rc = E.lib().ecs_batch_solve(1, (ctypes.c_void_p * 1)(S._h.value),
                                 (ctypes.POINTER(E.SolveDesc) * 1)(ctypes.pointer(d)),
                                 (ctypes.c_void_p * 1)(B.data_ptr()), (ctypes.c_void_p * 1)(xo.data_ptr()),
                                 (ctypes.c_int * 1)(10), (E.Stats * 1)())
    assert rc == -2 and "nrhs = 8" in E.lib().ecs_last_error(S._h).decode()


def test_batch_wide_tail_equals_single_solves():
    """FP32 cycles with the wide tail (a 65^2 level and below in one
    workgroup): the batched solve of three right-hand sides together equals
    the single solves bit for bit, and the residuals meet the tolerance by the
    oracle's operator."""
    import torch
    w = W.coulomb(E=2.5, n=257)
    rng = np.random.default_rng(91)
    rhs = [W.random_complex(w.shape, rng) for _ in range(3)]
    kr = E.Krylov(method="bicgstab", rtol=1e-8, maxit=5000)
    S = gpu_for(w, "f32", krylov=kr)
    S.set_tuning(tail_nodes=65)
    B = torch.stack([to_gpu(b) for b in rhs])
    xs, stats = E.batch_solve([S], [B], kr)
    torch.cuda.synchronize()
    assert stats[0]["status"] == 0, stats
    P = oracle_for(w)
    for r, b in enumerate(rhs):
        x1, _ = S.solve(to_gpu(b), krylov=kr)
        torch.cuda.synchronize()
        assert torch.equal(xs[0][r], x1), r
        res = np.linalg.norm((b - P.apply(to_np(xs[0][r])))[1:-1, 1:-1]) / np.linalg.norm(b[1:-1, 1:-1])
        assert res <= 1.05e-8, (r, res)
    with pytest.raises(E.EcsError):
        S.set_tuning(tail_nodes=66)


def test_batch_edge_cases():
    """A zero right-hand side yields x = 0; an empty system list is a no-op."""
    import torch
    w = W.coulomb(E=1.0, n=65)
    kr = E.Krylov(method="bicgstab", rtol=1e-8, maxit=5000)
    S = gpu_for(w, "f64", krylov=kr)
    b = torch.stack([torch.zeros(w.shape, dtype=torch.complex128, device="cuda"), to_gpu(w.rhs[0])])
    xs, stats = E.batch_solve([S], [b], kr)
    assert int(torch.count_nonzero(xs[0][0])) == 0
    assert stats[0]["status"] == 0
    xs, stats = E.batch_solve([], [], kr)
    assert xs == [] and stats == []


def test_autotune_schedule_keeps_results(tmp_path, monkeypatch):
    """Every candidate schedule gives the same cycle (to rounding) and the
    oracle's; the tuner applies and caches the fastest."""
    import torch
    from paper_1012_4307_amd import autotune
    monkeypatch.setenv("ECSMG_TUNING_CACHE", str(tmp_path / "tune.json"))
    w = W.coulomb(E=2.0, n=257)
    P = oracle_for(w)
    ref = P.mg_apply(w.rhs[0])
    for dt, tol in (("f64", 1e-12), ("f32", 2e-4)):
        S = gpu_for(w, dt)
        v = to_gpu(w.rhs[0])
        for cand in list(autotune.candidates(dt))[::5]:
            S.set_tuning(**cand)
            assert relerr(to_np(S.vcycle(v)), ref) < tol, cand
        best = autotune.autotune(S)
        assert S.get_tuning() == best
        assert (tmp_path / "tune.json").exists()
        S2 = gpu_for(w, dt)
        assert autotune.autotune(S2) == best   # from the cache
    with pytest.raises(E.EcsError):
        S.set_tuning(down_rows=7)


def test_autotune_group_one_schedule_for_the_batch(tmp_path, monkeypatch):
    """The throughput tuner for batches: one schedule from the candidate list,
    applied to every solver of the group, cached; solvers of another size are
    refused; the batched solve under that schedule still equals the single
    solves made under the same schedule."""
    import torch
    from paper_1012_4307_amd import autotune
    monkeypatch.setenv("ECSMG_TUNING_CACHE", str(tmp_path / "tune.json"))
    descs = [d for d in W.batch_systems(count=12, sizes=(129, 257)) if d["n"] == 129][:3]
    ws = [W.batch_inputs(d) for d in descs]
    kr = E.Krylov(method="bicgstab", rtol=1e-8, maxit=5000)
    streams = [torch.cuda.Stream() for _ in ws]
    solvers, rhs = [], []
    for st, w in zip(streams, ws):
        with torch.cuda.stream(st):
            solvers.append(gpu_for(w, "f64", krylov=kr))
        rhs.append(torch.stack([to_gpu(b) for b in w.rhs]))
    torch.cuda.synchronize()
    best = autotune.autotune_group(solvers, reps=2)
    assert best in list(autotune.candidates("f64"))
    assert all(S.get_tuning() == best for S in solvers)
    assert (tmp_path / "tune.json").exists()
    assert autotune.autotune_group(solvers) == best   # from the cache
    other = gpu_for(W.coulomb(E=1.0, n=65), "f64", krylov=kr)
    with pytest.raises(ValueError):
        autotune.autotune_group([solvers[0], other])
    xs, stats = E.batch_solve(solvers, rhs, kr)
    torch.cuda.synchronize()
    for q, w in enumerate(ws):
        assert stats[q]["status"] == 0, stats[q]
        with torch.cuda.stream(streams[q]):
            x1, _ = solvers[q].solve(to_gpu(w.rhs[0]), krylov=kr)
        torch.cuda.synchronize()
        assert torch.equal(xs[q][0], x1), q


def test_cycle_timer_times_the_solvers_own_stream():
    """The single-cycle tuner's timer brackets the cycles on the stream they
    run on: a solver made under a side stream times like one made on the
    current stream (2049^2 FP64, where a cycle's device time is several times
    the host's launch time)."""
    import torch
    from paper_1012_4307_amd import autotune
    w = W.large_coulomb(n=2049)
    v = to_gpu(w.rhs[0])
    S0 = gpu_for(w, "f64")
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        S1 = gpu_for(w, "f64")
    assert S1.stream == side and S0.stream == torch.cuda.current_stream()
    t0 = min(autotune.time_cycles(S0, v, reps=10) for _ in range(3))
    t1 = min(autotune.time_cycles(S1, v, reps=10) for _ in range(3))
    assert 0.8 < t1 / t0 < 1.25, (t0, t1)


def test_side_stream_solver_is_ordered_with_the_callers_stream():
    """A solver made under a side stream reads inputs the caller's stream has
    just written (behind a long FP64 product) and its outputs are read on the
    caller's stream, with no explicit synchronisation: the results equal those
    of a solver made on the caller's stream."""
    import torch
    w = W.coulomb(E=2.0, n=513)
    kr = E.Krylov(method="bicgstab", rtol=1e-8, maxit=5000)
    S0 = gpu_for(w, "f64", krylov=kr)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        S1 = gpu_for(w, "f64", krylov=kr)
    ref = to_gpu(w.rhs[0])
    z0, y0 = S0.vcycle(ref), S0.apply(ref)
    x0, _ = S0.solve(ref)
    a = torch.randn(4096, 4096, device="cuda", dtype=torch.float64)
    torch.cuda.synchronize()
    for _ in range(2):
        b = torch.zeros_like(ref)
        _ = a @ a                      # keeps the caller's stream busy for milliseconds
        b.copy_(ref)
        z1, y1 = S1.vcycle(b), S1.apply(b)
        assert float((z1 - z0).abs().max()) == 0 and float((y1 - y0).abs().max()) == 0
        b2 = torch.zeros_like(ref)
        _ = a @ a
        b2.copy_(ref)
        x1, st = S1.solve(b2)
        assert st["status"] == 0 and torch.equal(x1, x0)
    # larger Krylov settings make the side-stream solver reallocate its
    # workspace from the caller's stream pool while that stream is still
    # busy with memory it then frees: the set-up in the new workspace waits
    # for the caller's stream, so the solve equals the caller-stream solver's
    big = E.Krylov(method="fgmres", restart=40, rtol=1e-8, maxit=20000)
    xb0, _ = S0.solve(ref, krylov=big)
    scratch = torch.randn(64 << 20, device="cuda", dtype=torch.float64)
    _ = a @ a
    scratch.mul_(2.0)
    del scratch
    b3 = torch.zeros_like(ref)
    b3.copy_(ref)
    xb1, st = S1.solve(b3, krylov=big)
    assert st["status"] == 0 and torch.equal(xb1, xb0)


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("n,coarsest", [(81, 41), (49, 4)])
def test_batch_dense_end_equals_single_solves(dt, n, coarsest):
    """Five right-hand sides through one dense map (1521 unknowns: two stages of
    1024; 529: one) give the single solves' bits."""
    import torch
    w = W.coulomb(E=2.0, n=n, coarsest=coarsest)
    rng = np.random.default_rng(n)
    kr = E.Krylov(method="bicgstab", rtol=1e-8, maxit=500)
    S = gpu_for(w, dt, krylov=kr)
    B = torch.stack([to_gpu(W.random_complex(w.shape, rng)) for _ in range(5)])
    xs, stats = E.batch_solve([S], [B], kr)
    assert stats[0]["status"] == 0, stats
    for r in range(5):
        assert torch.equal(xs[0][r], S.solve(B[r].contiguous(), krylov=kr)[0]), r


def test_second_search_direction_only_where_the_cycle_forms_it():
    """The batched workspace holds a second p per right-hand side only when the
    cycles form the updates; a workspace sized while they did not still solves
    after they were switched on, with the same bits."""
    import ctypes
    import dataclasses
    import torch
    kr = E.Krylov(method="bicgstab", rtol=1e-9, maxit=5000)
    k8 = dataclasses.replace(kr, nrhs=8)

    def size(S):
        n = ctypes.c_size_t()
        assert E.lib().ecs_workspace_size(S._h, ctypes.byref(k8.to_c()), ctypes.byref(n)) == 0
        return n.value

    w = W.coulomb(E=1.5, n=257)
    S = gpu_for(w, "f64", krylov=kr)
    full = size(S)
    S.set_graphs(True)
    graphs = size(S)
    S.set_graphs("auto")
    S.set_tuning(fuse_updates=0)
    separate = size(S)
    assert full - separate >= 8 * 257 * 257 * 16 and graphs == separate
    rng = np.random.default_rng(78)
    B = torch.stack([to_gpu(W.random_complex(w.shape, rng)) for _ in range(8)])
    S.ws = None
    S._ensure_workspace(k8)
    S.set_tuning(fuse_updates=1)
    x = torch.empty_like(B)
    d = k8.to_c()
    torch.cuda.synchronize()
    rc = E.lib().ecs_batch_solve(1, (ctypes.c_void_p * 1)(S._h.value),
                                 (ctypes.POINTER(E.SolveDesc) * 1)(ctypes.pointer(d)),
                                 (ctypes.c_void_p * 1)(B.data_ptr()), (ctypes.c_void_p * 1)(x.data_ptr()),
                                 (ctypes.c_int * 1)(8), (E.Stats * 1)())
    assert rc == 0
    ref, _ = E.batch_solve([gpu_for(w, "f64", krylov=kr)], [B], kr)
    torch.cuda.synchronize()
    assert torch.equal(x, ref[0])
