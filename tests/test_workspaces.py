"""Workspace sizes and what a plan does in them.  qb_workspace_bytes is the
layout with one summation group per (cell, j); qb_workspace_bytes_preferred
adds the groups' buffers.  A plan in the smaller one sums in one group, or in
groups with I_3 cut into launches of fewer cells; both have to give the
oracle's operator and its transpose (1e-11 in float64), and with groups the
very numbers of the larger workspace."""
import ctypes
import functools

import numpy as np
import pytest

import paper_1408_1782_amd as qb
import workloads as wl
from oracle import adjoint as oad
from oracle import collision as oc
from oracle import pauli
from paper_1408_1782_amd import _lib
from test_gpu_adjoint import TOL, cot_api, cot_pauli, make_plan, rel, to_dev

FAKE_WS = ctypes.c_void_p(1 << 40)  # never dereferenced: the calls return before the device is touched


def _bytes(fn, N, J, M, Nx, precision="f64", max_cells=0):
    return getattr(qb.load(), fn)(ctypes.byref(qb.Problem(Nx, N, J, M, precision=precision)._c()), max_cells)


@pytest.mark.parametrize("N", [16, 32, 64])
@pytest.mark.parametrize("J,M", [(2, 1), (32, 64), (40, 71), (128, 256)])
def test_least_size_is_one_task_per_cell_and_direction(N, J, M):
    """Per cell: 46 planes and 14 per direction (12 in float32) of the padded
    grid, and four state arrays, whatever the number of nodes."""
    plane = (2 * N) ** 2
    for precision, size, per_j in (("f64", 8, 14), ("f32", 4, 12)):
        cell = ((46 + per_j * J) * plane + 16 * N * N) * size
        least = [_bytes("qb_workspace_bytes", N, J, M, Nx, precision) for Nx in (2, 38)]
        assert least[1] - least[0] == 36 * cell
        p = qb.Problem(38, N, J, M, precision=precision)._c()
        h = ctypes.c_void_p()
        assert qb.load().qb_plan_create(ctypes.byref(p), 0, FAKE_WS, least[1] - 1, ctypes.byref(h)) == _lib.QB_EWORKSPACE


@pytest.mark.parametrize("N,J,M", [(16, 32, 16), (32, 32, 32), (32, 40, 71), (64, 32, 64), (64, 40, 71)])
@pytest.mark.parametrize("Nx", [1, 37, 256, 600])
def test_preferred_size_stays_near_the_least(N, J, M, Nx):
    """At most a quarter and 8 GB more in float64, the same in float32."""
    least, pref = (_bytes(f, N, J, M, Nx) for f in ("qb_workspace_bytes", "qb_workspace_bytes_preferred"))
    assert least <= pref <= 1.25 * least + 8e9
    assert _bytes("qb_workspace_bytes_preferred", N, J, M, Nx, "f32") == _bytes("qb_workspace_bytes", N, J, M, Nx, "f32")


def test_sizes_of_very_many_cells_per_launch():
    """10^6 cells in one launch: more tasks than 32 bits count."""
    least, pref = (_bytes(f, 16, 128, 256, 10**6, max_cells=10**6)
                   for f in ("qb_workspace_bytes", "qb_workspace_bytes_preferred"))
    assert 10**6 * (46 + 14 * 128) * 32 * 32 * 8 < least <= pref <= 1.25 * least


def test_sizes_of_invalid_descriptions_are_zero():
    assert _bytes("qb_workspace_bytes_preferred", 24, 8, 8, 1) == 0
    assert _bytes("qb_workspace_bytes_preferred", 16, 8, 8, 1, max_cells=-1) == 0
    assert qb.load().qb_adjoint_workspace_bytes_preferred(None) == 0
    assert qb.load().qb_batch_workspace_bytes_preferred(None, 0) == 0


# ------------------------------------------------------------------ on the device
def _plan(monkeypatch, least, w, J, M, Nx):
    """A plan in its least or its preferred workspaces."""
    with monkeypatch.context() as m:
        if "ws" in least:
            m.setattr(_lib, "_workspace", lambda n, k: _alloc(k))
        plan = qb.Plan(qb.Problem(Nx, w.N, J, M, w.L, w.R, "f64"))
    with monkeypatch.context() as m:
        if "adj" in least:
            m.setattr(_lib, "_workspace", lambda n, k: _alloc(k))
        plan.enable_adjoint()
    return plan


def _alloc(n):
    import torch
    return torch.empty(int(n), dtype=torch.uint8, device="cuda")


def _run(plan, w, lam):
    import torch
    W = to_dev(w.W0[: plan.problem.Nx], "f64")
    C, G = plan.collision(W), plan.collision_vjp(W, to_dev(cot_api(lam), "f64"))
    torch.cuda.synchronize()
    return C, G


def _inputs(N, Nx):
    return wl.config(2, Nx=Nx, N=N), np.random.default_rng(N + Nx).standard_normal((Nx, N, N, 4))


@functools.lru_cache(maxsize=None)
def _reference(N, J, M, Nx, cells):
    w, lam = _inputs(N, Nx)
    t = oc.Tables(w.N, w.L, w.R, J, M)
    s = pauli.to_pauli(w.W0)
    return (np.stack([oc.collision(w.W0[c], w.L, w.R, J, M, t) for c in cells]),
            np.stack([oad.collision_pauli_vjp(s[c], lam[c], w.L, w.R, J, M, t) for c in cells]))


def _check(C, G, N, J, M, Nx, cells):
    ref, ref_vjp = _reference(N, J, M, Nx, cells)
    assert rel(C.cpu().numpy()[list(cells)], ref) < TOL["f64"]
    assert rel(cot_pauli(G)[list(cells)], ref_vjp) < TOL["f64"]


@pytest.mark.gpu
@pytest.mark.parametrize("least", ["ws adj", "adj", "ws", ""])
@pytest.mark.parametrize("N,J,M,Nx", [(16, 10, 9, 1), (16, 10, 9, 7), (32, 18, 17, 2), (64, 10, 9, 1)])
def test_every_workspace_gives_the_oracles_operator(monkeypatch, least, N, J, M, Nx):
    w, lam = _inputs(N, Nx)
    plan = _plan(monkeypatch, least, w, J, M, Nx)
    _check(*_run(plan, w, lam), N, J, M, Nx, tuple({0, Nx - 1}))
    plan.close()


@pytest.mark.gpu
@pytest.mark.parametrize("paired", [True, False])
@pytest.mark.parametrize("N,J,M,Nx", [(16, 32, 16, 23), (32, 16, 18, 11)])
def test_cells_of_every_i3_launch_are_the_same_numbers(monkeypatch, paired, N, J, M, Nx):
    """The least workspace of many cells holds the groups of a few: I_3 and its
    transpose run in several launches, and no cell notices."""
    import torch
    w, lam = _inputs(N, Nx)
    out = []
    for least in ("", "ws adj"):
        plan = _plan(monkeypatch, least, w, J, M, Nx)
        plan.set_pairing(paired)
        out.append(_run(plan, w, lam))
        plan.close()
    assert torch.equal(out[0][0], out[1][0])
    assert torch.equal(out[0][1], out[1][1])


@pytest.mark.gpu
def test_more_cells_than_one_i3_launch_in_the_preferred_workspace():
    """N = 16, J = 72, M = 72 runs I_3 in launches of at most 101 cells: cells of
    every launch against a plan of one cell and against the oracle."""
    import torch
    N, J, M, Nx = 16, 72, 72, 110
    w, lam = _inputs(N, Nx)
    plan = make_plan(w, "f64", J, M)
    C, G = _run(plan, w, lam)
    plan.close()
    _check(C, G, N, J, M, Nx, (100, 109))
    one = make_plan(w, "f64", J, M, Nx=1)
    for c in (0, 54, 55, 100, 101, 109):
        W, L = to_dev(w.W0[c : c + 1], "f64"), to_dev(cot_api(lam[c : c + 1]), "f64")
        assert torch.equal(one.collision(W)[0], C[c])
        assert torch.equal(one.collision_vjp(W, L)[0], G[c])
    one.close()


@pytest.mark.gpu
def test_batch_in_its_least_workspace(monkeypatch):
    import torch
    ws = [wl.config(2, Nx=n, N=N) for N, n in ((16, 1), (32, 3), (16, 4))]
    out = []
    for least in (False, True):
        if least:
            monkeypatch.setattr(_lib, "_workspace", lambda n, k: _alloc(k))
        b = qb.Batch([qb.Problem(w.Nx, w.N, 10, 9, w.L, w.R, "f64") for w in ws])
        W = [to_dev(w.W0, "f64") for w in ws]
        b.step(W, None, 1e-3, 2)
        torch.cuda.synchronize()
        out.append([x.cpu().numpy() for x in W])
        b.close()
    for a, c in zip(*out):
        assert rel(a, c) < TOL["f64"]


def test_python_takes_the_least_where_memory_is_short(monkeypatch):
    import torch

    def empty(n, **kw):
        if n > 1000:
            raise torch.cuda.OutOfMemoryError("no room")
        return n

    monkeypatch.setattr(torch, "empty", empty)
    assert _lib._workspace(900, 500) == 900
    assert _lib._workspace(5000, 500) == 500
    with pytest.raises(torch.cuda.OutOfMemoryError):
        _lib._workspace(5000, 2000)
