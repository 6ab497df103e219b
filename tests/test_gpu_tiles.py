"""GPU test of the tile the reverse mode runs on: its own until the program
chooses one; qb_plan_set_tile takes it along, unless it has been given a tile
or has been tuned."""
import numpy as np
import pytest

import workloads as wl
from oracle import adjoint as oad
from oracle import collision as oc
from oracle import pauli
from test_gpu_adjoint import TOL, cot_api, cot_pauli, make_plan, rel, to_dev

pytestmark = pytest.mark.gpu


def _choice(plan):
    c = plan.config()
    return c["tile"], c["adjoint_tile"], c["adjoint_variant"]


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("N,other", [(16, 16), (32, 32)])
def test_reverse_mode_follows_the_tile_that_is_set(precision, N, other):
    J, M = 4, 5
    w = wl.config(2, Nx=2, N=N)
    plan = make_plan(w, precision, J, M)
    first = (8, 1) if precision == "f64" else (16, 0)
    assert _choice(plan)[1:] == first
    plan.set_tile(other)
    assert _choice(plan) == (other, other, 0)
    lam = np.random.default_rng(N).standard_normal((2, N, N, 4))
    G = plan.collision_vjp(to_dev(w.W0, precision), to_dev(cot_api(lam), precision))
    t = oc.Tables(N, w.L, w.R, J, M)
    s = pauli.to_pauli(w.W0)
    ref = np.stack([oad.collision_pauli_vjp(s[c], lam[c], w.L, w.R, J, M, t) for c in range(2)])
    assert rel(cot_pauli(G), ref) < TOL[precision]
    plan.set_tile(8)
    assert _choice(plan) == (8, 8, 0)
    plan.set_adjoint_variant(1)
    plan.set_tile(other)
    assert _choice(plan) == (other, other, 1)
    plan.set_adjoint_tile(8)
    plan.set_tile(16)
    assert _choice(plan) == (16, 8, 1)
    plan.set_adjoint_tile(0)
    plan.set_tile(other)
    assert _choice(plan) == (other, other, 1)
    plan.close()


def test_a_tile_of_its_own_runs_kernel_0_unless_one_is_chosen():
    w = wl.config(2, Nx=1, N=32)
    plan = make_plan(w, "f64", 4, 4)
    plan.set_adjoint_tile(16)
    assert _choice(plan)[1:] == (16, 0)
    plan.close()


def test_a_tuned_reverse_tile_stays():
    w = wl.config(2, Nx=2, N=16)
    plan = make_plan(w, "f64", 4, 4)
    plan.tune()
    tuned = _choice(plan)[1:]
    plan.set_tile(16)
    plan.set_tile(8)
    assert _choice(plan)[1:] == tuned
    plan.close()
