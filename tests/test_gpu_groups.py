"""GPU tests of the node groups of I_3 and the direction groups of the other
terms, where the split can go wrong: one node, a last group that is short, an
odd middle node, one and two direction groups; float64 splits its sums into
groups, float32 keeps one sum per (cell, j).  The bars are those of every
collision test against the oracle (1e-11 and 2e-5)."""
import numpy as np
import pytest

import workloads as wl
from oracle import adjoint as oad
from oracle import collision as oc
from oracle import pauli
from test_gpu_adjoint import TOL, cot_api, cot_pauli, make_plan, rel, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("N,J,M", [(16, 2, 1), (16, 10, 2), (16, 10, 9), (16, 2, 17), (16, 8, 18),
                                   (32, 10, 9), (32, 2, 17)])
def test_groups_match_oracle(precision, N, J, M):
    import torch
    rng = np.random.default_rng(100 * N + 10 * J + M)
    w = wl.config(2, Nx=2, N=N)
    plan = make_plan(w, precision, J, M)
    W = to_dev(w.W0, precision)
    t = oc.Tables(N, w.L, w.R, J, M)
    C = plan.collision(W)
    lam = rng.standard_normal((2, N, N, 4))
    G = plan.collision_vjp(W, to_dev(cot_api(lam), precision))
    torch.cuda.synchronize()
    ref = np.stack([oc.collision(w.W0[c], w.L, w.R, J, M, t) for c in range(2)])
    assert rel(C.cpu().numpy().astype(np.complex128), ref) < TOL[precision]
    s = pauli.to_pauli(w.W0)
    ref = np.stack([oad.collision_pauli_vjp(s[c], lam[c], w.L, w.R, J, M, t) for c in range(2)])
    assert rel(cot_pauli(G), ref) < TOL[precision]
    plan.close()


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("N,M", [(16, 17), (32, 16)])
def test_a_cells_result_does_not_depend_on_the_number_of_cells(precision, N, M):
    """The groups depend on J and M alone, so one cell and the first of
    several are the same numbers."""
    import torch
    w = wl.config(2, Nx=3, N=N)
    out = []
    for cells in (1, 3):
        plan = make_plan(w, precision, 8, M, Nx=cells)
        out.append(plan.collision(to_dev(w.W0[:cells], precision))[0].cpu())
        plan.close()
    assert torch.equal(out[0], out[1])
