"""GPU test of qb_profile_read's launch counts: one of every kernel class per
collision launch and two groups of other reverse-mode kernels, however many
launches the I_3 buffers cut it into (110 cells with J = M = 72: two)."""
import pytest

import workloads as wl
from test_gpu_adjoint import make_plan, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["f64", "f32"])
@pytest.mark.parametrize("J,M,Nx", [(8, 8, 3), (72, 72, 110)])
def test_launches_count_once_per_collision(precision, J, M, Nx):
    w = wl.config(2, Nx=Nx, N=16)
    plan = make_plan(w, precision, J, M)
    W = to_dev(w.W0, precision)
    plan.profile(True)
    plan.collision(W)
    counts = {k: plan.profile_read(k) for k in ("dft_in", "terms", "i3", "combine")}
    assert {k: n for k, (_, n) in counts.items()} == dict(dft_in=1, terms=1, i3=1, combine=1)
    assert all(ms > 0 for ms, _ in counts.values())
    plan.collision_vjp(W, W)
    counts = {k: plan.profile_read(k) for k in ("dft_in", "i3_adjoint", "adjoint")}
    assert {k: n for k, (_, n) in counts.items()} == dict(dft_in=1, i3_adjoint=1, adjoint=2)
    assert all(ms > 0 for ms, _ in counts.values())
    plan.close()
