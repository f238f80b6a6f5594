"""rg_step without a schedule takes the tree's ghost mode: random states that
vary across every coarse-fine border, on which injection and interpolation
differ, against the oracle and the scheduled step.  rg_hydro_step_level, which
is given no tree, injects."""
import numpy as np
import pytest
import torch

from gpu_common import parity_metric, say
from oracle import oracle as O
from paper_2607_20704_amd import inputs as I

pytestmark = pytest.mark.gpu

CASES = [("periodic_3_5", 3, 5, I.PERIODIC), ("walls_3_6", 3, 6, I.OUTFLOW)]


@pytest.mark.parametrize("form", [0, 1], ids=["fp64", "mixed"])
@pytest.mark.parametrize("name,base,lmax,bc", CASES, ids=[c[0] for c in CASES])
def test_step_without_schedule_interpolates(name, base, lmax, bc, form):
    from paper_2607_20704_amd import api
    ijkl = I.sphere_tree(base, lmax, (0.35, 0.5, 0.6), 0.22, bc)
    T = {g: O.Tree(ijkl, bc, ghost=g) for g in (O.GHOST_INJECT, O.GHOST_LINEAR)}
    gam = 1.4
    rng = np.random.default_rng(11)
    n = 8 * len(ijkl)
    rho = np.exp(0.3 * rng.standard_normal(n))
    vel = 0.4 * rng.standard_normal((3, n))
    u0 = I.fill_split_cells(T[0].ijkl, I.conserved(rho, *vel, np.exp(0.3 * rng.standard_normal(n)), gam).reshape(-1, 5))
    u = torch.as_tensor(u0).cuda()
    got = {}
    for g in T:
        for schedule in (False, True):
            D = api.DeviceTree(ijkl, bc, schedule=schedule, ghost=g)
            v = torch.empty_like(u)
            dt = D.step(u, v, gam, 0.8, form=form)
            got[g, schedule] = v.cpu().numpy()
        assert np.array_equal(got[g, False], got[g, True])
        if form == api.RG_FP64:
            ref = u0.copy()
            T[g].run(ref, gam, 0.8, 1)
            worst = parity_metric(got[g, False], ref)[0]
            say("unscheduled step, ghost mode", g, name, "worst %.3g" % worst)
            assert worst <= 1e-12
    assert not np.array_equal(got[O.GHOST_INJECT, False], got[O.GHOST_LINEAR, False])
    # one level without a tree: injection, whatever the tree it belongs to says
    D = api.DeviceTree(ijkl, bc, schedule=False, ghost=O.GHOST_LINEAR)
    E = api.DeviceTree(ijkl, bc, schedule=True, ghost=O.GHOST_INJECT)
    ob, oe = int(D.level_begin[lmax]), int(D.level_begin[lmax + 1])
    a, b = torch.zeros_like(u), torch.zeros_like(u)
    D.hydro_level(lmax, dt, gam, u, a, form=form)
    E.hydro_level(lmax, dt, gam, u, b, form=form)
    assert torch.equal(a[8 * ob:8 * oe], b[8 * ob:8 * oe])
