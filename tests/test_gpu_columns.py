"""Columns of a complete level, slabs of bricks and the launches that serve
several levels, against the per-oct kernel: the same bits, state and next time
step, in both forms.

- Uniform boxes of one column up to 64 (16^3 to 128^3 cells), periodic and
  with outflow walls: segments of 2 planes, segments that do not divide the
  side (128^3 mixed: 12 planes, the last segment 8), bricks cut into 8, 4 and 1
  slabs.
- Graded trees with bricks on several levels, all levels in one launch per
  kernel."""
import numpy as np
import pytest
import torch

from paper_2607_20704_amd import inputs as I

pytestmark = pytest.mark.gpu


def _state(D, gam, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    n = 8 * D.n

    def rnd():
        return torch.randn(n, generator=g, dtype=torch.float64, device="cuda")

    rho = torch.exp(0.3 * rnd())
    vel = [0.5 * rnd() for _ in range(3)]
    e = torch.exp(0.3 * rnd()) / (gam - 1.0) + 0.5 * rho * (vel[0] ** 2 + vel[1] ** 2 + vel[2] ** 2)
    return torch.stack([rho] + [rho * v for v in vel] + [e], 1).contiguous()


def _step(D, u, gam, form, tune):
    from paper_2607_20704_amd import api
    dts = torch.zeros(2, dtype=torch.float64, device="cuda")
    api.cfl_dt(u, D.son_mask, D.level_begin, D.lmin, D.lmax, gam, 0.8, dts[:1])
    out = torch.full_like(u, float("nan"))
    D.step(u, out, gam, 0.8, form, dt=dts, tune=tune, chain=True)
    return out, dts


PER_OCT, BRICKS = (4, 256, 1), (4, 256, 0, 0, 0, 0, 0, 1)


@pytest.mark.parametrize("level", [4, 5, 6, 7])
@pytest.mark.parametrize("bc", [I.PERIODIC, I.OUTFLOW])
@pytest.mark.parametrize("form", [0, 1])
def test_complete_level(level, bc, form):
    from paper_2607_20704_amd import api
    D = api.DeviceTree(I.uniform_tree(level), bc)
    u = _state(D, 1.4, 40 + level)
    want, dt = _step(D, u, 1.4, form, PER_OCT)
    waves = (0, 2, 3) if form == api.RG_FP64 else (0, 3, 4)
    for w in waves:
        for tune in ((4, 256, 0, 0, w), BRICKS[:4] + (w,) + BRICKS[5:]):
            got, d = _step(D, u, 1.4, form, tune)
            assert torch.equal(got, want), tune
            assert torch.equal(d, dt), tune


@pytest.mark.parametrize("base,lmax,centre,radius,bc", [
    (5, 7, (0.5, 0.5, 0.5), 0.32, I.PERIODIC), (4, 6, (0.1, 0.5, 0.9), 0.4, I.OUTFLOW),
    (6, 7, (0.02, 0.97, 0.5), 0.25, I.PERIODIC)])
@pytest.mark.parametrize("form", [0, 1])
def test_levels_in_one_launch(base, lmax, centre, radius, bc, form):
    from paper_2607_20704_amd import api
    D = api.DeviceTree(I.sphere_tree(base, lmax, centre, radius, bc), bc)
    counts = D.schedule_counts()
    assert sum(counts[l][0] > 0 for l in counts) >= 2 and any(counts[l][2] for l in counts)
    u = _state(D, 1.4, base)
    for l in range(D.lmax, D.lmin, -1):
        api.restrict_level(u, D.father_cell, int(D.level_begin[l]), int(D.level_begin[l + 1]))
    want, dt = _step(D, u, 1.4, form, PER_OCT)
    for tune in (None, BRICKS, (2, 128), (7, 256, 0, 0, 0, 1), (4, 256, 0, 0, 0, 0, 256)):
        got, d = _step(D, u, 1.4, form, tune)
        assert torch.equal(got, want), tune
        assert torch.equal(d, dt), tune
    # level by level
    parts = torch.empty_like(u)
    nxt = torch.full((1,), float("inf"), dtype=torch.float64, device="cuda")
    for l in range(D.lmin, D.lmax + 1):
        D.hydro_level(l, dt[:1], 1.4, u, parts, form, cfl=0.8, dt_next=nxt)
    api.apply_coarse_corrections(parts, D.corr, D.corr_base, D.nbr27, D.corr_base, D.n)
    api.cfl_dt_corrected(parts, D.nbr27, D.level_begin, D.lmin, D.lmax, 1.4, 0.8, nxt)
    for l in range(D.lmax, D.lmin, -1):
        api.restrict_level(parts, D.father_cell, int(D.level_begin[l]), int(D.level_begin[l + 1]))
    assert torch.equal(parts, want)
    assert np.array_equal(nxt.cpu().numpy(), dt[1:].cpu().numpy())


@pytest.mark.parametrize("level", [5, 6])
@pytest.mark.parametrize("form", [0, 1])
def test_per_oct_default_shape(level, form):
    """The per-oct kernel as the library shapes it by form and number of octs
    (32768 octs, mixed: three octs to 128 threads, the last workgroup two)
    against four octs to 256 threads: the same bits."""
    from paper_2607_20704_amd import api
    D = api.DeviceTree(I.uniform_tree(level), I.OUTFLOW)
    u = _state(D, 1.4, 60 + level)
    want, dt = _step(D, u, 1.4, form, PER_OCT)
    got, d = _step(D, u, 1.4, form, (0, 0, 1))
    assert torch.equal(got, want) and torch.equal(d, dt)
