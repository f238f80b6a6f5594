"""The one-pass coarse-fine corrections of a step against the six passes and
the oracle, on trees where a coarse cell is bordered by fine octs on any set
of its six sides: cells split at random (opposite sides, all six, across the
periodic boundary, down to a coarse level of two octs a side), with and
without a schedule, single steps, chained time steps and subcycling."""
import numpy as np
import pytest
import torch

from gpu_common import parity_metric
from oracle import oracle as O
from paper_2607_20704_amd import inputs as I

pytestmark = pytest.mark.gpu


def random_tree(base, lmax, share, bc, seed):
    rng = np.random.default_rng(seed)
    drawn = {}

    def flag(l, cen):
        key = np.round(cen * (1 << l) - 0.5).astype(np.int64)
        out = np.empty(len(key), bool)
        for n, k in enumerate(map(tuple, key)):
            if (l, k) not in drawn:
                drawn[(l, k)] = rng.random() < share
            out[n] = drawn[(l, k)]
        return out

    return I.refined_tree(base, lmax, flag, bc)


def sides_of(T):
    """Per coarse leaf cell with any: the set of sides it receives, as bits."""
    got = {}
    slots = [12, 14, 10, 16, 4, 22]
    for o in range(int(T.level_begin[T.lmin + 1]), T.n):
        for s in range(6):
            e = T.nbr27[o, slots[s]]
            if e < 0 and e != -(1 << 31):
                got[-1 - e] = got.get(-1 - e, 0) | 1 << s
    return got


@pytest.mark.parametrize("base,lmax,share,bc,seed", [
    (1, 2, 0.5, I.PERIODIC, 1), (2, 3, 0.5, I.PERIODIC, 2), (3, 5, 0.4, I.PERIODIC, 3), (3, 4, 0.8, I.OUTFLOW, 4),
    (4, 6, 0.02, I.PERIODIC, 5), (4, 5, 0.9, I.PERIODIC, 6)])
@pytest.mark.parametrize("schedule", [True, False])
def test_one_pass_corrections(base, lmax, share, bc, seed, schedule):
    from paper_2607_20704_amd import api
    ijkl = random_tree(base, lmax, share, bc, seed)
    T = O.Tree(ijkl, bc)
    D = api.DeviceTree(ijkl, bc, schedule=schedule)
    if share in (0.8, 0.9):
        bits = set(sides_of(T).values())
        assert any(b & 3 == 3 or b & 12 == 12 or b & 48 == 48 for b in bits) and any(bin(b).count("1") >= 4 for b in bits)
    gam = 1.4
    rng = np.random.default_rng(seed)
    n = 8 * T.n
    rho = np.exp(0.3 * rng.standard_normal(n))
    vel = 0.4 * rng.standard_normal((3, n))
    u0 = I.fill_split_cells(T.ijkl, I.conserved(rho, *vel, np.exp(0.3 * rng.standard_normal(n)), gam).reshape(-1, 5))
    u = torch.as_tensor(u0).cuda()
    dts = torch.zeros(2, dtype=torch.float64, device="cuda")
    api.cfl_dt(u, D.son_mask, D.level_begin, D.lmin, D.lmax, gam, 0.8, dts[:1])
    one = torch.empty_like(u)
    D.step(u, one, gam, 0.8, dt=dts, chain=True)
    # the same step from its parts, six passes over all octs
    six = torch.empty_like(u)
    nxt = torch.full((1,), float("inf"), dtype=torch.float64, device="cuda")
    for l in range(D.lmin, D.lmax + 1):
        D.hydro_level(l, dts[:1], gam, u, six, cfl=0.8, dt_next=nxt)
    if D.lmax > D.lmin:
        api.apply_coarse_corrections(six, D.corr, D.corr_base, D.nbr27, D.corr_base, D.n)
        api.cfl_dt_corrected(six, D.nbr27, D.level_begin, D.lmin, D.lmax, gam, 0.8, nxt)
        for l in range(D.lmax, D.lmin, -1):
            api.restrict_level(six, D.father_cell, int(D.level_begin[l]), int(D.level_begin[l + 1]))
    assert torch.equal(one, six)
    assert torch.equal(dts[1:], nxt)
    ref = u0.copy()
    T.run(ref, gam, 0.8, 1)
    assert parity_metric(one.cpu().numpy(), ref)[0] <= 1e-12
    sub, _ = D.run_subcycled(u, gam, 0.8, 1)
    ref = u0.copy()
    T.run_subcycled(ref, gam, 0.8, 1)
    assert parity_metric(sub.cpu().numpy(), ref)[0] <= 1e-12
