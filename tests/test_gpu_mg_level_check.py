"""A level hierarchy used with a tree whose octs have changed: refused where
the counts differ, recorded as RG_EINVAL where they do not."""
import numpy as np
import pytest
import torch

from gpu_common import say
from paper_2607_20704_amd import inputs as I

pytestmark = pytest.mark.gpu


def _shift(ijkl, base):
    """The tree moved by one base-level oct along x (periodic): the same counts
    on every level, other octs above the base."""
    out = ijkl.copy()
    l = out[:, 3]
    out[:, 0] = (out[:, 0] + (1 << (l - base))) & ((1 << (l - 1)) - 1)
    return np.ascontiguousarray(out)


def test_changed_octs_are_reported():
    from paper_2607_20704_amd import api
    base, lmax = 4, 6
    ijkl = I.sphere_tree(base, lmax, (0.4, 0.55, 0.5), 0.16, I.PERIODIC)
    A = api.DeviceTree(ijkl, I.PERIODIC)
    B = api.DeviceTree(_shift(ijkl, base), I.PERIODIC)
    assert np.array_equal(A.level_begin, B.level_begin)
    f = torch.randn(8 * A.n, dtype=torch.float64, device="cuda")
    f[:8 * int(A.level_begin[base + 1])] -= f[:8 * int(A.level_begin[base + 1])].mean()
    phi = torch.zeros_like(f)
    api.check_ws(None)
    for l in range(base, lmax + 1):
        H = api.MgLevel(A, l)
        H.vcycles(phi, f, 1)
        assert api.check_ws(None)[0] == api.L.RG_OK, l
        H.tree = B
        H.vcycles(phi, f, 1)
        st, bad = api.check_ws(None)
        say("level multigrid, moved tree, level", l, "status", st, "oct", bad)
        if l == base:
            assert st == api.L.RG_OK     # complete: its octs are the same
        else:
            assert st == api.L.RG_EINVAL
            assert int(B.level_begin[l]) <= bad < int(B.level_begin[l + 1])
            assert int(A.keys.view(torch.int64)[bad]) != int(B.keys.view(torch.int64)[bad])
        H.tree = api.DeviceTree(I.sphere_tree(base, lmax, (0.4, 0.55, 0.5), 0.2, I.PERIODIC), I.PERIODIC)
        with pytest.raises(api.RgError):
            H.vcycles(phi, f, 1)
        H.close()
