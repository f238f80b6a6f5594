"""The level hierarchy's build: octs per level against the parents of the level's
octs, for levels of less than one and of several workgroups of faces, with and
without coarse levels."""
import numpy as np
import pytest

from gpu_common import say
from paper_2607_20704_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("base,lmax,radius,lcoarse", [(2, 3, 0.2, 1), (4, 6, 0.16, 1), (4, 6, 0.16, 4), (5, 8, 0.12, 2),
                                                      (3, 5, 0.3, 5)])
def test_hierarchy_counts(base, lmax, radius, lcoarse):
    from paper_2607_20704_amd import api
    D = api.DeviceTree(I.sphere_tree(base, lmax, (0.4, 0.55, 0.5), radius, I.PERIODIC), I.PERIODIC)
    keys = D.keys.cpu().numpy()
    for l in range(max(base, lcoarse), lmax + 1):
        octs = keys[int(D.level_begin[l]):int(D.level_begin[l + 1])]
        want = {l: len(octs)}
        for m in range(l - 1, lcoarse - 1, -1):
            octs = np.unique(octs >> np.uint64(3))
            want[m] = len(octs)
        H = api.MgLevel(D, l, lcoarse)
        say("hierarchy of level", l, "down to", lcoarse, want)
        assert H.counts() == want
        H.close()
