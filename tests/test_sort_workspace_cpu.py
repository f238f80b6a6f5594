"""rg_sort_workspace_bytes never falls: a workspace sized for a tree's capacity
serves every smaller tree.  At the sizes where the sort of a re-keyed step
changes its tiles (2^19 keys; 2^23, 2^24 ... keys: parts of a tile)."""
from paper_2607_20704_amd import _lib as L


def test_workspace_grows_with_the_keys():
    f = L.lib().rg_sort_workspace_bytes
    at = [0, 1, 2, 63, 64, 65, 255, 256, 257, 1000, 5000]
    at += [(k << 10) + d for k in range(1, 515) for d in (-1, 0, 1)]
    at += [(1 << k) + d for k in range(12, 31) for d in (-1, 0, 1)] + [3 << 23, (3 << 23) + 1, 2 ** 31 - 1]
    at = sorted(set(at))
    size = [f(n) for n in at]
    assert [(a, b) for a, b, s, t in zip(at, at[1:], size, size[1:]) if t < s] == []
