"""Re-keying of octs that are out of order (RG_STEP_REKEY): keys, permutation
and level ranges against a stable sort of the encoded keys, at the edges of the
sort's tiles (1024 and 2048 keys), groups of 64 tiles and parts of a tile, for
both digit widths; and its time beside the library sort that rg_sort_keys
runs."""
import ctypes
import statistics

import numpy as np
import pytest
import torch

from gpu_common import say

pytestmark = pytest.mark.gpu


def _octs(n, lmax, lmin=1, seed=0):
    """n distinct octs' worth of random coordinates of levels lmin..lmax (some
    octs repeat: equal keys keep their order)."""
    rng = np.random.default_rng(seed)
    l = rng.integers(lmin, lmax + 1, n)
    side = (1 << (l - 1))[:, None]
    xyz = (rng.random((n, 3)) * side).astype(np.int64)
    return torch.as_tensor(np.concatenate([xyz, l[:, None]], 1).astype(np.int32)).to("cuda").contiguous()


class _Rekey:
    def __init__(self, n, lmax):
        from paper_2607_20704_amd import api
        self.L = api.L
        lib = api.L.lib()
        self.keys = torch.empty(n, dtype=torch.uint64, device="cuda")
        self.scratch = torch.empty_like(self.keys)
        self.perm = torch.empty(n, dtype=torch.int32, device="cuda")
        self.ws = torch.empty(lib.rg_sort_workspace_bytes(n), dtype=torch.uint8, device="cuda")
        self.begin = torch.empty(api.RG_MAX_LEVEL + 2, dtype=torch.int64, device="cuda")
        t = self.t = api.L.RgTree()
        t.n_oct, t.lmin, t.lmax = n, 1, lmax
        t.d_keys, t.d_keys_scratch, t.d_perm = self.keys.data_ptr(), self.scratch.data_ptr(), self.perm.data_ptr()
        t.d_sort_ws, t.sort_ws_bytes, t.d_level_begin = self.ws.data_ptr(), self.ws.numel(), self.begin.data_ptr()

    def __call__(self, ijkl):
        self.t.d_ijkl = ijkl.data_ptr()
        self.L.check(self.L.lib().rg_prepare_tree(ctypes.byref(self.t), self.L.RG_STEP_REKEY,
                                                  torch.cuda.current_stream().cuda_stream))


# (octs, finest level): one tile and less; 64 tiles of 1024 keys, one more, one
# less; the change to tiles of 2048; a group of 64 of those; two parts a tile
SIZES = [(1, 3), (2, 21), (255, 6), (256, 9), (1023, 8), (1025, 7), (65535, 8), (65536, 9), (65537, 21),
         (524288, 8), (524289, 9), (655361, 10), (8388609, 9)]


@pytest.mark.parametrize("n,lmax", SIZES)
def test_octs_out_of_order(n, lmax):
    from paper_2607_20704_amd import api
    ijkl = _octs(n, lmax, seed=n)
    say("rekey:", n, "octs, levels 1 ..", lmax)
    R = _Rekey(n, lmax)
    keys = api.encode_keys(ijkl).view(torch.int64)
    ref, perm = torch.sort(keys, stable=True)
    for again in range(2):   # the second call finds the first one's counts in the workspace
        R(ijkl)
        assert torch.equal(R.keys.view(torch.int64), ref)
        assert torch.equal(R.perm.long(), perm)
        assert torch.equal(R.begin, api.level_ranges(ref.view(torch.uint64)))
    # in order, and in order but for the last pair
    ordered = ijkl[perm].contiguous()
    R(ordered)
    assert torch.equal(R.keys.view(torch.int64), ref)
    assert torch.equal(R.perm.long(), torch.arange(n, device="cuda"))
    if n > 2 and int(ref[-1]) != int(ref[-2]):
        ordered[[n - 2, n - 1]] = ordered[[n - 1, n - 2]]
        R(ordered.contiguous())
        assert torch.equal(R.keys.view(torch.int64), ref)
        assert R.perm[-2:].tolist() == [n - 1, n - 2]


def _us(f):
    for _ in range(3):
        f()
    t = []
    for _ in range(11):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        f()
        b.record()
        b.synchronize()
        t.append(1e3 * a.elapsed_time(b))
    return statistics.median(t)


@pytest.mark.parametrize("n,level", [(1 << 21, 8), (1 << 24, 9)])
def test_sorting_costs_no_more_than_the_library(n, level):
    """What octs in random order cost beyond octs in order, beside the library's
    passes over as many bits (rg_sort_keys sorts 64 bits, 8 a pass).  Bound: a
    tenth above the library."""
    from paper_2607_20704_amd import api
    ijkl = _octs(n, level, level, seed=3)
    keys = api.encode_keys(ijkl)
    order = torch.sort(keys.view(torch.int64), stable=True)[1]
    ordered = ijkl[order].contiguous()
    R = _Rekey(n, level)
    extra = _us(lambda: R(ijkl)) - _us(lambda: R(ordered))
    passes = (3 * level + 7) // 8
    library = _us(lambda: api.sort_keys(keys)) * passes / 8
    say("random order: %d octs, %.0f us beyond octs in order, library's %d passes %.0f us" %
        (n, extra, passes, library))
    assert extra <= 1.1 * library
