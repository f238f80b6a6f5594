"""rg_step and rg_refine refuse bad trees on the host: every call here returns
RG_EINVAL before anything is enqueued (pointers are made-up addresses, so a
call that went on would end in a launch)."""
import ctypes

import pytest

from paper_2607_20704_amd import _lib as L

FLAGS = [0, L.RG_STEP_CHAIN_DT]


def _tree(lmax=3):
    t = L.RgTree()
    t.n_oct, t.lmin, t.lmax = (72, 2, 3) if lmax == 3 else (8, 2, 2)
    t.level_begin[2], t.level_begin[3], t.level_begin[4] = 0, 8, 72
    t.d_keys, t.d_nbr27, t.d_father_cell, t.d_son_mask, t.d_corr = 256, 512, 768, 1024, 1280
    return t


def _step(t, u=4096, unew=8192, form=0, flags=0, dt=2048):
    return L.lib().rg_step(ctypes.byref(t), u, unew, 1.4, 0.8, form, flags, dt, None, None)


@pytest.mark.parametrize("flags", FLAGS)
@pytest.mark.parametrize("lmax", [2, 3])
@pytest.mark.parametrize("missing", ["d_nbr27", "d_son_mask"])
def test_step_without_schedule_needs_the_lists(missing, lmax, flags):
    t = _tree(lmax)
    setattr(t, missing, None)
    assert _step(t, flags=flags) == L.RG_EINVAL


@pytest.mark.parametrize("flags", FLAGS)
@pytest.mark.parametrize("bad", [{"u": 4100}, {"unew": 8196}, {"dt": 2052}, {"u": 8192}, {"form": 7}])
def test_step_without_schedule_refuses_bad_buffers(bad, flags):
    assert _step(_tree(), flags=flags, **bad) == L.RG_EINVAL


@pytest.mark.parametrize("flags", FLAGS)
def test_step_without_schedule_refuses_bad_level_ranges(flags):
    t = _tree()
    t.level_begin[3] = 80          # level 3 would end before it begins
    assert _step(t, flags=flags) == L.RG_EINVAL
    t = _tree()
    t.n_oct = t.level_begin[4] = (1 << 28) + 8
    assert _step(t, flags=flags) == L.RG_EINVAL


@pytest.mark.parametrize("flags", FLAGS)
def test_step_with_schedule_refuses_bad_buffers(flags):
    t = _tree()
    sched = L.RgSchedule()
    t.sched = ctypes.pointer(sched)
    assert _step(t, flags=flags) == L.RG_EINVAL          # no list
    sched.d_list = 16384
    assert _step(t, dt=2052, flags=flags) == L.RG_EINVAL
    assert _step(t, u=8192, flags=flags) == L.RG_EINVAL
    assert _step(t, form=7, flags=flags) == L.RG_EINVAL


def _refine(**kw):
    lib = L.lib()
    t = _tree()
    t.capacity = 72
    t.d_hash_ws, t.hash_ws_bytes = 1 << 16, lib.rg_hash_workspace_bytes(72)
    t.d_sort_ws, t.sort_ws_bytes = 1 << 17, lib.rg_sort_workspace_bytes(72)
    t.d_ijkl, t.d_keys_scratch, t.d_perm, t.d_level_begin = 1 << 18, 1 << 19, 1 << 20, 1 << 21
    for k, v in kw.items():
        setattr(t, k, v)
    p = L.RgRefineParams()
    p.rho_thresh, p.lmax = 1.0, 4
    return lib.rg_refine(ctypes.byref(t), 1 << 22, 1 << 23, ctypes.byref(p), 1 << 24,
                         lib.rg_refine_workspace_bytes(72), None)


@pytest.mark.parametrize("bad", [{"d_keys": None}, {"d_keys_scratch": 256}, {"d_sort_ws": (1 << 17) + 8},
                                 {"d_keys_scratch": (1 << 19) + 4}, {"d_hash_ws": (1 << 16) + 8}])
def test_refine_refuses_bad_buffers(bad):
    """d_keys_scratch = 256 is d_keys: the new keys would be written over the
    ones they come from."""
    assert _refine(**bad) == L.RG_EINVAL
