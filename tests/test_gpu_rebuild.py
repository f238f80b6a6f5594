"""The rebuild of a tree on the device at the sizes where its pieces meet,
bit for bit against the oracle: neighbour lists of short lists (octs one by
one) and, in a batch and in long lists, by sibling groups; schedules; refined
trees whose flags leave any subset of an oct's cells, states and coordinates at
any alignment their types allow; keys of octs in any order."""
import numpy as np
import pytest
import torch

from gpu_common import say
from oracle import oracle as O
from paper_2607_20704_amd import inputs as I

pytestmark = pytest.mark.gpu


def _holed(base, lmax, bc, seed):
    """A graded tree whose finest level lacks about a third of its octs: groups
    of one to eight octs, complete ones at every offset of a 64-entry chunk."""
    ijkl = I.sphere_tree(base, lmax, (0.3, 0.45, 0.6), 0.2, bc)
    drop = (ijkl[:, 3] == lmax) & (np.random.default_rng(seed).random(len(ijkl)) < 0.06)
    return np.ascontiguousarray(ijkl[~drop])


TREES = [
    ("one_oct", lambda: I.uniform_tree(1), I.PERIODIC),
    ("two_per_side_periodic", lambda: I.uniform_tree(2), I.PERIODIC),
    ("two_per_side_walls", lambda: I.uniform_tree(2), I.OUTFLOW),
    ("levels_1_3", lambda: np.concatenate([I.uniform_tree(1), I.uniform_tree(2), I.uniform_tree(3)]), I.PERIODIC),
    ("levels_2_4_walls", lambda: np.concatenate([I.uniform_tree(l) for l in (2, 3, 4)]), I.OUTFLOW),
    ("holes_3_5", lambda: _holed(3, 5, I.PERIODIC, 5), I.PERIODIC),
    ("holes_3_6_walls", lambda: _holed(3, 6, I.OUTFLOW, 6), I.OUTFLOW),
    ("holes_4_8", lambda: _holed(4, 8, I.PERIODIC, 7), I.PERIODIC),   # > 40000 octs outside bricks
]


def _tree(name):
    mk, bc = next((t[1], t[2]) for t in TREES if t[0] == name)
    return np.ascontiguousarray(mk(), dtype=np.int32), bc


def _check_lists(D, T):
    from paper_2607_20704_amd import api
    assert api.check_ws(D.hash_ws)[0] == 0
    assert np.array_equal(D.nbr27.cpu().numpy(), T.nbr27)
    assert np.array_equal(D.father_cell.cpu().numpy(), T.father_cell)
    assert np.array_equal(D.son_mask.cpu().numpy(), T.son_mask.astype(np.int32))


@pytest.mark.parametrize("schedule", [False, True])
@pytest.mark.parametrize("name", [t[0] for t in TREES])
def test_neighbour_lists(name, schedule):
    from paper_2607_20704_amd import api
    ijkl, bc = _tree(name)
    T = O.Tree(ijkl, bc)
    D = api.DeviceTree(ijkl, bc, schedule=schedule)
    say("neighbours:", name, len(ijkl), "outside bricks", D.sched.nbr_rest_count if schedule else D.n)
    for again in (False, True):
        if again:
            for x in (D.nbr27, D.father_cell, D.son_mask):
                x.fill_(-7)
            D.prepare()
        _check_lists(D, T)


def test_neighbour_lists_of_a_batch():
    from paper_2607_20704_amd import api
    trees = [_tree(t[0]) for t in TREES]
    D = [api.DeviceTree(*t) for t in trees]
    u = []
    for d in D:
        x = torch.ones((8 * d.n, 5), dtype=torch.float64, device="cuda")
        x[:, 4] = 2.5
        u.append(x)
    B = api.Batch(D, u, [1.4] * len(D), [0.8] * len(D), 1, rebuild=True)
    for d in D:
        for x in (d.nbr27, d.father_cell, d.son_mask):
            x.fill_(-7)
    B.run()
    torch.cuda.synchronize()
    for d, t in zip(D, trees):
        say("batch:", len(t[0]))
        _check_lists(d, O.Tree(*t))
    B.close()


@pytest.mark.parametrize("name", [t[0] for t in TREES])
def test_device_schedule_equals_host(name):
    from paper_2607_20704_amd import api
    D = api.DeviceTree(*_tree(name))
    dev = D.schedule_lists()
    D.build_schedule(on_host=True)
    host = D.schedule_lists()
    say("schedule:", name, D.schedule_counts())
    assert dev.keys() == host.keys()
    for k in dev:
        for a, b in zip(dev[k], host[k]):
            assert np.array_equal(a, b), (name, k)


@pytest.mark.parametrize("odd", [False, True])
@pytest.mark.parametrize("share", [0.02, 0.3, 1.0])
@pytest.mark.parametrize("name", [t[0] for t in TREES[1:-1]])
def test_refine(name, share, odd):
    """A share of the cells above the density threshold, in no order; odd: both
    states 8 bytes and the coordinates 4 bytes past a 16-byte boundary."""
    from paper_2607_20704_amd import api
    ijkl, bc = _tree(name)
    T = O.Tree(ijkl, bc)
    rng = np.random.default_rng(len(ijkl))
    ref = rng.random((8 * T.n, 5)) + 0.5
    ref[:, 0] = np.where(rng.random(8 * T.n) < share, 2.0, 1.0) * (0.9 + 0.2 * rng.random(8 * T.n))
    lmax = min(T.lmax + 1, 6)
    _, ni, nu = T.refine(ref, 1.5, 0.0, lmax)
    T2 = O.Tree(ni, bc)
    say("refine:", name, T.n, "->", T2.n)
    D = api.DeviceTree(ijkl, bc, capacity=9 * T.n)
    shift = 1 if odd else 0
    u = torch.empty(40 * D.capacity + 1, dtype=torch.float64, device="cuda")[shift:shift + 40 * T.n].view(-1, 5)
    out = torch.empty(40 * D.capacity + 1, dtype=torch.float64, device="cuda")[shift:shift + 40 * D.capacity]
    u.copy_(torch.as_tensor(ref))
    if odd:
        buf = torch.empty(4 * D.capacity + 1, dtype=torch.int32, device="cuda")[1:].view(-1, 4)
        buf[:D.n] = D.ijkl_sorted
        D._ijkl = buf
        D._desc.d_ijkl = buf.data_ptr()
    got = D.refine(u, 1.5, 0.0, lmax, out=out.view(-1, 5))
    torch.cuda.synchronize()
    assert D.n == T2.n and np.array_equal(D.keys.cpu().numpy(), T2.keys)
    assert np.array_equal(D.ijkl_sorted.cpu().numpy(), T2.ijkl)
    assert [int(x) for x in D.level_begin] == [int(x) for x in D.level_begin_dev.cpu()]
    assert all(int(D.level_begin[l]) == T2.level_begin[l] for l in range(T2.lmin, T2.lmax + 2))
    assert np.array_equal(got.cpu().numpy(), T2.permute_cells(nu))
    _check_lists(D, T2)


@pytest.mark.parametrize("how", ["sorted", "one_swap", "repeats", "shuffled"])
@pytest.mark.parametrize("level", [1, 2, 5, 6, 7, 8, 9])
def test_rekey(level, how):
    """Keys and places of octs in any order: one tile of 1024 keys and
    several, whole and in part (of 4096 beyond 524288 keys, of two parts
    beyond 2097152), one to three passes of 8 bits, equal keys in
    the order they came."""
    from paper_2607_20704_amd import api, _lib as L
    if level == 7:   # 4096-key tiles: complete levels 6 and 7 and a part of level 8
        ijkl = np.concatenate([I.uniform_tree(6), I.uniform_tree(7), I.uniform_tree(8)[:8 * 40001]])
    elif level == 9:
        ijkl = np.concatenate([I.uniform_tree(8), I.uniform_tree(9)[:8 * 1001]])
    else:
        ijkl = _tree("holes_4_8")[0] if level == 8 else I.uniform_tree(level)
    D = api.DeviceTree(ijkl, I.PERIODIC)
    rng = np.random.default_rng(level)
    c = D.ijkl_sorted.cpu().numpy()
    if how == "one_swap" and D.n > 1:
        at = min(254, D.n - 2)   # the last key of one workgroup's stretch and the first of the next
        c[[at, at + 1]] = c[[at + 1, at]]
    elif how == "repeats":
        c = c[rng.integers(0, D.n, D.n)]
    elif how == "shuffled":
        c = c[rng.permutation(D.n)]
    D._ijkl[:D.n] = torch.as_tensor(np.ascontiguousarray(c))
    want = O.keys(c)
    order = np.argsort(want, kind="stable")
    for _ in range(2):
        D.keys.view(torch.int64).fill_(-1)
        D.perm_scratch.fill_(-1)
        D.prepare(L.RG_STEP_REKEY)
        torch.cuda.synchronize()
        assert np.array_equal(D.keys_scratch[:D.n].cpu().numpy(), want)
        assert np.array_equal(D.keys.cpu().numpy(), want[order])
        assert np.array_equal(D.perm_scratch[:D.n].cpu().numpy(), order)


def test_ungraded_group_is_reported():
    """A complete sibling group on level 9 whose outside neighbours exist
    neither there nor on level 8, behind enough octs for the lists to go by
    groups: reported, naming an oct of the group."""
    from paper_2607_20704_amd import api, _lib as L

    def group(at, level):
        return np.array([[at + i, at + j, at + k, level] for i in range(2) for j in range(2) for k in range(2)])

    tree = np.concatenate([I.uniform_tree(7), group(64, 8), group(128, 9)]).astype(np.int32)
    tree = tree[O.tree_order(tree)]
    st_o, bad_o, *_ = O.neighbours(tree, I.PERIODIC)
    keys = torch.as_tensor(O.keys(tree).astype(np.int64)).cuda().view(torch.uint64)
    ws = api.hash_build(keys)
    api.build_neighbours(ws, keys, 7, I.PERIODIC)
    st, bad = api.check_ws(ws)
    say("ungraded group: oct named", bad, "by the oracle", bad_o)
    assert st == L.RG_EUNGRADED == st_o
    assert tree[bad, 3] == 9


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("n", [1, 262144, 262145])
def test_hash_table(n, noalloc):
    """Tables on either side of the size from which segments are built in LDS:
    every key found at its index, others absent, a repeated key reported."""
    from paper_2607_20704_amd import api, _lib as L
    ijkl = np.concatenate([I.uniform_tree(7), [[0, 0, 0, 8]]]).astype(np.int32)[:n]
    hk = O.keys(ijkl).astype(np.int64)
    keys = torch.as_tensor(hk).cuda().view(torch.uint64)

    def build(k):
        if not noalloc:
            return api.hash_build(k)
        table = torch.empty(api.hash_workspace_bytes(n), dtype=torch.uint8, device="cuda")
        api.hash_build_noalloc(k, table)
        return table

    ws = build(keys)
    assert api.check_ws(ws) == (L.RG_OK, -1)
    assert np.array_equal(api.hash_lookup(ws, keys).cpu().numpy(), np.arange(n))
    absent = torch.as_tensor(np.concatenate([8 * hk + 7, [0]])).cuda().view(torch.uint64)
    assert np.all(api.hash_lookup(ws, absent).cpu().numpy() == -1)
    if n > 1:
        hk[n // 2] = hk[5]
        st, bad = api.check_ws(build(torch.as_tensor(hk).cuda().view(torch.uint64)))
        assert st == L.RG_EDUPKEY and bad in (5, n // 2)
