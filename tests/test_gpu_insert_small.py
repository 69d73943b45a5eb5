"""The insert of small calls (up to 5 * 2^16 vertices): its workgroups grow at 192
of 128, 256, 512 and 1024 threads and merge vertices by key in LDS.  Table, flags,
counts and averages equal the oracle's bit for bit; a call whose vertices share
few cells must not wait for every vertex's own claim."""
import numpy as np
import pytest
import torch

import oracle
import paper_1902_05942_amd as pf
from gpu_util import check_frame_against_oracle, gpu_frame, table_contents, to_dev
from test_gpu_insert_windows import _insert_and_compare, _keys

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [127, 129, 192 * 128, 192 * 128 + 1, 192 * 256, 192 * 256 + 1, 192 * 512, 192 * 512 + 1, 192 * 1024,
                               192 * 1024 + 1, 5 << 16])
@pytest.mark.parametrize("distinct", [1, 3, 0])
def test_edges_of_workgroup_sizes(gpu, n, distinct):
    """All vertices in one cell, in three, and each in its own; one key has every
    bit set (the LDS table's mark of an empty entry)."""
    rng = np.random.default_rng(n + distinct)
    ids = np.arange(n) % distinct if distinct else rng.permutation(n)
    key = _keys(ids + 1)
    if distinct != 1:
        key[ids == 1] = ~np.uint64(0)
    _insert_and_compare(key, (rng.random((3, n)) * 300 - 150).astype(np.float32), max(10, int(2 * n).bit_length()))


def edge_frame(n, seed, s, m, probe=64):
    """Vertices of every kind side by side: valid and masked, non-finite positions
    and normals, positions beyond the key range, contributions that are not finite
    or out of range."""
    rng = np.random.default_rng(seed)
    f = {a: rng.random(n, dtype=np.float32) for a in ("px", "py", "pz", "r", "g", "b")}
    axis = rng.integers(0, 3, n)
    for a, c in enumerate(("nx", "ny", "nz")):
        f[c] = np.where(axis == a, rng.choice([-1.0, 1.0], n), 0.0).astype(np.float32)
    f["valid"] = (rng.random(n) < 0.9).astype(np.uint8)
    odd = rng.integers(0, 40, n)  # one vertex in 40 of each kind
    f["px"][odd == 0] = np.nan
    f["py"][odd == 1] = -np.inf
    f["nz"][odd == 2] = np.nan
    f["pz"][odd == 3] = 3.0e9  # level 15, yet more than 2^16 cells from the origin at cell size 0.01 and below
    f["r"][odd == 4] = np.inf
    f["g"][odd == 5] = np.nan
    f["b"][odd == 6] = 1.0e15
    f["r"][odd == 7] = -1.0e15
    f.update(cam=(0.5, 0.5, 4.0), s=s, seed=seed, log2_slots=m, max_probe=probe, frac_bits=24)
    return f


@pytest.mark.parametrize("n", [300, 192 * 256 + 1, 192 * 512 + 1, 192 * 1024 + 1, 5 << 16])
def test_flagged_vertices_beside_valid_ones(gpu, n):
    f = edge_frame(n, n, 0.01, 20)
    t = pf.Table(20)
    pf.table_init(t)
    R = oracle.filter_frame(f, temporal=False)
    assert {0, pf.V_INVALID, pf.V_KEYRANGE, pf.V_RADRANGE} <= set(np.unique(R.flags))
    for agg in ("fused", "binned"):
        check_frame_against_oracle(gpu_frame(f, to_dev(f), t, agg=agg), R, t)


def us(call, before, reps=9):
    """Median time of a call on the GPU."""
    out = []
    for _ in range(reps + 2):
        before()
        e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
        e[0].record()
        call()
        e[1].record()
        e[1].synchronize()
        out.append(e[0].elapsed_time(e[1]) * 1e3)
    return sorted(out[2:])[reps // 2]


def times_of_cells(n, m, cells, insert):
    t = pf.Table(m)
    pf.table_init(t)
    k = torch.from_numpy(_keys(np.arange(n) % cells + 1).view(np.int64)).cuda()
    c = torch.ones(n, device="cuda")
    fl = torch.zeros(n, dtype=torch.uint8, device="cuda")
    slot = torch.empty(n, dtype=torch.int32, device="cuda")
    ws = torch.empty(pf.insert_workspace_bytes(n, m), dtype=torch.uint8, device="cuda")
    return us(lambda: insert(t, k, c, fl, slot, ws), lambda: pf.clear(t))


@pytest.mark.parametrize("n", [50000, 300000])
def test_binned_insert_of_one_cell_is_not_slow(gpu, n):
    """It has a thousandth of the claims and of the memory traffic of a call whose
    vertices all have cells of their own; three times that call's time leaves room
    for the adds to one address (a claim by every vertex took twenty times)."""
    def insert(t, k, c, fl, slot, ws):
        pf.insert_accumulate_binned(t, k, c, c, c, fl, slot, ws)

    one, many = (times_of_cells(n, 20, cells, insert) for cells in (1, n))
    print(f"{n} vertices: one cell {one:.1f} us, each its own {many:.1f} us", flush=True)
    assert one < 3 * many


@pytest.mark.parametrize("n", [50000, 300000])
def test_atomic_insert_of_one_cell_is_not_slow(gpu, n):
    """As above for the insert by device atomics, 64 lanes combined."""
    def insert(t, k, c, fl, slot, ws):
        pf.insert_accumulate(t, k, c, c, c, fl, slot, 64)

    one, many = (times_of_cells(n, 20, cells, insert) for cells in (1, n))
    print(f"{n} vertices: one cell {one:.1f} us, each its own {many:.1f} us", flush=True)
    assert one < 3 * many


@pytest.mark.parametrize("agg", [0, 64])
@pytest.mark.parametrize("n,run", [(1, 1), (64, 64), (65, 5), (130, 63), (1000, 64), (4097, 200)])
def test_atomic_insert_of_runs(gpu, agg, n, run):
    """Neighbouring vertices with the same key claim once: runs within, across and
    around wavefronts, cut by flagged vertices."""
    ids = np.arange(n) // run
    key = _keys(ids + 1)
    flags = (np.arange(n) % 11 == 3).astype(np.uint8)
    t = pf.Table(13, 64)
    pf.table_init(t)
    fl, slot = torch.from_numpy(flags).cuda(), torch.empty(n, dtype=torch.int32, device="cuda")
    c = torch.from_numpy((np.arange(n) % 100 - 50).astype(np.float32)).cuda()
    pf.insert_accumulate(t, torch.from_numpy(key.view(np.int64)).cuda(), c, c, c, fl, slot, agg)
    live = flags == 0
    assert np.array_equal(fl.cpu().numpy(), flags)
    cells, counts = np.unique(key[live], return_counts=True)
    tc = table_contents(t)
    order = np.argsort(tc["key"])
    assert np.array_equal(tc["key"][order], cells) and np.array_equal(tc["count"][order], counts)
    at = slot.cpu().numpy()
    assert (at[~live] == -1).all() and np.array_equal(t.keys().cpu().numpy().view(np.uint64)[at[live]], key[live])
    want = [int((np.arange(n)[live & (key == k)] % 100 - 50).sum()) << 24 for k in cells]
    assert np.array_equal(tc["sum"][order][:, 0], np.array(want, np.int64))
