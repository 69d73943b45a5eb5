"""The binned insert where its windows, buckets and bins have their edges: the
size up to which a call is one launch, steps of 1024 vertices, windows that fill the LDS table, groups whose count or sums
need more than one record, a bucket that runs full (its groups then go to their
cells by device atomics) and bins of more cells than one pass sums.  All sums are
integers: table, averages and counts equal the oracle's group-by bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_1902_05942_amd as pf
from gpu_util import assert_bits_equal, table_contents

pytestmark = pytest.mark.gpu


def _insert_and_compare(key, rgb, m, frac_bits=24, agg=None):
    n = key.size
    probe = min(64, 1 << m)
    R = oracle.filter_keys(key, rgb[0], rgb[1], rgb[2], np.ones(n, np.uint8), m, probe, frac_bits)
    t = pf.Table(m, probe, frac_bits)
    pf.table_init(t)
    k = torch.from_numpy(key.view(np.int64)).cuda()
    r, g, b = (torch.from_numpy(x).cuda() for x in rgb)
    fl = torch.zeros(n, dtype=torch.uint8, device="cuda")
    slot = torch.empty(n, dtype=torch.int32, device="cuda")
    cnt = torch.empty(n, dtype=torch.int32, device="cuda")
    ws = torch.empty(pf.insert_workspace_bytes(n, m), dtype=torch.uint8, device="cuda")
    out = [torch.empty(n, device="cuda") for _ in range(3)]
    if agg is None:
        pf.insert_accumulate_binned(t, k, r, g, b, fl, slot, ws)
    else:
        slot = slot if agg else None
        pf.insert_accumulate(t, k, r, g, b, fl, slot, agg)
    pf.query_average(t, k, slot, r, g, b, fl, False, *out, cnt)
    torch.cuda.synchronize()
    assert R.table.order_free and not R.flags.any()
    assert_bits_equal(fl.cpu().numpy(), R.flags, "flags")
    assert_bits_equal(cnt.cpu().numpy().view(np.uint32), R.cnt, "count")
    assert_bits_equal(np.stack([o.cpu().numpy() for o in out], 1), R.out, "average")
    tc = table_contents(t)
    order = np.argsort(tc["key"])
    assert_bits_equal(tc["key"][order], R.gkey, "table keys")
    assert_bits_equal(tc["count"][order], R.gcnt, "table counts")
    assert_bits_equal(tc["sum"][order], R.gsum, "table sums")
    assert_bits_equal(tc["occupied"], R.table.occupied, "occupied slots")
    bits = np.unpackbits(t.occupancy().cpu().numpy().view(np.uint8), bitorder="little")[:1 << m]
    assert_bits_equal(bits, R.table.occupied, "occupancy bitmap")


def _keys(ids):
    return ids.astype(np.uint64) * np.uint64(2654435761)


@pytest.mark.parametrize("n,distinct,m", [
    (1, 1, 4), (63, 9, 5), (1023, 1023, 12), (1024, 1, 4), (1025, 700, 12), (4097, 4097, 14), (5000, 3, 6),
    (64 * 1024, 30000, 17), (5 << 16, 60000, 18), ((5 << 16) + 1, (5 << 16) + 1, 20), (330001, 3, 6), (350000, 1, 4),
    (512 * 1024, 512 * 1024, 20), (525000, 1793, 17), (1 << 21, 900000, 22)])
def test_edges_of_steps_windows_and_bins(gpu, n, distinct, m):
    rng = np.random.default_rng(n + m)
    ids = np.concatenate([np.arange(distinct), rng.integers(0, distinct, n - distinct)])
    rng.shuffle(ids)
    _insert_and_compare(_keys(ids), rng.random((3, n), dtype=np.float32), m)


@pytest.mark.parametrize("frac_bits,scale,per", [
    (40, 900.0, 1),        # every sum needs its high part
    (24, 150.0, 65),       # counts on both sides of 64, some sums beyond 2^31
    (24, -150.0, 64),
    (8, 1.0e13, 2000),     # sums near the top of 64 bits
    (24, 1.0, 4096)])      # one cell for a whole window
def test_groups_of_more_than_one_record(gpu, frac_bits, scale, per):
    n = 330000
    rng = np.random.default_rng(per)
    rgb = (rng.random((3, n), dtype=np.float32) * np.float32(scale)).astype(np.float32)
    rgb[1] = -rgb[1]
    _insert_and_compare(_keys(np.arange(n) // per), rgb, 20, frac_bits)


def test_full_bucket_and_several_passes(gpu):
    # every home slot lies in one 256th of the table: that bin's buckets run
    # full, and it holds more cells than are summed in one pass
    m, cells, n = 22, 5000, 1 << 20
    cand = _keys(np.arange(1, 3000000))
    home, _ = oracle.key_hashes(cand, m)
    chosen = cand[(home >> np.uint32(m - 8)) == 17][:cells]
    assert len(chosen) == cells
    rng = np.random.default_rng(3)
    _insert_and_compare(chosen[rng.integers(0, cells, n)], rng.random((3, n), dtype=np.float32), m)


@pytest.mark.parametrize("n,distinct,m,agg", [
    ((1 << 19) - 1, 1, 4, 64), (1 << 19, 1, 4, 64), (1 << 19, 200000, 20, 0), ((1 << 19) + 77, 1793, 17, 256)])
def test_atomic_insert_by_windows(gpu, n, distinct, m, agg):
    """The insert by device atomics on both sides of the size from which it
    merges by windows; among its keys one with every bit set."""
    rng = np.random.default_rng(n)
    ids = np.concatenate([np.arange(distinct), rng.integers(0, distinct, n - distinct)])
    rng.shuffle(ids)
    key = _keys(ids)
    key[ids == 0] = ~np.uint64(0)
    _insert_and_compare(key, rng.random((3, n), dtype=np.float32) - np.float32(0.5), m, agg=agg)


def test_atomic_insert_by_windows_overflows(gpu):
    # 16 slots, 2 probes, 40 keys: whole groups overflow, and every vertex of a
    # placed key is counted
    n = 1 << 19
    key = _keys(np.arange(n) % 40)
    t = pf.Table(4, 2)
    pf.table_init(t)
    k = torch.from_numpy(key.view(np.int64)).cuda()
    r = torch.ones(n, device="cuda")
    fl = torch.zeros(n, dtype=torch.uint8, device="cuda")
    slot = torch.empty(n, dtype=torch.int32, device="cuda")
    pf.insert_accumulate(t, k, r, r, r, fl, slot, 64)
    torch.cuda.synchronize()
    flags, slots = fl.cpu().numpy(), slot.cpu().numpy()
    over = flags == pf.V_OVERFLOW
    assert 0 < over.sum() < n and not flags[~over].any()
    assert (slots[over] == -1).all() and (slots[~over] >= 0).all()
    tc = table_contents(t)
    placed = np.unique(key[~over])
    assert np.array_equal(np.sort(tc["key"]), placed) and not np.isin(key[over], placed).any()
    assert int(tc["count"].sum()) == int((~over).sum())
    assert int(pf.read_stats(t)[pf.STAT_OVERFLOW]) == int(over.sum())


@pytest.mark.parametrize("agg", [0, 2, 64, 256])
@pytest.mark.parametrize("n,distinct", [(1, 1), (15, 15), (65, 40), (300, 2), (5000, 4000)])
def test_atomic_insert_of_partial_wavefronts(gpu, n, distinct, agg):
    """Four lanes of a wavefront add the words of one cell: wavefronts that are
    not full, cells with and without a contribution side by side, sums of both
    signs (the fingerprint beside the count stays as it is)."""
    rng = np.random.default_rng(n + agg)
    ids = np.concatenate([np.arange(distinct), rng.integers(0, distinct, n - distinct)])
    rng.shuffle(ids)
    _insert_and_compare(_keys(ids), (rng.random((3, n)) * 300 - 150).astype(np.float32), 13, agg=agg)


@pytest.mark.parametrize("n,agg", [(1, 0), (65, 0), (700, 0), (700, 64), (700, 256), ((1 << 19) + 3, 64)])
def test_atomic_insert_of_binary32_sums(gpu, n, agg):
    """Whole numbers whose sums stay below 2^24 are exact in any order; every
    seventh vertex is flagged."""
    rng = np.random.default_rng(n)
    ids = rng.integers(0, max(1, n // 9), n)
    rgb = rng.integers(-40, 41, (3, n)).astype(np.float32)
    t = pf.Table(17, 64, sum_format=pf.SUMS_FLOAT32)
    pf.table_init(t)
    fl = (np.arange(n) % 7 == 6).astype(np.uint8)
    out = [torch.empty(n, device="cuda") for _ in range(3)]
    cnt = torch.empty(n, dtype=torch.int32, device="cuda")
    slot = torch.empty(n, dtype=torch.int32, device="cuda")
    k, d_fl = torch.from_numpy(_keys(ids).view(np.int64)).cuda(), torch.from_numpy(fl).cuda()
    r, g, b = (torch.from_numpy(x).cuda() for x in rgb)
    pf.insert_accumulate(t, k, r, g, b, d_fl, slot, agg)
    pf.query_average(t, k, slot, r, g, b, d_fl, False, *out, cnt)
    torch.cuda.synchronize()
    live = fl == 0
    want_cnt = np.bincount(ids[live], minlength=ids.max() + 1)[ids]
    assert np.array_equal(cnt.cpu().numpy()[live], want_cnt[live])
    for c in range(3):
        total = np.bincount(ids[live], weights=rgb[c][live].astype(np.float64), minlength=ids.max() + 1)[ids]
        want = (total.astype(np.float32) / want_cnt.clip(1).astype(np.float32))
        assert_bits_equal(out[c].cpu().numpy()[live], want[live], "average")


@pytest.mark.parametrize("m", [4, 7, 9, 13, 14, 18, 19, 21])
def test_blend_visits_every_cell_once(gpu, m):
    """Ranges of 8 to 64 bitmap words: with the same cells in the previous table
    every one is found, and the blend of equal values returns them."""
    n = (1 << m) // 2
    key = _keys(np.arange(n))
    k = torch.from_numpy(key.view(np.int64)).cuda()
    c = torch.from_numpy(np.arange(n, dtype=np.float32) % 1024).cuda()  # halves and doubles of them are exact
    fl = torch.zeros(n, dtype=torch.uint8, device="cuda")
    tabs = [pf.Table(m, 1 << min(m, 10)) for _ in range(2)]
    for t in tabs:
        pf.table_init(t)
        pf.insert_accumulate(t, k, c, c, c, fl, None, 0)
    pf.temporal_update(tabs[1], None, 0.5)
    pf.temporal_update(tabs[0], tabs[1], 0.5)
    out = [torch.empty(n, device="cuda") for _ in range(3)]
    pf.query_average(tabs[0], k, None, c, c, c, fl, True, *out)
    torch.cuda.synchronize()
    assert not fl.any().item()
    assert int(pf.read_stats(tabs[0])[pf.STAT_TEMPORAL_HIT]) == n
    for o in out:
        assert torch.equal(o, c)


@pytest.mark.parametrize("probe", [1, 2, 3, 4, 5, 6, 9, 16])
def test_small_call_claims_within_max_probe(gpu, probe):
    """A small call reads the slots after the home slot four at a time: placed
    keys lie less than max_probe slots from home with no empty slot before them,
    and the others find all of their slots taken."""
    m, n = 5, 96
    key = _keys(np.arange(n) % 48 + 1000 * probe)
    t = pf.Table(m, probe)
    pf.table_init(t)
    k = torch.from_numpy(key.view(np.int64)).cuda()
    one = torch.ones(n, device="cuda")
    fl = torch.zeros(n, dtype=torch.uint8, device="cuda")
    slot = torch.empty(n, dtype=torch.int32, device="cuda")
    ws = torch.empty(pf.insert_workspace_bytes(n, m), dtype=torch.uint8, device="cuda")
    pf.insert_accumulate_binned(t, k, one, one, one, fl, slot, ws)
    torch.cuda.synchronize()
    flags, slots = fl.cpu().numpy(), slot.cpu().numpy()
    taken = table_contents(t)["occupied"].astype(bool)
    home, _ = oracle.key_hashes(key, m)
    for i in range(n):
        window = (int(home[i]) + np.arange(probe)) % (1 << m)
        if flags[i] == 0:
            d = (int(slots[i]) - int(home[i])) % (1 << m)
            assert d < probe and taken[window[:d + 1]].all()
        else:
            assert flags[i] == pf.V_OVERFLOW and slots[i] == -1 and taken[window].all()
    assert (flags != 0).any() or probe == 16


def test_bins_of_more_cells_than_passes_pay(gpu):
    # half of the table's bins hold ~13,300 cells each: their records go to the
    # cells by device atomics
    m = 24
    cand = _keys(np.arange(1, 3400000))
    home, _ = oracle.key_hashes(cand, m)
    chosen = cand[home < np.uint32(1 << (m - 1))]
    rng = np.random.default_rng(9)
    key = np.concatenate([chosen, chosen[rng.integers(0, len(chosen), 200000)]])
    rng.shuffle(key)
    assert len(chosen) > 128 * 6 * 2048 and len(key) < 1 << 22
    _insert_and_compare(key, (rng.random((3, len(key))) * 300 - 150).astype(np.float32), m)


@pytest.mark.parametrize("max_samples", [None, 3])
def test_blend_of_bins_of_many_cells(gpu, max_samples):
    """3.5M vertices, nearly every one a cell of its own: the fused insert with
    the blend against the atomic insert and the temporal pass."""
    n, m = 3500000, 23
    g = torch.Generator(device="cuda").manual_seed(4)
    f = {c: torch.rand(n, device="cuda", generator=g) for c in ("px", "py", "pz", "r", "g", "b")}
    f.update(nx=torch.zeros(n, device="cuda"), ny=torch.zeros(n, device="cuda"), nz=torch.ones(n, device="cuda"),
             valid=torch.ones(n, dtype=torch.uint8, device="cuda"), cam=(0.0, 0.0, 3.0), s=0.0008)
    fused = pf.FrameFilter(n, m, fused=True, max_samples=max_samples)
    apart = pf.FrameFilter(n, m, agg_width=64, max_samples=max_samples)
    for seed in (5, 5, 6):
        a = fused.filter(**f, seed=seed, with_count=True)
        b = apart.filter(**f, seed=seed, with_count=True)
        used = int(pf.read_stats(fused.tables[1])[pf.STAT_USED])
        assert used > 256 * 6 * 2048 and used == int(pf.read_stats(apart.tables[1])[pf.STAT_USED])
        assert int(pf.read_stats(fused.tables[1])[pf.STAT_TEMPORAL_HIT]) == \
            int(pf.read_stats(apart.tables[1])[pf.STAT_TEMPORAL_HIT])
        assert not fused.vflags.any().item() and torch.equal(fused.count, apart.count)
        for x, y in zip(a, b):
            assert torch.equal(x.view(torch.int32), y.view(torch.int32))
