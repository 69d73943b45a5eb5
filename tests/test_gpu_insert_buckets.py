"""The insert through buckets (more than 5 * 2^16 vertices) with vertices that are
flagged where it computes their keys and contributions: masked, not finite, beyond
the key range, out of range, without room in the table, beside valid ones in the
same windows; a caller's key that equals the LDS table's mark of an empty entry;
keys of one skewed bin.  Against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_1902_05942_amd as pf
from gpu_util import assert_bits_equal, check_frame_against_oracle, gpu_frame, table_contents, to_dev
from test_gpu_insert_small import edge_frame
from test_gpu_insert_windows import _insert_and_compare, _keys

pytestmark = pytest.mark.gpu
N = (5 << 16) + 1  # the smallest call that takes this way


@pytest.mark.parametrize("n,s,m", [(N, 0.01, 20), (N + 1023, 0.5, 16), (1 << 20, 0.003, 22)])
@pytest.mark.parametrize("agg", ["fused", "binned"])
def test_flagged_vertices_beside_valid_ones(gpu, agg, n, s, m):
    f = edge_frame(n, n, s, m)
    t = pf.Table(m)
    pf.table_init(t)
    R = oracle.filter_frame(f, temporal=False)
    kinds = set(np.unique(R.flags))
    assert {0, pf.V_INVALID, pf.V_RADRANGE} <= kinds and (pf.V_KEYRANGE in kinds or s > 0.1)
    check_frame_against_oracle(gpu_frame(f, to_dev(f), t, agg=agg), R, t)


@pytest.mark.parametrize("max_samples", [None, 5])
def test_flagged_vertices_and_the_temporal_blend(gpu, max_samples):
    """Two frames, the second blended in the insert's own launches."""
    n, m = N + 5000, 20
    tabs = [pf.Table(m), pf.Table(m)]
    for t in tabs:
        pf.table_init(t)
    state = None
    for frame in range(2):
        f = edge_frame(n, 7 + frame, 0.05, m)
        res = gpu_frame(f, to_dev(f), tabs[frame], prev=tabs[0] if frame else None, agg="fused", temporal=True,
                        alpha=0.2, clear=False, max_samples=max_samples, temporal_in_insert=True)
        R = oracle.filter_frame(f, prev_state=state, temporal=True, alpha_old=0.2, max_samples=max_samples)
        check_frame_against_oracle(res, R, tabs[frame])
        state = R.state


@pytest.mark.parametrize("temporal", [False, True])
def test_batches_into_one_table(gpu, temporal):
    """Three calls through buckets and a small one accumulate into one table."""
    n, m = 3 * N + 1000, 20
    rng = np.random.default_rng(4)
    key = _keys(rng.integers(0, 70000, n))
    rgb = (rng.random((3, n)) * 300 - 150).astype(np.float32)
    R = oracle.filter_keys(key, rgb[0], rgb[1], rgb[2], np.ones(n, np.uint8), m)
    t = pf.Table(m)
    pf.table_init(t)
    k = torch.from_numpy(key.view(np.int64)).cuda()
    r, g, b = (torch.from_numpy(x).cuda() for x in rgb)
    fl = torch.zeros(n, dtype=torch.uint8, device="cuda")
    slot, cnt = (torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2))
    ws = torch.empty(pf.insert_workspace_bytes(N, m), dtype=torch.uint8, device="cuda")
    for i0 in range(0, n, N):
        part = slice(i0, min(n, i0 + N))
        pf.insert_accumulate_binned(t, k[part].clone(), r[part].clone(), g[part].clone(), b[part].clone(), fl[part],
                                    slot[part], ws)
    if temporal:
        pf.temporal_update(t, None, 0.5)
    out = [torch.empty(n, device="cuda") for _ in range(3)]
    pf.query_average(t, k, slot, r, g, b, fl, temporal, *out, cnt)
    torch.cuda.synchronize()
    assert not fl.any().item()
    assert_bits_equal(cnt.cpu().numpy().view(np.uint32), R.cnt, "count")
    assert_bits_equal(np.stack([o.cpu().numpy() for o in out], 1), R.out, "average")


@pytest.mark.parametrize("n,distinct,m", [(N, 5000, 14), (N, N, 20), (1 << 20, 3, 6)])
def test_key_with_every_bit_set(gpu, n, distinct, m):
    rng = np.random.default_rng(n)
    ids = np.concatenate([np.arange(distinct), rng.integers(0, distinct, n - distinct)])
    rng.shuffle(ids)
    key = _keys(ids + 1)
    key[ids % 7 == 0] = ~np.uint64(0)
    _insert_and_compare(key, (rng.random((3, n)) * 300 - 150).astype(np.float32), m)


@pytest.mark.parametrize("m,probe", [(6, 2), (10, 1), (13, 4)])
def test_keys_built_in_the_window_overflow(gpu, m, probe):
    """Tables of far fewer slots than voxels: a vertex's cell holds its key, or the
    probe limit kept it out and it is flagged."""
    f = edge_frame(N, 3, 0.02, m, probe)
    t = pf.Table(m, probe)
    pf.table_init(t)
    res = gpu_frame(f, to_dev(f), t, agg="fused")
    R = oracle.filter_frame(f, temporal=False)
    over = res["flags"] == pf.V_OVERFLOW
    assert over.any() and np.array_equal(res["flags"][~over] != 0, R.flags[~over] & ~np.uint8(pf.V_OVERFLOW) != 0)
    assert np.array_equal(res["key"], R.key)
    placed = res["flags"] == 0
    keys = t.keys().cpu().numpy().view(np.uint64)
    assert np.array_equal(keys[res["slot"][placed]], res["key"][placed])
    assert (res["slot"][~placed] == 0xffffffff).all()
    home, _ = oracle.key_hashes(res["key"][placed], m)
    assert (((res["slot"][placed] - home) & ((1 << m) - 1)) < probe).all()
    tc = table_contents(t)
    assert int(tc["count"].sum()) == int(placed.sum())
    assert int(res["stats"][pf.STAT_OVERFLOW]) == int(over.sum())
    assert not np.isin(res["key"][over], res["key"][placed]).any()


def test_every_record_in_one_bin(gpu):
    """700 cells whose home slots all lie in the first of the 256 bins of a 2^22-slot
    table (16384 slots each), over 600 windows' worth of vertices."""
    m, n, cells = 22, 600 * 4096, 700
    cand = _keys(np.arange(1, 400000))
    home, _ = oracle.key_hashes(cand, m)
    chosen = cand[home < np.uint32(1 << (m - 8))][:cells]
    assert len(chosen) == cells
    rng = np.random.default_rng(5)
    _insert_and_compare(chosen[(np.arange(n) * 7919) % cells], rng.random((3, n), dtype=np.float32), m)
