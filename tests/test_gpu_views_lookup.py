"""The lookup after the persistent multi-view launch: every lane of a wavefront
holds one view's items, so the most views a call takes, of sizes around its items
of 512 vertices and 8192 slots; and the launch's resident workgroups."""
import numpy as np
import pytest
import torch

import paper_1902_05942_amd as pf

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("temporal", [True, False])
@pytest.mark.parametrize("nviews", [1, 2, 63, 64])
def test_many_views_equal_single_calls(gpu, nviews, temporal):
    rng = np.random.default_rng(nviews)
    sizes = [(int(n), int(np.clip(np.ceil(np.log2(2 * n)), 7, 16)))
             for n in rng.choice([1, 7, 511, 512, 513, 1024, 1500, 9000], nviews)]
    mv = pf.MultiViewFilter(sizes, temporal=temporal, mode="persistent")
    single = [pf.FrameFilter(n, m, temporal=temporal, fused=True) for n, m in sizes]
    for frame in range(3):
        frames = []
        for n, _ in sizes:
            f = {c: torch.from_numpy(rng.random(n, dtype=np.float32) * np.float32(0.05)).cuda()
                 for c in ("px", "py", "pz", "r", "g", "b")}
            f.update(nx=torch.zeros(n, device="cuda"), ny=torch.zeros(n, device="cuda"),
                     nz=torch.ones(n, device="cuda"), cam=(0.0, 0.0, 2.0), s=0.01, seed=17 + frame,
                     valid=torch.from_numpy((rng.random(n) < 0.9).astype(np.uint8)).cuda())
            frames.append(f)
        got = mv.filter(frames, block=256, with_count=True)
        assert mv.status() == 0
        for v, (f, flt) in enumerate(zip(frames, single)):
            a = {x: f[x] for x in ("px", "py", "pz", "nx", "ny", "nz", "valid", "r", "g", "b", "cam", "s", "seed")}
            want = flt.filter(**a, with_count=True)
            assert torch.equal(mv.bufs[v]["vflags"], flt.vflags) and torch.equal(mv.bufs[v]["count"], flt.count)
            for x, y in zip(got[v], want):
                assert torch.equal(x.view(torch.int32), y.view(torch.int32))
            if temporal:  # the next frame's table is empty
                assert not mv.tables[v][0].cells()[:, 0].any().item()
                assert not mv.tables[v][0].occupancy().any().item()
    phases = mv.phase_us()
    assert all(0 <= x < 1e6 for x in phases), phases


@pytest.mark.parametrize("block,groups", [(64, 13), (128, 8), (256, 4), (512, 2)])
def test_resident_workgroups(gpu, block, groups):
    """LDS bounds the persistent launch: 160 KB hold this many workgroups of each
    size (16 waves a compute unit from 128 lanes on)."""
    n = 3000
    mv = pf.MultiViewFilter([(n, 13)], mode="persistent")
    f = {c: torch.rand(n, device="cuda") for c in ("px", "py", "pz", "r", "g", "b")}
    f.update(nx=torch.zeros(n, device="cuda"), ny=torch.zeros(n, device="cuda"), nz=torch.ones(n, device="cuda"),
             cam=(0.0, 0.0, 2.0), s=0.01, seed=1, valid=torch.ones(n, dtype=torch.uint8, device="cuda"))
    mv.filter([f], block=block)
    assert mv.status() == 0
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert mv.status_words()[1] == groups * cus
