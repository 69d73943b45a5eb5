"""The neighbourhood search where nearly every neighbour is there: a filled
cube of voxels under one normal at a table load of 0.4, so that a workgroup
takes several batches of voxels and lists more slots to probe than it has room
for; cell values and lookup equal the oracle's bit for bit."""
import numpy as np
import pytest
import torch

import oracle
import paper_1902_05942_amd as pf
import synth
from gpu_util import assert_bits_equal, check_frame_against_oracle, gpu_frame, table_contents, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,below", [(40000, 6), (40000, 1 << 30), (3000, 2)])
def test_filled_cube(gpu, n, below):
    f = synth.mixed_normals_frame(n, 21, 0.0125)
    f["nx"], f["ny"], f["nz"] = np.zeros(n, np.float32), np.ones(n, np.float32), np.zeros(n, np.float32)
    t = pf.Table(f["log2_slots"], f["max_probe"], f["frac_bits"])
    pf.table_init(t)
    res = gpu_frame(f, to_dev(f), t, agg="fused", low_density=(below, pf.LD_NEIGHBOURS))
    R = oracle.filter_frame(f, temporal=False, low_density_fallback=(below, pf.LD_NEIGHBOURS))
    assert n < 40000 or 0.3 < len(R.gkey) / (1 << f["log2_slots"]) < 0.6
    check_frame_against_oracle(res, R, t)
    tc = table_contents(t)
    assert_bits_equal(tc["blend"][np.argsort(tc["key"])][:, :3], R.gval[R.table.gslot >= 0], "cell values")
