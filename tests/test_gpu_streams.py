"""The stream a call is enqueued on: torch's current one unless one is given."""
import pytest
import torch

import paper_1902_05942_amd as pf

pytestmark = pytest.mark.gpu


def test_calls_follow_the_current_stream(gpu):
    side = torch.cuda.Stream()
    assert pf._lib._stream(None) == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert pf._lib._stream(None) == side.cuda_stream
        t = pf.Table(10)
        pf.table_init(t)  # ordered with the side stream's own work, no synchronisation between
        k = torch.arange(100, device="cuda")
        c = torch.ones(100, device="cuda")
        fl = torch.zeros(100, dtype=torch.uint8, device="cuda")
        pf.insert_accumulate(t, k, c, c, c, fl, None, 0)
        out = [torch.empty(100, device="cuda") for _ in range(3)]
        pf.query_average(t, k, None, c, c, c, fl, False, *out)
    assert pf._lib._stream(side) == side.cuda_stream
    side.synchronize()
    assert not fl.any().item() and all(torch.equal(o, c) for o in out)
