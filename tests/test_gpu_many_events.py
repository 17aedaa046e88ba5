"""The event kernels take a workgroup an event (GPU): 17 million events are more work items than one
launch holds. Observables and truth selection of events of one particle are those of a small call."""

import numpy as np
import pytest

from tests._gpu import fmd_lib, torch_cuda

pytestmark = pytest.mark.gpu


def test_seventeen_million_events():
    torch, fmd = torch_cuda(), fmd_lib()
    E = 17_000_000
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    feat = torch.randn((E, 9), generator=g, device="cuda")
    off = np.arange(E + 1, dtype=np.int64)
    # leave other values where the results go
    junk = torch.full((3 * E,), float("nan"), device="cuda")
    del junk
    ht, met, iso = fmd.event_observables(off, feat)
    o, rows = fmd.truth_select(off, feat, 10.0, 4)          # x0 > 0: about half of them
    keep = feat[:, 0] > 0
    assert np.array_equal(np.diff(o), keep.cpu().numpy())
    assert torch.equal(rows, feat[keep])
    for a in (0, 1 << 22, 16_700_000, E - 1000):
        part = feat[a:a + 1000].contiguous()
        h, m, i = fmd.event_observables(off[:1001], part)
        assert torch.equal(h, ht[a:a + 1000]) and torch.equal(m, met[a:a + 1000])
        assert torch.equal(i.nan_to_num(-1), iso[a:a + 1000].nan_to_num(-1))
