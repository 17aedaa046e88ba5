"""The serving loop on many resident rows (GPU): iterations hand the block kernels the 64-row tiles
of resident requests. Up to 128 tiles (8,192 rows) run 32-row workgroups of eight waves, up to 256
tiles (16,384 rows) 64-row ones, above that the throughput kernels. Requests that finish early leave
gaps between the others. Every result must be bitwise that of the request alone, which runs other
forms of the kernels."""

import time

import numpy as np
import pytest

from tests._gpu import fmd_lib, torch_cuda
from workload import configs, events, params

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", [configs.BF16, configs.FP8])
@pytest.mark.parametrize("rows,least", [(21000, 16384 + 64), (13500, 8192 + 64)],
                         ids=["throughput", "64-row"])
def test_many_resident_rows_equal_alone(precision, rows, least):
    torch, fmd = torch_cuda(), fmd_lib()
    cfg = configs.BASE_MODEL.with_precision(precision)
    flat = params.draw(cfg, 12, perturbed=True)
    rng = np.random.default_rng(rows)
    # nine requests; every second one ends early, the others run long enough that all are
    # resident together and then run on among the gaps; one has its own reco counts
    reqs = []
    for i in range(9):
        n = rng.integers(1, 300, size=64)
        n = n[:int(np.searchsorted(np.cumsum(n), rows / 9))]
        off = np.r_[0, np.cumsum(n)].astype(np.int64)
        roff = np.r_[0, np.cumsum(np.maximum(n - 7, 0))].astype(np.int64) if i == 4 else None
        sched = configs.Schedule(configs.EULER, 8) if i % 2 else configs.Schedule(configs.RK4, 18)
        reqs.append((off, events.particles(rng, int(off[-1])), 500 + i, sched, roff))
    m = fmd.Model(cfg, flat)
    alone = [m.simulate(o, f, s, sc, reco_offsets=ro) for o, f, s, sc, ro in reqs]
    srv = fmd.Server(m, hbm_budget_bytes=1 << 30)
    ids = [srv.submit(o, f, s, sc, reco_offsets=ro) for o, f, s, sc, ro in reqs]
    most, seen = 0, set()
    left = dict(zip(ids, range(len(ids))))
    deadline = time.monotonic() + 60
    while left:
        assert time.monotonic() < deadline
        info = srv.info()
        most = max(most, info["resident_tokens"])
        seen.add(info["resident_requests"])
        for rid in list(left):
            got = srv.poll(rid)
            if got is not None:
                k = left.pop(rid)
                assert np.array_equal(got[0], alone[k]), k
    srv.close()
    m.close()
    assert most >= least, most
    assert len(seen - {0, 9}) >= 1, seen            # iterations with some of the requests gone
