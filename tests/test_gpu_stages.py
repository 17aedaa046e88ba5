"""The stage loop of the sampler (GPU): stages captured one or four a graph, the rest of a
schedule launched one by one."""

import time

import numpy as np
import pytest

from tests._gpu import fmd_lib, torch_cuda
from workload import configs, events, params

pytestmark = pytest.mark.gpu


def _events(torch, sizes, seed=0):
    off = np.r_[0, np.cumsum(sizes)].astype(np.int64)
    return off, torch.from_numpy(events.particles(np.random.default_rng(seed), int(off[-1]))).cuda()


def test_alternating_short_and_long_schedules_keep_their_graphs():
    """Schedules below and above 16 stages use graphs of one and of four stages. A caller that
    alternates them on the same events must not pay a capture per call: the host time of the
    long call alternating with short ones against the same call repeated. Capturing its 100
    kernels takes some 2 us each, 200 us with nothing else; the bar is half of that, on the
    fastest of 15 calls of each kind."""
    torch, fmd = torch_cuda(), fmd_lib()
    cfg = configs.BASE_MODEL.with_precision(configs.BF16)
    m = fmd.Model(cfg, params.draw(cfg, 0))
    off, feat = _events(torch, [50, 40])
    out = torch.empty((int(off[-1]), 9), device="cuda")
    short, long = configs.Schedule(configs.EULER, 12), configs.Schedule(configs.EULER, 16)

    def host_seconds(sched):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        m.simulate(off, feat, 1, sched, out=out)
        return time.perf_counter() - t0

    for s in (short, long, short, long):       # tuning, captures
        host_seconds(s)
    repeated = min(host_seconds(long) for _ in range(15))
    alternating = min([host_seconds(s) for _ in range(15) for s in (short, long)][1::2])
    torch.cuda.synchronize()
    m.close()
    assert alternating < repeated + 100e-6, (alternating, repeated)
