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


SCHEDULES = [configs.Schedule(configs.EULER, 50), configs.Schedule(configs.EULER, 15),
             configs.Schedule(configs.EULER, 17), configs.Schedule(configs.MIDPOINT, 9),
             configs.Schedule(configs.EULER, 19), configs.Schedule(configs.RK4, 4),
             configs.Schedule(configs.MIDPOINT, 3)]
NETS = {"d64-fp32": configs.SMALL_MODEL, "d128-fp32": configs.ModelCfg(128, 1, 4, n_max=64),
        "base-bf16": configs.BASE_MODEL.with_precision(configs.BF16),
        "base-fp8": configs.BASE_MODEL.with_precision(configs.FP8),
        "d64-bf16": configs.SMALL_MODEL.with_precision(configs.BF16), "linear": None}


@pytest.mark.parametrize("net", list(NETS))
def test_groups_of_four_and_the_rest_equal_eager_launches(net):
    """Schedules of 16 stages and more whose stages are no multiple of four (the default 50 among
    them) replay groups of four and launch the rest; shorter ones replay single stages. Every
    schedule in turn on one model, into two output buffers, several times with eager calls,
    other work and synchronizations between, equals eager launches bit for bit."""
    torch, fmd = torch_cuda(), fmd_lib()
    cfg = NETS[net]
    m = fmd.linear_field(0.7, -0.4) if cfg is None else fmd.Model(cfg, params.draw(cfg, 2, perturbed=True))
    off, feat = _events(torch, [33, 1, 0, 60, 17], seed=3)
    m.graphs_enable(False)
    eager = [m.simulate(off, feat, 4, s) for s in SCHEDULES]
    m.graphs_enable(True)
    outs = [torch.full_like(eager[0], float("nan")) for _ in range(2)]
    for round_ in range(3):
        for s, ref in zip(SCHEDULES, eager):
            for out in outs:
                out.fill_(float("nan"))
                m.simulate(off, feat, 4, s, out=out)
                if round_ == 1:
                    torch.cuda.synchronize()
                    m.graphs_enable(False)
                    assert torch.equal(m.simulate(off, feat, 4, SCHEDULES[-1]), eager[-1])
                    m.graphs_enable(True)
                assert torch.equal(out, ref), (s, round_)
    assert all(torch.isfinite(e).all() for e in eager)
    m.close()
