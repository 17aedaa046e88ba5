"""The fused block kernels' forms for few rows (GPU): calls of at most 8192 padded rows run
32-row tiles, calls of at most 16384 rows 64-row tiles of eight waves, larger ones the
throughput kernels. A row's bits must not depend on which form computed it, so events taken out
of a large call and run in small ones must give the same rows bit for bit, in BF16 and FP8, for
the sampler's stages (embedding and output head inside the block kernels) and for single
evaluations (per-event times, statistics tail), around the tile edges and at the largest call of
each form. The linear algebra itself is compared with the oracle in the parity tests; here the
reference is the large call."""

import numpy as np
import pytest

from tests._gpu import fmd_lib, torch_cuda
from workload import configs, events, params

pytestmark = pytest.mark.gpu


def _cut(off, ids):
    rows = np.concatenate([np.arange(off[e], off[e + 1]) for e in ids])
    return np.r_[0, np.cumsum([off[e + 1] - off[e] for e in ids])].astype(np.int64), rows


@pytest.mark.parametrize("precision", [configs.BF16, configs.FP8])
def test_rows_do_not_depend_on_the_kernel_form(precision):
    torch, fmd = torch_cuda(), fmd_lib()
    cfg = configs.BASE_MODEL.with_precision(precision)
    rng = np.random.default_rng(21)
    edge = [1, 31, 32, 33, 63, 64, 65, 127, 129, 300]
    sizes = np.r_[edge, rng.integers(20, 201, size=170)]
    off = np.r_[0, np.cumsum(sizes)].astype(np.int64)
    assert off[-1] > 16384 + 256                      # the throughput kernels
    feat = torch.from_numpy(events.particles(rng, int(off[-1]))).cuda()
    x = torch.from_numpy(rng.standard_normal((int(off[-1]), 9)).astype(np.float32)).cuda()
    t = torch.from_numpy(rng.uniform(0, 1, len(sizes)).astype(np.float32)).cuda()
    m = fmd.Model(cfg, params.draw(cfg, seed=0, perturbed=True))
    scheds = [configs.Schedule(configs.EULER, 2), configs.Schedule(configs.RK4, 1)]
    big = [m.simulate_from_state(off, feat, x, s) for s in scheds] + [m.velocity(off, feat, x, t)]
    cum = np.cumsum(sizes)
    groups = [[0], [1], [2], [3], [5], [6], [9], list(range(10)),
              list(range(int(np.searchsorted(cum, 8192, "right")))),     # the largest of each form
              list(range(int(np.searchsorted(cum, 8192, "right")) + 3)),
              list(range(int(np.searchsorted(cum, 16384, "right"))))]
    for ids in groups:
        o, rows = _cut(off, ids)
        r = torch.from_numpy(rows).cuda()
        f, xs, te = feat[r].contiguous(), x[r].contiguous(), t[torch.tensor(ids, device="cuda")]
        got = [m.simulate_from_state(o, f, xs, s) for s in scheds] + [m.velocity(o, f, xs, te.contiguous())]
        for g, b in zip(got, big):
            assert torch.equal(g, b[r]), (len(ids), int(o[-1]))
    m.close()
