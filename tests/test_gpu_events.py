"""Event kernels at the sizes where their work splits change (GPU): the observables with one
lepton more or less than a batch of lepton threads, events at the edges of a workgroup and of the
decoded tile, and event counts on both sides of the choice of workgroup size, against the FP64
oracle within the tolerance of the observables' parity tests; the truth selection with equal keys
at the limit, signed zeros, infinities and events longer than the keys kept in LDS, and event
counts at the edges of the offset scan, exactly."""

import numpy as np
import pytest

from oracle import observables as ob
from oracle import select as osel
from tests._gpu import fmd_lib, torch_cuda
from workload import events

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 2, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256]
LONG = [257, 511, 513, 1023, 1024, 1025, 2049]


@pytest.mark.parametrize("sizes,repeat", [(EDGES, 1), (EDGES, 40), (EDGES, 150), (EDGES + LONG, 1),
                                          (EDGES * 20 + LONG, 8)])
def test_observables_at_the_edges(sizes, repeat):
    torch, fmd = torch_cuda(), fmd_lib()
    rng = np.random.default_rng(len(sizes) * repeat)
    n = np.array(sizes * repeat)
    off = np.r_[0, np.cumsum(n)].astype(np.int64)
    feat = events.particles(rng, int(off[-1]))
    feat[:, 1] *= np.float32(0.3)                     # more particles inside the cones
    for e in range(0, len(n), 3):                     # events of leptons only
        feat[off[e]:off[e + 1], 3:8] = 0
        feat[off[e]:off[e + 1], 4 + e % 2] = 1
    ht, met, iso = (a.cpu().numpy() for a in fmd.event_observables(off, torch.from_numpy(feat).cuda()))
    # the oracle on the first copy; the other copies hold other particles of the same sizes
    k = len(sizes) if repeat > 1 else len(n)
    o = off[:k + 1]
    rht, rmet, riso = ob.observables(o, feat[:o[-1]])
    assert np.allclose(ht[:k], rht, rtol=1e-6, atol=1e-6)
    assert np.allclose(met[:k], rmet, rtol=1e-6, atol=1e-4)
    assert np.allclose(iso[:o[-1]], riso, rtol=1e-6, atol=1e-7, equal_nan=True)
    # and each event the same in a call of its own (another workgroup size) to the last bit but
    # for the order of the sums
    for e in (len(n) - 1, len(n) // 2):
        a, b = off[e], off[e + 1]
        h1, m1, i1 = fmd.event_observables(np.array([0, b - a]), torch.from_numpy(feat[a:b].copy()).cuda())
        assert np.allclose(i1.cpu().numpy(), iso[a:b], rtol=1e-6, atol=0, equal_nan=True)
        assert np.allclose(h1.cpu().numpy(), ht[e], rtol=1e-6)


@pytest.mark.parametrize("n_events,limit", [(1, 1), (1, 0), (63, 100), (64, 255), (4095, 20),
                                            (4096, 64), (4097, 128), (40, 2047), (40, 2500)])
def test_selection_at_the_edges(n_events, limit):
    torch, fmd = torch_cuda(), fmd_lib()
    rng = np.random.default_rng(n_events + limit)
    top = 300 if n_events < 1000 else 80
    n = rng.integers(0, top, size=n_events)
    n[:min(n_events, 12)] = [limit, limit + 1, 0, 1, 255, 256, 257, 512, 2047, 2048, 2049, 3000][:n_events]
    off = np.r_[0, np.cumsum(n)].astype(np.int64)
    feat = events.particles(rng, int(off[-1]))
    # few distinct values: ties at the limit; zeros of both signs, infinities, values at the cut
    vals = np.array([0.0, -0.0, 1.5, -1.25, np.inf, -np.inf, np.log(0.05), 3e38, 1e-40], np.float32)
    pick = rng.integers(0, 2 * len(vals), size=len(feat))
    feat[:, 0] = np.where(pick < len(vals), vals[pick % len(vals)], feat[:, 0])
    o, out = fmd.truth_select(off, torch.from_numpy(feat).cuda(), 0.5, limit)
    ro, rout = osel.select(off, feat, 0.5, limit)
    assert np.array_equal(o, ro)
    assert np.array_equal(out.cpu().numpy().view(np.uint32), np.asarray(rout, np.float32).view(np.uint32))
    ho, hout = fmd.truth_select(off, feat, 0.5, limit)             # host memory in and out
    assert np.array_equal(ho, ro) and np.array_equal(hout.view(np.uint32), out.cpu().numpy().view(np.uint32))
