"""Attention of heads of 32 at the ends of its range of work lists (GPU). FP32, few and large events:
the work items of an event that is large against the call are dealt to all XCDs instead of one.
Millions of small events: more workgroups than one launch holds."""

import numpy as np
import pytest

from oracle import net
from tests._gpu import fmd_lib, torch_cuda
from workload import configs, errors, events, params

pytestmark = pytest.mark.gpu


def _inputs(torch, sizes, seed=0):
    rng = np.random.default_rng(seed)
    off = np.r_[0, np.cumsum(sizes)].astype(np.int64)
    T = int(off[-1])
    dev = [events.particles(rng, T), rng.standard_normal((T, 9)).astype(np.float32),
           rng.uniform(0, 1, len(sizes)).astype(np.float32)]
    return off, [torch.from_numpy(a).cuda() for a in dev]


def test_one_large_event_uses_the_whole_chip():
    """One event of 4,000 particles has 63 query tiles in 8 heads, two workgroups a CU; eight such
    events have eight times that. On one XCD each, both take the time of one event on 32 CUs;
    dealt, one event takes a small part of the time of eight (an eighth if the chip is full in
    both). The bar is two fifths."""
    torch, fmd = torch_cuda(), fmd_lib()
    cfg = configs.ModelCfg(d_model=256, n_blocks=1, n_heads=8, n_max=4096)
    m = fmd.Model(cfg, params.draw(cfg, 0))
    ms = []
    for k in (1, 8):
        off, (feat, x, t) = _inputs(torch, [4000] * k)
        m.velocity(off, feat, x, t)
        best = []
        for _ in range(3):
            m.timing_enable(True)
            m.velocity(off, feat, x, t)
            torch.cuda.synchronize()
            best.append([m.timing_read(c)[0] for c in (fmd.K_ATTN_SELF, fmd.K_ATTN_CROSS)])
            m.timing_enable(False)
        ms.append(np.min(best, axis=0))
    m.close()
    assert (ms[0] < 0.4 * ms[1]).all(), ms


@pytest.mark.parametrize("d,heads", [(64, 2), (256, 8)])
def test_dealt_events_keep_their_bits(d, heads):
    """Events whose tiles are dealt in a small call, and that stay whole behind enough others; reco
    counts on both sides of the truth counts; the oracle within the bar of the parity tests."""
    torch, fmd = torch_cuda(), fmd_lib()
    cfg = configs.ModelCfg(d_model=d, n_blocks=1, n_heads=heads, n_max=2100)
    flat = params.draw(cfg, 3, perturbed=True)
    m = fmd.Model(cfg, flat)
    sizes = [600, 1, 0, 64, 65, 257] if d == 256 else [2100, 1, 0, 64, 65, 257]
    off, (feat, x, t) = _inputs(torch, sizes)
    alone = m.velocity(off, feat, x, t)
    more = 1200 if d == 256 else 12000            # the large event then stays whole
    off2, (feat2, x2, t2) = _inputs(torch, sizes + [100] * more, seed=1)
    n = int(off[-1])
    feat2[:n], x2[:n], t2[:len(sizes)] = feat, x, t
    assert torch.equal(m.velocity(off2, feat2, x2, t2)[:n], alone)
    P = net.unpack(flat, cfg)
    f, xs = feat.cpu().numpy(), x.cpu().numpy()
    ref = np.concatenate([net.velocity(P, f[off[e]:off[e + 1]], xs[off[e]:off[e + 1]], float(t[e]))
                          for e in range(len(sizes)) if sizes[e]])
    assert errors.normwise_rel_err(alone.cpu().numpy(), ref).max() < 1e-5
    # reco counts of their own: the cross-attention list is another one
    sched = configs.Schedule(configs.EULER, 3)
    reco = np.array([100, 3, 0, 600, 1, 257] + [90] * more)
    roff = np.r_[0, np.cumsum(reco)].astype(np.int64)
    small = m.simulate(off, feat, 5, sched, reco_offsets=roff[:len(sizes) + 1])
    big = m.simulate(off2, feat2, 5, sched, reco_offsets=roff)
    assert torch.equal(big[:int(roff[len(sizes)])], small)
    m.close()


@pytest.mark.parametrize("precision", [configs.FP32, configs.BF16])
def test_millions_of_small_events(precision):
    """2.2 million events of one particle are 17.6 million (item, head) workgroups at 8 heads, more
    than the 2^32 - 1 work items of one launch. Each event's velocity is that of a small call; in BF16 as well."""
    torch, fmd = torch_cuda(), fmd_lib()
    cfg = configs.ModelCfg(d_model=256, n_blocks=1, n_heads=8, n_max=16, precision=precision)
    m = fmd.Model(cfg, params.draw(cfg, 3, perturbed=True))
    E = 2_200_000
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    off = np.arange(E + 1, dtype=np.int64)
    feat, x = (torch.randn((E, 9), generator=g, device="cuda") for _ in range(2))
    t = torch.rand(E, generator=g, device="cuda")
    v = m.velocity(off, feat, x, t)
    for a in (0, E // 2, E - 1000):
        part = [q[a:a + 1000].contiguous() for q in (feat, x, t)]
        assert torch.equal(m.velocity(off[:1001], *part), v[a:a + 1000])
    assert torch.isfinite(v).all()
    m.close()
    torch.cuda.empty_cache()
