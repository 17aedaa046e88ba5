"""Event observables do not depend on the events around an event (GPU). The kernel takes 128, 256
or 512 threads an event by the number and the longest of a call's events; H_T and the vector pT
sum have one order of summation whatever that choice, so an event's values are the same bits in
any call. Events whose momenta balance to the last bit show it: their MET is nothing but the
rounding of the sums, different for every order (checked here on the host)."""

import numpy as np
import pytest

from tests._gpu import fmd_lib, torch_cuda
from workload import events


def balanced(rng, n):
    """n particles (n even): pairs of equal pT at +-phi, phi one of the two float32 values next to
    pi/2, so that the y components cancel exactly; the last pairs cancel the x components, which
    are small and of either sign, down to below the rounding of the sums."""
    up = np.float32(np.pi / 2)
    phis = (np.nextafter(up, np.float32(0)), up)                  # cos > 0, cos < 0
    rows = events.particles(rng, n)
    rows[:, 3:8] = 0
    rows[:, 3] = 1                                                # no leptons
    pt = lambda x0: 10.0 * np.exp(np.float64(x0))                 # noqa: E731
    left, px = n // 2, 0.0
    for k in range(left):
        fix = left - k <= 5
        phi = phis[int(px > 0)] if fix else phis[k % 2]
        x0 = rows[2 * k, 0]
        if fix and px:
            x0 = np.float32(np.log(abs(px) / (2 * abs(np.cos(np.float64(phi)))) / 10.0))
        rows[2 * k:2 * k + 2, 0] = x0
        rows[2 * k, 2], rows[2 * k + 1, 2] = phi, -phi
        px += 2 * pt(x0) * np.cos(np.float64(phi))
    return rows[rng.permutation(n)]


def _met(rows, threads):
    pt, phi = 10.0 * np.exp(rows[:, 0].astype(np.float64)), rows[:, 2].astype(np.float64)
    parts = [(0.0, 0.0)] * threads
    for i in range(len(rows)):
        x, y = parts[i % threads]
        parts[i % threads] = (x + pt[i] * np.cos(phi[i]), y + pt[i] * np.sin(phi[i]))
    return np.float32(np.hypot(sum(p[0] for p in parts), sum(p[1] for p in parts)))


def test_balanced_events_show_the_order():
    rng = np.random.default_rng(0)
    for n in (200, 700):
        rows = balanced(rng, n)
        m = [_met(rows, t) for t in (128, 256, 512)]
        assert max(m) < 1e-9 and len(set(m)) > 1, m


@pytest.mark.gpu
def test_an_event_is_the_same_in_any_call():
    torch, fmd = torch_cuda(), fmd_lib()
    rng = np.random.default_rng(1)
    short = [balanced(rng, n) for n in (60, 128, 130, 200, 254, 256)]
    long = [balanced(rng, n) for n in (258, 510, 514, 700, 1024, 1026, 1500, 2050)]

    def run(batch):
        off = np.r_[0, np.cumsum([len(r) for r in batch])].astype(np.int64)
        ht, met, iso = fmd.event_observables(off, torch.from_numpy(np.concatenate(batch)).cuda())
        return ht.cpu().numpy(), met.cpu().numpy()

    def fill(k):
        return [events.particles(rng, int(n)) for n in rng.integers(1, 90, size=k)]

    for group, others in ((short, (0, 600, 2100)), (long, (0, 600, 2100)),
                          (short + long, (600, 2100))):
        alone = [run([r]) for r in group]
        for k in others:
            ht, met = run(group + fill(k))
            for e, (h, m) in enumerate(alone):
                assert ht[e] == h[0] and met[e] == m[0], (len(group[e]), k, met[e], m[0])
