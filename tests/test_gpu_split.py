"""FP32 products by three-way BF16 splits (GPU, d_model <= 256): one velocity evaluation against
the FP64 oracle at every width of the kernels (and 320, which keeps the FP32 matrix instruction),
around the row-tile edges; rows that do not depend on the tile or the call around them; operands
far from 1.

Tolerance: a partial product left out is below 2^-23 of its product and of either sign, and a
dot product of K terms rounds about K / 16 + 6 times at 2^-24 of its size: for K up to 1024 some
70 roundings, or 8 x 2^-24 = 5e-7 normwise where they add in quadrature, through about 50 products
in sequence that enter the residual at equal weight: 5e-7 x sqrt(50) = 3.5e-6 at most, against
1e-4 where one plane of an operand (2^-16 of it) were lost in each. The bar is 5e-6, half the bar
of the parity tests."""

import numpy as np
import pytest

from oracle import net
from tests._gpu import fmd_lib, torch_cuda
from workload import configs, errors, events, params

pytestmark = pytest.mark.gpu

SIZES = [1, 31, 0, 33, 64, 65, 100, 2, 129, 200]


def _case(d, heads, blocks=2, seed=4):
    cfg = configs.ModelCfg(d_model=d, n_blocks=blocks, n_heads=heads, n_max=1000)
    rng = np.random.default_rng(seed)
    off = np.r_[0, np.cumsum(SIZES)].astype(np.int64)
    feat = events.particles(rng, int(off[-1]))
    x = rng.standard_normal(feat.shape).astype(np.float32)
    t = rng.uniform(0, 1, len(SIZES)).astype(np.float32)
    return cfg, params.draw(cfg, seed, perturbed=True), off, feat, x, t


def _velocity(torch, m, off, *arrays):
    return m.velocity(off, *[torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrays]).cpu().numpy()


@pytest.mark.parametrize("d,heads,blocks", [(64, 4, 2), (64, 1, 1), (128, 4, 2), (192, 6, 2),
                                            (256, 8, 6), (256, 16, 1), (320, 10, 1)])
def test_velocity_matches_oracle(d, heads, blocks):
    torch, fmd = torch_cuda(), fmd_lib()
    cfg, flat, off, feat, x, t = _case(d, heads, blocks)
    m = fmd.Model(cfg, flat)
    v = _velocity(torch, m, off, feat, x, t)
    P = net.unpack(flat, cfg)
    ref = np.concatenate([net.velocity(P, feat[off[e]:off[e + 1]], x[off[e]:off[e + 1]], float(t[e]))
                          for e in range(len(SIZES)) if SIZES[e]])
    assert errors.normwise_rel_err(v, ref).max() < 5e-6
    m.close()


@pytest.mark.parametrize("d,heads", [(64, 4), (256, 8)])
def test_rows_do_not_depend_on_tile_or_batch(d, heads):
    torch, fmd = torch_cuda(), fmd_lib()
    cfg, flat, off, feat, x, t = _case(d, heads)
    m = fmd.Model(cfg, flat)
    small = _velocity(torch, m, off, feat, x, t)          # tuned candidates
    m.autotune_enable(False)
    assert np.array_equal(small, _velocity(torch, m, off, feat, x, t))
    # the same events behind enough others that 64-row tiles fill the chip
    rng = np.random.default_rng(9)
    pre = rng.integers(20, 201, size=160)
    off2 = np.r_[0, np.cumsum(np.r_[pre, SIZES])].astype(np.int64)
    assert off2[-1] > 64 * 256
    k = int(pre.sum())
    feat2 = np.concatenate([events.particles(rng, k), feat])
    x2 = np.concatenate([rng.standard_normal((k, 9)).astype(np.float32), x])
    t2 = np.r_[rng.uniform(0, 1, len(pre)).astype(np.float32), t]
    for tuned in (False, True):
        m.autotune_enable(tuned)
        assert np.array_equal(_velocity(torch, m, off2, feat2, x2, t2)[k:], small)
    # a row that is not finite stays in its event
    bad = x.copy()
    bad[off[6]] = np.inf
    bad[off[6] + 1] = np.nan
    v = _velocity(torch, m, off, feat, bad, t)
    keep = np.ones(len(x), bool)
    keep[off[6]:off[7]] = False
    assert np.array_equal(v[keep], small[keep]) and np.isnan(v[~keep]).all()
    m.close()


def test_powers_of_two_move_exactly():
    """Values of the self-attention times 2^40 and W_o times 2^-40: every split, product and sum
    scales exactly, so the result is the same bit for bit."""
    torch, fmd = torch_cuda(), fmd_lib()
    cfg, flat, off, feat, x, t = _case(256, 8)
    m = fmd.Model(cfg, flat)
    v = _velocity(torch, m, off, feat, x, t)
    m.close()
    scaled = flat.copy()
    P = params.named(cfg, scaled)
    for i in range(cfg.n_blocks):
        P[f"blk{i}.W_qkv"][:, 512:] *= np.float32(2.0 ** 40)
        P[f"blk{i}.b_qkv"][512:] *= np.float32(2.0 ** 40)
        P[f"blk{i}.W_o"][...] *= np.float32(2.0 ** -40)
    m = fmd.Model(cfg, scaled)
    assert np.array_equal(_velocity(torch, m, off, feat, x, t), v)
    m.close()


@pytest.mark.parametrize("blocks,heads", [(1, 4), (2, 4), (3, 1)])
def test_chained_blocks_match_the_separate_products(blocks, heads):
    """Width 64 runs a block's six products as two kernels, the separate ones while per-kernel
    timing is on: the same bits, for single evaluations and sampler stages, at the edges of the
    32-row tiles and in a call that fills the chip."""
    torch, fmd = torch_cuda(), fmd_lib()
    cfg, flat, off, feat, x, t = _case(64, heads, blocks)
    rng = np.random.default_rng(3)
    m = fmd.Model(cfg, flat)
    for n in ([1], [31], [32], [33], SIZES, list(rng.integers(20, 201, size=160))):
        o = np.r_[0, np.cumsum(n)].astype(np.int64)
        f = torch.from_numpy(events.particles(rng, int(o[-1]))).cuda()
        xs = torch.from_numpy(rng.standard_normal((int(o[-1]), 9)).astype(np.float32)).cuda()
        te = torch.from_numpy(rng.uniform(0, 1, len(n)).astype(np.float32)).cuda()
        got = []
        for timing in (True, False):
            m.timing_enable(timing)
            got.append((m.velocity(o, f, xs, te),
                        m.simulate_from_state(o, f, xs, configs.Schedule(configs.RK4, 2))))
        assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1]), int(o[-1])
    m.close()
