"""The workspace that a model's own calls, its server and its captured stage graphs share (GPU):
buffers that move under a cached graph, growths that fail, tables that stay bounded."""

import numpy as np
import pytest

from oracle import sample
from tests._gpu import fmd_lib, torch_cuda
from workload import configs, errors, events, params

pytestmark = pytest.mark.gpu

CFG = configs.SMALL_MODEL


def _events(torch, sizes, seed=0):
    off = np.r_[0, np.cumsum(sizes)].astype(np.int64)
    return off, torch.from_numpy(events.particles(np.random.default_rng(seed), int(off[-1]))).cuda()


def test_a_server_that_grows_the_stage_table_does_not_leave_a_graph_behind():
    """The server's iterations hold one stage-table entry per event. One with more events than
    the stages of the model's last call moves the table, and nothing else here: the pool, the
    events and the work items fit the workspace of that call, and nothing is tuned. The same
    call afterwards has the key of the graph captured before."""
    torch, fmd = torch_cuda(), fmd_lib()
    m = fmd.Model(CFG, params.draw(CFG, 5, perturbed=True))
    m.autotune_enable(False)
    off, feat = _events(torch, [40] * 200)
    sched = configs.Schedule(configs.EULER, 20)
    first = m.simulate(off, feat, 3, sched)
    probe = fmd.Server(m, hbm_budget_bytes=4 << 20)
    bpt = probe.info()["bytes_per_token"]
    probe.close()
    req_off, req_feat = _events(torch, [20] * 60, seed=1)       # 60 entries, more than 20
    short = configs.Schedule(configs.EULER, 3)
    srv = fmd.Server(m, hbm_budget_bytes=bpt * (2048 + 256 + 8))
    assert srv.info()["pool_tokens"] + 256 <= 8000
    got, _ = srv.wait(srv.submit(req_off, req_feat.cpu().numpy(), 9, short))
    srv.close()
    again = m.simulate(off, feat, 3, sched)                     # another output buffer
    assert torch.equal(first, again)
    assert np.array_equal(got, m.simulate(req_off, req_feat, 9, short).cpu().numpy())
    assert torch.equal(first, m.simulate(off, feat, 3, sched))
    m.close()


@pytest.mark.parametrize("cfg", [CFG, configs.BASE_MODEL.with_precision(configs.BF16)],
                         ids=["small-fp32", "base-bf16"])
def test_a_workspace_that_could_not_grow_is_grown_by_the_next_call(cfg):
    """A server whose pool no device can hold is refused with the workspace half exchanged (the
    first buffer is already given up). The model's next calls get their buffers back."""
    torch, fmd = torch_cuda(), fmd_lib()
    m = fmd.Model(cfg, params.draw(cfg, 5, perturbed=True))
    off, feat = _events(torch, [30] * 20)
    sched = configs.Schedule(configs.RK4, 4)
    first = m.simulate(off, feat, 3, sched)
    t = torch.full((20,), 0.25, device="cuda")
    v = m.velocity(off, feat, first, t)
    torch.cuda.synchronize()
    with pytest.raises(fmd.FmdError) as e:
        fmd.Server(m, hbm_budget_bytes=1 << 48)       # its ODE state alone is above 1 TiB
    assert e.value.status == fmd.E_NOMEM
    assert torch.equal(m.simulate(off, feat, 3, sched), first)
    assert torch.equal(m.velocity(off, feat, first, t), v)
    m.close()


def test_time_embeddings_of_a_long_schedule_are_bounded():
    """A schedule of 60,000 stages needs 16 bytes of the stage table each (0.96 MB); the time
    embeddings, 256 bytes a stage at this width, are formed 1,024 stages at a time instead of
    taking 15 MB more. The device's free memory moves by less than 6 MB (allocations come in units
    of 2 MB), and a short call afterwards is unchanged."""
    torch, fmd = torch_cuda(), fmd_lib()
    m = fmd.Model(CFG, params.draw(CFG, 5, perturbed=True))
    off, feat = _events(torch, [3, 2])
    out = torch.empty((5, 9), device="cuda")
    short = m.simulate(off, feat, 3, configs.Schedule(configs.EULER, 20)).clone()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    m.simulate(off, feat, 3, configs.Schedule(configs.EULER, 60000), out=out)
    torch.cuda.synchronize()
    assert free - torch.cuda.mem_get_info()[0] < 6 << 20
    assert torch.isfinite(out).all()
    assert torch.equal(m.simulate(off, feat, 3, configs.Schedule(configs.EULER, 20)), short)
    m.close()


@pytest.mark.parametrize("graphs", [True, False])
def test_a_schedule_longer_than_the_time_rows_matches_the_oracle(graphs):
    """1,100 Euler stages (two sets of time embeddings) on one event, against the oracle within
    the bar of the FP32 parity tests."""
    torch, fmd = torch_cuda(), fmd_lib()
    cfg = configs.ModelCfg(d_model=64, n_blocks=1, n_heads=4, n_max=64)
    flat = params.draw(cfg, 6, perturbed=True)
    off, feat = _events(torch, [3], seed=4)
    sched = configs.Schedule(configs.EULER, 1100)
    m = fmd.Model(cfg, flat)
    m.graphs_enable(graphs)
    got = m.simulate(off, feat, 8, sched).cpu().numpy()
    m.close()
    ref = sample.simulate(flat, cfg, off, feat.cpu().numpy(), sched, seed=8)
    assert errors.normwise_rel_err(got, ref).max() < 1e-4


@pytest.mark.parametrize("cfg,stats,encoding", [
    (configs.BASE_MODEL.with_precision(configs.BF16), 8, 0),        # k_truth_kv keeps the encoding
    (configs.BASE_MODEL, 0, 1),                                     # split products: own statistics
    (configs.ModelCfg(d_model=128, n_blocks=2, n_heads=4, n_max=64, precision=configs.BF16), 8, 1),
    (configs.ModelCfg(d_model=320, n_blocks=1, n_heads=10, n_max=64), 8, 1)],
    ids=["base-bf16", "base-fp32", "d128-bf16", "d320-fp32"])
def test_a_row_of_the_server_pool_costs_the_buffers_the_model_uses(cfg, stats, encoding):
    """bytes_per_token is the sum of a row's buffers: three state arrays of 16 floats, the residual
    row, its event index, Q/K/V, attention output, cross query, hidden layer, cross K/V of every
    block, features and output; the LayerNorm statistics and the rows of the truth encoding only
    where the model has them. The device memory of a pool of a gibibyte is that per row, within 2%."""
    torch, fmd = torch_cuda(), fmd_lib()
    m = fmd.Model(cfg, params.draw(cfg, 0))
    d, es = cfg.d_model, 2 if cfg.precision == configs.BF16 else 4
    row = 3 * 64 + 4 * d + 4 + 9 * d * es + 2 * d * cfg.n_blocks * es + 72 + stats + encoding * d * es
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    srv = fmd.Server(m, hbm_budget_bytes=1 << 30)
    used = free - torch.cuda.mem_get_info()[0]
    info = srv.info()
    assert info["bytes_per_token"] == row
    assert 0.98 < used / (row * (info["pool_tokens"] + 256)) < 1.02, used
    off, feat = events.truth_events(5, ("uniform", 1, 50), seed=8)
    sched = configs.Schedule(configs.EULER, 3)
    got, _ = srv.wait(srv.submit(off, feat, 9, sched))
    srv.close()
    assert np.array_equal(got, m.simulate(off, feat, 9, sched))
    m.close()
