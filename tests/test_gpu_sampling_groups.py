"""Sampling where the lanes per particle change (half a wavefront up to k = 32,
a whole one beyond, several slots a lane above 64), with lists of odd length,
chains longer than the draws made at a time and none at all, against the
oracle: events, partners and channels exactly outside near-ties, masses to
1e-12 (the tolerance of the physical rates); the many-run table form gives the
same bits."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from paper_2609_35967_amd import Engine
from paper_2609_35967_amd.binding import ManyRuns

pytestmark = pytest.mark.gpu


def _engine(params, st, **kw):
    eng = Engine(params, st, seed=6, **kw)
    eng.build_neighbors()
    return eng


@pytest.mark.parametrize("k", [2, 17, 31, 32, 33, 64, 65, 200])
@pytest.mark.parametrize("n, eps", [(3, 1.0), (257, 4.0), (3001, 0.3), (3001, 1e-9)])
def test_sampling(k, n, eps):
    params, st = workloads.by_name("disk3d_warm", 12, n)
    st["M"] = st["M"] * (n / 2.0 ** 20)  # as dense in grains as the million-particle disk
    params = dict(params, k=min(k, n), eps=eps)
    eng = _engine(params, st)
    eng.collision_rates()
    s = eng.state_numpy()
    log = torch.full((n, 40), -1, dtype=torch.int32, device="cuda")
    dt = eng.interval_state()["dt_exe"]
    eng.sample_collisions(log=log, log_cap=40, flip=False)
    torch.cuda.synchronize()
    P = oracle.make_problem(params)
    res = oracle.mc(P, s["id"], eng.nbr.cpu().numpy(), eng.cnt.cpu().numpy(), eng.dmax.cpu().numpy(), s["m"], s["M"],
                    s["x"], s["y"], s["z"], dt, 6, 0, log_cap=40)
    ok = ~res["near_tie"]
    m_new = eng.A.t["m1" if eng.A.cur == 0 else "m0"].cpu().numpy()
    ev, lg = eng.events.cpu().numpy(), log.cpu().numpy()
    assert np.array_equal(ev[ok], res["events"][ok])
    np.testing.assert_allclose(m_new[ok], res["m"][ok], rtol=1e-12, atol=0)
    assert np.array_equal(np.where(lg >= 0, lg & 0xFFFF, -1)[ok], res["log_slot"][ok])
    assert np.array_equal(np.where(lg >= 0, (lg >> 16) & 0xFF, -1)[ok], res["log_chan"][ok])
    assert eng.interval_state()["n_events"] == ev.sum()
    assert eng.status() & 0x21 == 0


def test_many_runs_give_the_same_bits():
    runs = [("disk3d_warm", 1501, 32), ("disk3d_warm", 777, 20), ("disk3d", 300, 33), ("disk3d_warm", 2000, 48)]
    alone, many = [], []
    for name, n, k in runs:
        params, st = workloads.by_name(name, 12, n)
        params = dict(params, k=k, eps=1.0)
        alone.append(Engine(params, st, seed=6, device_interval=True))
        many.append(Engine(params, st, seed=6, device_interval=True))
    M = ManyRuns(many)
    for _ in range(4):
        M.interval()
        for e in alone:
            e.step()
    torch.cuda.synchronize()
    for a, b in zip(alone, many):
        assert torch.equal(a.events, b.events) and torch.equal(a.A.m(), b.A.m())
        assert a.interval_state()["n_events"] == b.interval_state()["n_events"]
