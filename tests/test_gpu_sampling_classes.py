"""Sampling of short, long and very long chains side by side: particles that
expect fewer than 16 events, up to 1024, and more are listed apart and run by
different loops.  Sets just below and above the sizes up to which a run alone
sends all but the short ones to the last of them, alone and in the many-run
form, against the oracle: events exactly outside near-ties; masses to 1e-12
an event, the bound of a single event's outcome."""
import functools

import numpy as np
import pytest
import torch

import oracle
import workloads
from paper_2609_35967_amd import Engine
from paper_2609_35967_amd.binding import ManyRuns

pytestmark = pytest.mark.gpu

CASES = [(1500, 17, 16.0), (1500, 32, 16.0), (1500, 48, 16.0), (1500, 128, 16.0), (1500, 200, 16.0), (8192, 32, 16.0),
         (8193, 32, 16.0), (9001, 17, 16.0), (32768, 48, 4.0), (32769, 48, 4.0), (33001, 100, 4.0)]


def _engine(n, k, dense, **kw):
    params, st = workloads.by_name("disk3d_warm", 12, n)
    st["M"] = st["M"] * dense
    return Engine(dict(params, k=k, eps=1.0), st, seed=6, device_interval=True, **kw)


@functools.lru_cache(maxsize=None)
def _alone(n, k, dense):
    """Masses and events of the first interval, checked against the oracle."""
    eng = _engine(n, k, dense)
    eng.build_neighbors()
    eng.collision_rates()
    s = eng.state_numpy()
    dt = eng.interval_state()["dt_exe"]
    x = eng.lam.cpu().numpy() * dt
    sizes = [int(((x >= a) & (x < b)).sum()) for a, b in ((0.1, 16.0), (16.0, 1024.0), (1024.0, np.inf))]
    print("[gpu]", n, k, "chains", sizes, flush=True)
    assert sizes[0] > 500 and sizes[1] > 50 and sizes[2] > 2
    eng.sample_collisions()
    torch.cuda.synchronize()
    m, ev = eng.A.m().cpu().numpy(), eng.events.cpu().numpy()
    P = oracle.make_problem(eng.params)
    res = oracle.mc(P, s["id"], eng.nbr.cpu().numpy(), eng.cnt.cpu().numpy(), eng.dmax.cpu().numpy(), s["m"], s["M"],
                    s["x"], s["y"], s["z"], dt, 6, 0)
    ok = ~res["near_tie"]
    assert ok.sum() > 0.99 * n and (ev[ok] > 1024).any()
    assert np.array_equal(ev[ok], res["events"][ok])
    err = np.abs(m - res["m"]) / res["m"]
    assert (err <= 1e-12 * (1 + ev))[ok].all()
    assert eng.interval_state()["n_events"] == ev.sum()
    assert eng.status() & 0x21 == 0
    return m, ev


@pytest.mark.parametrize("n, k, dense", CASES)
def test_alone(n, k, dense):
    _alone(n, k, dense)


@pytest.mark.parametrize("ks", [(1, 17, 32), (33, 64), (65, 128), (129, 256)])
def test_many(ks):
    cases = [c for c in CASES if ks[0] <= c[1] <= ks[-1]]
    many = [_engine(*c) for c in cases]
    ManyRuns(many).interval()
    torch.cuda.synchronize()
    for c, e in zip(cases, many):
        m, ev = _alone(*c)
        assert np.array_equal(e.A.m().cpu().numpy(), m) and np.array_equal(e.events.cpu().numpy(), ev), c
        assert e.status() & 0x21 == 0, c
