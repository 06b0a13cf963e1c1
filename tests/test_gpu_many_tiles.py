"""Many runs stepped as one above the total size from which the search goes
through the shared tiles (160,000 open particles, 400,000 periodic ones),
small runs among them (so few that the wavefronts of their hand-back pass are
fewer than the dies): every run bit-equal to itself alone, in its first search,
in later ones with positions moved, and with previous distances too short for
most queries (which are then handed back)."""
import pytest
import torch

import workloads
from paper_2609_35967_amd import Engine
from paper_2609_35967_amd.binding import ManyRuns

pytestmark = pytest.mark.gpu

RUNS = {
    "disk3d_warm": [(150_001, 32), (1024, 32), (300, 20), (1793, 33), (1152, 8), (9001, 32)],
    "additive_col": [(390_007, 32), (1024, 32), (1452, 17), (7169, 33), (3000, 32)],
}


@pytest.mark.parametrize("fallback_div", [64, 256, 1024])
@pytest.mark.parametrize("name", sorted(RUNS))
def test_runs_match_alone(name, fallback_div):
    alone, many = [], []
    for n, k in RUNS[name]:
        params, st = workloads.by_name(name, 21, n)
        if name == "disk3d_warm":
            st["M"] = st["M"] * (n / 2.0 ** 20)  # as dense in grains as the million-particle disk
        params = dict(params, k=k)
        alone.append(Engine(params, st, seed=n, device_interval=True))
        many.append(Engine(params, st, seed=n, device_interval=True))
    runs = ManyRuns(many, dict(fallback_div=fallback_div))
    for it in range(4):
        print("[gpu]", name, fallback_div, "interval", it, flush=True)
        if it == 3:
            for e in alone + many:
                e.dmax.mul_(0.6)
        for e in alone:
            e.step()
        runs.interval()
        torch.cuda.synchronize()
        for a, b in zip(alone, many):
            where = (name, fallback_div, it, a.n)
            assert torch.equal(a.nbr, b.nbr) and torch.equal(a.cnt, b.cnt) and torch.equal(a.dmax, b.dmax), where
            assert torch.equal(a.A.t["id"], b.A.t["id"]) and torch.equal(a.A.m(), b.A.m()), where
            assert torch.equal(a.A.t["z"], b.A.t["z"]) and torch.equal(a.events, b.events), where
            assert b.status() & 0x21 == 0, where
