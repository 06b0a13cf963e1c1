"""Rates where the lanes that share a particle's pairs change (4, 2, 1), with
neighbourhoods that end inside a group of lanes, against the oracle: the
dimensionless rates bit for bit (the additions stay in slot order), the
physical ones to 1e-12, and the sum over the pairs exactly in both forms (the
single-precision pairs themselves are compared in the tests of that form)."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from paper_2609_35967_amd import Engine

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [7, 49_152, 49_153, 98_304, 98_305])
@pytest.mark.parametrize("name, k, fp32", [("additive_col", 3, 0), ("additive_col", 33, 0), ("disk3d_warm", 6, 0),
                                           ("disk3d_warm", 33, 0), ("disk3d_warm", 33, 1)])
def test_lanes(n, name, k, fp32):
    params, st = workloads.by_name(name, 4, n)
    params = dict(params, k=min(k, n), rates_fp32=fp32)
    g = np.random.Generator(np.random.PCG64(n))
    st["M"] = np.where(g.random(n) < 0.05, 0.0, st["M"])
    st["M"][:3] = 1.0 / n
    eng = Engine(params, st, seed=1)
    eng.build_neighbors()
    lp = torch.empty((n, params["k"]), dtype=torch.float64, device="cuda")
    ab = torch.empty((2, n), dtype=torch.float64, device="cuda")
    eng.collision_rates(lam_pair=lp, ab=ab)
    torch.cuda.synchronize()
    s = eng.state_numpy()
    na = int(eng.n_active.item())
    q = np.unique(np.concatenate([g.integers(0, n, min(n, 2000)), [0, na - 1, n - 1]]))
    P = oracle.make_problem(params)
    lam, a, b, pairs = oracle.rates(P, eng.nbr.cpu().numpy(), eng.cnt.cpu().numpy(), eng.dmax.cpu().numpy(), s["m"],
                                    s["M"], s["x"], s["y"], s["z"], want_pairs=True, queries=q)
    got = [eng.lam.cpu().numpy()[q], lp.cpu().numpy()[q], ab[0].cpu().numpy()[q], ab[1].cpu().numpy()[q]]
    if name == "additive_col":
        assert np.array_equal(got[0], lam) and np.array_equal(got[1], pairs)
        np.testing.assert_allclose(got[2], a, rtol=1e-12, atol=1e-300)
        np.testing.assert_allclose(got[3], b, rtol=1e-12, atol=1e-300)
    elif not fp32:
        for x, y in zip(got, (lam, pairs, a, b)):
            np.testing.assert_allclose(x, y, rtol=1e-12, atol=1e-300)
    # lambda*_i is the sum of the pair rates in slot order, rounding by rounding
    total = np.zeros(len(q))
    for j in range(params["k"]):
        total = total + got[1][:, j]
    assert np.array_equal(got[0], total)
    assert eng.status() & 0x21 == 0
