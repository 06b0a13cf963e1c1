"""Morton order where the radix sort's shape changes (keys per thread, blocks
per group of the digit counts) and the controller's sums where its grid does,
against the oracle: the order and the interval's ticks exactly, the sums to a
few roundings."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from paper_2609_35967_amd import Engine

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 63, 255, 256, 257, 32767, 32768, 32769, 65537, 131073, 262145, 524289, 1048577])
def test_order(n):
    g = np.random.Generator(np.random.PCG64(n))
    p = np.where(g.random(n) < 0.5, g.random((3, n)), np.round(g.random((3, n)) * 8) / 8)  # many equal keys
    M = np.where(g.random(n) < 0.1, 0.0, 1.0 / n)
    M[0] = 1.0 / n
    st = dict(id=np.arange(n, dtype=np.uint32), x=p[0], y=p[1], z=p[2], M=M, m=np.ones(n))
    eng = Engine(dict(workloads.const_box_params(n, k=2), periodic=(0, 0, 0)), st, seed=1)
    for _ in range(2):
        x, y, z, M = (eng.A.t[a].cpu().numpy() for a in ("x", "y", "z", "M"))
        ids = eng.A.t["id"].cpu().numpy()
        eng.build_neighbors()
        torch.cuda.synchronize()
        perm = oracle.sort_perm(oracle.morton_keys(x, y, z, M))
        assert np.array_equal(eng.A.t["id"].cpu().numpy(), ids[perm])
        assert int(eng.n_active.item()) == int((M > 0).sum())


@pytest.mark.parametrize("n", [2, 511, 512, 513, 5000, 131072, 131073, 200001])
@pytest.mark.parametrize("warm", [False, True])
def test_controller_sums(n, warm):
    """Two intervals: the plan's and the audit's sums over one and many blocks."""
    params, st = workloads.by_name("disk3d_warm" if warm else "disk3d", 3, n)
    params = dict(params, k=min(8, n))
    eng = Engine(params, st, seed=2)
    eng.build_neighbors()
    for it in range(2):
        ab = torch.empty((2, n), dtype=torch.float64, device="cuda")
        iv0 = eng.interval_state()
        eng.collision_rates(ab=ab)
        iv = eng.interval_state()
        s = eng.state_numpy()
        a, b = ab.cpu().numpy()
        P = oracle.make_problem(params)
        plan = oracle.plan(P, s["m"], s["M"], a, b, params["dt_coll"], iv0["ticks"], iv0["C"])
        assert iv["exe_ticks"] == plan["exe_ticks"] and iv["n_groups"] == plan["group_of"].max() + 1
        np.testing.assert_allclose(iv["dt_req"], plan["dt_req"], rtol=1e-13)
        eng.sample_collisions()
        m1 = eng.state_numpy()["m"]
        done = eng.interval_state()
        au = oracle.audit(P, s["m"], m1, s["M"], plan["group_of"], plan["gM"], iv0["C"])
        assert done["C"] == au["C"]
        np.testing.assert_allclose(done["audit_worst"], au["worst"], rtol=1e-13, atol=1e-300)
    assert eng.status() & 0x21 == 0
