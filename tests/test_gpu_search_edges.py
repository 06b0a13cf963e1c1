"""The wavefront-per-query search at its edges: neighbourhoods just beyond the
shared lists, at the change of list length, and sets smaller than k, against
brute force (exact lists; distances within one rounding)."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from paper_2609_35967_amd import Engine

pytestmark = pytest.mark.gpu


def _check(params, st):
    eng = Engine(params, st, seed=3)
    for _ in range(2):  # without previous distances, then with them
        eng.build_neighbors()
        torch.cuda.synchronize()
        s = eng.state_numpy()
        P = oracle.make_problem(params)
        nbr, cnt, dmax = oracle.knn(P, s["x"], s["y"], s["z"], s["M"])
        assert np.array_equal(eng.cnt.cpu().numpy(), cnt)
        assert np.array_equal(eng.nbr.cpu().numpy(), nbr)
        np.testing.assert_allclose(eng.dmax.cpu().numpy(), dmax, rtol=1e-15)
    assert eng.status() & 0x21 == 0


@pytest.mark.parametrize("k", [34, 48, 64, 65, 129, 130])
@pytest.mark.parametrize("n", [37, 130, 3001])
def test_disk(k, n):
    params, st = workloads.by_name("disk3d", 5, n)
    _check(dict(params, k=k), st)


@pytest.mark.parametrize("k", [40, 64, 129])
def test_many_equal_distances(k):
    """A lattice: shells of equal distance larger than the bin the ranking takes."""
    st = workloads.lattice_box(13)
    _check(dict(workloads.const_box_params(13 ** 3, k=k)), st)


@pytest.mark.parametrize("k", [50, 200])
def test_clustered_first_search(k):
    """Dense clumps in a sparse set: the first radius holds far more than the list."""
    g = np.random.Generator(np.random.PCG64(11))
    n = 4000
    c = g.random((3, 8))
    p = np.where(g.random(n) < 0.9, c[:, g.integers(0, 8, n)] + 1e-4 * g.standard_normal((3, n)), g.random((3, n))) % 1.0
    st = dict(id=np.arange(n, dtype=np.uint32), x=p[0], y=p[1], z=p[2], M=np.full(n, 1.0 / n), m=np.ones(n))
    _check(dict(workloads.const_box_params(n, k=k)), st)


@pytest.mark.parametrize("hint", [None, 0.6, 1.0, 1.5, 2.5])
@pytest.mark.parametrize("name, n, k", [("disk3d", 160_001, 32), ("disk3d", 163_841, 33), ("disk3d", 200_003, 5),
                                        ("const_box", 400_001, 32), ("additive_col", 400_003, 32),
                                        ("additive_col", 400_100, 20)])
def test_tiles(name, n, k, hint):
    """The shared tiles just above the sizes they start at, with previous
    distances absent, short and long, inactive slots among the others:
    open, periodic on every axis (groups at the faces meet several images)
    and on two, against brute force for sampled rows."""
    params, st = workloads.by_name(name, 9, n)
    params = dict(params, k=k)
    g = np.random.Generator(np.random.PCG64(n))
    st["M"] = np.where(g.random(n) < 0.05, 0.0, st["M"])
    eng = Engine(params, st, seed=3)
    eng.build_neighbors()
    if hint is not None:
        eng.dmax.mul_(hint)
        eng.build_neighbors()
    torch.cuda.synchronize()
    s = eng.state_numpy()
    na = int(eng.n_active.item())
    face = np.flatnonzero(np.minimum(s["x"][:na], s["y"][:na]) < 0.02 * abs(s["x"][:na]).max())
    q = np.concatenate([g.choice(na, 300, replace=False), g.choice(face, 200), [0, na - 1, na, n - 1]])
    P = oracle.make_problem(params)
    nbr, cnt, dmax = oracle.knn(P, s["x"], s["y"], s["z"], s["M"], queries=q)
    assert np.array_equal(eng.cnt.cpu().numpy()[q], cnt)
    assert np.array_equal(eng.nbr.cpu().numpy()[q], nbr)
    np.testing.assert_allclose(eng.dmax.cpu().numpy()[q], dmax, rtol=1e-15)
    assert eng.status() & 0x21 == 0


@pytest.mark.parametrize("kept", ["one in 50", "blocks 1 to 15 of 16", "block 0"])
@pytest.mark.parametrize("name, n", [("disk3d", 163_841), ("additive_col", 400_003)])
def test_some_previous_distances(name, n, kept):
    """Previous distances for a part of the particles only: the search that a
    sample of them picks finds the same lists as with all of them."""
    params, st = workloads.by_name(name, 9, n)
    eng = Engine(params, st, seed=3)
    eng.build_neighbors()
    eng.build_neighbors()
    want = [t.clone() for t in (eng.nbr, eng.cnt, eng.dmax)]
    i = torch.arange(n, device=eng.dmax.device)
    keep = {"one in 50": i % 50 == 7, "blocks 1 to 15 of 16": (i // 256) % 16 != 0, "block 0": i < 256}[kept]
    eng.dmax.mul_(keep)
    eng.build_neighbors()
    for a, b in zip((eng.nbr, eng.cnt, eng.dmax), want):
        assert torch.equal(a, b)
    assert eng.status() & 0x21 == 0
