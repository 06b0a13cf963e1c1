"""The frozen neighbourhood: gd_collision_rates keeps a copy of the masses in
the workspace, and what follows reads the neighbours from that copy, for every
kernel.  Masses that change in m[cur] after the rates call change no other
particle's sampling, and a spatial group's rates without a new snapshot
(snapshot = 0) see the same neighbours as the whole set's."""
import ctypes as C

import pytest
import torch

import workloads
from paper_2609_35967_amd import Engine

pytestmark = pytest.mark.gpu

KERNELS = ["const", "additive", "product", "physical"]


def _engine(kernel, n, k, **kw):
    if kernel == "physical":
        params, st = workloads.by_name("disk3d_warm", 4, n)
    else:
        params, st = workloads.by_name("additive_col", 4, n)
        params = dict(params, kernel=kernel)
    eng = Engine(dict(params, k=k, eps=1.0, **kw), st, seed=8)
    eng.build_neighbors()
    return eng


@pytest.mark.parametrize("table", [False, True])
@pytest.mark.parametrize("fp32", [0, 1])
@pytest.mark.parametrize("kernel", KERNELS)
@pytest.mark.parametrize("n, k", [(3001, 20), (70_001, 40), (100_001, 32)])
def test_sampling_reads_the_copy(kernel, fp32, n, k, table):
    out = []
    for edit in (False, True):
        eng = _engine(kernel, n, k, rates_fp32=fp32)
        odd = eng.A.t["id"] % 2 == 1
        eng.collision_rates()
        if edit:  # (the odd particles' own start state, and nothing else)
            eng.A.m().mul_(torch.where(odd, 3.0, 1.0))
        if table:
            sz = C.c_size_t()
            assert eng.lib.gd_sample_table_size(1, C.byref(sz)) == 0
            tab = torch.empty(sz.value, dtype=torch.uint8, device="cuda")
            eng.sample_deferred(tab.data_ptr(), sz.value, 0)
            assert eng.lib.gd_sample_table_run(C.c_void_p(tab.data_ptr()), sz.value, 1, k, fp32, eng._s()) == 0
            eng.sample_audit()
        else:
            eng.sample_collisions()
        torch.cuda.synchronize()
        assert eng.status() & 0x21 == 0
        out.append((eng.A.m().clone(), eng.events.clone(), odd))
    (m0, e0, odd), (m1, e1, _) = out
    assert int(e0[~odd].sum()) > 100
    assert torch.equal(e0[~odd], e1[~odd]) and torch.equal(m0[~odd], m1[~odd])


@pytest.mark.parametrize("kernel", KERNELS)
@pytest.mark.parametrize("n", [3001, 70_001, 100_001])
def test_group_rates_on_the_whole_sets_copy(kernel, n):
    eng = _engine(kernel, n, 32)
    eng.set_groups(1)
    eng._group_layout()
    rows, sched = C.c_void_p(eng.gmask.data_ptr()), C.c_void_p(eng.gsched.data_ptr())
    ws = C.c_void_p(eng.ws_ptr)
    own = eng.A.m().clone()
    eng.A.m().mul_(2.0)
    eng._rates_group(0, eng.group_lo, rows, sched, True, ws, eng._s())  # a copy of other masses
    eng.A.m().copy_(own)
    eng.collision_rates()
    whole = eng.lam.clone()
    eng.lam.zero_()
    eng._rates_group(0, eng.group_lo, rows, sched, False, ws, eng._s())
    torch.cuda.synchronize()
    assert torch.equal(eng.lam[:eng.group_lo[1]], whole[:eng.group_lo[1]])
    assert eng.status() & 0x21 == 0
