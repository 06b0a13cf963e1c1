"""The sampling calls of one workspace in any order: a deferred call that no
table run and no audit followed leaves the next sampling, of either form, as
if it had not been made."""
import ctypes as C

import pytest
import torch

import workloads
from paper_2609_35967_amd import Engine

pytestmark = pytest.mark.gpu


def _engine(n, k, kernel):
    if kernel == "physical":
        params, st = workloads.by_name("disk3d_warm", 4, n)
    else:
        params, st = workloads.by_name("additive_col", 4, n)
    eng = Engine(dict(params, k=k, eps=1.0), st, seed=8)
    eng.build_neighbors()
    eng.collision_rates()
    return eng


@pytest.mark.parametrize("then", ["direct", "table"])
@pytest.mark.parametrize("kernel", ["additive", "physical"])
@pytest.mark.parametrize("n, k", [(777, 20), (3001, 48)])
def test_abandoned_deferred_call(n, k, kernel, then):
    ref = _engine(n, k, kernel)
    ref.sample_collisions()
    eng = _engine(n, k, kernel)
    sz = C.c_size_t()
    assert eng.lib.gd_sample_table_size(2, C.byref(sz)) == 0
    tab = torch.empty(sz.value, dtype=torch.uint8, device="cuda")
    for _ in range(3):
        eng.sample_deferred(tab.data_ptr(), sz.value, 1)
    if then == "direct":
        eng.sample_collisions()
    else:
        eng.sample_deferred(tab.data_ptr(), sz.value, 0)
        assert eng.lib.gd_sample_table_run(C.c_void_p(tab.data_ptr()), sz.value, 1, k, 0, eng._s()) == 0
        eng.sample_audit()
    torch.cuda.synchronize()
    assert int(ref.events.sum()) > n // 4
    assert torch.equal(eng.events, ref.events) and torch.equal(eng.A.m(), ref.A.m())
    assert eng.interval_state() == ref.interval_state()
    eng.collision_rates()
    eng.sample_collisions()
    ref.collision_rates()
    ref.sample_collisions()
    torch.cuda.synchronize()
    assert torch.equal(eng.events, ref.events) and torch.equal(eng.A.m(), ref.A.m())
    assert eng.status() & 0x21 == 0
