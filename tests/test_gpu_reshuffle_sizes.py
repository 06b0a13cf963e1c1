"""Relabelling of the neighbours at the sizes where a thread takes more than
one slot of pi's table, inactive particles among the others: every slot of the
table is written (seen through rows of the active particles), against the
oracle's pi."""
import numpy as np
import pytest
import torch

import oracle
import workloads
from paper_2609_35967_amd import Engine

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("static", [False, True])
@pytest.mark.parametrize("n", [131_072, 131_073, 262_145, 1_048_577])
def test_sizes(n, static):
    params, st = workloads.by_name("const_box", 3, n)
    st["M"] = np.where(np.arange(n) % 5 == 2, 0.0, st["M"])
    eng = Engine(dict(params, kernel="product", k=8), st, seed=11)
    eng.build_neighbors()
    torch.cuda.synchronize()
    before, cnt, N = eng.nbr.cpu().numpy(), eng.cnt.cpu().numpy(), int(eng.n_active.item())
    (eng.reshuffle_neighbors_static if static else eng.reshuffle_neighbors)(4)
    torch.cuda.synchronize()
    assert np.array_equal(eng.nbr.cpu().numpy(), oracle.reshuffle(before, cnt, N, 11, 4))
    assert eng.status() & 0x21 == 0
