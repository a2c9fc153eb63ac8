"""Serving in batches large enough for the class kernels: the same answers as in
small ones, and a sample of them the oracle's."""
import numpy as np
import pytest

import oracle
from paper_2606_06386_amd import inputs as I

pytestmark = pytest.mark.gpu


def test_large_batches_give_the_answers_of_small_ones():
    import torch
    from paper_2606_06386_amd import serve
    small = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    c = I.config_c5(1e8, count=1600)                       # (all arrive within the first launches)
    a = serve.serve(c["u"], c["v"], c["arrival"], max_batch=4096, depth=2)
    b = serve.serve(c["u"], c["v"], c["arrival"], max_batch=64, depth=2)
    assert max(a["batches"]) > small >= max(b["batches"])
    qa, ra, sa = a["requests"].results()
    qb, rb, sb = b["requests"].results()
    assert (sa == 0).all() and (sb == 0).all()
    assert all((x == y).all() for x, y in zip(qa, qb)) and all((x == y).all() for x, y in zip(ra, rb))
    for j in range(0, 1600, 41):
        u, v = c["u"][j], c["v"][j]
        qo, ro, so = oracle.divrem(u[None, :], v[None, :], nq=len(u), nr=len(v))
        assert so[0] == 0 and (qa[j] == qo[0]).all() and (ra[j] == ro[0]).all(), j
