"""Inverses in batches of every kind of kernel: up to three per compute unit,
one round, several rounds, of 256, 512 and 1024 threads and at half the waves,
against the oracle."""
import random

import numpy as np
import pytest

import oracle
from paper_2606_06386_amd import inputs as I

pytestmark = pytest.mark.gpu
B = 1 << 32


# h, divisor row (on both sides of the length up to which large batches take half the waves), instances per compute unit
@pytest.mark.parametrize("h,nv,per_cu", [
    (2048, 1024, 3), (2048, 1024, 4), (2048, 1024, 5), (300, 12, 4), (300, 12, 5), (1030, 70, 5),
    (2500, 1300, 1), (2500, 1790, 3), (2500, 1791, 3), (4096, 300, 3),
    (4500, 2000, 1), (4500, 3838, 2), (4500, 3839, 2), (8192, 8192, 1), (8192, 8192, 2)])
def test_every_kind_of_batch(h, nv, per_cu):
    import torch
    from paper_2606_06386_amd import binding
    rng = random.Random(h * 10000 + nv)
    ks = [nv - 1, max(nv - 2, 0), nv // 2, max(0, h - 252), max(0, h - 253), max(0, h - 505), 0]
    vals = [v for k in ks if k < nv
            for v in (rng.getrandbits(32 * k + 32) | 1 << (32 * k + 31), B ** k + 1 + k, B ** (k + 1) - 1, B ** k)]
    v = np.stack([I.from_int(x, nv) for x in vals])
    rows = np.arange(per_cu * torch.cuda.get_device_properties(0).multi_processor_count) % len(v)
    for nw in (h + 1, max(1, h - nv // 2)):
        w, st = binding.shinv(torch.from_numpy(v.view(np.int32)).cuda()[torch.from_numpy(rows).cuda()].contiguous(), h, nw=nw)
        wo, so = oracle.shinv(v, h, nw=nw)
        assert (st.cpu().numpy() == so[rows]).all(), f"status nw={nw}"
        bad = np.nonzero((w.cpu().numpy().view(np.uint32) != wo[rows]).any(axis=1))[0]
        assert not len(bad), f"nw={nw}: {len(bad)} instances differ, operands {sorted(set(rows[bad]))[:8]}"
