"""The division kernels of small, middle and large batches give the same results.

Up to three instances per compute unit share their quotient products among four
waves, batches of one round of 256-thread workgroups run kernels with more
registers, larger ones a third kind.  The same operands, at the lengths where
blocks and strips end, repeated to batches of each kind, against the oracle."""
import random

import numpy as np
import pytest

import oracle
from paper_2606_06386_amd import inputs as I

pytestmark = pytest.mark.gpu
B = 1 << 32


def _operands(d, k):
    rng = random.Random(1000 * d + k)
    h = d + k
    us, vs = [], []
    for v in (rng.getrandbits(32 * k + 32) | 1 << (32 * k + 31), B ** k + 1, B ** (k + 1) - 1, B ** k + rng.getrandbits(32 * k)):
        w = rng.getrandbits(32 * max(d - 1, 1)) | 1
        for u in (rng.getrandbits(32 * h) | 1 << (32 * h - 1), B ** h - 1, v * w + v - 1, v * w, v - 1):
            us.append(min(u, B ** h - 1))
            vs.append(v)
    return us, vs, h


# quotient limbs at the ends of one and two blocks (and of those whose carries may be late), divisors of one to three strips
@pytest.mark.parametrize("d,k", [(1, 1), (8, 3), (39, 60), (132, 254), (243, 255), (244, 247), (245, 300), (252, 260),
                                 (253, 510), (504, 247), (505, 520), (1030, 700), (1, 1020)])
@pytest.mark.parametrize("per_cu", [0, 3, 4, 5])
def test_every_kind_of_batch(d, k, per_cu):
    import torch
    from paper_2606_06386_amd import binding
    us, vs, h = _operands(d, k)
    n = max(len(us), per_cu * torch.cuda.get_device_properties(0).multi_processor_count)
    u, v = (np.stack([I.from_int(x, w) for x in xs]) for xs, w in ((us, h), (vs, k + 1)))
    rows = torch.arange(n, device="cuda") % len(us)
    dev = [torch.from_numpy(x.view(np.int32)).cuda()[rows].contiguous() for x in (u, v)]
    got = [x.cpu().numpy().view(np.uint32) for x in binding.divrem(dev[0], dev[1], nq=d + 1)]
    want = oracle.divrem(u, v, nq=d + 1, nr=k + 1)
    rows = rows.cpu().numpy()
    for g, w, name in zip(got, want, ("quotient", "remainder", "status")):
        assert (g == np.asarray(w).view(np.uint32)[rows]).all(), name


# wide operands: divisors on both sides of the length up to which large batches take half the waves
@pytest.mark.parametrize("d,k", [(1990, 300), (300, 1789), (300, 1790), (260, 3837), (260, 3838), (4000, 500)])
@pytest.mark.parametrize("per_cu", [1, 3])
def test_wide_batches(d, k, per_cu):
    test_every_kind_of_batch(d, k, per_cu)


@pytest.mark.parametrize("nu,nv,batch", [(100, 8192, 2), (2048, 8192, 1100), (600, 2100, 3)])
def test_divisor_rows_wider_than_the_dividend(nu, nv, batch):
    import torch
    from paper_2606_06386_amd import binding
    rng = random.Random(nv)
    us = [rng.getrandbits(32 * nu) | 1 for _ in range(3)]
    vs = [rng.getrandbits(32 * n) | 1 << (32 * n - 1) for n in (5, nu // 2, min(nv, nu + 1))]
    rows = np.arange(batch) % 3
    u, v = (np.stack([I.from_int(x, w) for x in xs])[rows] for xs, w in ((us, nu), (vs, nv)))
    q, r, st = (x.cpu().numpy().view(np.uint32) for x in binding.divrem(
        torch.from_numpy(u.view(np.int32)).cuda(), torch.from_numpy(v.view(np.int32)).cuda()))
    for j in range(3):
        want = divmod(us[j], vs[j])
        for row in (np.nonzero(rows == j)[0][[0, -1]] if batch > j else []):
            assert st[row] == 0 and (q[row] == I.from_int(want[0], nu)).all() and (r[row] == I.from_int(want[1], nv)).all()
