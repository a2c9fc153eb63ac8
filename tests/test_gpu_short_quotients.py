"""Divisions that need no inverse: quotients that a comparison shows to be 0 or
1, and numbers of up to three limbs by one limb.

Both sides of every condition (the divisor's top limb at 2^31, equal operands,
operands that differ in their lowest limb only, B^h on either side of v and of
2v), quotients one limb longer than their row, in batches of every kind of
kernel, against the oracle; and that they cost less than divisions that do need
an inverse."""
import itertools
import random

import numpy as np
import pytest

import oracle
from paper_2606_06386_amd import inputs as I

pytestmark = pytest.mark.gpu
B = 1 << 32


@pytest.fixture(scope="module")
def mp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2606_06386_amd import binding
    binding.lib()
    return binding


def _stack(vals, n):
    return np.stack([I.from_int(x, n) for x in vals])


def _dev(x, batch):
    """the rows of x, repeated to a batch of at least `batch`"""
    import torch
    rows = torch.arange(max(batch, len(x)), device="cuda") % len(x)
    return torch.from_numpy(x.view(np.int32)).cuda()[rows].contiguous()


def _same(got, want, label):
    for g, w, name in zip(got, want, ("q", "r", "status") if len(want) == 3 else ("w", "status")):
        g = g.cpu().numpy().view(np.uint32)
        w = np.asarray(w).view(np.uint32)
        bad = np.nonzero((g != w[np.arange(len(g)) % len(w)]).reshape(len(g), -1).any(axis=1))[0]
        assert not len(bad), f"{label}: {name} of {len(bad)} instances differ, first {bad[:6]} (operands {bad[:6] % len(w)})"


def _check(mp, u, v, nq, per_cu, label):
    import torch
    n = per_cu * torch.cuda.get_device_properties(0).multi_processor_count
    _same(mp.divrem(_dev(u, n), _dev(v, n), nq=nq), oracle.divrem(u, v, nq=nq, nr=v.shape[1]), label)


@pytest.mark.parametrize("per_cu", [0, 4, 5])
@pytest.mark.parametrize("nu,nv,nq", [(3, 1, 3), (3, 1, 2), (3, 1, 1), (2, 1, 1), (1, 1, 1), (5, 3, 4), (70, 70, 3)])
def test_one_limb_divisors(mp, nu, nv, nq, per_cu):
    rng = random.Random(nu * 100 + nv)
    limbs = [0, 1, 2 ** 31, 2 ** 32 - 1, rng.getrandbits(32)]
    us = [sum(x << (32 * i) for i, x in enumerate(u)) for u in itertools.product(limbs, repeat=min(nu, 4))]
    vs = [1, 2, 3, 2 ** 16 + 1, 2 ** 31 - 1, 2 ** 31, 2 ** 31 + 1, 2 ** 32 - 2, 2 ** 32 - 1, rng.getrandbits(32) | 1]
    pairs = [(u, v) for u in us for v in vs]
    pairs += [(min(v * w + e, B ** min(nu, 3) - 1), v) for v in vs for w in (1, 2 ** 32 - 1, rng.getrandbits(40))
              for e in (0, v - 1)]
    _check(mp, _stack([u for u, _ in pairs], nu), _stack([v for _, v in pairs], nv), nq, per_cu, f"{nu}/{nv} nq={nq}")


@pytest.mark.parametrize("per_cu", [0, 4, 5])
@pytest.mark.parametrize("k", [1, 2, 62, 63, 64, 255, 300, 2047])
def test_operands_of_one_length(mp, k, per_cu):
    rng = random.Random(k)
    low = rng.getrandbits(32 * k)
    vs = [top * B ** k + x for top in (1, 2, 2 ** 31 - 1, 2 ** 31, 2 ** 31 + 1, 2 ** 32 - 1) for x in (0, 1, low, B ** k - 1)]
    pairs = [(u, v) for v in vs for u in (v, v - 1, v + 1, 2 * v - 1, 2 * v, B ** (k + 1) - 1, B ** k, 3 * v + 2)
             if u < B ** (k + 1)]
    u, v = [u for u, _ in pairs], [v for _, v in pairs]
    _check(mp, _stack(u, k + 1), _stack(v, k + 1), 1, per_cu, f"k={k}")
    _check(mp, _stack(u, k + 4), _stack(v, k + 9), 3, per_cu, f"wide k={k}")


@pytest.mark.parametrize("per_cu", [0, 4, 5])
@pytest.mark.parametrize("h", [0, 1, 2, 3, 4, 7, 64, 300])
def test_shinv_of_long_divisors(mp, h, per_cu):
    import torch
    n = per_cu * torch.cuda.get_device_properties(0).multi_processor_count
    rng = random.Random(h)
    vs = [top * B ** k + x for k in {0, max(h - 2, 0), max(h - 1, 0), h, h + 1}
          for top in (1, 2, 2 ** 31 - 1, 2 ** 31, 2 ** 31 + 1, 2 ** 32 - 1)
          for x in ({0, 1, rng.getrandbits(32 * k), B ** k - 1} if k else {0})]
    v = _stack(vs, h + 2)
    for nw in {h + 1, 1, 2, 3}:
        _same(mp.shinv(_dev(v, n), h, nw=nw), oracle.shinv(v, h, nw=nw), f"h={h} nw={nw}")


def _us(fns, reps=40, rounds=8):
    """the shortest mean time of each call, in turn"""
    import torch
    best = [float("inf")] * len(fns)
    for _ in range(rounds):
        for i, f in enumerate(fns):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            f()
            e0.record()
            for _ in range(reps):
                f()
            e1.record()
            e1.synchronize()
            best[i] = min(best[i], e0.elapsed_time(e1) / reps * 1e3)
    return best


def test_cost_below_that_of_an_inverse(mp):
    """By three quarters at most of what the same widths cost where the inverse is needed."""
    rng = random.Random(5)
    rows = lambda xs, n: _dev(_stack(xs, n), 4096)  # noqa: E731
    v64 = [B ** 63 * top + rng.getrandbits(32 * 63) for top in (3, 2 ** 32 - 5)]
    u64 = rows([B ** 64 - 1], 64)
    vr, vn, one = rows(v64[:1], 64), rows(v64[1:], 64), rows([2 ** 31 + 11], 1)
    u4, u3 = rows([B ** 4 - 1], 4), rows([B ** 3 - 1], 3)
    ws = rows([B ** 8 - 3], 9)
    calls = {"64 by 64 limbs, inverse": lambda: mp.divrem(u64, vr, nq=1), "64 by 64 limbs, 0 or 1": lambda: mp.divrem(u64, vn, nq=1),
             "4 limbs by 1": lambda: mp.divrem(u4, one, nq=4), "3 limbs by 1": lambda: mp.divrem(u3, one, nq=3),
             "shinv, h = 11": lambda: mp.shinv(ws, 11), "shinv, h = 8": lambda: mp.shinv(ws, 8), "shinv, h = 7": lambda: mp.shinv(ws, 7)}
    t = dict(zip(calls, _us(list(calls.values()))))
    assert t["64 by 64 limbs, 0 or 1"] < 0.75 * t["64 by 64 limbs, inverse"], t
    assert t["3 limbs by 1"] < 0.75 * t["4 limbs by 1"], t
    assert t["shinv, h = 8"] < 0.75 * t["shinv, h = 11"] and t["shinv, h = 7"] < 0.75 * t["shinv, h = 11"], t
