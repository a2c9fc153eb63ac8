"""Block division at the sizes where its splits change, against the oracle.

The quotient's d = h - k limbs are found in blocks of at most 252 limbs, the
remainder is updated in strips of 256 columns of k + 2 limbs, digits are
converted in rows of 64 limbs and 8-limb blocks, and the inverse's precision
follows the longest block.  Quotient and divisor lengths on both sides of each
of these, one-limb divisors, and quotients one limb longer than their row;
random and structured operands, bit-exact."""
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


def _dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.uint32).view(np.int32)).cuda()


def _divisors(rng, k):
    """divisors of k + 1 limbs"""
    rnd = rng.getrandbits(32 * k + 32) | 1
    return [rnd | 1 << (32 * k + 31), B ** k + rnd % B ** k, B ** k + 1, B ** (k + 1) - 1, B ** k + B ** k // 2 + 1]


def _cases(rng, d, k):
    h = d + k
    out = []
    for v in _divisors(rng, k):
        w = rng.getrandbits(32 * max(d - 1, 1)) | 1
        out += [(rng.getrandbits(32 * h) | 1 << (32 * h - 1), v), (B ** h - 1, v), (min(v * w + v - 1, B ** h - 1), v),
                (min(v * w, B ** h - 1), v)]
    return out


def _check(mp, u, v, nq, label):
    import torch
    q, r, st = mp.divrem(_dev(u), _dev(v), nq=nq)
    torch.cuda.synchronize()
    q, r, st = q.cpu().numpy().view(np.uint32), r.cpu().numpy().view(np.uint32), st.cpu().numpy()
    qo, ro, so = oracle.divrem(u, v, nq=nq, nr=v.shape[1])
    bad = [j for j in range(len(u)) if st[j] != so[j] or (q[j] != qo[j]).any() or (r[j] != ro[j]).any()]
    assert not bad, f"{label}: {len(bad)} mismatching instances {bad[:8]}, status {st[bad[:8]]}"


def _stack(vals, n):
    return np.stack([I.from_int(x, n) for x in vals])


# quotient lengths around one, two, three and four blocks (and the even split of the rest)
@pytest.mark.parametrize("d", [1, 2, 3, 4, 17, 255, 256, 257, 258, 259, 513, 514, 515, 769, 770, 1025, 1026, 1030])
def test_quotient_lengths(mp, d):
    rng = random.Random(d)
    for k in (1, 62, 255, 700):
        c = _cases(rng, d, k)
        _check(mp, _stack([u for u, _ in c], d + k), _stack([v for _, v in c], k + 1), d, f"d={d} k={k}")


# divisor lengths around rows, blocks and strips (k + 2 limbs are updated)
@pytest.mark.parametrize("k", [0, 1, 2, 6, 7, 8, 61, 62, 63, 64, 253, 254, 255, 256, 510, 511, 1021, 1022, 1023, 2046])
def test_divisor_lengths(mp, k):
    rng = random.Random(100 + k)
    for d in (5, 300):
        c = _cases(rng, d, k)
        n = d + k
        _check(mp, _stack([u for u, _ in c], n), _stack([v for _, v in c], k + 1), d, f"k={k} d={d}")
        # the same in wider rows: leading zero limbs in u, v and q
        _check(mp, _stack([u for u, _ in c], n + 5), _stack([v for _, v in c], k + 9), d + 3, f"wide k={k} d={d}")


@pytest.mark.parametrize("nq,nv", [(257, 1024), (257, 257), (40, 12), (12, 40), (8, 8), (26, 20), (27, 20), (300, 3)])
def test_row_widths(mp, nq, nv):
    """Long and short q and r rows; quotients that fit nq limbs, that need one more, and that need many more."""
    rng = random.Random(nq * 1000 + nv)
    k = nv - 1
    us, vs = [], []
    for d in (nq, nq + 1, nq + 2, nq + 40):
        for u, v in _cases(rng, d, k):
            us.append(u)
            vs.append(v)
            us.append(min(v * (B ** min(nq, d) - 1) + v - 1, B ** (d + k) - 1))
            vs.append(v)
    n = nq + 40 + k
    _check(mp, _stack(us, n), _stack(vs, nv), nq, f"nq={nq} nv={nv}")


@pytest.mark.parametrize("h", [1, 26, 256, 257, 300, 1000])
def test_shinv_blocks(mp, h):
    import torch
    rng = random.Random(h)
    vals = [v for k in (0, 1, 5, h // 2, h - 1, h) if k >= 0 for v in _divisors(rng, k)]
    v = _stack(vals, max(h, 5) + 2)
    for nw in (h + 1, max(1, h // 2)):
        w, st = mp.shinv(_dev(v), h, nw=nw)
        torch.cuda.synchronize()
        wo, so = oracle.shinv(v, h, nw=nw)
        assert (st.cpu().numpy() == so).all(), f"shinv h={h} nw={nw}"
        assert (w.cpu().numpy().view(np.uint32) == wo).all(), f"shinv h={h} nw={nw}"
