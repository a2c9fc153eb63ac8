"""Workloads of the batched multi-precision division library, as data.

Each case is a dict of plain values; ``prepare`` makes its device-resident
operands, ``run`` is one call (or launch sequence) through the public binding
``paper_2606_06386_amd.binding``, ``work`` counts the bytes and operations the
result cannot do without, and ``exact`` gives the same results with Python
integers.  ``draw`` gives further cases of the same ranges.

Kinds of case (the binding's four operations):
  divrem   (q, r) of `batch` divisions of one shape: u of nu limbs, v in an
           nv-limb buffer.  vlen "full" fills the buffer; "spread" draws each
           divisor's length uniformly in [vmin, nv] limbs, zero-padded.
           hard = 1 makes every fourth instance adversarial: v = B^nv - 1,
           v = B^(nv-1) + 1, v with top limb 1, u = v w + v - 1, u < v.
  mul      products of na x nb limbs.
  shinv    w = floor(B^h / v), v of nv limbs.
  ragged   (q, r) of `count` divisions of uneven precision from packed pools:
           the dividend's width is one of four classes ("classes") or
           2^x / 32 limbs with x uniform in [15, 18] ("spread"); the
           divisor's length is uniform in [n / part, n].
Limbs are uniformly random with a nonzero top limb; precisions are 2^15 to
2^18 bits (1024 to 8192 limbs of 32 bits), the range of the library.
"""
import math

import numpy as np
import torch

# --------------------------------------------------------------------- cases


def listed():
    return [
        # one division on its own: the latency of a single call
        {"name": "divrem_2p15_one", "kind": "divrem", "nu": 1024, "nv": 512, "batch": 1, "vlen": "full", "hard": 0},
        # the smallest precision of the range, one round of workgroups
        {"name": "divrem_2p15_b1024", "kind": "divrem", "nu": 1024, "nv": 512, "batch": 1024, "vlen": "full",
         "hard": 0},
        # the benchmark's shape, adversarial divisors included
        {"name": "divrem_2p16_b4096", "kind": "divrem", "nu": 2048, "nv": 1024, "batch": 4096, "vlen": "full",
         "hard": 1},
        # random divisors of any length up to half the dividend (long quotients), as a table of random integers has
        {"name": "divrem_2p16_spread", "kind": "divrem", "nu": 2044, "nv": 1024, "batch": 2048, "vlen": "spread",
         "vmin": 4, "hard": 0},
        # odd widths between the power-of-two sizes, a batch that does not fill its last round
        {"name": "divrem_odd_3001", "kind": "divrem", "nu": 3001, "nv": 1777, "batch": 700, "vlen": "full",
         "hard": 0},
        # the largest precision, divisors from a quarter of the dividend to all of it
        {"name": "divrem_2p18_b256", "kind": "divrem", "nu": 8192, "nv": 8192, "batch": 256, "vlen": "spread",
         "vmin": 2048, "hard": 0},
        # full products at the benchmark's precision, and at the largest
        {"name": "mul_2p16_b4096", "kind": "mul", "na": 2048, "nb": 2048, "batch": 4096},
        {"name": "mul_2p18_b256", "kind": "mul", "na": 8192, "nb": 8192, "batch": 256},
        # an unbalanced product of odd widths
        {"name": "mul_odd_1531x333", "kind": "mul", "na": 1531, "nb": 333, "batch": 2000},
        # inverses of divisors that are used many times
        {"name": "shinv_2p16_b1024", "kind": "shinv", "nv": 1024, "h": 2048, "batch": 1024},
        # mixed precisions in one launch sequence
        {"name": "ragged_mixed_4096", "kind": "ragged", "count": 4096, "widths": "classes", "part": 4},
        # what a serving loop launches at a low arrival rate: a few requests of any width
        {"name": "ragged_serve_5", "kind": "ragged", "count": 5, "widths": "spread", "part": 8},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_MOST = 4096 * 2048 * 2048     # batch x width^2 of a drawn case: at most the benchmark's batch


def draw(rng):
    kind = rng.choice(["divrem", "divrem", "divrem", "mul", "shinv", "ragged"])
    if kind == "ragged":
        if rng.random() < 0.5:
            return {"kind": kind, "count": _log_int(rng, 1, 700), "widths": "classes", "part": rng.choice([2, 4, 8])}
        return {"kind": kind, "count": _log_int(rng, 1, 1200), "widths": "spread", "part": rng.choice([2, 4, 8])}
    n = _log_int(rng, 1000, 8192)
    if rng.random() < 0.3:
        n = rng.choice([1024, 2048, 4096, 8192])
    top = max(2, min(8192, _MOST // (n * n)))
    batch = _log_int(rng, 1, top) if rng.random() < 0.5 else _log_int(rng, max(1, top // 8), top)
    m = max(64, int(n * rng.uniform(0.125, 1.0)))
    if kind == "mul":
        return {"kind": kind, "na": n, "nb": m, "batch": batch}
    if kind == "shinv":
        return {"kind": kind, "nv": m, "h": n, "batch": batch}
    c = {"kind": kind, "nu": n, "nv": m, "batch": batch, "vlen": "full", "hard": int(rng.random() < 0.25)}
    if rng.random() < 0.3:
        c["vlen"], c["vmin"], c["hard"] = "spread", max(4, m // rng.choice([2, 4, 64])), 0
    return c


# -------------------------------------------------------------------- inputs


def _limbs(gen, batch, n):
    x = torch.randint(-2 ** 31, 2 ** 31, (batch, n), dtype=torch.int32, device="cuda", generator=gen)
    x[:, n - 1] = torch.where(x[:, n - 1] == 0, torch.ones_like(x[:, n - 1]), x[:, n - 1])
    return x


def _to_int(row):
    return int.from_bytes(np.ascontiguousarray(row).view("<u4").tobytes(), "little")


def _from_int(x, n):
    return np.frombuffer(int(x).to_bytes(4 * n, "little"), dtype="<i4")


def _adversarial(gen, u, v):
    """Every fourth instance: one of five families of divisors or dividends that stress the method."""
    nu, nv, batch = u.shape[1], v.shape[1], u.shape[0]
    w = _limbs(gen, batch, max(nu - nv - 1, 1)).cpu().numpy() if nu - nv >= 2 else None
    f = [torch.arange(3 + 4 * i, batch, 20, device="cuda") for i in range(5)]
    v[f[0]] = -1                                        # v = B^nv - 1
    v[f[1]] = 0                                         # v = B^(nv-1) + 1
    v[f[1], 0] = 1
    v[f[1], nv - 1] = 1
    v[f[2], nv - 1] = 1                                 # top limb 1
    if w is not None:
        for j in f[3].tolist():                         # u = v w + v - 1
            vi = _to_int(v[j].cpu().numpy())
            u[j] = torch.from_numpy(_from_int(vi * _to_int(w[j]) + vi - 1, nu).copy()).cuda()
    if nu >= nv:                                        # u < v
        u[f[4], nv - 1:] = 0


def _divrem_inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    u = _limbs(gen, case["batch"], case["nu"])
    v = _limbs(gen, case["batch"], case["nv"])
    if case["vlen"] == "spread":
        ln = torch.randint(case["vmin"], case["nv"] + 1, (case["batch"],), device="cuda", generator=gen)
        col = torch.arange(case["nv"], device="cuda")[None, :]
        v = torch.where(col >= ln[:, None], torch.zeros_like(v), v)
        top = torch.gather(v, 1, ln[:, None] - 1)
        v.scatter_(1, ln[:, None] - 1, torch.where(top == 0, torch.ones_like(top), top))
    if case["hard"]:
        _adversarial(gen, u, v)
    return u.contiguous(), v.contiguous()


def _divrem_nq(case):
    return max(1, case["nu"] - (case["vmin"] if case["vlen"] == "spread" else case["nv"]) + 1) \
        if not case["hard"] else max(1, case["nu"] - case["nv"] + 1)


def _ragged_inputs(case, seed):
    count = case["count"]
    shape = np.random.default_rng(1000 * count + case["part"])     # the widths belong to the case, the limbs to the seed
    if case["widths"] == "classes":
        ns = shape.choice([1024, 2048, 4096, 8192], count)
    else:
        ns = np.rint(2.0 ** shape.uniform(15.0, 18.0, count) / 32.0).astype(np.int64)
    nvs = shape.integers((ns + case["part"] - 1) // case["part"], ns + 1)
    rng = np.random.default_rng(seed)

    def rows(widths):
        ends = np.cumsum(widths)
        flat = np.frombuffer(rng.bytes(4 * int(ends[-1])), dtype="<u4").copy()
        flat[ends - 1] |= np.uint32(1)
        return np.split(flat, ends[:-1])
    return rows(ns), rows(nvs)


def prepare(case, seed):
    from paper_2606_06386_amd import binding
    kind = case["kind"]
    binding.lib()
    state = {"kind": kind, "mp": binding}
    if kind == "divrem":
        state["u"], state["v"] = _divrem_inputs(case, seed)
        state["nq"] = _divrem_nq(case)
    elif kind == "ragged":
        from paper_2606_06386_amd import ragged
        us, vs = _ragged_inputs(case, seed)
        state["batch"] = binding.Ragged(ragged.pack(us, vs))
    else:
        gen = torch.Generator(device="cuda")
        gen.manual_seed(seed)
        if kind == "mul":
            state["a"], state["b"] = (_limbs(gen, case["batch"], case[k]) for k in ("na", "nb"))
        else:
            state["v"] = _limbs(gen, case["batch"], case["nv"])
            state["h"], state["nw"] = case["h"], max(1, case["h"] - case["nv"] + 2)
    return state


def run(state):
    mp, kind = state["mp"], state["kind"]
    if kind == "divrem":
        return mp.divrem(state["u"], state["v"], nq=state["nq"])
    if kind == "mul":
        return mp.mul(state["a"], state["b"])
    if kind == "shinv":
        return mp.shinv(state["v"], state["h"], nw=state["nw"])
    b = state["batch"]
    b.run()
    return b.q, b.r, b.status


# ---------------------------------------------------------------------- work

_OPS = 32     # operations of one 32 x 32-bit limb product in 8-bit pieces: 16 multiply-adds


def _div_products(h, n):
    """limb products of a classical division of h by n limbs (the remainder's: one per quotient and divisor limb)"""
    return np.maximum(h - n + 1, 0) * n


def work(case):
    kind = case["kind"]
    if kind == "mul":
        na, nb, b = case["na"], case["nb"], case["batch"]
        return {"bytes": 8 * b * (na + nb), "flops": _OPS * b * na * nb}
    if kind == "shinv":
        b, h, nv = case["batch"], case["h"], case["nv"]
        nw = max(1, h - nv + 2)
        return {"bytes": 4 * b * (nv + nw + 1), "flops": _OPS * b * int(_div_products(h + 1, nv))}
    if kind == "divrem":
        b, nu, nv = case["batch"], case["nu"], case["nv"]
        lens = np.arange(case["vmin"], nv + 1) if case["vlen"] == "spread" else np.array([nv])
        mean = float(np.mean(_div_products(nu, lens)))
        return {"bytes": 4 * b * (nu + 2 * nv + _divrem_nq(case) + 1), "flops": _OPS * b * mean}
    if case["widths"] == "classes":
        ns = np.array([1024, 2048, 4096, 8192], dtype=np.float64)
    else:
        ns = 2.0 ** np.linspace(15.0, 18.0, 64) / 32.0
    part = case["part"]
    f = np.linspace(1.0 / part, 1.0, 64)[:, None]       # divisor length as a fraction of the dividend's
    limbs = float(np.mean(2 * ns + 0 * f + 2 * f * ns))
    return {"bytes": case["count"] * (4 * limbs + 52),
            "flops": _OPS * case["count"] * float(np.mean(_div_products(ns, f * ns)))}


# --------------------------------------------------------------------- exact


def exact(case, seed):
    """The results with Python integers (whole numbers); None where that takes long."""
    kind = case["kind"]
    if kind == "ragged" or work(case)["flops"] / _OPS > 1.5e9:
        return None
    state = prepare(case, seed)
    host = lambda t: [_to_int(r) for r in t.cpu().numpy()]  # noqa: E731
    stack = lambda xs, n: np.stack([_from_int(x, n) for x in xs])  # noqa: E731
    if kind == "mul":
        return stack([a * b for a, b in zip(host(state["a"]), host(state["b"]))], case["na"] + case["nb"])
    if kind == "shinv":
        ws = [(1 << (32 * case["h"])) // v for v in host(state["v"])]
        return stack(ws, state["nw"]), np.zeros(len(ws), dtype=np.int32)
    qr = [divmod(u, v) for u, v in zip(host(state["u"]), host(state["v"]))]
    return (stack([q for q, _ in qr], state["nq"]), stack([r for _, r in qr], case["nv"]),
            np.zeros(len(qr), dtype=np.int32))
