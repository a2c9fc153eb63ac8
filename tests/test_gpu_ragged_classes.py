"""The class kernels of ragged batches (more than two instances per compute
unit) with divisors of many strips and long quotients, every distinct instance
against the oracle: under each kind of class configuration, through both entry
points, eager and captured on a stream the library has not seen."""
import random

import numpy as np
import pytest

import oracle
from paper_2606_06386_amd import inputs as I
from paper_2606_06386_amd import ragged as R

pytestmark = pytest.mark.gpu
B = 1 << 32
DEFAULTS = [(256, 4), (256, 4), (512, 2), (1024, 2)]
CONFIGS = [DEFAULTS, [(256, 1), (256, 1), (512, 1), (1024, 1)], [(1024, 8), (512, 2), (1024, 3), (1024, 2)],
           [(512, 4), (1024, 2), (512, 8), (1024, 8)], [(256, 8), (512, 8), (1024, 1), (1024, 3)]]


@pytest.fixture
def mp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2606_06386_amd import binding
    binding.lib()
    knob = binding.get_knob(binding.MP_KNOB_SMALL_LIMIT)
    binding.set_knob(binding.MP_KNOB_SMALL_LIMIT, binding.MP_SMALL_LIMIT_AUTO)
    _configure(binding, DEFAULTS)
    yield binding
    _configure(binding, DEFAULTS)
    binding.set_knob(binding.MP_KNOB_SMALL_LIMIT, knob)


def _configure(binding, config):
    for cls, (threads, wgs_per_cu) in enumerate(config):
        binding.ragged_config(cls, threads, wgs_per_cu)


def _instances(widths):
    """(u, v, nq) of distinct instances: per width, divisors from one limb to all of
    the dividend's, structured ones among them, and the cases without a division"""
    rng = random.Random(sum(widths))
    rnd = lambda n: rng.getrandbits(32 * n) | 1 << (32 * n - 1)  # noqa: E731
    out = []
    for n in widths:
        for k in (0, 60, 299, n // 4, n // 2, n - 300, n - 2, n - 1):
            v = [rnd(k + 1), B ** k + 1, B ** (k + 1) - 1, B ** k + rng.getrandbits(32 * k) if k else 3][len(out) % 4]
            u = [rnd(n), B ** n - 1, min(v * (rnd(n - k) >> 1) + v - 1, B ** n - 1)][len(out) % 3]
            out.append((I.from_int(u, n), I.from_int(v, min(k + 1 + len(out) % 3, 8192)), n))
        out += [(I.from_int(rnd(n), n), np.zeros(n // 3, dtype=np.uint32), n),           # v = 0
                (I.from_int(rnd(n - 9), n), I.from_int(rnd(n - 8), n), 5),               # u < v
                (I.from_int(rnd(n), n), I.from_int(B ** (n // 2), n // 2 + 1), n),       # v = B^k
                (I.from_int(rnd(n), n), I.from_int(rnd(n // 2), n // 2), n // 3)]        # q wider than its row
    return out


def _batch(inst, count):
    """`count` instances, the distinct ones in turn (and what each has to give)"""
    want = [[np.asarray(x)[0] for x in oracle.divrem(u[None], v[None], nq=nq, nr=len(v))] for u, v, nq in inst]
    ids = np.arange(count) % len(inst)
    return R.pack([inst[j][0] for j in ids], [inst[j][1] for j in ids], [inst[j][2] for j in ids]), ids, want


def _check(rb, packed, ids, want, label):
    import torch
    torch.cuda.synchronize()
    q, r, st = (x.cpu().numpy().view(np.uint32) for x in (rb.q, rb.r, rb.status))
    qs, rs = R.unpack(q, packed["desc"], "q"), R.unpack(r, packed["desc"], "r")
    bad = [j for j, i in enumerate(ids)
           if st[j] != want[i][2] or (qs[j] != want[i][0]).any() or (rs[j] != want[i][1]).any()]
    assert not bad, f"{label}: {len(bad)} instances differ, first {[(j, int(ids[j]), int(st[j])) for j in bad[:6]]}"
    rb.q.fill_(-5)
    rb.r.fill_(-5)
    rb.status.fill_(-1)


def _cus():
    import torch
    return torch.cuda.get_device_properties(0).multi_processor_count


def test_every_class_and_configuration(mp):
    packed, ids, want = _batch(_instances((701, 1024, 1025, 2048, 2049, 4096, 4097, 8192)), 2 * _cus() + 41)
    rb = mp.Ragged(packed)
    for config in CONFIGS:
        _configure(mp, config)
        for entry in ("run", "run_static"):
            getattr(rb, entry)()
            _check(rb, packed, ids, want, f"{entry} {config}")


@pytest.mark.parametrize("widths", [(8192,), (4096, 8192)])
def test_widest_class_two_and_three_workgroups_per_two_units(mp, widths):
    """(more than 1.5 instances of it per compute unit, without and with the next class beside)"""
    packed, ids, want = _batch(_instances(widths), len(widths) * (2 * _cus() + 1))
    rb = mp.Ragged(packed)
    for config in (DEFAULTS, CONFIGS[3]):
        _configure(mp, config)
        rb.run()
        _check(rb, packed, ids, want, f"{widths} {config}")


@pytest.mark.parametrize("small", [16, 100])
def test_shorter_blocks(mp, small):
    packed, ids, want = _batch(_instances((1024, 2049, 8192)), 2 * _cus() + 41)
    mp.set_knob(mp.MP_KNOB_SMALL_LIMIT, small)
    rb = mp.Ragged(packed)
    rb.run()
    _check(rb, packed, ids, want, f"small_limit {small}")


def test_captured_on_a_stream_not_seen_before(mp):
    import torch
    packed, ids, want = _batch(_instances((1000, 2048, 4096, 8192)), 2 * _cus() + 41)
    rb = mp.Ragged(packed)
    rb.run()
    _check(rb, packed, ids, want, "eager")
    g, s = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            rb.run()
    torch.cuda.current_stream().wait_stream(s)
    for rep in range(3):
        torch.arange(1 << 16, device="cuda").sum().item()      # unrelated eager work
        g.replay()
        _check(rb, packed, ids, want, f"replay {rep}")
